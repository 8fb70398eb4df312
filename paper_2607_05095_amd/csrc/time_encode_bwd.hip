// time_encode_bwd.hip -- backward of the TGAT time features (Sec. 6.1; the
// frequencies and phases of the time encoder are trained with the model):
//   a_ej      = fmaf(omega[j], dt_e, phi[j])            (the forward's argument)
//   dphi[j]   = sum_e dte[e,j] * (-sin a_ej)
//   domega[j] = sum_e dte[e,j] * (-sin a_ej) * dt_e
//
// Each output is a sum over every edge of the block (millions of terms of
// both signs).  An fp32 sine (a few ulp per term) leaves the sum of a column
// that nearly cancels with a relative error far above 1e-5, so the sine is
// evaluated in fp64 on the exact fp32 argument and every product and sum is
// fp64: a one-step Cody-Waite reduction by pi (x = k*pi + r, |r| <= pi/2,
// one fused multiply-add with the fp64 rounding of pi) and an odd polynomial
// of degree 11 for sin(r), whose coefficients were fitted near-minimax
// (Lawson's iteratively reweighted least squares on Chebyshev nodes of
// [0, (pi/2)^2] in r^2, on the relative error of sin): its relative error is
// below 2.4e-11 on |r| <= pi/2, and the one-step reduction adds at most
// 4e-11 absolute for |x| <= 1e6.  Terms of a cancelling column need about
// 1e-8 (the 1e-5 target on a sum 1e-3 of the sum of its magnitudes).
// The range is checked once per row: a row whose bound
// fmaf(max|omega|, |dt|, max|phi|) exceeds 1e6 (or is not finite) is left
// to the library sine in a cold second pass of the workgroups that met one.
//
// Determinism: the reduction order depends only on N, E, the first and last
// offset, d_t and the width of a thread's accesses.  Workgroup b of
// nblk = tb_grid(N, E, VEC) owns the b-th of nblk equal ranges of edges; each thread accumulates its column chunk over its rows in a fixed
// order, the row lanes are added in lane order through LDS, and a second
// kernel adds the per-workgroup partials in a fixed tree.  Repeated calls give
// bitwise-identical results.
//
// About 23 vector instructions per element, most of them fp64: 153 us of issue
// for 2.64 M edges x 100, against 170 of their bytes.  Neither is reached: the
// vector units are busy in 56 % of the kernel's cycles, and the five waves of a
// SIMD wait in 73 % of theirs, for rows of dte and at the three barriers of a
// tile.  So the chip has to stay full to the end: as many workgroups as are
// resident at once where N allows them, all with the same number of edges.  Groups of 32 segments dealt out to 2048
// workgroups left some with five groups and most with four, in two rounds of
// residence: 2.64 M edges of 264,000 segments x 100 fp32 286 -> 258 us, 0.19 M of
// ragged ones x 128 bf16 52 -> 41 us.  More rows of dte in flight per thread
// (2, 4, 5) change nothing or cost registers: 268 / 265 / 263 us.
#include "common.h"

namespace fast {

constexpr int TB_THREADS = 256;
constexpr int TB_SEGS = 8;           // fewest destination segments per workgroup, on average
constexpr int TB_MAX_BLOCKS = 1280;  // 5 workgroups per CU, what the registers hold at once
constexpr int TB_WIN = TB_THREADS;   // segments whose ends and times a tile stages
constexpr int TB_TILE_MAX = 256;     // rows staged per tile
constexpr int TB_MAX_VEC = 8;

__host__ __device__ inline int64_t tb_blocks(int64_t N) {
  const int64_t g = (N + TB_SEGS - 1) / TB_SEGS;
  return g < TB_MAX_BLOCKS ? g : TB_MAX_BLOCKS;
}
// Workgroups of a call.  A workgroup pays for its start and for 2 d_t partials
// that are written and read again: 128 edges each while the chip is not full
// (20,000 edges 12 us with 156 workgroups, 18 with 62), 192 beyond or 320 where a
// thread has 8 columns and twice the sums (0.24 M edges x 100 fp32: 32 us so, 33.5
// with 320 edges; x 128 bf16: 39 us so, 46 with 192), up to the workgroups
// resident at once (8 columns per thread: 4 per CU) and up to tb_blocks(N), for
// which the workspace has room: 1e5 edges of 8 segments are left to one (4.5 ms).
inline int64_t tb_grid(int64_t N, int64_t E, int vec) {
  const int64_t most = tb_blocks(N), cap = vec >= 8 ? 1024 : TB_MAX_BLOCKS;
  const int64_t few = (E + 127) / 128 < 512 ? (E + 127) / 128 : 512, many = E / (vec >= 8 ? 320 : 192);
  int64_t g = few > many ? few : many;
  g = g < cap ? g : cap;
  return g < most ? g : most;
}

// sin(x) in fp64 for an fp32 x with |x| <= 1e6.  k = round(x / pi) comes
// from the magic-number rounding fma(x, 1/pi, 1.5*2^52), whose low word
// holds k in two's complement; r = x - k*pi in one fused multiply-add
// (k <= 3.2e5, so the neglected k*(pi - PI_HI) stays below 4e-11), and the
// parity of k flips the sign of r, since sin x = (-1)^k sin r = sin((-1)^k r).
__device__ __forceinline__ double sin_reduced(float xf) {
  const double x = double(xf);
  const double PI_HI = 0x1.921fb54442d18p+1;
  const double INV_PI = 0x1.45f306dc9c883p-2, MAGIC = 0x1.8p52;
  const double t = fma(x, INV_PI, MAGIC);
  const double k = t - MAGIC;
  double r = fma(-k, PI_HI, x);
  const uint32_t flip = uint32_t(__double2loint(t)) << 31;
  r = __hiloint2double(int(uint32_t(__double2hiint(r)) ^ flip), __double2loint(r));
  const double r2 = r * r;
  double p = -0x1.9a6887b9bb2dbp-26;
  p = fma(p, r2, 0x1.71708023de99ap-19);
  p = fma(p, r2, -0x1.a017d9a03cff9p-13);
  p = fma(p, r2, 0x1.11110c4a00de9p-7);
  p = fma(p, r2, -0x1.555555476965fp-3);
  return fma(r * r2, p, r);                   // r + r^3 p(r^2)
}

// A row is reduced in-line when every |fmaf(omega[j], dt, phi[j])| of its
// columns is at most 1e6 * (1 + 2^-22) < 2^20: fmaf(max|omega|, |dt|,
// max|phi|) bounds them up to two roundings.  Not-less-than sends a NaN
// bound (a NaN time) to the library path too.
constexpr float TB_ROW_LIMIT = 1.0e6f;
__device__ __forceinline__ bool tb_row_ok(float om_max, float ph_max, float dt) {
  return fmaf(om_max, fabsf(dt), ph_max) <= TB_ROW_LIMIT;
}
__device__ __attribute__((noinline)) double sin_library(double x) { return sin(x); }

// Last segment that begins at or before edge e (64 probes at a time; every
// lane of the wave takes part and returns it); in [0, N) whatever off holds.
__device__ __forceinline__ int64_t tb_segment(const int32_t* __restrict__ off, int64_t N, int64_t e) {
  const int lane = threadIdx.x & 63;
  int64_t lo = 0, hi = N;                      // offsets before lo are at most e, from hi on above
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) >> 6;
    const int64_t p = lo + int64_t(lane + 1) * step - 1;
    const bool below = p < hi && int64_t(off[p]) <= e;
    const int c = __popcll(__ballot(below));
    const int64_t cap = lo + int64_t(c + 1) * step - 1;
    lo += int64_t(c) * step;
    hi = cap < hi ? cap : hi;
  }
  return lo > 0 ? lo - 1 : 0;
}

struct TbTile {
  int32_t end[TB_WIN];                         // of the window's segments
  float tdst[TB_WIN], dt[TB_TILE_MAX];
  int64_t next;                                // the last row's segment, from the window's first
};

// Calls f(t0, nrows) for tiles of up to `tile` rows that cover the edges
// [t0, t1), with the rows' time differences in s.dt.  Every thread of the
// workgroup calls it.  A tile's rows find their segments in a window of TB_WIN
// segments in LDS, and the tile ends with the window -- unless that leaves less
// than a quarter of it, as in blocks of mostly empty segments: then each row
// searches the offsets in memory by itself, and empty segments cost nothing
// (1000 edges x 100 fp32 of 1e6 segments: 320 us with the windows walked one
// after the other, 15 so; no difference in dense blocks).
template <class F>
__device__ __forceinline__ void tb_tiles(TbTile& s, const int32_t* __restrict__ off, int64_t N, int64_t E,
                                         const float* __restrict__ dst_t, const float* __restrict__ edge_t,
                                         int64_t t0, int64_t t1, int tile, F&& f) {
  if (t0 >= t1) return;
  int64_t seg = tb_segment(off, N, t0);
  while (t0 < t1) {
    const int ns = int(N - seg < TB_WIN ? N - seg : TB_WIN);
    const int64_t e = t0 + threadIdx.x;
    const float te = int(threadIdx.x) < tile && e < t1 ? edge_t[e] : 0.f;
    if (int(threadIdx.x) < ns) {
      s.end[threadIdx.x] = int32_t(clamp64(off[seg + threadIdx.x + 1], 0, E));
      s.tdst[threadIdx.x] = dst_t[seg + threadIdx.x];
    }
    __syncthreads();
    // rows behind the last segment's end, if any, belong to it
    const int64_t w1 = seg + ns == N || s.end[ns - 1] > t1 ? t1 : s.end[ns - 1];
    int nrows = int(w1 - t0 < tile ? w1 - t0 : tile);
    if (nrows > tile / 4 || w1 == t1) {
      if (int(threadIdx.x) < nrows) {
        int lo = 0, hi = ns - 1;               // first segment of the window that ends behind e
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (s.end[mid] > e) hi = mid; else lo = mid + 1;
        }
        s.dt[threadIdx.x] = s.tdst[lo] - te;
        if (int(threadIdx.x) == nrows - 1) s.next = lo;
      }
    } else {                                   // the same in memory, over all segments from seg on
      nrows = int(t1 - t0 < tile ? t1 - t0 : tile);
      if (int(threadIdx.x) < nrows) {
        int64_t lo = seg, hi = N - 1;
        while (lo < hi) {
          const int64_t mid = (lo + hi) >> 1;
          if (int64_t(off[mid + 1]) > e) hi = mid; else lo = mid + 1;
        }
        s.dt[threadIdx.x] = dst_t[lo] - te;
        if (int(threadIdx.x) == nrows - 1) s.next = lo - seg;
      }
    }
    __syncthreads();
    f(t0, nrows);
    t0 += nrows;
    seg += s.next;
    __syncthreads();
  }
}

// Grid: tb_grid(N, E, VEC) workgroups.  Thread t owns the column chunk t % cpr of
// the rows t / cpr, t / cpr + rpp, ... of every tile, as in the forward.
// partial: [2 * d_t][nblk] fp64 (domega rows first, then dphi).
template <typename TG, int VEC, bool NT>
__global__ void __launch_bounds__(TB_THREADS) k_time_encode_bwd(
    const int32_t* __restrict__ off, int64_t N, int64_t E, const float* __restrict__ dst_t,
    const float* __restrict__ edge_t, const float* __restrict__ omega,
    const float* __restrict__ phi, int d_t, const TG* __restrict__ dte,
    double* __restrict__ partial) {
  __shared__ TbTile s_tile;
  __shared__ double s_red[TB_THREADS * VEC * 2];

  const int64_t nblk = gridDim.x;
  const int cpr = d_t / VEC;               // vector chunks per row (<= TB_THREADS)
  const int rpp = TB_THREADS / cpr;        // rows per pass
  const int rsub = int(threadIdx.x) / cpr;
  const int c0 = int(threadIdx.x) - rsub * cpr;
  const bool active = rsub < rpp;
  const int tile = (TB_TILE_MAX / rpp) * rpp;

  float om[VEC], ph[VEC], om_max = 0.f, ph_max = 0.f;
  double acc_w[VEC], acc_p[VEC];
  bool big = false;                        // a row beyond the reduction's range
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    om[k] = active ? omega[c0 * VEC + k] : 0.f;
    ph[k] = active ? phi[c0 * VEC + k] : 0.f;
    om_max = fmaxf(om_max, fabsf(om[k]));
    ph_max = fmaxf(ph_max, fabsf(ph[k]));
    acc_w[k] = 0.0;
    acc_p[k] = 0.0;
  }

  const int64_t e0 = clamp64(off[0], 0, E), e1 = clamp64(off[N], e0, E);
  const int64_t t0 = e0 + (e1 - e0) * int64_t(blockIdx.x) / nblk;
  const int64_t t1 = e0 + (e1 - e0) * (int64_t(blockIdx.x) + 1) / nblk;
  const float* s_dt = s_tile.dt;
  tb_tiles(s_tile, off, N, E, dst_t, edge_t, t0, t1, tile, [&](int64_t r0, int nrows) {
    if (!active) return;
    for (int row = rsub; row < nrows; row += rpp) {
      const float dt = s_dt[row];
      if (__builtin_expect(!tb_row_ok(om_max, ph_max, dt), 0)) {
        big = true;                        // left to the cold pass
        continue;
      }
      Raw<TG, VEC> raw;
      raw.template load<NT>(dte + (r0 + row) * d_t + c0 * VEC);
      float g[VEC];
      raw.unpack(g);
      const double dtd = double(dt);
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        // the term is -g sin x
        const double q = double(g[k]) * sin_reduced(fmaf(om[k], dt, ph[k]));
        acc_p[k] -= q;
        acc_w[k] = fma(-q, dtd, acc_w[k]);
      }
    }
  });

  // Cold pass, only in a workgroup that met a row beyond the reduction's
  // range (or not finite): the same rows again, adding just those rows with
  // the library sine.  The order stays a fixed function of the inputs.
  if (__syncthreads_or(big)) {
    tb_tiles(s_tile, off, N, E, dst_t, edge_t, t0, t1, tile, [&](int64_t r0, int nrows) {
      if (!active || !big) return;
      for (int row = rsub; row < nrows; row += rpp) {
        const float dt = s_dt[row];
        if (tb_row_ok(om_max, ph_max, dt)) continue;
        Raw<TG, VEC> raw;
        raw.template load<false>(dte + (r0 + row) * d_t + c0 * VEC);
        float g[VEC];
        raw.unpack(g);
        for (int k = 0; k < VEC; ++k) {
          const float x = fmaf(om[k], dt, ph[k]);
          const double gs = -double(g[k]) * sin_library(double(x));
          acc_p[k] += gs;
          acc_w[k] = fma(gs, double(dt), acc_w[k]);
        }
      }
    });
  }

  // row lanes of one column chunk, added in lane order
  if (active) {
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
      s_red[(rsub * d_t + c0 * VEC + k) * 2 + 0] = acc_w[k];
      s_red[(rsub * d_t + c0 * VEC + k) * 2 + 1] = acc_p[k];
    }
  }
  __syncthreads();
  for (int j = threadIdx.x; j < d_t; j += TB_THREADS) {
    double w = 0.0, p = 0.0;
    for (int r = 0; r < rpp; ++r) {
      w += s_red[(r * d_t + j) * 2 + 0];
      p += s_red[(r * d_t + j) * 2 + 1];
    }
    partial[int64_t(j) * nblk + blockIdx.x] = w;
    partial[int64_t(d_t + j) * nblk + blockIdx.x] = p;
  }
}

// One workgroup per output value: out[j] for j < d_t is domega, then dphi.
// Strided fp64 partial sums per thread, then a fixed LDS tree.
__global__ void __launch_bounds__(TB_THREADS) k_time_encode_bwd_final(
    const double* __restrict__ partial, int64_t nblk, int d_t, float* __restrict__ domega,
    float* __restrict__ dphi) {
  __shared__ double s[TB_THREADS];
  const int row = blockIdx.x;
  double acc = 0.0;
  for (int64_t b = threadIdx.x; b < nblk; b += TB_THREADS) acc += partial[row * nblk + b];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int w = TB_THREADS / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (row < d_t) domega[row] = float(s[0]);
    else dphi[row - d_t] = float(s[0]);
  }
}

template <typename TG, int VEC>
static void launch_tb(const fast_tcsr_t* g, const float* omega, const float* phi, int d_t,
                      const void* dte, double* partial, hipStream_t st) {
  const int64_t nb = tb_grid(g->num_dst, g->num_edges, VEC);
  const bool nt = (size_t(d_t) * sizeof(TG)) % CACHE_LINE == 0 && aligned(dte, CACHE_LINE);
  if (nt)
    hipLaunchKernelGGL((k_time_encode_bwd<TG, VEC, true>), dim3(uint32_t(nb)), dim3(TB_THREADS),
                       0, st, g->dst_offsets, g->num_dst, g->num_edges, g->dst_t, g->edge_t,
                       omega, phi, d_t, static_cast<const TG*>(dte), partial);
  else
    hipLaunchKernelGGL((k_time_encode_bwd<TG, VEC, false>), dim3(uint32_t(nb)), dim3(TB_THREADS),
                       0, st, g->dst_offsets, g->num_dst, g->num_edges, g->dst_t, g->edge_t,
                       omega, phi, d_t, static_cast<const TG*>(dte), partial);
}

// Widest vector of VEC elements that divides d_t, keeps the row's chunks
// within one workgroup and matches the pointer's alignment; 0 if none.
static int pick_vec(int d_t, int esz, const void* p) {
  for (int v = TB_MAX_VEC; v >= 1; v >>= 1) {
    if (v * esz > 16) continue;
    if (d_t % v == 0 && d_t / v <= TB_THREADS && aligned(p, size_t(v) * esz)) return v;
  }
  return 0;
}

}  // namespace fast

using namespace fast;

extern "C" size_t fast_time_encode_bwd_workspace(int64_t num_dst, int d_t) {
  if (num_dst < 0 || d_t <= 0) return 0;
  return align_up(size_t(2) * size_t(d_t) * size_t(tb_blocks(num_dst)) * sizeof(double), 256) + 256;
}

extern "C" fast_status_t fast_time_encode_bwd(const fast_tcsr_t* g, const float* omega,
                                              const float* phi, int d_t, const void* dte,
                                              fast_dtype_t dte_dtype, float* domega, float* dphi,
                                              void* ws, size_t ws_bytes, fast_stream_t stream) {
  const char* fn = "fast_time_encode_bwd";
  if (!g) return fail(FAST_ERR_INVALID_ARG, "%s: graph is NULL", fn);
  if (g->num_dst < 0 || g->num_edges < 0) return fail(FAST_ERR_INVALID_ARG, "%s: negative size", fn);
  if (g->num_edges >= (int64_t(1) << 31)) return fail(FAST_ERR_UNSUPPORTED, "%s: E >= 2^31", fn);
  if (d_t <= 0) return fail(FAST_ERR_INVALID_ARG, "%s: d_t = %d <= 0", fn, d_t);
  if (dte_dtype != FAST_F32 && dte_dtype != FAST_BF16) return fail(FAST_ERR_INVALID_ARG, "%s: bad dtype", fn);
  if (g->num_dst == 0 && g->num_edges > 0)
    return fail(FAST_ERR_INVALID_ARG, "%s: E > 0 edges but no destination", fn);
  if (!domega || !dphi) return fail(FAST_ERR_INVALID_ARG, "%s: NULL domega/dphi", fn);
  if (!aligned(domega, 4) || !aligned(dphi, 4))
    return fail(FAST_ERR_UNSUPPORTED, "%s: domega/dphi not 4-byte aligned", fn);
  const size_t need = fast_time_encode_bwd_workspace(g->num_dst, d_t);
  if (!ws || ws_bytes < need)
    return fail(FAST_ERR_WORKSPACE, "%s: workspace of %zu bytes < %zu", fn, ws_bytes, need);
  if (!aligned(ws, 8)) return fail(FAST_ERR_UNSUPPORTED, "%s: workspace not 8-byte aligned", fn);
  const int esz = elem_size(dte_dtype);
  int vec = 1;
  if (g->num_edges > 0) {
    if (!g->dst_offsets || !g->dst_t || !g->edge_t || !omega || !phi || !dte)
      return fail(FAST_ERR_INVALID_ARG, "%s: NULL dst_offsets/dst_t/edge_t/omega/phi/dte", fn);
    vec = pick_vec(d_t, esz, dte);
    if (vec == 0)
      return fail(FAST_ERR_UNSUPPORTED,
                  "%s: d_t = %d needs more than %d vector chunks per row, or dte is misaligned",
                  fn, d_t, TB_THREADS);
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  double* partial = static_cast<double*>(ws);
  int64_t nblk = 0;
  if (g->num_edges > 0) {
    nblk = tb_grid(g->num_dst, g->num_edges, vec);
    if (dte_dtype == FAST_F32) {
      switch (vec) {
        case 4: launch_tb<float, 4>(g, omega, phi, d_t, dte, partial, st); break;
        case 2: launch_tb<float, 2>(g, omega, phi, d_t, dte, partial, st); break;
        default: launch_tb<float, 1>(g, omega, phi, d_t, dte, partial, st); break;
      }
    } else {
      switch (vec) {
        case 8: launch_tb<uint16_t, 8>(g, omega, phi, d_t, dte, partial, st); break;
        case 4: launch_tb<uint16_t, 4>(g, omega, phi, d_t, dte, partial, st); break;
        case 2: launch_tb<uint16_t, 2>(g, omega, phi, d_t, dte, partial, st); break;
        default: launch_tb<uint16_t, 1>(g, omega, phi, d_t, dte, partial, st); break;
      }
    }
  }
  // with no edges every sum is empty: the final pass writes zeros
  hipLaunchKernelGGL(k_time_encode_bwd_final, dim3(uint32_t(2 * d_t)), dim3(TB_THREADS), 0, st,
                     partial, nblk, d_t, domega, dphi);
  return check_launch(fn);
}
