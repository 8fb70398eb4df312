// indexed_rows.hip -- the two reductions that indexed operands need (Sec. 4.2:
// many positions of a batch read one de-duplicated row through the inverse
// index; the gradient of that row is the sum over those positions).
//
// fast_occurrence_csr: for every row, its positions in ascending order -- a
// stable counting sort of the index, done as an LSD radix sort of (key,
// position) pairs over digits of at most 8 bits.  Each pass: per-tile digit
// histograms, one scan of the (digit, tile) counts, and a scatter in which
// every item finds its rank among the tile's items with the same digit from
// wave ballots, in position order -- stable, so after the last pass each
// row's positions are ascending.  Positions whose index is outside the row range
// get the key num_rows and sort behind every valid one.
//
// fast_index_add_rows: dst[u] = sum of src rows over the occurrences of u,
// in occurrence order, accumulated in fp64 and rounded once to fp32.  A row
// with at most IA_PIECE occurrences is summed by one group of lanes; a row
// read by more positions (a hub id of a skewed batch) is summed as a fixed
// three-level tree: pieces of consecutive occurrences, each summed by its own
// group, then (when there are many pieces) groups of consecutive piece sums,
// then the row adds its group (or piece) sums in order -- each level about
// cbrt(count) long, so no group walks a long chain of dependent loads.  The
// tree depends only on the counts, so the result is the same on every run.
#include "scan.h"

namespace fast {

// ------------------------------------------------------------------ radix sort
// A pass is bound by its scattered writes and by launch latency, not by its
// bytes (8 read and 8 written per item): a tile is sorted by digit in LDS
// first, so that the items of one digit leave as one contiguous run, and the
// digits are as narrow as the pass count allows (7 + 6 + 6 bits for 19-bit
// keys), so that a run of a tile is 32-64 items.  Items are loaded once and
// keep their rank in registers; the counts' prefixes take one launch, a
// workgroup per digit.  Against tiles of 2048 items scattered straight from
// registers with 8-bit digits and a two-launch scan, one list of 2.64 M Zipf
// positions over 4e5 rows went from 174 to 85 us (first scatter 56 -> 15),
// of 1.32 M uniform positions over 1.2e6 rows from 133 to 66 us.
constexpr int RS_THREADS = 512;
constexpr int RS_WAVES = RS_THREADS / 64;
constexpr int RS_ROUNDS = 8;                        // 64-item rounds per wave
constexpr int RS_TILE = RS_THREADS * RS_ROUNDS;     // 4096 items per tile
constexpr int RS_MAX_BITS = 8;
constexpr int RS_DIGITS = 1 << RS_MAX_BITS;

inline int64_t rs_tiles(int64_t n) { return (n + RS_TILE - 1) / RS_TILE; }

// Items of a tile: wave w takes items [w*512, (w+1)*512) in rounds of 64
// consecutive items, so (wave, round, lane) order is position order.
__device__ __forceinline__ int64_t rs_item(int64_t tile, int w, int r, int lane) {
  return tile * RS_TILE + int64_t(w) * (RS_ROUNDS * 64) + r * 64 + lane;
}

// Keys and values of a thread's items: in the first pass the key comes from
// the index (num_rows for a position outside the row range) and the value is
// the position.  Positions past n read the last item; the caller masks them.
struct RsSrc {
  const int32_t* index;   // first pass
  const int32_t* keys;    // later passes
  const int32_t* vals;
  int32_t num_rows;
  __device__ void load_keys(int64_t tile, int w, int lane, int64_t n, uint32_t (&k)[RS_ROUNDS]) const {
    const int32_t* __restrict__ p = index ? index : keys;
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) {
      const int64_t i = rs_item(tile, w, r, lane);
      k[r] = uint32_t(p[i < n ? i : n - 1]);
    }
    if (index) {
#pragma unroll
      for (int r = 0; r < RS_ROUNDS; ++r) k[r] = k[r] < uint32_t(num_rows) ? k[r] : uint32_t(num_rows);
    }
  }
  __device__ void load_vals(int64_t tile, int w, int lane, int64_t n, int32_t (&v)[RS_ROUNDS]) const {
#pragma unroll
    for (int r = 0; r < RS_ROUNDS; ++r) {
      const int64_t i = rs_item(tile, w, r, lane);
      v[r] = index ? int32_t(i) : vals[i < n ? i : n - 1];
    }
  }
};

// Lanes of the wave holding the same digit as this lane (inactive lanes excluded).
template <int BITS>
__device__ __forceinline__ uint64_t digit_match(uint32_t d, bool valid) {
  uint64_t m = __ballot(valid);
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t bal = __ballot(bit);
    m &= bit ? bal : ~bal;
  }
  return m;
}

// hist[d * T + tile] = items of the tile whose digit is d.  The lanes that
// share the first lane's digit add up to one LDS atomic: after a first pass
// a hub row's items lie side by side, and 64 atomics on one digit serialise.
template <int BITS>
__global__ void __launch_bounds__(RS_THREADS) k_rs_hist(RsSrc src, int64_t n, int shift,
                                                       uint32_t* hist, int64_t T) {
  constexpr int BINS = 1 << BITS;
  __shared__ uint32_t s_h[BINS];
  if (threadIdx.x < BINS) s_h[threadIdx.x] = 0;
  const int64_t tile = blockIdx.x;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t key[RS_ROUNDS];
  src.load_keys(tile, w, lane, n, key);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const bool valid = rs_item(tile, w, r, lane) < n;     // a prefix of the lanes
    const uint32_t d = (key[r] >> shift) & (BINS - 1);
    const uint32_t d0 = uint32_t(__builtin_amdgcn_readfirstlane(int(d)));
    const uint64_t same = __ballot(valid && d == d0);
    if (lane == 0 && same) atomicAdd(&s_h[d0], uint32_t(__popcll(same)));
    else if (valid && d != d0) atomicAdd(&s_h[d], 1u);
  }
  __syncthreads();
  if (threadIdx.x < BINS) hist[int64_t(threadIdx.x) * T + tile] = s_h[threadIdx.x];
}

// One workgroup per digit d: hist[d * T ...] becomes its exclusive prefix
// over the tiles, total[d] the digit's count.
constexpr int RS_ROW_ITEMS = 4;
__global__ void __launch_bounds__(SCAN_THREADS) k_rs_rowscan(uint32_t* hist, int64_t T, uint32_t* total) {
  __shared__ uint32_t lds4[4];
  uint32_t* row = hist + int64_t(blockIdx.x) * T;
  uint32_t carry = 0;
  for (int64_t t0 = 0; t0 < T; t0 += SCAN_THREADS * RS_ROW_ITEMS) {
    const int64_t i0 = t0 + int64_t(threadIdx.x) * RS_ROW_ITEMS;
    uint32_t c[RS_ROW_ITEMS], sum = 0;
#pragma unroll
    for (int k = 0; k < RS_ROW_ITEMS; ++k) {
      c[k] = i0 + k < T ? row[i0 + k] : 0u;
      sum += c[k];
    }
    uint32_t tot;
    uint32_t run = carry + block_exclusive_scan(sum, lds4, tot);
#pragma unroll
    for (int k = 0; k < RS_ROW_ITEMS; ++k) {
      if (i0 + k < T) row[i0 + k] = run;
      run += c[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// Exclusive prefixes of x and of y over the workgroup's RS_THREADS threads.
__device__ __forceinline__ void rs_block_scan2(uint32_t& x, uint32_t& y, uint2* lds) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t ix = x, iy = y;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t ux = __shfl_up(ix, o, 64), uy = __shfl_up(iy, o, 64);
    if (lane >= o) {
      ix += ux;
      iy += uy;
    }
  }
  if (lane == 63) lds[w] = make_uint2(ix, iy);
  __syncthreads();
  uint32_t bx = 0, by = 0;
#pragma unroll
  for (int j = 0; j < RS_WAVES; ++j) {
    bx += j < w ? lds[j].x : 0u;
    by += j < w ? lds[j].y : 0u;
  }
  x = bx + ix - x;
  y = by + iy - y;
}

// base[d * T + tile]: items of digit d in the tiles before this one; total[d]:
// items of digit d.  The tile is sorted by digit in LDS (stable: wave, round,
// lane order), then written out run by run.
template <int BITS>
__global__ void __launch_bounds__(RS_THREADS) k_rs_scatter(RsSrc src, int64_t n, int shift,
                                                          const uint32_t* __restrict__ base,
                                                          const uint32_t* __restrict__ total,
                                                          int64_t T, int32_t* __restrict__ keys_out,
                                                          int32_t* __restrict__ vals_out) {
  constexpr int BINS = 1 << BITS;
  static_assert(BINS <= RS_THREADS, "a thread per digit");
  __shared__ uint32_t s_cnt[RS_WAVES][BINS];
  __shared__ uint2 s_scan[RS_WAVES];
  __shared__ uint32_t s_base[BINS];
  __shared__ int32_t s_key[RS_TILE], s_val[RS_TILE];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, b = threadIdx.x;
  const int64_t tile = blockIdx.x;
  const uint64_t lt = (uint64_t(1) << lane) - 1;
  uint32_t key[RS_ROUNDS], rank[RS_ROUNDS];
  int32_t val[RS_ROUNDS];
  src.load_keys(tile, w, lane, n, key);
  src.load_vals(tile, w, lane, n, val);
  const uint32_t before = b < BINS ? base[int64_t(b) * T + tile] : 0u;
  uint32_t dbase = b < BINS ? total[b] : 0u;
  for (int j = b; j < RS_WAVES * BINS; j += RS_THREADS) (&s_cnt[0][0])[j] = 0u;
  __syncthreads();
  // rank of each item among the wave's items of its digit
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    const bool valid = rs_item(tile, w, r, lane) < n;
    const uint32_t d = (key[r] >> shift) & (BINS - 1);
    const uint64_t m = digit_match<BITS>(d, valid);
    const uint32_t seen = s_cnt[w][d];
    rank[r] = seen + uint32_t(__popcll(m & lt));
    if (valid && (m & lt) == 0) s_cnt[w][d] = seen + uint32_t(__popcll(m));   // lowest lane of its digit
  }
  __syncthreads();
  // prefix over the waves, then over the digits: s_cnt[w][d] becomes the
  // tile position of wave w's first item of digit d
  uint32_t c[RS_WAVES], start = 0;
  if (b < BINS) {
#pragma unroll
    for (int j = 0; j < RS_WAVES; ++j) {
      c[j] = start;
      start += s_cnt[j][b];
    }
  }
  rs_block_scan2(start, dbase, s_scan);
  if (b < BINS) {
#pragma unroll
    for (int j = 0; j < RS_WAVES; ++j) s_cnt[j][b] = start + c[j];
    s_base[b] = dbase + before - start;        // output slot of tile position p: s_base[d] + p
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RS_ROUNDS; ++r) {
    if (rs_item(tile, w, r, lane) < n) {
      const uint32_t p = s_cnt[w][(key[r] >> shift) & (BINS - 1)] + rank[r];
      s_key[p] = int32_t(key[r]);
      s_val[p] = val[r];
    }
  }
  __syncthreads();
  const int64_t left = n - tile * RS_TILE;
  const int m = int(left < RS_TILE ? left : RS_TILE);
  for (int p = b; p < m; p += RS_THREADS) {
    const uint32_t k = uint32_t(s_key[p]);
    const uint32_t pos = s_base[(k >> shift) & (BINS - 1)] + uint32_t(p);
    keys_out[pos] = int32_t(k);
    vals_out[pos] = s_val[p];
  }
}

template <int BITS>
static void rs_pass(const RsSrc& src, int64_t n, int shift, uint32_t* hist, uint32_t* total,
                    int32_t* keys_out, int32_t* vals_out, hipStream_t st) {
  const int64_t T = rs_tiles(n);
  hipLaunchKernelGGL(k_rs_hist<BITS>, dim3(uint32_t(T)), dim3(RS_THREADS), 0, st, src, n, shift, hist, T);
  hipLaunchKernelGGL(k_rs_rowscan, dim3(1u << BITS), dim3(SCAN_THREADS), 0, st, hist, T, total);
  hipLaunchKernelGGL(k_rs_scatter<BITS>, dim3(uint32_t(T)), dim3(RS_THREADS), 0, st, src, n, shift,
                     hist, total, T, keys_out, vals_out);
}

// Number of sorted keys below u, for u = u_first + i, i in [0, count): the
// row offsets of the sorted positions (keys outside the row range carry the
// key num_rows), and the segment of each edge (the offsets at or below it,
// less one).  No atomics: a hub row's count costs nothing extra.
// A workgroup takes OO_ROWS consecutive rows: two of its waves find where its
// rows' keys begin and end, 64 probes at a time, and every row is then searched
// for in that range alone -- in LDS when it is short, as it is but for hub
// rows.  (A search over all n keys per row is bound by its probes: 22 us for
// 1.25 M rows, 12 this way; 0.41 M rows with a hub 9.6 and 11.5.)
constexpr int OO_THREADS = 256;
constexpr int OO_PER = 2;
constexpr int OO_ROWS = OO_PER * OO_THREADS;
constexpr int OO_KEYS = 4096;

// First position in [0, n) whose key is not below u, n if there is none;
// every lane of the wave takes part and returns it.
__device__ __forceinline__ int64_t wave_lower_bound(const int32_t* __restrict__ keys, int64_t n,
                                                    int64_t u) {
  const int lane = threadIdx.x & 63;
  int64_t lo = 0, hi = n;                      // keys before lo are below u, keys from hi on are not
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) >> 6;  // probes lo + step - 1, lo + 2 step - 1, ...
    const int64_t p = lo + int64_t(lane + 1) * step - 1;
    const bool below = p < hi && int64_t(keys[p]) < u;
    const int c = __popcll(__ballot(below));   // the probes below u come first
    const int64_t cap = lo + int64_t(c + 1) * step - 1;
    lo += int64_t(c) * step;
    hi = cap < hi ? cap : hi;
  }
  return lo;
}

struct OutBound {
  int32_t* __restrict__ out;
  // m results from i0 on, in LDS
  __device__ void operator()(const int32_t* below, int64_t i0, int m) const {
    for (int j = threadIdx.x; j < m; j += OO_THREADS) out[i0 + j] = below[j];
  }
};
// rec[e] = (segment of edge e, its H coefficients), 1 + H words: a sum reads
// the two together, from one line mostly, not from two arrays (bf16 4 x 32
// sums of 1.32 M edges into 0.74 M / 1.25 M rows: 168 -> 138 / 203 -> 183 us,
// for 13 us more here).
struct OutEdgeRec {
  const float* __restrict__ scal;
  int32_t* __restrict__ rec;
  int H;
  int32_t last;
  __device__ void operator()(const int32_t* below, int64_t i0, int m) const {
    const int w = 1 + H, de = OO_THREADS / w, dk = OO_THREADS - de * w;
    int e = int(threadIdx.x) / w, k = int(threadIdx.x) - e * w;
    int32_t* __restrict__ r = rec + i0 * w;
    for (int j = threadIdx.x; j < m * w; j += OO_THREADS) {
      if (k) {
        r[j] = __float_as_int(scal[(i0 + e) * H + k - 1]);
      } else {                                       // in range whatever the offsets hold
        const int32_t v = below[e] - 1;
        r[j] = v < 0 ? 0 : (v > last ? last : v);
      }
      e += de;
      k += dk;
      if (k >= w) {
        k -= w;
        ++e;
      }
    }
  }
};

template <class Out>
__global__ void __launch_bounds__(OO_THREADS) k_lower_bounds(const int32_t* __restrict__ keys,
                                                            int64_t n, int64_t u_first,
                                                            int64_t count, Out out) {
  __shared__ int64_t s_range[2];
  __shared__ int32_t s_key[OO_KEYS], s_below[OO_ROWS];
  const int64_t i0 = int64_t(blockIdx.x) * OO_ROWS, u0 = u_first + i0;
  const int w = threadIdx.x >> 6;
  if (w < 2) {
    const int64_t p = wave_lower_bound(keys, n, u0 + w * OO_ROWS);
    if ((threadIdx.x & 63) == 0) s_range[w] = p;
  }
  __syncthreads();
  const int64_t a = s_range[0], b = s_range[1];
  const bool small = b - a <= OO_KEYS;
  if (small) {
    for (int j = threadIdx.x; j < int(b - a); j += OO_THREADS) s_key[j] = keys[a + j];
    __syncthreads();
  }
  // a thread's searches advance together: their probes are independent
  int64_t lo[OO_PER], hi[OO_PER];
#pragma unroll
  for (int r = 0; r < OO_PER; ++r) {
    lo[r] = 0;
    hi[r] = b - a;
  }
  for (int64_t len = b - a; len > 0; len >>= 1) {
#pragma unroll
    for (int r = 0; r < OO_PER; ++r) {
      const int64_t u = u0 + r * OO_THREADS + threadIdx.x;
      const int64_t mid = (lo[r] + hi[r]) >> 1;
      if (lo[r] < hi[r]) {
        const int32_t k = small ? s_key[mid] : keys[a + mid];
        if (int64_t(k) < u) lo[r] = mid + 1; else hi[r] = mid;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < OO_PER; ++r) s_below[r * OO_THREADS + threadIdx.x] = int32_t(a + lo[r]);
  __syncthreads();
  out(s_below, i0, int(count - i0 < OO_ROWS ? count - i0 : OO_ROWS));
}

template <class Out>
static void launch_lower_bounds(const int32_t* keys, int64_t n, int64_t u_first, int64_t count,
                                const Out& out, hipStream_t st) {
  hipLaunchKernelGGL(k_lower_bounds<Out>, dim3(uint32_t((count + OO_ROWS - 1) / OO_ROWS)),
                     dim3(OO_THREADS), 0, st, keys, n, u_first, count, out);
}

__global__ void __launch_bounds__(RS_THREADS) k_ir_fill(int32_t* p, int64_t n, int32_t v) {
  for (int64_t i = int64_t(blockIdx.x) * RS_THREADS + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * RS_THREADS)
    p[i] = v;
}

struct OccWs {
  int32_t* keys[2];
  int32_t* vals[2];
  uint32_t* hist;
  uint32_t* total;
};

static size_t occ_layout(int64_t n, int64_t num_rows, char* base, OccWs* ws) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align_up(bytes, 256);
    return base ? base + o : nullptr;
  };
  const int64_t T = rs_tiles(n);
  char* k0 = take(size_t(n) * 4);
  char* k1 = take(size_t(n) * 4);
  char* v0 = take(size_t(n) * 4);
  char* v1 = take(size_t(n) * 4);
  char* h = take(size_t(T) * RS_DIGITS * 4);
  char* tt = take(size_t(RS_DIGITS) * 4);
  if (ws) {
    ws->keys[0] = reinterpret_cast<int32_t*>(k0);
    ws->keys[1] = reinterpret_cast<int32_t*>(k1);
    ws->vals[0] = reinterpret_cast<int32_t*>(v0);
    ws->vals[1] = reinterpret_cast<int32_t*>(v1);
    ws->hist = reinterpret_cast<uint32_t*>(h);
    ws->total = reinterpret_cast<uint32_t*>(tt);
  }
  return off;
}

static uint32_t grid_cap(int64_t n, int64_t per, uint32_t cap = 8192) {
  int64_t g = (n + per - 1) / per;
  if (g < 1) g = 1;
  return uint32_t(g < cap ? g : cap);
}

// ------------------------------------------------------------------ index add
constexpr int IA_THREADS = 256;
constexpr int IA_PIECE = 64;   // occurrences summed by one group
constexpr int IA_ROWS = 4;   // rows per group of lanes on large outputs
constexpr int64_t IA_GROUPS_FILL = 16384;   // groups that fill the chip twice at 64 lanes, half of it at 16
constexpr int IA_PART_UNROLL = 4;   // partial sums in flight per lane of a long row

constexpr int IA_GROUP_MIN = 16;   // fewest pieces per group of the second level

// The smallest power of two p >= lo with p^3 >= c (c < 2^31: p <= 2048).
__device__ __forceinline__ int64_t ia_cbrt_pow2(int64_t c, int64_t lo) {
  int64_t p = lo;
  while (p * p * p < c) p <<= 1;
  return p;
}
// Tree of a row with c > IA_PIECE occurrences: pieces of ia_piece_len(c)
// occurrences and, when there are more than ia_group_len(c) pieces, groups of
// that many consecutive pieces.  For c = 3e5 (a hub of the 1e7-node batch):
// 2344 pieces of 128, 19 groups of 128 pieces.  Functions of c alone.
__device__ __forceinline__ int64_t ia_piece_len(int64_t c) { return ia_cbrt_pow2(c, IA_PIECE); }
__device__ __forceinline__ int64_t ia_group_len(int64_t c) { return ia_cbrt_pow2(c, IA_GROUP_MIN); }

// Pieces of a row (0 for c <= IA_PIECE, which one group sums directly); at
// most 2 c / IA_PIECE.
__device__ __forceinline__ int64_t ia_multi_pieces(int64_t c) {
  if (c <= IA_PIECE) return 0;
  const int64_t p = ia_piece_len(c);
  return (c + p - 1) / p;
}
// Groups of the second level (0 when the row has at most ia_group_len(c)
// pieces); at most 2 pieces / IA_GROUP_MIN.
__device__ __forceinline__ int64_t ia_multi_groups(int64_t c) {
  const int64_t m = ia_multi_pieces(c), g = ia_group_len(c);
  return m > g ? (m + g - 1) / g : 0;
}

// Both counts of row u in one 64-bit item (pieces high, groups low) for one
// scan; item num_rows is 0, so the prefix at num_rows is the pair of totals.
struct InMulti {
  const int32_t* occ_off;
  int64_t n, num_rows;
  __device__ uint64_t operator()(int64_t u) const {
    if (u >= num_rows) return 0u;
    const int64_t c = clamp64(int64_t(occ_off[u + 1]) - occ_off[u], 0, n);
    return (uint64_t(ia_multi_pieces(c)) << 32) | uint64_t(ia_multi_groups(c));
  }
};
struct OutMulti {
  int32_t* multi_off;
  int32_t* group_off;
  __device__ void operator()(int64_t u, uint64_t prefix, uint64_t) const {
    multi_off[u] = int32_t(prefix >> 32);
    group_off[u] = int32_t(prefix & 0xffffffffu);
  }
};

// acc += fp64 rows part[m0 .. m1) (chunk c of VE values, rows of D), in
// order, U rows loaded before they are added.
template <int VE, int U>
__device__ __forceinline__ void ia_sum_partials(const double* __restrict__ part, int64_t m0,
                                                int64_t m1, int D, int c, double (&acc)[VE]) {
  int64_t m = m0;
  for (; m + U <= m1; m += U) {
    double x[U][VE];
#pragma unroll
    for (int r = 0; r < U; ++r)
#pragma unroll
      for (int t = 0; t < VE; ++t) x[r][t] = part[(m + r) * D + c * VE + t];
#pragma unroll
    for (int r = 0; r < U; ++r)
#pragma unroll
      for (int t = 0; t < VE; ++t) acc[t] += x[r][t];
  }
  for (; m < m1; ++m)
#pragma unroll
    for (int t = 0; t < VE; ++t) acc[t] += part[m * D + c * VE + t];
}

// Row sources of the index-add kernels.  Position p = occ[j] contributes, to
// chunk c (VE values) of its row's sum:
//   PlainRows:  src row p;
//   ScaledRows: coefficient scal[p, head] times src row seg[p] -- the
//               coefficient of edge p and the destination segment it belongs
//               to, one head coefficient per element (a chunk spans at most
//               two heads, since VE <= dh).
// Products are formed in fp64 (exact for fp32 factors), sums in fp64.
template <typename T, int VE>
struct PlainRows {
  // rows in flight per lane in the pieces of long rows, whose sums are
  // chains of up to a thousand occurrences
  static constexpr int PIECE_UNROLL = 16, ROW_UNROLL = 8;
  const T* __restrict__ src;
  int D;
  int64_t n;
  struct Pos {
    int32_t p;
  };
  struct Item {
    Raw<T, VE> r;
  };
  __device__ void chunk(int) {}
  __device__ Pos pos(int32_t p) const { return Pos{int32_t(clamp64(p, 0, n - 1))}; }
  __device__ static Pos from_lane(const Pos& k, int r, int lanes) { return Pos{__shfl(k.p, r, lanes)}; }
  template <bool SPACED>
  __device__ Item fetch(const Pos& k, int c) const {
    // each source row is read once per call: streaming (non-temporal)
    // loads, as for the output rows below (1e7-node batch, K / V indices 0.41 /
    // 0.43 -> 0.39 / 0.41 ms; the large batch's V index 1.30 -> 1.21 ms)
    Item it;
    it.r.template load<true>(src + int64_t(k.p) * D + c * VE);
    return it;
  }
  __device__ void add(double (&acc)[VE], const Item& it) const {
    float x[VE];
    it.r.unpack(x);
#pragma unroll
    for (int t = 0; t < VE; ++t) acc[t] += double(x[t]);
  }
};

template <typename T, int VE>
struct ScaledRows {
  static constexpr int PIECE_UNROLL = 8, ROW_UNROLL = 4;
  const T* __restrict__ src;          // [N, H, dh]
  const int32_t* __restrict__ rec;    // [n, 1 + H]: segment, coefficients
  int D, H, dh;
  int64_t n, N;
  int h0, h1, split;                  // heads of the chunk; elements t < split use h0
  struct Pos {
    int32_t p, v;
  };
  struct Item {
    Raw<T, VE> r;
    float s0, s1;
  };
  __device__ void chunk(int c) {
    const int c0 = c * VE;
    h0 = c0 / dh;
    h1 = (c0 + VE - 1) / dh;
    split = (h0 + 1) * dh - c0;
  }
  __device__ Pos pos(int32_t p) const {
    const int32_t e = int32_t(clamp64(p, 0, n - 1));
    return Pos{e, rec[int64_t(e) * (1 + H)]};
  }
  __device__ static Pos from_lane(const Pos& k, int r, int lanes) {
    return Pos{__shfl(k.p, r, lanes), __shfl(k.v, r, lanes)};
  }
  template <bool SPACED>
  __device__ Item fetch(const Pos& k, int c) const {
    Item it;
    it.r.template load<false>(src + int64_t(k.v) * D + c * VE);
    const int32_t* __restrict__ s = rec + int64_t(k.p) * (1 + H) + 1;
    it.s0 = __int_as_float(s[h0]);
    // The branch waits for s0 before the next row is asked for.  A stream of
    // short rows is faster so (1.32 M edges into 1.25 M rows, bf16 4 x 32: 227 us,
    // 257 without), long rows slower (6000 positions in 100 rows 49 us, 36
    // without): they load s1 also where it is s0.
    it.s1 = !SPACED || dh % VE ? __int_as_float(s[h1]) : it.s0;
    return it;
  }
  __device__ void add(double (&acc)[VE], const Item& it) const {
    float x[VE];
    it.r.unpack(x);
#pragma unroll
    for (int t = 0; t < VE; ++t) acc[t] = fma(double(t < split ? it.s0 : it.s1), double(x[t]), acc[t]);
  }
};

// acc += the contributions of positions occ[j0 .. j1) in order, chunk c of
// the group's lane l (on: the lane holds a chunk); every lane of the group
// calls it.  The group's lanes look up a position each -- one load, whatever
// its count -- and then pass them round, so that the rows of U positions are
// in flight together, also where a row has fewer than U of them.  In groups
// of fewer than 16 lanes every lane looks up all: as many positions as lanes
// are too few in flight for a hub's pieces, and a mask per position in the
// loop breaks up the loads (2.64 M positions x 1 in 65,536 rows 202 -> 133 us,
// 600 x 20 bf16 in 100 rows 30 -> 25).  WIDE: groups of 16 lanes and more only.
template <int VE, class Src, int U, bool WIDE = false>
__device__ __forceinline__ void ia_sum(const int32_t* __restrict__ occ, int64_t j0, int64_t j1, int c,
                                       bool on, int l, int lanes, const Src& src, double (&acc)[VE]) {
  if (!WIDE && lanes < 16) {
    constexpr int S = U < 16 ? 4 : U;           // more in flight cost the short rows their occupancy
    typename Src::Item x[S];
    int64_t j = j0;
    for (; j + S <= j1; j += S) {
#pragma unroll
      for (int r = 0; r < S; ++r) x[r] = src.template fetch<false>(src.pos(occ[j + r]), c);
#pragma unroll
      for (int r = 0; r < S; ++r) src.add(acc, x[r]);
    }
    for (; j < j1; j += 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (j + r < j1) x[r] = src.template fetch<false>(src.pos(occ[j + r]), c);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (j + r < j1) src.add(acc, x[r]);
    }
    return;
  }
  for (int64_t jb = j0; jb < j1; jb += lanes) {
    const int m = int(j1 - jb < lanes ? j1 - jb : lanes);
    const typename Src::Pos mine = src.pos(occ[jb + (l < m ? l : m - 1)]);
    for (int r0 = 0; r0 < m; r0 += U) {
      typename Src::Item x[U];
      if (r0 + U <= m) {
#pragma unroll
        for (int r = 0; r < U; ++r) x[r] = src.template fetch<false>(Src::from_lane(mine, r0 + r, lanes), c);
#pragma unroll
        for (int r = 0; r < U; ++r) src.add(acc, x[r]);
      } else {
#pragma unroll
        for (int r = 0; r < U; ++r) {
          const typename Src::Pos k = Src::from_lane(mine, (r0 + r) & (lanes - 1), lanes);
          if (on && r0 + r < m) x[r] = src.template fetch<false>(k, c);
        }
#pragma unroll
        for (int r = 0; r < U; ++r)
          if (r0 + r < m) src.add(acc, x[r]);
      }
    }
  }
}

// Pieces of the long rows: one group of `lanes` lanes per piece q in
// [0, multi_off[num_rows]); its sum goes to partial[q].
template <int VE, class Src>
__global__ void __launch_bounds__(IA_THREADS) k_ia_pieces(
    const int32_t* __restrict__ occ_off, const int32_t* __restrict__ occ,
    const int32_t* __restrict__ multi_off, int64_t num_rows, int64_t multi_bound, int64_t n,
    int lanes, int D, Src src, double* __restrict__ partial) {
  const int64_t q = (int64_t(blockIdx.x) * IA_THREADS + threadIdx.x) / lanes;
  const int l = int(threadIdx.x) % lanes;
  if (q >= multi_bound || q >= multi_off[num_rows]) return;
  // the long row u with multi_off[u] <= q < multi_off[u + 1]
  int64_t lo = 0, hi = num_rows - 1;
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) >> 1;
    if (multi_off[mid] <= q) lo = mid; else hi = mid - 1;
  }
  const int64_t u = lo, k = q - multi_off[u];
  // offsets and positions are clamped into range, so malformed occurrence
  // lists give wrong sums but never an out-of-bounds access
  const int64_t r0 = clamp64(occ_off[u], 0, n);
  const int64_t r1 = clamp64(occ_off[u + 1], r0, n);
  const int64_t len = ia_piece_len(r1 - r0);
  const int64_t j0 = clamp64(r0 + k * len, r0, r1);
  const int64_t j1 = j0 + len < r1 ? j0 + len : r1;
  const int chunks = D / VE;
  for (int c0 = 0; c0 < chunks; c0 += lanes) {
    const int c = c0 + l;
    const bool on = c < chunks;
    src.chunk(on ? c : 0);
    double acc[VE];
#pragma unroll
    for (int t = 0; t < VE; ++t) acc[t] = 0.0;
    ia_sum<VE, Src, Src::PIECE_UNROLL>(occ, j0, j1, on ? c : 0, on, l, lanes, src, acc);
#pragma unroll
    for (int t = 0; t < VE; ++t)
      if (on) partial[q * D + c * VE + t] = acc[t];
  }
}

// Second level of the long rows: one group of `lanes` lanes per group g in
// [0, group_off[num_rows]) of ia_group_len(c) consecutive piece sums, added
// in piece order into partial2[g].
template <int VE>
__global__ void __launch_bounds__(IA_THREADS) k_ia_groups(
    const int32_t* __restrict__ occ_off, const int32_t* __restrict__ multi_off,
    const int32_t* __restrict__ group_off, int64_t num_rows, int64_t multi_bound,
    int64_t group_bound, int64_t n, int lanes, int D, const double* __restrict__ partial,
    double* __restrict__ partial2) {
  const int64_t g = (int64_t(blockIdx.x) * IA_THREADS + threadIdx.x) / lanes;
  const int l = int(threadIdx.x) % lanes;
  if (g >= group_bound || g >= group_off[num_rows]) return;
  // the long row u with group_off[u] <= g < group_off[u + 1]
  int64_t lo = 0, hi = num_rows - 1;
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) >> 1;
    if (group_off[mid] <= g) lo = mid; else hi = mid - 1;
  }
  const int64_t u = lo, k = g - group_off[u];
  const int64_t r0 = clamp64(occ_off[u], 0, n);
  const int64_t r1 = clamp64(occ_off[u + 1], r0, n);
  const int64_t len = ia_group_len(r1 - r0);
  const int64_t p0 = clamp64(multi_off[u], 0, multi_bound);
  const int64_t p1 = clamp64(multi_off[u + 1], p0, multi_bound);
  const int64_t m0 = clamp64(p0 + k * len, p0, p1);
  const int64_t m1 = m0 + len < p1 ? m0 + len : p1;
  const int chunks = D / VE;
  for (int c = l; c < chunks; c += lanes) {
    double acc[VE];
#pragma unroll
    for (int t = 0; t < VE; ++t) acc[t] = 0.0;
    ia_sum_partials<VE, 8>(partial, m0, m1, D, c, acc);
#pragma unroll
    for (int t = 0; t < VE; ++t) partial2[g * D + c * VE + t] = acc[t];
  }
}

// Rounds a row's sum once and stores its chunk.  Output rows are written
// once: streamed (scaled sums of the large batch's V index 1.61 -> 1.46 ms
// with both policies).
template <int VE>
__device__ __forceinline__ void ia_store(float* __restrict__ dst, const double (&acc)[VE]) {
  float o[VE];
#pragma unroll
  for (int t = 0; t < VE; ++t) o[t] = float(acc[t]);
  if constexpr (VE == 8) {
    StreamIO<float, 4, true>::store(dst, o);
    StreamIO<float, 4, true>::store(dst + 4, o + 4);
  } else {
    StreamIO<float, VE, true>::store(dst, o);
  }
}

// Chunk c of a long row, added from the level below: its groups, or its
// pieces (ranges clamped: the counts of malformed lists may wrap).
template <int VE>
__device__ __forceinline__ void ia_long_row(
    const int32_t* __restrict__ multi_off, const int32_t* __restrict__ group_off, int64_t u,
    int64_t multi_bound, int64_t group_bound, int c, int D, const double* __restrict__ partial,
    const double* __restrict__ partial2, float* __restrict__ dst) {
  int64_t p0 = clamp64(group_off[u], 0, group_bound);
  int64_t p1 = clamp64(group_off[u + 1], p0, group_bound);
  const double* __restrict__ part = partial2;
  if (p1 == p0) {
    p0 = clamp64(multi_off[u], 0, multi_bound);
    p1 = clamp64(multi_off[u + 1], p0, multi_bound);
    part = partial;
  }
  double acc[VE];
#pragma unroll
  for (int t = 0; t < VE; ++t) acc[t] = 0.0;
  ia_sum_partials<VE, IA_PART_UNROLL>(part, p0, p1, D, c, acc);
  ia_store<VE>(dst + u * D + c * VE, acc);
}

// R consecutive rows by one group of lanes: zeros for a row without
// occurrences, a long row added from the level below.  The rows' occurrences
// lie side by side in occ, so with R > 1 the group walks them as one stream:
// the lanes look up as many positions at once as there are lanes, ROW_UNROLL
// source rows are in flight whichever output rows they belong to, and a row's
// sum is stored where its last position has been added.  A row of one or two positions by itself waits
// for offset, position, segment and row one after the other: with 1 / 2 / 4 /
// 8 rows per group the fp32 sums of 0.44 M and 0.58 M rows (half of 2.64 M
// positions in hub rows) took 174 / 141 / 125 / 131 and 218 / 169 / 146 / 151
// us.  A group that meets a long row goes row by row.
template <int VE, class Src, int R>
__global__ void __launch_bounds__(IA_THREADS) k_ia_rows(
    const int32_t* __restrict__ occ_off, const int32_t* __restrict__ occ,
    const int32_t* __restrict__ multi_off, const int32_t* __restrict__ group_off,
    int64_t num_rows, int64_t multi_bound, int64_t group_bound, int64_t n, int lanes, int D,
    Src src, const double* __restrict__ partial, const double* __restrict__ partial2,
    float* __restrict__ dst) {
  const int64_t u0 = (int64_t(blockIdx.x) * IA_THREADS + threadIdx.x) / lanes * R;
  const int l = int(threadIdx.x) % lanes;
  if (u0 >= num_rows) return;
  const int nr = int(num_rows - u0 < R ? num_rows - u0 : R);
  const int chunks = D / VE;
  bool stream = false;
  int64_t lo = 0, hi = 0;                       // lane l < nr: the bounds of row l
  if constexpr (R > 1) {                        // then lanes > R
    lo = clamp64(occ_off[u0 + (l < nr ? l : nr)], 0, n);
    hi = clamp64(occ_off[u0 + (l + 1 < nr ? l + 1 : nr)], 0, n);
    // every row short and in order: any other sends the group row by row
    bool bad = hi < lo || hi - lo > IA_PIECE;
    for (int o = 1; o < lanes; o <<= 1) bad |= __shfl_xor(int(bad), o, lanes) != 0;
    stream = !bad;
  }
  if (!stream) {
    for (int64_t u = u0; u < u0 + nr; ++u) {
      const int64_t j0 = clamp64(occ_off[u], 0, n);
      const int64_t j1 = clamp64(occ_off[u + 1], j0, n);
      const bool longrow = j1 - j0 > IA_PIECE;
      for (int c0 = 0; c0 < chunks; c0 += lanes) {
        const int c = c0 + l;
        const bool on = c < chunks;
        if (longrow) {
          if (on)
            ia_long_row<VE>(multi_off, group_off, u, multi_bound, group_bound, c, D, partial, partial2,
                            dst);
          continue;
        }
        src.chunk(on ? c : 0);
        double acc[VE];
#pragma unroll
        for (int t = 0; t < VE; ++t) acc[t] = 0.0;
        ia_sum<VE, Src, Src::ROW_UNROLL, (R > 1)>(occ, j0, j1, on ? c : 0, on, l, lanes, src, acc);
        if (on) ia_store<VE>(dst + u * D + c * VE, acc);
      }
    }
    return;
  }
  const int64_t j0 = __shfl(lo, 0, lanes);
  const int ends = int(hi - j0);                            // lane r: end of row r, from the first position
  const int total = __shfl(ends, nr - 1, lanes);            // at most R * IA_PIECE
  if constexpr (VE >= 4) {
    if (total == 0) {   // rows without occurrences: one run of zeros (3e6 such rows x 128: 715 -> 300 us)
      const float zero[4] = {0.f, 0.f, 0.f, 0.f};
      for (int k = l; k < nr * D / 4; k += lanes) StreamIO<float, 4, true>::store(dst + u0 * D + 4 * k, zero);
      return;
    }
  }
  for (int c0 = 0; c0 < chunks; c0 += lanes) {
    const int c = c0 + l;
    const bool on = c < chunks;
    src.chunk(on ? c : 0);
    double acc[VE];
#pragma unroll
    for (int t = 0; t < VE; ++t) acc[t] = 0.0;
    int row = 0, end = __shfl(ends, 0, lanes);
    float* out = dst + u0 * D + c * VE;
    for (int b = 0; b < total; b += lanes) {
      const int m = total - b < lanes ? total - b : lanes;
      const typename Src::Pos mine = src.pos(occ[j0 + b + (l < m ? l : m - 1)]);
      for (int r0 = 0; r0 < m; r0 += Src::ROW_UNROLL) {
        typename Src::Item x[Src::ROW_UNROLL];
#pragma unroll
        for (int r = 0; r < Src::ROW_UNROLL; ++r) {
          const typename Src::Pos k = Src::from_lane(mine, (r0 + r) & (lanes - 1), lanes);
          if (on && r0 + r < m) x[r] = src.template fetch<true>(k, c);
        }
#pragma unroll
        for (int r = 0; r < Src::ROW_UNROLL; ++r) {
          if (r0 + r < m) {
            while (b + r0 + r == end) {                     // the rows that end before this position
              if (on) ia_store<VE>(out, acc);
#pragma unroll
              for (int t = 0; t < VE; ++t) acc[t] = 0.0;
              out += D;
              end = __shfl(ends, ++row, lanes);
            }
            src.add(acc, x[r]);
          }
        }
      }
    }
    for (; row < nr; ++row) {
      if (on) ia_store<VE>(out, acc);
#pragma unroll
      for (int t = 0; t < VE; ++t) acc[t] = 0.0;
      out += D;
    }
  }
}

struct IaWs {
  int32_t* multi_off;
  int32_t* group_off;
  void* scan;
  double* partial;
  double* partial2;
};

static int64_t ia_multi_bound(int64_t n) { return (2 * n) / IA_PIECE + 1; }
// pieces of rows with groups, over IA_GROUP_MIN / 2
static int64_t ia_group_bound(int64_t n) { return ia_multi_bound(n) * 2 / IA_GROUP_MIN + 1; }

static size_t ia_layout(int64_t n, int64_t num_rows, int D, char* base, IaWs* ws) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align_up(bytes, 256);
    return base ? base + o : nullptr;
  };
  char* mo = take(size_t(num_rows + 1) * 4);
  char* go = take(size_t(num_rows + 1) * 4);
  char* sc = take(scan_workspace<uint64_t>(num_rows + 1));
  char* pa = take(size_t(ia_multi_bound(n)) * size_t(D) * 8);
  char* pb = take(size_t(ia_group_bound(n)) * size_t(D) * 8);
  if (ws) {
    ws->multi_off = reinterpret_cast<int32_t*>(mo);
    ws->group_off = reinterpret_cast<int32_t*>(go);
    ws->scan = sc;
    ws->partial = reinterpret_cast<double*>(pa);
    ws->partial2 = reinterpret_cast<double*>(pb);
  }
  return off;
}

static int pow2_at_least(int x, int cap) {
  int p = 1;
  while (p < x && p < cap) p <<= 1;
  return p;
}

}  // namespace fast

using namespace fast;

extern "C" size_t fast_occurrence_csr_workspace(int64_t n, int64_t num_rows) {
  if (n < 0 || num_rows < 0 || n >= (int64_t(1) << 31) || num_rows >= (int64_t(1) << 31) - 1)
    return 0;
  return occ_layout(n, num_rows, nullptr, nullptr);
}

extern "C" fast_status_t fast_occurrence_csr(const int32_t* index, int64_t n, int64_t num_rows,
                                             int32_t* occ_off, int32_t* occ, void* ws,
                                             size_t ws_bytes, fast_stream_t stream) {
  const char* fn = "fast_occurrence_csr";
  if (n < 0 || num_rows < 0) return fail(FAST_ERR_INVALID_ARG, "%s: negative size", fn);
  if (n >= (int64_t(1) << 31) || num_rows >= (int64_t(1) << 31) - 1)
    return fail(FAST_ERR_UNSUPPORTED, "%s: n or num_rows beyond 2^31", fn);
  if (!occ_off) return fail(FAST_ERR_INVALID_ARG, "%s: occ_off is NULL", fn);
  if (n > 0 && (!index || !occ)) return fail(FAST_ERR_INVALID_ARG, "%s: index/occ is NULL", fn);
  const size_t need = fast_occurrence_csr_workspace(n, num_rows);
  if (!ws || ws_bytes < need)
    return fail(FAST_ERR_WORKSPACE, "%s: workspace of %zu bytes < %zu", fn, ws_bytes, need);
  if (!aligned(ws, 256)) return fail(FAST_ERR_UNSUPPORTED, "%s: workspace not 256-byte aligned", fn);
  hipStream_t st = static_cast<hipStream_t>(stream);
  OccWs w;
  occ_layout(n, num_rows, static_cast<char*>(ws), &w);
  if (n == 0) {
    hipLaunchKernelGGL(k_ir_fill, dim3(grid_cap(num_rows + 1, RS_THREADS * 4)), dim3(RS_THREADS), 0,
                       st, occ_off, num_rows + 1, 0);
    return check_launch(fn);
  }
  // positions sorted stably by key (keys <= num_rows), the key's bits split
  // evenly over the passes
  int bits = 1;
  while ((int64_t(1) << bits) <= num_rows) ++bits;
  const int passes = (bits + RS_MAX_BITS - 1) / RS_MAX_BITS;
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    const RsSrc src{p == 0 ? index : nullptr, w.keys[(p + 1) & 1], w.vals[(p + 1) & 1], int32_t(num_rows)};
    int32_t* kout = w.keys[p & 1];
    int32_t* vout = p == passes - 1 ? occ : w.vals[p & 1];
    const int width = (bits - shift + passes - p - 1) / (passes - p);
    switch (width) {
      case 8: rs_pass<8>(src, n, shift, w.hist, w.total, kout, vout, st); break;
      case 7: rs_pass<7>(src, n, shift, w.hist, w.total, kout, vout, st); break;
      case 6: rs_pass<6>(src, n, shift, w.hist, w.total, kout, vout, st); break;
      case 5: rs_pass<5>(src, n, shift, w.hist, w.total, kout, vout, st); break;
      default: rs_pass<4>(src, n, shift, w.hist, w.total, kout, vout, st); break;   // keys of 1-4 bits
    }
    shift += width;
  }
  // row offsets from the sorted keys
  launch_lower_bounds(w.keys[(passes - 1) & 1], n, 0, num_rows + 1, OutBound{occ_off}, st);
  return check_launch(fn);
}

// Launches the row sums over occurrence lists for a row source: one scan of
// the (piece, group) counts, the long rows' pieces, their groups, then one
// group of lanes per row.
template <int VE, class Src>
static hipError_t ia_launch(const int32_t* occ_off, const int32_t* occ, int64_t n,
                            int64_t num_rows, int D, const Src& src, const IaWs& w, float* dst,
                            hipStream_t st) {
  hipError_t e = scan_launch<InMulti, OutMulti, uint64_t>(
      InMulti{occ_off, n, num_rows}, OutMulti{w.multi_off, w.group_off}, num_rows + 1, w.scan,
      nullptr, nullptr, st);
  if (e != hipSuccess) return e;
  const int lanes = pow2_at_least(D / VE, 64);
  const int64_t groups_per_block = IA_THREADS / lanes;
  const int64_t mb = ia_multi_bound(n), gb = ia_group_bound(n);
  const int64_t np_blocks = (mb + groups_per_block - 1) / groups_per_block;
  const int64_t ng_blocks = (gb + groups_per_block - 1) / groups_per_block;
  // IA_ROWS rows per group where that leaves the chip enough groups (below,
  // a group per row fills it better) and a group has a lane for each bound;
  // rows of 8 positions and more fill a group's loads by themselves (2.64 M
  // fp32 2 x 50 positions over 65,536 / 200,000 / 400,000 / 1e6 uniform rows, a
  // row / 4 rows per group: 260 / 282, 268 / 294, 314 / 309, 460 / 343 us)
  const bool many = lanes >= 4 * IA_ROWS && num_rows >= IA_ROWS * IA_GROUPS_FILL && n < 8 * num_rows;
  const int R = many ? IA_ROWS : 1;
  const int64_t nr_blocks = ((num_rows + R - 1) / R + groups_per_block - 1) / groups_per_block;
  if (n > IA_PIECE) {
    hipLaunchKernelGGL((k_ia_pieces<VE, Src>), dim3(uint32_t(np_blocks)), dim3(IA_THREADS), 0, st,
                       occ_off, occ, w.multi_off, num_rows, mb, n, lanes, D, src, w.partial);
    hipLaunchKernelGGL((k_ia_groups<VE>), dim3(uint32_t(ng_blocks)), dim3(IA_THREADS), 0, st,
                       occ_off, w.multi_off, w.group_off, num_rows, mb, gb, n, lanes, D, w.partial,
                       w.partial2);
  }
  if (many)
    hipLaunchKernelGGL((k_ia_rows<VE, Src, IA_ROWS>), dim3(uint32_t(nr_blocks)), dim3(IA_THREADS), 0,
                       st, occ_off, occ, w.multi_off, w.group_off, num_rows, mb, gb, n, lanes, D, src,
                       w.partial, w.partial2, dst);
  else
    hipLaunchKernelGGL((k_ia_rows<VE, Src, 1>), dim3(uint32_t(nr_blocks)), dim3(IA_THREADS), 0, st,
                       occ_off, occ, w.multi_off, w.group_off, num_rows, mb, gb, n, lanes, D, src,
                       w.partial, w.partial2, dst);
  return hipGetLastError();
}

// Widest vector (8 values for bf16 sources, else 4, 2 or 1) that divides D,
// is at most `cap` and fits the alignment of both row pointers.
static int ia_vector(int D, int cap, const void* src, int esz, const float* dst) {
  if (esz == 2 && 8 <= cap && D % 8 == 0 && aligned(src, 16) && aligned(dst, 16)) return 8;
  for (int v : {4, 2})
    if (v <= cap && D % v == 0 && aligned(src, size_t(v) * esz) && aligned(dst, size_t(v) * 4))
      return v;
  return 1;
}

static fast_status_t ia_common_checks(const char* fn, int64_t n, int64_t num_rows, int D,
                                      fast_dtype_t src_dtype) {
  if (n < 0 || num_rows < 0 || D < 1) return fail(FAST_ERR_INVALID_ARG, "%s: bad size", fn);
  if (n >= (int64_t(1) << 31) || num_rows >= (int64_t(1) << 31) - 1)
    return fail(FAST_ERR_UNSUPPORTED, "%s: n or num_rows beyond 2^31", fn);
  if (src_dtype != FAST_F32 && src_dtype != FAST_BF16) return fail(FAST_ERR_INVALID_ARG, "%s: bad dtype", fn);
  return FAST_OK;
}

extern "C" size_t fast_index_add_rows_workspace(int64_t n, int64_t num_rows, int D) {
  if (n < 0 || num_rows < 0 || D < 1 || n >= (int64_t(1) << 31) || num_rows >= (int64_t(1) << 31) - 1)
    return 0;
  return ia_layout(n, num_rows, D, nullptr, nullptr);
}

extern "C" fast_status_t fast_index_add_rows(const int32_t* occ_off, const int32_t* occ,
                                             int64_t n, int64_t num_rows, int D,
                                             fast_dtype_t src_dtype, const void* src, float* dst,
                                             void* ws, size_t ws_bytes, fast_stream_t stream) {
  const char* fn = "fast_index_add_rows";
  if (fast_status_t c = ia_common_checks(fn, n, num_rows, D, src_dtype)) return c;
  if (num_rows == 0) return ok();
  if (!occ_off || !dst) return fail(FAST_ERR_INVALID_ARG, "%s: occ_off/dst is NULL", fn);
  if (n > 0 && (!occ || !src)) return fail(FAST_ERR_INVALID_ARG, "%s: occ/src is NULL", fn);
  const size_t need = fast_index_add_rows_workspace(n, num_rows, D);
  if (!ws || ws_bytes < need)
    return fail(FAST_ERR_WORKSPACE, "%s: workspace of %zu bytes < %zu", fn, ws_bytes, need);
  if (!aligned(ws, 256)) return fail(FAST_ERR_UNSUPPORTED, "%s: workspace not 256-byte aligned", fn);
  const int esz = elem_size(src_dtype);
  if (!aligned(src, size_t(esz)) || !aligned(dst, 4))
    return fail(FAST_ERR_UNSUPPORTED, "%s: src/dst misaligned", fn);
  const int VE = ia_vector(D, 8, src, esz, dst);
  hipStream_t st = static_cast<hipStream_t>(stream);
  IaWs w;
  ia_layout(n, num_rows, D, static_cast<char*>(ws), &w);
  hipError_t e = hipSuccess;
#define FAST_IA(T_, VE_) \
  e = ia_launch<VE_>(occ_off, occ, n, num_rows, D, PlainRows<T_, VE_>{static_cast<const T_*>(src), D, n}, w, dst, st)
  if (src_dtype == FAST_F32) {
    if (VE == 4) FAST_IA(float, 4); else if (VE == 2) FAST_IA(float, 2); else FAST_IA(float, 1);
  } else {
    if (VE == 8) FAST_IA(uint16_t, 8); else if (VE == 4) FAST_IA(uint16_t, 4);
    else if (VE == 2) FAST_IA(uint16_t, 2); else FAST_IA(uint16_t, 1);
  }
#undef FAST_IA
  if (e != hipSuccess) return fail(FAST_ERR_HIP, "%s: %s", fn, hipGetErrorString(e));
  return check_launch(fn);
}

static size_t ias_layout(int64_t n, int64_t num_rows, int H, int D, char* base, int32_t** rec,
                         IaWs* ws) {
  const size_t head = align_up(size_t(n) * size_t(1 + H) * 4, 256);
  if (rec) *rec = reinterpret_cast<int32_t*>(base);
  return head + ia_layout(n, num_rows, D, base ? base + head : nullptr, ws);
}

extern "C" size_t fast_index_add_scaled_rows_workspace(int64_t n, int64_t num_rows, int H, int dh) {
  if (H < 1 || dh < 1 || int64_t(H) * dh >= (int64_t(1) << 31)) return 0;
  const int D = H * dh;
  if (n < 0 || num_rows < 0 || n >= (int64_t(1) << 31) || num_rows >= (int64_t(1) << 31) - 1)
    return 0;
  return ias_layout(n, num_rows, H, D, nullptr, nullptr, nullptr);
}

extern "C" fast_status_t fast_index_add_scaled_rows(
    const int32_t* occ_off, const int32_t* occ, int64_t n, int64_t num_rows,
    const int32_t* dst_offsets, int64_t num_dst, int H, int dh, fast_dtype_t src_dtype,
    const float* scal, const void* src, float* dst, void* ws, size_t ws_bytes,
    fast_stream_t stream) {
  const char* fn = "fast_index_add_scaled_rows";
  if (H < 1 || dh < 1 || int64_t(H) * dh >= (int64_t(1) << 31))
    return fail(FAST_ERR_INVALID_ARG, "%s: bad H = %d or dh = %d", fn, H, dh);
  const int D = H * dh;
  if (fast_status_t c = ia_common_checks(fn, n, num_rows, D, src_dtype)) return c;
  if (num_dst < 0) return fail(FAST_ERR_INVALID_ARG, "%s: negative num_dst", fn);
  if (num_dst >= (int64_t(1) << 31)) return fail(FAST_ERR_UNSUPPORTED, "%s: num_dst >= 2^31", fn);
  if (n > 0 && num_dst == 0) return fail(FAST_ERR_INVALID_ARG, "%s: edges but no destination", fn);
  if (num_rows == 0) return ok();
  if (!occ_off || !dst) return fail(FAST_ERR_INVALID_ARG, "%s: occ_off/dst is NULL", fn);
  if (n > 0 && (!occ || !src || !scal || !dst_offsets))
    return fail(FAST_ERR_INVALID_ARG, "%s: occ/dst_offsets/scal/src is NULL", fn);
  const size_t need = fast_index_add_scaled_rows_workspace(n, num_rows, H, dh);
  if (!ws || ws_bytes < need)
    return fail(FAST_ERR_WORKSPACE, "%s: workspace of %zu bytes < %zu", fn, ws_bytes, need);
  if (!aligned(ws, 256)) return fail(FAST_ERR_UNSUPPORTED, "%s: workspace not 256-byte aligned", fn);
  const int esz = elem_size(src_dtype);
  if (!aligned(src, size_t(esz)) || !aligned(dst, 4) || !aligned(scal, 4))
    return fail(FAST_ERR_UNSUPPORTED, "%s: src/dst/scal misaligned", fn);
  const int VE = ia_vector(D, dh, src, esz, dst);   // a chunk spans at most two heads
  hipStream_t st = static_cast<hipStream_t>(stream);
  int32_t* rec = nullptr;
  IaWs w;
  ias_layout(n, num_rows, H, D, static_cast<char*>(ws), &rec, &w);
  if (n > 0)
    launch_lower_bounds(dst_offsets, num_dst, 1, n, OutEdgeRec{scal, rec, H, int32_t(num_dst - 1)}, st);
  hipError_t e = hipSuccess;
#define FAST_IAS(T_, VE_)                                                                          \
  e = ia_launch<VE_>(occ_off, occ, n, num_rows, D,                                                 \
                     ScaledRows<T_, VE_>{static_cast<const T_*>(src), rec, D, H, dh, n,             \
                                         num_dst, 0, 0, 0},                                        \
                     w, dst, st)
  if (src_dtype == FAST_F32) {
    if (VE == 4) FAST_IAS(float, 4); else if (VE == 2) FAST_IAS(float, 2); else FAST_IAS(float, 1);
  } else {
    if (VE == 8) FAST_IAS(uint16_t, 8); else if (VE == 4) FAST_IAS(uint16_t, 4);
    else if (VE == 2) FAST_IAS(uint16_t, 2); else FAST_IAS(uint16_t, 1);
  }
#undef FAST_IAS
  if (e != hipSuccess) return fail(FAST_ERR_HIP, "%s: %s", fn, hipGetErrorString(e));
  return check_launch(fn);
}
