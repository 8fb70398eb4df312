// sample.hip -- most-recent-k temporal neighbour sampling (Sec. 6.1: the
// experiments sample the k = 10 most recent neighbours of each root) over a
// T-CSR temporal graph, producing the sampled block in the CSR-by-destination
// form every other operator takes.
//
// A root (node v, query time t) may use only events strictly earlier than t.
// v's entries are in time order, so those events are a prefix of its list;
// a search finds its end and the root keeps the last min(k, length) entries
// of it, in entry order.  Up to SR_TILED roots the calls are bound by
// latency, not by bytes, and take two launches:
//   * 16 or 4 lanes search for one root, that many probes at a time: a hub's
//     4e6 entries take 6 or 11 dependent loads instead of 22;
//   * a workgroup's roots are one scan tile: the search leaves the tile's sum,
//     and the fill adds up the sums of the tiles before its own, scans its
//     own counts, writes the offsets and copies its roots' neighbours, times
//     and edge ids (16 lanes per root; one root's entries are contiguous).
// 6,000 roots and then their 60,000 places, k = 10, 2e7 events, the same roots
// again and again: 40.6 us with a thread per search and a scan of its own (4
// launches a hop), 23.5 now; fresh roots in swept caches, hop 1 / hop 2, 24.8 /
// 30.2 and 12.9 / 22.2.  More roots are bound by the probes and copies
// themselves (24,000 roots and their 240,000 places: 16 / 4 / 1 lanes a search
// 73 / 59 / 56 us): they keep a thread per search and the scan of its own.
// The output is a function of the inputs alone.
#include "scan.h"

namespace fast {

constexpr int SR_THREADS = 256;
constexpr int SR_GROUP = 16;   // lanes copying one root's entries
// Tiles of 16 roots (256 threads of the fill) spread small batches over the
// chip, tiles of 64 (1024 threads) keep the tile sums few; each up to
// SR_MAX_TILES tiles, whose sums the fill's workgroups add up themselves.
constexpr int SR_SMALL = 16, SR_LARGE = 64;
constexpr int64_t SR_MAX_TILES = 2048;
constexpr int64_t SR_TILED = SR_MAX_TILES * SR_LARGE;
// 16 lanes per search while they are too few to be bound by their probes
// (6,000 roots: 5.0 us against 6.5 with 4 lanes; 60,000: 12.9 against 7.8; the
// call on fresh roots, 16 / 4 lanes: 600 of them 11.6 / 13.7 us, 6,000 12.9 / 14.8,
// 12,000 14.2 / 15.8, 18,000 15.6 / 16.7, 36,000 18.6 / 18.6).
constexpr int64_t SR_WIDE_SEARCH = 8192;

// First p in [a, b) with !(ts[p] < t), b if none; every lane of the group of
// L lanes calls it and returns it.  Stays in [a, b] whatever ts holds.
template <int L>
__device__ __forceinline__ int64_t group_lower_bound(const float* __restrict__ ts, int64_t a, int64_t b,
                                                     float t, int lane) {
  const int shift = int(threadIdx.x & 63) & ~(L - 1);
  while (a < b) {
    const int64_t len = b - a;
    const int64_t step = L == 1 ? (len >> 1) + 1 : (len + L - 1) / L;   // probes a + step - 1, a + 2 step - 1, ...
    const int64_t p = a + int64_t(lane + 1) * step - 1;
    const bool below = p < b && ts[p] < t;
    const int c = L == 1 ? int(below) : __popc(uint32_t(__ballot(below) >> shift) & ((1u << L) - 1u));
    const int64_t cap = a + int64_t(c + 1) * step - 1;
    a += int64_t(c) * step;
    b = cap < b ? cap : b;
  }
  return a;
}

// One tile of ROOTS roots, L lanes per root.
template <int ROOTS, int L>
__global__ void __launch_bounds__(ROOTS * L) k_sample_count(
    const int64_t* __restrict__ indptr, int64_t num_nodes, int64_t num_entries,
    const float* __restrict__ ts, const int64_t* __restrict__ roots,
    const float* __restrict__ root_t, int64_t R, int k, int32_t* __restrict__ count,
    int64_t* __restrict__ start, uint32_t* __restrict__ tsum) {
  __shared__ uint32_t s_c[ROOTS];
  const int sub = int(threadIdx.x) / L, lane = int(threadIdx.x) % L;
  const int64_t i = int64_t(blockIdx.x) * ROOTS + sub;
  int32_t c = 0;
  if (i < R) {
    const int64_t v = roots[i];
    int64_t s = 0;
    if (k > 0 && v >= 0 && v < num_nodes) {
      const int64_t lo = clamp64(indptr[v], 0, num_entries);
      const int64_t hi = clamp64(indptr[v + 1], lo, num_entries);
      const int64_t a = group_lower_bound<L>(ts, lo, hi, root_t[i], lane);
      c = int32_t(a - lo < k ? a - lo : k);
      s = a - c;
    }
    if (lane == 0) {
      count[i] = c;
      start[i] = s;
    }
  }
  if (!tsum) return;                         // uniform: no tile sums wanted
  static_assert(ROOTS <= 64 || L == 1, "a wave adds up the tile");
  if (lane == 0) s_c[sub] = uint32_t(c);
  __syncthreads();
  if (threadIdx.x < 64) {
    uint32_t x = int(threadIdx.x) < ROOTS ? s_c[threadIdx.x] : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    if (threadIdx.x == 0) tsum[blockIdx.x] = x;
  }
}

// Offsets and neighbours of one tile.  off[i] holds root i's count on entry:
// only the root's own tile reads it, and writes the offset in its place.
template <int ROOTS>
__global__ void __launch_bounds__(ROOTS * SR_GROUP) k_sample_fill(
    const int64_t* __restrict__ nbr, const float* __restrict__ ts,
    const int64_t* __restrict__ eid, const int64_t* __restrict__ start,
    const uint32_t* __restrict__ tsum, int64_t R, int32_t* __restrict__ off,
    int64_t* __restrict__ src_ids, float* __restrict__ edge_t, int64_t* __restrict__ edge_ids) {
  constexpr int THREADS = ROOTS * SR_GROUP;
  __shared__ uint32_t s_part[THREADS / 64], s_off[ROOTS];
  const int sub = int(threadIdx.x) / SR_GROUP, lane = int(threadIdx.x) % SR_GROUP;
  const int64_t r0 = int64_t(blockIdx.x) * ROOTS, i = r0 + sub;
  const int32_t c = i < R ? off[i] : 0;
  const int64_t s = i < R ? start[i] : 0;
  uint32_t before = 0;
  for (int j = threadIdx.x; j < int(blockIdx.x); j += THREADS) before += tsum[j];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = before;
  if (lane == 0) s_off[sub] = uint32_t(c);
  __syncthreads();
  if (threadIdx.x < 64) {
    uint32_t base = 0u;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) base += s_part[w];
    const uint32_t x = int(threadIdx.x) < ROOTS ? s_off[threadIdx.x] : 0u;
    uint32_t inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(inc, o, 64);
      if (int(threadIdx.x) >= o) inc += y;
    }
    const int64_t r = r0 + threadIdx.x;
    if (int(threadIdx.x) < ROOTS) s_off[threadIdx.x] = base + inc - x;
    if (int(threadIdx.x) < ROOTS && r < R) {
      off[r] = int32_t(base + inc - x);
      if (r == R - 1) off[R] = int32_t(base + inc);
    }
  }
  __syncthreads();
  if (i >= R) return;
  const int64_t o = s_off[sub];
  for (int j = lane; j < c; j += SR_GROUP) {
    src_ids[o + j] = nbr[s + j];
    edge_t[o + j] = ts[s + j];
    edge_ids[o + j] = eid[s + j];
  }
}

struct InRootCount {
  const int32_t* c;
  __device__ uint32_t operator()(int64_t i) const { return uint32_t(c[i]); }
};
struct OutRootOffset {
  int32_t* off;
  __device__ void operator()(int64_t i, uint32_t prefix, uint32_t) const { off[i] = int32_t(prefix); }
};

// Neighbours of every root, its offset known: groups of SR_GROUP lanes, one
// root each.
__global__ void __launch_bounds__(SR_THREADS) k_sample_copy(
    const int64_t* __restrict__ nbr, const float* __restrict__ ts,
    const int64_t* __restrict__ eid, const int32_t* __restrict__ count,
    const int64_t* __restrict__ start, const int32_t* __restrict__ off, int64_t R,
    int64_t* __restrict__ src_ids, float* __restrict__ edge_t, int64_t* __restrict__ edge_ids) {
  const int64_t i = (int64_t(blockIdx.x) * SR_THREADS + threadIdx.x) / SR_GROUP;
  const int lane = int(threadIdx.x) % SR_GROUP;
  if (i >= R) return;
  const int32_t c = count[i];
  const int64_t s = start[i], o = off[i];
  for (int j = lane; j < c; j += SR_GROUP) {
    src_ids[o + j] = nbr[s + j];
    edge_t[o + j] = ts[s + j];
    edge_ids[o + j] = eid[s + j];
  }
}

struct SrWs {
  int32_t* count;      // or the tile sums, where the counts lie in dst_offsets
  int64_t* start;
  void* scan;
};

static size_t sr_layout(int64_t R, char* base, SrWs* ws) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align_up(bytes, 256);
    return base ? base + o : nullptr;
  };
  char* c = take(size_t(R) * 4);
  char* s = take(size_t(R) * 8);
  char* sc = take(scan_workspace(R));
  if (ws) {
    ws->count = reinterpret_cast<int32_t*>(c);
    ws->start = reinterpret_cast<int64_t*>(s);
    ws->scan = sc;
  }
  return off;
}

}  // namespace fast

using namespace fast;

extern "C" size_t fast_sample_recent_workspace(int64_t num_roots) {
  if (num_roots < 0 || num_roots >= (int64_t(1) << 31)) return 0;
  return sr_layout(num_roots, nullptr, nullptr);
}

extern "C" fast_status_t fast_sample_recent(const fast_temporal_graph_t* g, const int64_t* roots,
                                            const float* root_t, int64_t num_roots, int k,
                                            int32_t* dst_offsets, int64_t* src_ids, float* edge_t,
                                            int64_t* edge_ids, void* ws, size_t ws_bytes,
                                            fast_stream_t stream) {
  const char* fn = "fast_sample_recent";
  if (!g) return fail(FAST_ERR_INVALID_ARG, "%s: graph is NULL", fn);
  if (g->num_nodes < 0 || g->num_entries < 0 || num_roots < 0 || k < 0)
    return fail(FAST_ERR_INVALID_ARG, "%s: negative size or k", fn);
  if (num_roots >= (int64_t(1) << 31))   // also with k = 0: the workspace is sized per root
    return fail(FAST_ERR_UNSUPPORTED, "%s: num_roots >= 2^31", fn);
  if (num_roots * int64_t(k) >= (int64_t(1) << 31))
    return fail(FAST_ERR_UNSUPPORTED, "%s: num_roots * k >= 2^31", fn);
  if (!dst_offsets) return fail(FAST_ERR_INVALID_ARG, "%s: dst_offsets is NULL", fn);
  if (num_roots > 0 && (!roots || !root_t))
    return fail(FAST_ERR_INVALID_ARG, "%s: roots/root_t is NULL", fn);
  if (num_roots > 0 && k > 0 && (!src_ids || !edge_t || !edge_ids))
    return fail(FAST_ERR_INVALID_ARG, "%s: NULL src_ids/edge_t/edge_ids", fn);
  if (g->num_nodes > 0 && !g->indptr) return fail(FAST_ERR_INVALID_ARG, "%s: indptr is NULL", fn);
  if (g->num_entries > 0 && (!g->nbr || !g->ts || !g->eid))
    return fail(FAST_ERR_INVALID_ARG, "%s: NULL nbr/ts/eid", fn);
  const size_t need = fast_sample_recent_workspace(num_roots);
  if (!ws || ws_bytes < need)
    return fail(FAST_ERR_WORKSPACE, "%s: workspace of %zu bytes < %zu", fn, ws_bytes, need);
  if (!aligned(ws, 256)) return fail(FAST_ERR_UNSUPPORTED, "%s: workspace not 256-byte aligned", fn);
  hipStream_t st = static_cast<hipStream_t>(stream);
  SrWs w;
  sr_layout(num_roots, static_cast<char*>(ws), &w);
  const int64_t R = num_roots;
  const int kk = (g->num_nodes > 0 && g->num_entries > 0) ? k : 0;   // no entries: all empty
  // tiled: the counts go to dst_offsets and the tile sums (at most R) to their
  // place in the workspace, which a smaller batch never needs more of than a
  // larger one
  const bool tiled = R <= SR_TILED;
  int32_t* counts = tiled ? dst_offsets : w.count;
  uint32_t* tsum = tiled ? reinterpret_cast<uint32_t*>(w.count) : nullptr;
  const auto count = [&](auto kernel, int64_t roots_per_wg, int lanes) {
    hipLaunchKernelGGL(kernel, dim3(uint32_t((R + roots_per_wg - 1) / roots_per_wg)),
                       dim3(uint32_t(roots_per_wg * lanes)), 0, st, g->indptr, g->num_nodes,
                       g->num_entries, g->ts, roots, root_t, R, kk, counts, w.start, tsum);
  };
  const auto fill = [&](auto kernel, int64_t roots_per_wg) {
    hipLaunchKernelGGL(kernel, dim3(uint32_t((R + roots_per_wg - 1) / roots_per_wg)),
                       dim3(uint32_t(roots_per_wg * SR_GROUP)), 0, st, g->nbr, g->ts, g->eid, w.start, tsum,
                       R, dst_offsets, src_ids, edge_t, edge_ids);
  };
  if (R > 0 && R <= SR_MAX_TILES * SR_SMALL) {
    if (R <= SR_WIDE_SEARCH) count(k_sample_count<SR_SMALL, 16>, SR_SMALL, 16);
    else count(k_sample_count<SR_SMALL, 4>, SR_SMALL, 4);
    fill(k_sample_fill<SR_SMALL>, SR_SMALL);
  } else if (R > 0 && R <= SR_TILED) {
    count(k_sample_count<SR_LARGE, 4>, SR_LARGE, 4);
    fill(k_sample_fill<SR_LARGE>, SR_LARGE);
  } else {
    if (R > 0) count(k_sample_count<SR_THREADS, 1>, SR_THREADS, 1);   // a thread per search, no tile sums
    const hipError_t e = scan_launch(InRootCount{w.count}, OutRootOffset{dst_offsets}, R, w.scan, nullptr,
                                     dst_offsets + R, st);
    if (e != hipSuccess) return fail(FAST_ERR_HIP, "%s: %s", fn, hipGetErrorString(e));
    if (R > 0 && kk > 0)
      hipLaunchKernelGGL(k_sample_copy, dim3(uint32_t((R * SR_GROUP + SR_THREADS - 1) / SR_THREADS)),
                         dim3(SR_THREADS), 0, st, g->nbr, g->ts, g->eid, w.count, w.start, dst_offsets, R,
                         src_ids, edge_t, edge_ids);
  }
  return check_launch(fn);
}
