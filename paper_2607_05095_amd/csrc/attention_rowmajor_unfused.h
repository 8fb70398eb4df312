// attention_rowmajor_unfused.h -- the separate edge softmax and aggregation
// operators in the row-major lane layout of attention_rowmajor.h (fp32, two
// heads off the 16-byte grid: the 2 x 50 heads of 100-wide rows), so that
// their rows move as 16-byte accesses too.
//
// Each kernel reads or writes its per-edge rows once and is bound by HBM.  A
// chunk of RU_CH edges is loaded back to back; slots that no segment of the
// wave needs load nothing.  The per-edge scalars of a chunk (alpha, dalpha: RU_CH x H
// consecutive floats) move as one access, a lane per float, and are passed
// between lanes by shuffles.  The softmax keeps the logits of the first
// RU_SAVE chunks in registers, so that a segment of up to 20 edges reads its
// K rows once; its backward has the first chunk's rows in flight before it
// forms D.  66,000 segments of 10 edges, 2 x 50 heads, against the head-major
// lanes' 8-byte accesses: softmax forward 91 -> 66 us, aggregation forward
// 59 -> 48, aggregation backward 125 -> 100, softmax backward 145 -> 109 us
// (138 with D formed first).
#pragma once

#include "attention_rowmajor.h"

namespace fast {

constexpr int RU_CH = 10;
constexpr int RU_SAVE = 2;

// Rows [base, min(base + RU_CH, e1)) of a per-edge array, streamed: each is
// read once per call.  Slots past the end hold the segment's last row again,
// or zeros where no segment of the wave needs the slot.
template <int H>
__device__ __forceinline__ void ru_load(const float* __restrict__ rows, int64_t base, int64_t e1, int F,
                                        const RmMap<H>& m, float (&x)[RU_CH][4]) {
  const int64_t last = e1 > 0 ? e1 - 1 : 0;   // also of an empty segment: a row of the array
#pragma unroll
  for (int i = 0; i < RU_CH; ++i) {
    if (!__any(base + i < e1)) x[i][0] = x[i][1] = x[i][2] = x[i][3] = 0.f;
    else rm_load_row<true, H>(rows, base + i < e1 ? base + i : last, F, m, x[i]);
  }
}

// The chunk's scalars of a per-edge [E, H] array: entry k = i * H + h lives in
// lane k % G, slot k / G (0 past the segment's end).
template <int H, int G>
struct RuScalars {
  static constexpr int N = (RU_CH * H + G - 1) / G;
  float v[N];
  __device__ __forceinline__ void load(const float* __restrict__ p, int64_t base, int64_t e1, int lane) {
#pragma unroll
    for (int s = 0; s < N; ++s) {
      const int k = s * G + lane;
      v[s] = k < RU_CH * H && base + k / H < e1 ? p[base * H + k] : 0.f;
    }
  }
  __device__ __forceinline__ float get(int k) const { return __shfl(v[k / G], k % G, G); }
  // Sets entry k of the lane that holds it.
  __device__ __forceinline__ void put(int k, float x, int lane) { v[k / G] = lane == k % G ? x : v[k / G]; }
  __device__ __forceinline__ void store(float* __restrict__ p, int64_t base, int64_t e1, int lane) const {
#pragma unroll
    for (int s = 0; s < N; ++s) {
      const int k = s * G + lane;
      if (k < RU_CH * H && base + k / H < e1) p[base * H + k] = v[s];
    }
  }
};

// Logits (base 2) of a chunk, -inf past the segment's end, and their running max.
template <int H, int G>
__device__ __forceinline__ void ru_logits(const float (&q)[4], const float (&kx)[RU_CH][4],
                                          const RmMap<H>& m, int64_t base, int64_t e1, float sl2,
                                          float slope, float (&t)[RU_CH][H]) {
#pragma unroll
  for (int i = 0; i < RU_CH; ++i) {
    if (i == RU_CH / 2 && !__any(base + i < e1)) {
#pragma unroll
      for (int k = RU_CH / 2; k < RU_CH; ++k)
#pragma unroll
        for (int h = 0; h < H; ++h) t[k][h] = -INFINITY;
      break;
    }
    float d[H];
    rm_dots<H, G>(q, kx[i], m, d);
#pragma unroll
    for (int h = 0; h < H; ++h) t[i][h] = base + i < e1 ? lrelu(d[h] * sl2, slope) : -INFINITY;
  }
}

template <int H, int G>
__global__ void __launch_bounds__(ATT_MAX_BLOCK) k_softmax_fwd_rm(AttnArgs a) {
  RmMap<H> m;
  if (!rm_setup<H, G>(a, m)) return;
  const int F = a.L.F;
  const float* K = static_cast<const float*>(a.K);
  const float sl2 = a.scale * LOG2E;
  float q[4];
  rm_load_row<true, H>(static_cast<const float*>(a.Q), m.seg, F, m, q);
  int64_t e0, e1;
  seg_range(a, m.seg, e0, e1);
  float mx[H], Z[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    mx[h] = -INFINITY;
    Z[h] = 0.f;
  }
  auto fold = [&](const float (&t)[RU_CH][H]) {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      float mn = mx[h];
#pragma unroll
      for (int i = 0; i < RU_CH; ++i) mn = fmaxf(mn, t[i][h]);
      Z[h] *= exp2_hw(mx[h] - mn);
#pragma unroll
      for (int i = 0; i < RU_CH; ++i) Z[h] += exp2_hw(t[i][h] - mn);
      mx[h] = mn;
    }
  };
  // pass 1: running max and normaliser; the first RU_SAVE chunks keep their logits
  float t[RU_SAVE][RU_CH][H];
#pragma unroll
  for (int c = 0; c < RU_SAVE; ++c) {
    const int64_t base = e0 + c * RU_CH;
    if (base < e1) {
      float kx[RU_CH][4];
      ru_load<H>(K, base, e1, F, m, kx);
      ru_logits<H, G>(q, kx, m, base, e1, sl2, a.slope, t[c]);
      fold(t[c]);
    }
  }
  for (int64_t base = e0 + RU_SAVE * RU_CH; base < e1; base += RU_CH) {
    float kx[RU_CH][4], tt[RU_CH][H];
    ru_load<H>(K, base, e1, F, m, kx);
    ru_logits<H, G>(q, kx, m, base, e1, sl2, a.slope, tt);
    fold(tt);
  }
  float invZ[H];
#pragma unroll
  for (int h = 0; h < H; ++h) invZ[h] = Z[h] > 0.f ? 1.f / Z[h] : 0.f;
  if (a.lse_out && m.c < H) {
    float lse = 0.f;
#pragma unroll
    for (int h = 0; h < H; ++h)
      if (m.c == h) lse = Z[h] > 0.f ? (mx[h] + log2f(Z[h])) * LN2 : -INFINITY;
    a.lse_out[m.seg * H + m.c] = lse;
  }
  // pass 2: alpha (past the saved chunks K is read again, normally from L2)
  auto emit = [&](const float (&x)[RU_CH][H], int64_t base) {
    RuScalars<H, G> s;
#pragma unroll
    for (int j = 0; j < s.N; ++j) s.v[j] = 0.f;
#pragma unroll
    for (int i = 0; i < RU_CH; ++i)
#pragma unroll
      for (int h = 0; h < H; ++h) s.put(i * H + h, exp2_hw(x[i][h] - mx[h]) * invZ[h], m.c);
    s.store(a.alpha_out, base, e1, m.c);
  };
#pragma unroll
  for (int c = 0; c < RU_SAVE; ++c)
    if (e0 + c * RU_CH < e1) emit(t[c], e0 + c * RU_CH);
  for (int64_t base = e0 + RU_SAVE * RU_CH; base < e1; base += RU_CH) {
    float kx[RU_CH][4], tt[RU_CH][H];
    ru_load<H>(K, base, e1, F, m, kx);
    ru_logits<H, G>(q, kx, m, base, e1, sl2, a.slope, tt);
    emit(tt, base);
  }
}

template <int H, int G>
__global__ void __launch_bounds__(ATT_MAX_BLOCK) k_softmax_bwd_rm(AttnArgs a) {
  RmMap<H> m;
  if (!rm_setup<H, G>(a, m)) return;
  const int F = a.L.F;
  const float* K = static_cast<const float*>(a.K);
  float q[4];
  rm_load_row<true, H>(static_cast<const float*>(a.Q), m.seg, F, m, q);
  int64_t e0, e1;
  seg_range(a, m.seg, e0, e1);
  // The first chunk is loaded before D is known.  D = sum alpha dalpha: lane c
  // holds the entries c, c + G, ... of the segment, all of head c % H.
  static_assert(G % H == 0 && RU_CH * H <= G * RuScalars<H, G>::N, "lanes keep their head");
  RuScalars<H, G> al, da;
  float kx[RU_CH][4];
  al.load(a.alpha_in, e0, e1, m.c);
  da.load(a.dalpha_in, e0, e1, m.c);
  ru_load<H>(K, e0, e1, F, m, kx);
  float part = 0.f;
#pragma unroll
  for (int s = 0; s < al.N; ++s) part = fmaf(al.v[s], da.v[s], part);
  for (int64_t base = e0 + RU_CH; base < e1; base += RU_CH) {
    RuScalars<H, G> x, y;
    x.load(a.alpha_in, base, e1, m.c);
    y.load(a.dalpha_in, base, e1, m.c);
#pragma unroll
    for (int s = 0; s < x.N; ++s) part = fmaf(x.v[s], y.v[s], part);
  }
  float D[H];
#pragma unroll
  for (int h = 0; h < H; ++h) D[h] = group_sum_ct<G>(m.c % H == h ? part : 0.f);
  float dq[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t base = e0; base < e1; base += RU_CH) {
    if (base != e0) {
      al.load(a.alpha_in, base, e1, m.c);
      da.load(a.dalpha_in, base, e1, m.c);
      ru_load<H>(K, base, e1, F, m, kx);
    }
    // the lane's own entries: alpha (dalpha - D) scale, the rest of g is LReLU'
#pragma unroll
    for (int s = 0; s < al.N; ++s) {
      float Dl = D[0];
#pragma unroll
      for (int h = 1; h < H; ++h) Dl = m.c % H == h ? D[h] : Dl;
      al.v[s] *= (da.v[s] - Dl);
    }
#pragma unroll
    for (int i = 0; i < RU_CH; ++i) {
      if (base + i >= e1) break;
      float d[H], g[H];
      rm_dots<H, G>(q, kx[i], m, d);
#pragma unroll
      for (int h = 0; h < H; ++h)
        g[h] = al.get(i * H + h) * lrelu_grad(d[h] * a.scale, a.slope) * a.scale;
      float dk[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float gk = pick<H>(g, m.hs[k]);
        dq[k] = fmaf(gk, kx[i][k], dq[k]);
        dk[k] = gk * q[k];
      }
      rm_store_row<false, H>(static_cast<float*>(a.dK), base + i, F, m, dk);
    }
  }
  rm_store_row<true, H>(static_cast<float*>(a.dQ), m.seg, F, m, dq);
}

template <int H, int G>
__global__ void __launch_bounds__(ATT_MAX_BLOCK) k_agg_fwd_rm(AttnArgs a) {
  RmMap<H> m;
  if (!rm_setup<H, G>(a, m)) return;
  const int F = a.L.F;
  const float* V = static_cast<const float*>(a.V);
  int64_t e0, e1;
  seg_range(a, m.seg, e0, e1);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t base = e0; base < e1; base += RU_CH) {
    RuScalars<H, G> al;
    float vx[RU_CH][4];
    al.load(a.alpha_in, base, e1, m.c);
    ru_load<H>(V, base, e1, F, m, vx);
#pragma unroll
    for (int i = 0; i < RU_CH; ++i) {
      float w[H];
#pragma unroll
      for (int h = 0; h < H; ++h) w[h] = al.get(i * H + h);
      if (base + i < e1) {                               // a masked slot's row may be infinite
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = fmaf(pick<H>(w, m.hs[k]), vx[i][k], acc[k]);
      }
    }
  }
  rm_store_row<true, H>(static_cast<float*>(a.out), m.seg, F, m, acc);
}

// Four waves per SIMD, not the five that the registers hold: 66,000 segments of
// 10 edges, the four operators 311 -> 308 us.
template <int H, int G>
__global__ void __launch_bounds__(ATT_MAX_BLOCK) __attribute__((amdgpu_waves_per_eu(4, 4))) k_agg_bwd_rm(AttnArgs a) {
  RmMap<H> m;
  if (!rm_setup<H, G>(a, m)) return;
  const int F = a.L.F;
  const float* V = static_cast<const float*>(a.V);
  float go[4];
  rm_load_row<true, H>(static_cast<const float*>(a.dO), m.seg, F, m, go);
  int64_t e0, e1;
  seg_range(a, m.seg, e0, e1);
  for (int64_t base = e0; base < e1; base += RU_CH) {
    RuScalars<H, G> al, da;
    float vx[RU_CH][4];
    al.load(a.alpha_in, base, e1, m.c);
    ru_load<H>(V, base, e1, F, m, vx);
#pragma unroll
    for (int j = 0; j < da.N; ++j) da.v[j] = 0.f;
#pragma unroll
    for (int i = 0; i < RU_CH; ++i) {
      if (i == RU_CH / 2 && !__any(base + i < e1)) break;
      float d[H], w[H], dv[4];
      rm_dots<H, G>(go, vx[i], m, d);
#pragma unroll
      for (int h = 0; h < H; ++h) {
        da.put(i * H + h, d[h], m.c);
        w[h] = al.get(i * H + h);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) dv[k] = pick<H>(w, m.hs[k]) * go[k];
      if (base + i < e1) rm_store_row<false, H>(static_cast<float*>(a.dV), base + i, F, m, dv);
    }
    da.store(a.dalpha_out, base, e1, m.c);
  }
}

}  // namespace fast
