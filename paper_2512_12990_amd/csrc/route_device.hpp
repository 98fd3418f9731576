// Cache-aware top-k routing (paper Section 2.1: experts whose slices are resident get their
// gating score boosted before selection): device routines shared by the routing entry points.
#pragma once
#include "common.hpp"

struct RouteArgs {
  int E, k, d_model;
  const float* logits;     // [T, E] or null
  const void* x;           // [T, d_model] act dtype (used when logits is null)
  const float* w_router;   // [E, d_model]
  const float* bias;       // [E] or null
  int norm_topk;
  float routed_scale;
  float* logits_out;       // [T, E] or null
  int32_t* idx;            // [T, k]
  float* w;                // [T, k]
};

// Monotone map float -> uint32 (a < b  <=>  map(a) < map(b)); -0 is first folded onto +0 so
// equal scores compare equal.
__device__ __forceinline__ uint32_t orderable(float f) {
  if (f == 0.0f) f = 0.0f;
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float unorderable(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o ^ 0x80000000u) : ~o);
}

template <int CTRL, int ROWM, int BANKM> __device__ __forceinline__ uint32_t dpp_umax(uint32_t v) {
  const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWM, BANKM, true);
  return t > v ? t : v;
}
// Unsigned maximum over the wave, returned in every lane.
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {
  v = dpp_umax<0xB1, 0xF, 0xF>(v);
  v = dpp_umax<0x4E, 0xF, 0xF>(v);
  v = dpp_umax<0x114, 0xF, 0xE>(v);
  v = dpp_umax<0x118, 0xF, 0xC>(v);
  v = dpp_umax<0x142, 0xA, 0xF>(v);
  v = dpp_umax<0x143, 0xC, 0xF>(v);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Top-k selection of one token by ONE wave.  z[0..E) are the token's logits (LDS); lane l keeps the experts l,
// l + 64, ... (NJ of them) in registers, and every pick is one reduction over the wave's lanes.
// Rule: k largest z + bias from the highest down, equal scores to the lower expert index; weights
// = softmax of the unbiased logits at the selected experts (optionally renormalised), * scale.
template <int NJ>
__device__ __forceinline__ void select_topk_wave(const RouteArgs& a, int t, const float* z, int lane) {
  const int E = a.E;
  float zv[NJ], p[NJ];
  uint32_t ord[NJ], zmax = 0;      // ord: orderable biased score; 0 = absent or already taken
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    const int e = lane + 64 * j;
    const bool ok = e < E;
    zv[j] = ok ? z[e] : 0.0f;
    const float score = zv[j] + (ok && a.bias ? a.bias[e] : 0.0f);          // one fp32 add
    const uint32_t os = orderable(score), oz = orderable(zv[j]);
    ord[j] = ok ? (os > 1u ? os : 1u) : 0u;
    zmax = ok && oz > zmax ? oz : zmax;
  }
  const float m = unorderable(wave_umax(zmax));
  float den = 0.0f;
#pragma unroll
  for (int j = 0; j < NJ; j++) { p[j] = lane + 64 * j < E ? expf(zv[j] - m) : 0.0f; den += p[j]; }
  den = wave_sum(den);
  float wsum = 0.0f, myw = 0.0f;
  int mysel = 0;
  for (int r = 0; r < a.k; r++) {
    uint32_t best = ord[0];
    int jb = 0;
#pragma unroll
    for (int j = 1; j < NJ; j++) if (ord[j] > best) { best = ord[j]; jb = j; }
    const uint32_t top = wave_umax(best);
    int ls, js;
    if (NJ == 1) {                                            // lowest lane among equal scores
      ls = (int)__builtin_ctzll(__ballot(best == top)); js = 0;
    } else {
      const int e_star = (int)~wave_umax(~(best == top ? (uint32_t)(lane + 64 * jb) : 0xFFFFFFFFu));      // lowest index among equal scores
      ls = e_star & 63; js = e_star >> 6;
    }
    float pw = 0.0f;
#pragma unroll
    for (int j = 0; j < NJ; j++) {
      const float u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p[j]), ls));
      if (js == j) pw = u;
      if (js == j && lane == ls) ord[j] = 0u;
    }
    const float wj = pw / den;
    wsum += wj;
    if (lane == r) { mysel = ls + 64 * js; myw = wj; }      // slot r belongs to lane r
  }
  const float mul = (a.norm_topk ? 1.0f / wsum : 1.0f) * a.routed_scale;
  if (lane < a.k) {
    a.idx[(size_t)t * a.k + lane] = mysel;
    a.w[(size_t)t * a.k + lane] = myw * mul;
  }
}

// Router logits of NT tokens by a work-group of RT_NW waves, then the selection, one wave per token.
// Lane l of a wave sums columns l, l + 64, ... of a row in that order by fused multiply-add, then comes the wave
// sum; router_logits_kernel does the same, so logits are bit-identical between entry points.
// Bound: vector issue (T * E * d / 64 fused multiply-adds of a wave, and a conversion per four of them) with many
// tokens, the latency of the router rows (E * d * 4 bytes per work-group out of L2) with few.  A wave takes RT_R rows at
// a time against all NT vectors, 512 columns per batch, the next batch's weights in flight while one is summed.  The
// vectors stand in LDS column by column, so that one LDS read feeds NT * RT_R multiply-adds.  NT is the
// smallest of 1, 2, 4, 8 (fp32: 4) that needs no more work-groups than there are CUs.  64 experts, d 2048, bf16, top-6:
// 173 / 1000 / 2048 / 4096 tokens in 18.7 / 18.7 / 19.4 / 36 us with eight tokens per work-group, cold batches and a
// selection over LDS keys; 11.6 (what the host needs to send it off) / 12.1 / 16.4 / 30.5 us now.
#define RT_R 4
#define RT_NW 16
#define RT_THREADS (RT_NW * 64)
// Position of column i of the staged activations, in columns: one column of padding after every eight, so that the
// blocks of columns that the staging threads of a wave write start in different banks.
__device__ __forceinline__ int rt_col(int i) { return i + (i >> 3); }

template <int ACT, int NT> struct RouteLds {      // NT * E logits, then (without given logits) the activations
  static size_t bytes(int E, int d, bool given_logits) {
    return (size_t)((NT * E * 4 + 15) & ~15) + (given_logits ? 0 : (size_t)(d + d / 8 + 1) * NT * (ACT == SMOE_BF16 ? 2 : 4));
  }
};

template <int ACT, int NT>
__device__ __forceinline__ void router_logits_block(const RouteArgs& a, int t0, int nt, float* zt, uint8_t* xs) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int E = a.E, d = a.d_model;
  constexpr int ESZ = ACT == SMOE_BF16 ? 2 : 4, VEC = 16 / ESZ, CB = NT * ESZ;      // elements of a 16-byte load, bytes of a column
  const int nb = d >> 9;                                        // whole batches of 512 columns
  float w0[RT_R][8], w1[RT_R][8];
  const float* wrow[RT_R];
  auto rows_of = [&](int e0) {
#pragma unroll
    for (int r = 0; r < RT_R; r++) wrow[r] = a.w_router + (size_t)min(e0 + r, E - 1) * d;      // (rows past E repeat the last one)
  };
  auto fetch = [&](int i, float (&w)[RT_R][8]) {
    const int i0 = min(i, nb - 1) * 512 + lane;
#pragma unroll
    for (int r = 0; r < RT_R; r++)
#pragma unroll
      for (int u = 0; u < 8; u++) w[r][u] = wrow[r][i0 + u * 64];
  };
  rows_of(wave * RT_R);
  constexpr bool AHEAD = NT * ESZ < 16;                         // the widest form has no registers for a second batch, and plenty of sums per batch
  if (AHEAD && nb) fetch(0, w0);                                // on their way while the activations are staged
  if (d % VEC == 0) {
    // a thread moves VEC consecutive columns of one vector
    for (int i = tid; i < NT * (d / VEC); i += RT_THREADS) {
      const int q = i % NT, cb = i / NT;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (q < nt) v = *(const uint4*)((const uint8_t*)a.x + ((size_t)(t0 + q) * d + (size_t)cb * VEC) * ESZ);
      const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < VEC; j++) {
        uint8_t* dst = xs + (size_t)rt_col(cb * VEC + j) * CB + q * ESZ;
        if (ACT == SMOE_BF16) *(uint16_t*)dst = (uint16_t)(u[j / 2] >> ((j & 1) * 16));
        else *(uint32_t*)dst = u[j % 4];
      }
    }
  } else {
    for (int i = tid; i < NT * d; i += RT_THREADS) {
      const int q = i / d, c = i - q * d;
      uint8_t* dst = xs + (size_t)rt_col(c) * CB + q * ESZ;
      if (ACT == SMOE_BF16) *(uint16_t*)dst = q < nt ? ((const uint16_t*)a.x)[(size_t)t0 * d + i] : (uint16_t)0;
      else *(float*)dst = q < nt ? ((const float*)a.x)[(size_t)t0 * d + i] : 0.0f;
    }
  }
  __syncthreads();
  auto column = [&](int i, float (&xf)[NT]) {
    const uint8_t* c = xs + (size_t)rt_col(i) * CB;
    if constexpr (ACT == SMOE_BF16) {
      if constexpr (NT == 1) {
        xf[0] = bf16_bits_to_f32(*(const uint16_t*)c);
      } else {
        struct alignas(CB) Words { uint32_t u[NT / 2 ? NT / 2 : 1]; };
        const Words w = *(const Words*)c;
#pragma unroll
        for (int j = 0; j < NT / 2; j++) { xf[2 * j] = __uint_as_float(w.u[j] << 16); xf[2 * j + 1] = __uint_as_float(w.u[j] & 0xFFFF0000u); }
      }
    } else {
      struct alignas(CB) Vals { float f[NT]; };
      const Vals w = *(const Vals*)c;
#pragma unroll
      for (int j = 0; j < NT; j++) xf[j] = w.f[j];
    }
  };
  for (int e0 = wave * RT_R; e0 < E; e0 += RT_NW * RT_R) {
    float p[RT_R][NT];
#pragma unroll
    for (int r = 0; r < RT_R; r++)
#pragma unroll
      for (int q = 0; q < NT; q++) p[r][q] = 0.0f;
    auto batch = [&](int i, const float (&w)[RT_R][8]) {
#pragma unroll
      for (int u = 0; u < 8; u++) {
        float xf[NT];
        column(i * 512 + u * 64 + lane, xf);
#pragma unroll
        for (int r = 0; r < RT_R; r++)
#pragma unroll
          for (int q = 0; q < NT; q++) p[r][q] = fmaf(w[r][u], xf[q], p[r][q]);
      }
    };
    if (e0 != wave * RT_R) {
      rows_of(e0);
      if (AHEAD && nb) fetch(0, w0);
    }
    if constexpr (AHEAD) {
      for (int i = 0; i < nb; i += 2) {
        fetch(i + 1, w1);
        batch(i, w0);
        if (i + 1 < nb) {
          fetch(i + 2, w0);
          batch(i + 1, w1);
        }
      }
    } else {
      for (int i = 0; i < nb; i++) {
        fetch(i, w0);
        batch(i, w0);
      }
    }
    for (int i = nb * 512 + lane; i < d; i += 64) {
      float xf[NT];
      column(i, xf);
#pragma unroll
      for (int r = 0; r < RT_R; r++) {
        const float w = wrow[r][i];
#pragma unroll
        for (int q = 0; q < NT; q++) p[r][q] = fmaf(w, xf[q], p[r][q]);
      }
    }
#pragma unroll
    for (int r = 0; r < RT_R; r++)
#pragma unroll
      for (int q = 0; q < NT; q++) {
        const float s = wave_sum(p[r][q]);
        if (lane == 0 && e0 + r < E) zt[q * E + e0 + r] = s;
      }
  }
}

template <int ACT, int NT>
__device__ __forceinline__ void route_tokens_block(const RouteArgs& a, int T, uint8_t* dyn) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int E = a.E, t0 = blockIdx.x * NT, nt = min(NT, T - t0);
  float* zt = (float*)dyn;                                            // [NT][E]
  if (a.logits) {
    for (int i = tid; i < nt * E; i += RT_THREADS) zt[i] = a.logits[(size_t)t0 * E + i];
  } else {
    router_logits_block<ACT, NT>(a, t0, nt, zt, dyn + ((NT * E * 4 + 15) & ~15));
  }
  __syncthreads();
  if (a.logits_out)
    for (int i = tid; i < nt * E; i += RT_THREADS) a.logits_out[(size_t)t0 * E + i] = zt[i];
  for (int q = wave; q < nt; q += RT_NW) {
    if (E <= 64) select_topk_wave<1>(a, t0 + q, zt + q * E, lane);
    else select_topk_wave<4>(a, t0 + q, zt + q * E, lane);
  }
}
