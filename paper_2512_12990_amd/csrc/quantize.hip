// AMAT quantise + slice (paper Section 4.2 and its equation; Table 1 note 1).
//
// Two kernels of the same arithmetic.  quantize_flat_kernel takes groups of 32 * 2^n <= 512 columns
// (every group the decode kernels accept and the sizes in use): eight columns per lane in one wide
// load.  quantize_rows_kernel takes every other group (96, 1024, ...): one wavefront per group.
// All arithmetic that decides an integer (scale, zero-point, code) is plain IEEE fp32 with
// round-to-nearest-even, no contraction and correctly rounded division, so codes are reproducible
// bit for bit.
#include "common.hpp"
#include <type_traits>

#pragma clang fp contract(off)

template <int WDT> __device__ __forceinline__ float load_w(const void* p, size_t i) {
  if (WDT == SMOE_F32) return ((const float*)p)[i];
  return bf16_bits_to_f32(((const uint16_t*)p)[i]);
}

__device__ __forceinline__ float wave_min(float v) {
  for (int m = 32; m >= 1; m >>= 1) v = fminf(v, __shfl_xor(v, m));
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
  for (int m = 32; m >= 1; m >>= 1) v = fmaxf(v, __shfl_xor(v, m));
  return v;
}

// Any group: one work-group per destination row, one wavefront per group.
// w0/w1: source matrices of the n experts being converted ([n, N/2, K] each when `interleave`,
// else w0 is [n, N, K]).  Destination family `m` already points at expert 0 of the bank.
template <int WDT>
__global__ __launch_bounds__(256) void quantize_rows_kernel(const void* __restrict__ w0, const void* __restrict__ w1,
                                                            MatDev m, int e0, int group, int sc_bf16, int interleave, int symmetric) {
  const int row = blockIdx.x, el = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int K = m.K, ng = m.ng;
  const void* src;
  size_t src_row;
  if (interleave) {
    src = (row & 1) ? w1 : w0;
    src_row = (size_t)el * (m.N / 2) + (row >> 1);
  } else {
    src = w0;
    src_row = (size_t)el * m.N + row;
  }
  const size_t sbase = src_row * (size_t)K;
  const size_t e = (size_t)(e0 + el);
  const int bits = m.bits;                             // 4: 8-bit codes, nibble planes; 3: 6-bit codes; 2: 4-bit codes, 2-bit planes
  const float qmax = bits == 4 ? 255.0f : bits == 3 ? 63.0f : 15.0f;
  uint8_t* pm = const_cast<uint8_t*>(m.msb) + e * m.plane_stride + (size_t)row * (K * bits / 8);
  uint8_t* pl = const_cast<uint8_t*>(m.lsb) + e * m.plane_stride + (size_t)row * (K * bits / 8);
  uint8_t* pz = const_cast<uint8_t*>(m.zp) + e * m.zp_stride + (size_t)row * ng;
  uint8_t* ps = const_cast<uint8_t*>(m.sc) + e * m.sc_stride;

  for (int g = wave; g < ng; g += 4) {
    const int k0 = g * group;
    const int gsz = min(group, K - k0);
    const int np = gsz >> 1;
    float lo = 0.0f, hi = 0.0f;                       // the range always contains 0
    for (int p = lane; p < np; p += 64) {
      const float a = load_w<WDT>(src, sbase + k0 + 2 * p), b = load_w<WDT>(src, sbase + k0 + 2 * p + 1);
      lo = fminf(lo, fminf(a, b));
      hi = fmaxf(hi, fmaxf(a, b));
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    // symmetric variant (Section 6.1 item 1: symmetric integer weights): step from the largest magnitude, the
    // zero-point fixed at mid-range of the unsigned store
    const float half = 0.5f * (qmax + 1.0f);
    float s = symmetric ? fmaxf(hi, -lo) / (half - 1.0f) : (hi - lo) / qmax;
    if (sc_bf16) s = bf16_bits_to_f32(f32_to_bf16_bits(s));
    if (!(s > 0.0f)) s = 1.0f;
    const int zp = symmetric ? (int)half : (int)fminf(fmaxf(rintf((-lo) / s), 0.0f), qmax);
    if (bits == 3) {
      // 6-bit codes: upper three bits = the low-bit code.  A plane keeps the 32 three-bit values of a
      // chunk of 32 columns in 12 bytes, laid out so that a nibble word (one value per nibble, columns
      // 8t .. 8t+7 in word t) comes out of it with a shift and a mask: column 8t + j has its two low
      // bits in word t >> 1 at bits 4j + 2(t & 1), 4j + 2(t & 1) + 1 and its third bit in word 2 at
      // bit 4j + t.  Eight lanes build a chunk: lane j of them takes the columns 8t + j.
      const int nchunk = gsz >> 5, j = lane & 7;
      for (int cb = 0; cb < nchunk; cb += 8) {
        const int c = cb + (lane >> 3);
        uint32_t wm[3] = {0, 0, 0}, wl[3] = {0, 0, 0};
        if (c < nchunk) {
#pragma unroll
          for (int t = 0; t < 4; t++) {
            const float a = load_w<WDT>(src, sbase + k0 + 32 * c + 8 * t + j);
            const int q = min(max((int)rintf(a / s) + zp, 0), 63);
            const uint32_t mv = (uint32_t)q >> 3, lv = (uint32_t)q & 7u;
            wm[t >> 1] |= (mv & 3u) << (4 * j + 2 * (t & 1));
            wl[t >> 1] |= (lv & 3u) << (4 * j + 2 * (t & 1));
            wm[2] |= (mv >> 2) << (4 * j + t);
            wl[2] |= (lv >> 2) << (4 * j + t);
          }
        }
#pragma unroll
        for (int i = 0; i < 3; i++)
          for (int x = 1; x < 8; x <<= 1) {
            wm[i] |= (uint32_t)__shfl_xor((int)wm[i], x);
            wl[i] |= (uint32_t)__shfl_xor((int)wl[i], x);
          }
        if (c < nchunk && j == 0) {
          uint32_t* dm = (uint32_t*)(pm + (size_t)((k0 >> 5) + c) * 12);
          uint32_t* dl = (uint32_t*)(pl + (size_t)((k0 >> 5) + c) * 12);
#pragma unroll
          for (int i = 0; i < 3; i++) { dm[i] = wm[i]; dl[i] = wl[i]; }
        }
      }
    } else if (bits == 2) {
      // 4-bit codes: upper two bits = the low-bit code; four codes per plane byte, column 4j in bits 0-1
      for (int p = lane; p < (gsz >> 2); p += 64) {
        int bm = 0, bl = 0;
#pragma unroll
        for (int c = 0; c < 4; c++) {
          const float a = load_w<WDT>(src, sbase + k0 + 4 * p + c);
          const int q = min(max((int)rintf(a / s) + zp, 0), 15);
          bm |= (q >> 2) << (2 * c);
          bl |= (q & 3) << (2 * c);
        }
        pm[(k0 >> 2) + p] = (uint8_t)bm;
        pl[(k0 >> 2) + p] = (uint8_t)bl;
      }
    } else
    for (int p = lane; p < np; p += 64) {
      const float a = load_w<WDT>(src, sbase + k0 + 2 * p), b = load_w<WDT>(src, sbase + k0 + 2 * p + 1);
      const int qa = min(max((int)rintf(a / s) + zp, 0), 255);
      const int qb = min(max((int)rintf(b / s) + zp, 0), 255);
      // planes keep every nibble n as n - 8 in 4-bit two's complement (n ^ 8): signed 4-bit dot products
      // read them directly
      pm[(k0 >> 1) + p] = (uint8_t)(((qa >> 4) | (qb & 0xF0)) ^ 0x88);          // floor(q/16): the low-bit code
      pl[(k0 >> 1) + p] = (uint8_t)(((qa & 15) | ((qb & 15) << 4)) ^ 0x88);     // the bits truncation drops
    }
    if (lane == 0) {
      pz[g] = (uint8_t)zp;
      const size_t si = (size_t)row * m.sng + g;
      if (sc_bf16) ((uint16_t*)ps)[si] = (uint16_t)f32_to_bf16_bits(s);
      else ((float*)ps)[si] = s;
    }
  }
}

// ---------------------------------------------------------------------------------- eight columns per lane
// Bound: HBM (2 or 4 bytes read and 1 byte written per weight) with vector issue close behind (about
// 17 instructions per weight).  A matrix is a flat list of units of eight columns, every row padded to
// whole groups, so a group is L = group / 8 neighbouring lanes (4 .. 64) and its range is a few lane
// exchanges.  A lane holds QF_U units 64 lanes apart, all fetched (16 bytes bf16, 32 bytes fp32 a unit)
// before the first is used; the three divisions of a group (scale, zero-point, reciprocal) are made by
// one lane per unit -- lane u of every quad takes unit u -- and handed round inside the quad, so a wave
// issues them once for all its units.  gate/up and down of all experts are one launch.
// 8 experts of d_model 2048, d_ff 1408 into the 8/4 store, bf16, groups of 128: 50.7 us (4.1 TB/s) against
// 160 us with the general kernel; 3 experts, fp32, 6/3 store, groups of 32: 29.4 us (4.3 TB/s) against 321.
#define QF_U 4
#define QF_WAVES 4
#define QF_UNITS (QF_U * QF_WAVES * 64)      // units per work-group

struct QuantFam {
  MatDev m;
  uint32_t upr, magic;      // units per padded row, ceil(2^32 / upr)
  int interleave;           // source rows come in turn from w0 and w1
  const void* w0; const void* w1;
};
struct QuantArgs {
  QuantFam gu, dn;
  uint32_t nb_gu;           // work-groups of the gate/up family; the rest belong to down
  int e0, lanes, sc_bf16, symmetric;      // lanes = group / 8
};

// value of lane U of the quad, in all four of its lanes
template <int U> __device__ __forceinline__ float quad_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), U * 0x55, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ float dpp_min(float v) { return fminf(v, dpp_f32<CTRL>(v)); }
template <int CTRL> __device__ __forceinline__ float dpp_max(float v) { return fmaxf(v, dpp_f32<CTRL>(v)); }

// RN(a / s) for s in [2^-90, 2^90] and y = RN(1 / s): two residual corrections of a * y.  The first
// leaves a faithful quotient, the second then rounds correctly (Markstein's theorem: the residual of a
// faithful quotient is exact).  Quotients below 1/4 may come out inexact when their residual underflows; they
// round to code offset 0 all the same.
__device__ __forceinline__ float div_rn(float a, float s, float y) {
  const float q0 = a * y;
  const float q1 = fmaf(fmaf(-q0, s, a), y, q0);
  return fmaf(fmaf(-q1, s, a), y, q1);
}

template <int WDT, int BITS>
__global__ __launch_bounds__(QF_WAVES * 64) void quantize_flat_kernel(QuantArgs a) {
  const bool is_dn = blockIdx.x >= a.nb_gu;
  const QuantFam& F = is_dn ? a.dn : a.gu;
  const MatDev& m = F.m;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, el = blockIdx.y;
  const uint32_t b0 = (blockIdx.x - (is_dn ? a.nb_gu : 0u)) * QF_UNITS;
  const uint32_t row0 = b0 / F.upr, rem0 = b0 - row0 * F.upr;      // (uniform)
  const int L = a.lanes, K = m.K;
  const size_t e = (size_t)(a.e0 + el);
  constexpr float QMAX = (float)((1 << (2 * BITS)) - 1), HALF = (float)(1 << (2 * BITS - 1));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

  uint32_t row[QF_U], col[QF_U];
  bool live[QF_U];
  constexpr int NV = WDT == SMOE_F32 ? 2 : 1;      // 16-byte loads of a unit
  u32x4 raw[QF_U][NV];
#pragma unroll
  for (int u = 0; u < QF_U; u++) {
    const uint32_t v = rem0 + (wave * QF_U + u) * 64 + lane, q = __umulhi(v, F.magic);
    row[u] = row0 + q;
    col[u] = (v - q * F.upr) * 8;
    live[u] = row[u] < (uint32_t)m.N && col[u] < (uint32_t)K;      // (K is a multiple of 32: a unit is in or out as a whole)
    const uint32_t r = F.interleave ? row[u] >> 1 : row[u], n_src = F.interleave ? (uint32_t)m.N >> 1 : (uint32_t)m.N;
    const void* src = F.interleave && (row[u] & 1) ? F.w1 : F.w0;
    const size_t i0 = ((size_t)el * n_src + r) * (size_t)K + col[u];
    // (padding units fetch the matrix's first values and drop them: no branch, so all loads go out together)
    const uint8_t* p = (const uint8_t*)src + (live[u] ? i0 : 0) * (WDT == SMOE_F32 ? 4 : 2);
#pragma unroll
    for (int j = 0; j < NV; j++) raw[u][j] = *(const u32x4*)(p + 16 * j);
  }
#pragma unroll
  for (int u = 0; u < QF_U; u++)
#pragma unroll
    for (int j = 0; j < NV; j++)
#pragma unroll
      for (int i = 0; i < 4; i++) raw[u][j][i] = live[u] ? raw[u][j][i] : 0u;
  auto val = [&](int u, int i) __attribute__((always_inline)) {
    if (WDT == SMOE_F32) return __uint_as_float(raw[u][NV == 2 ? i >> 2 : 0][i & 3]);
    const uint32_t w = raw[u][0][i >> 1];
    return __uint_as_float((i & 1) ? w & 0xFFFF0000u : w << 16);
  };
  // ---- range of every unit's group (it always contains 0; padding units hold zeros)
  float mylo = 0.0f, myhi = 0.0f;      // of the unit this lane divides for
#pragma unroll
  for (int u = 0; u < QF_U; u++) {
    float lo = 0.0f, hi = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; i++) { const float v = val(u, i); lo = fminf(lo, v); hi = fmaxf(hi, v); }
    lo = dpp_min<0xB1>(lo); hi = dpp_max<0xB1>(hi);                              // quads
    lo = dpp_min<0x4E>(lo); hi = dpp_max<0x4E>(hi);
    if (L >= 8) { lo = dpp_min<0x141>(lo); hi = dpp_max<0x141>(hi); }           // row_half_mirror: eight lanes
    if (L >= 16) { lo = dpp_min<0x140>(lo); hi = dpp_max<0x140>(hi); }          // row_mirror: sixteen
    if (L >= 32) { lo = fminf(lo, __shfl_xor(lo, 16)); hi = fmaxf(hi, __shfl_xor(hi, 16)); }
    if (L >= 64) { lo = fminf(lo, __shfl_xor(lo, 32)); hi = fmaxf(hi, __shfl_xor(hi, 32)); }
    if ((lane & 3) == u) { mylo = lo; myhi = hi; }
  }
  // ---- scale, zero-point and reciprocal of the group of unit (lane & 3)
  // symmetric variant (Section 6.1 item 1: symmetric integer weights): step from the largest magnitude, the
  // zero-point fixed at mid-range of the unsigned store
  float ms = a.symmetric ? fmaxf(myhi, -mylo) / (HALF - 1.0f) : (myhi - mylo) / QMAX;
  if (a.sc_bf16) ms = bf16_bits_to_f32(f32_to_bf16_bits(ms));
  if (!(ms > 0.0f)) ms = 1.0f;
  const float mz = a.symmetric ? HALF : fminf(fmaxf(rintf((-mylo) / ms), 0.0f), QMAX);
  const float my = 1.0f / ms;
  const bool plain = ms >= 0x1p-90f && ms <= 0x1p90f;      // div_rn applies (an infinite range fails this, too)
  const bool all_plain = __ballot(plain) == ~0ull;
  // metadata: lane u of a group's first quad writes the group of unit u
#pragma unroll
  for (int u = 0; u < QF_U; u++) {
    if ((lane & (L - 1)) == u && row[u] < (uint32_t)m.N) {
      const uint32_t g = col[u] / 8 / (uint32_t)L;      // (L is a power of two)
      const_cast<uint8_t*>(m.zp)[e * m.zp_stride + (size_t)row[u] * m.ng + g] = (uint8_t)(int)mz;
      uint8_t* ps = const_cast<uint8_t*>(m.sc) + e * m.sc_stride;
      const size_t si = (size_t)row[u] * m.sng + g;
      if (a.sc_bf16) ((uint16_t*)ps)[si] = (uint16_t)f32_to_bf16_bits(ms);
      else ((float*)ps)[si] = ms;
    }
  }
  // ---- codes and planes
  auto unit = [&](auto uc, auto plain_c) __attribute__((always_inline)) {
    constexpr int u = decltype(uc)::value;
    const float s = quad_bcast<u>(ms), y = quad_bcast<u>(my);
    const int zp = (int)quad_bcast<u>(mz);
    uint32_t qe = 0, qo = 0;      // codes of the even / odd columns, one per byte
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const float v = val(u, i);
      const float d = decltype(plain_c)::value ? div_rn(v, s, y) : v / s;
      const uint32_t q = (uint32_t)min(max((int)rintf(d) + zp, 0), (int)QMAX);
      if (i & 1) qo |= q << (4 * (i - 1)); else qe |= q << (4 * i);
    }
    uint8_t* pm = const_cast<uint8_t*>(m.msb) + e * m.plane_stride;
    uint8_t* pl = const_cast<uint8_t*>(m.lsb) + e * m.plane_stride;
    const size_t at = (size_t)row[u] * (K * BITS / 8);
    if (BITS == 4) {
      // planes keep every nibble n as n - 8 in 4-bit two's complement (n ^ 8): signed 4-bit dot products
      // read them directly
      const uint32_t mw = (((qe >> 4) & 0x0F0F0F0Fu) | (qo & 0xF0F0F0F0u)) ^ 0x88888888u;      // floor(q/16): the low-bit code
      const uint32_t lw = ((qe & 0x0F0F0F0Fu) | ((qo & 0x0F0F0F0Fu) << 4)) ^ 0x88888888u;      // the bits truncation drops
      if (live[u]) { *(uint32_t*)(pm + at + (col[u] >> 1)) = mw; *(uint32_t*)(pl + at + (col[u] >> 1)) = lw; }
    } else if (BITS == 3) {
      // 6-bit codes, 12 bytes per 32 columns: column 8t + j has its two low bits in word t >> 1 at bits
      // 4j + 2(t & 1) and its third bit in word 2 at bit 4j + t.  Lane t of a quad holds columns 8t .. 8t + 7;
      // lanes 0 .. 2 store a word each.
      const int t = lane & 3;
      auto plane = [&](uint32_t n, uint8_t* p) __attribute__((always_inline)) {      // n: one three-bit value per nibble
        uint32_t lo = (n & 0x33333333u) << (2 * (t & 1)), hi = ((n >> 2) & 0x11111111u) << t;
        lo |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0xB1, 0xF, 0xF, true);      // words 0 (lanes 0, 1) and 1 (lanes 2, 3)
        hi |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0xB1, 0xF, 0xF, true);
        hi |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x4E, 0xF, 0xF, true);
        const uint32_t lo2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x4E, 0xF, 0xF, true);      // lane 1 gets word 1
        if (live[u] && t < 3) *(uint32_t*)(p + at + (size_t)(col[u] >> 5) * 12 + 4 * t) = t == 0 ? lo : t == 1 ? lo2 : hi;
      };
      plane(((qe >> 3) & 0x07070707u) | ((qo << 1) & 0x70707070u), pm);
      plane((qe & 0x07070707u) | ((qo & 0x07070707u) << 4), pl);
    } else {
      // 4-bit codes: upper two bits = the low-bit code; four codes per plane byte, column 4j in bits 0-1
      auto plane = [&](uint32_t n, uint8_t* p) __attribute__((always_inline)) {      // n: one two-bit value per nibble
        n = (n | (n >> 2)) & 0x0F0F0F0Fu;
        n = (n | (n >> 4)) & 0x00FF00FFu;
        n |= n >> 8;
        if (live[u]) *(uint16_t*)(p + at + (col[u] >> 2)) = (uint16_t)n;
      };
      plane(((qe >> 2) & 0x03030303u) | ((qo << 2) & 0x30303030u), pm);
      plane((qe & 0x03030303u) | ((qo & 0x03030303u) << 4), pl);
    }
  };
  auto units = [&](auto plain_c) __attribute__((always_inline)) {
    unit(std::integral_constant<int, 0>(), plain_c); unit(std::integral_constant<int, 1>(), plain_c);
    unit(std::integral_constant<int, 2>(), plain_c); unit(std::integral_constant<int, 3>(), plain_c);
  };
  static_assert(QF_U == 4, "one unit per lane of a quad");
  if (all_plain) units(std::true_type());
  else units(std::false_type());
}

// The flat kernel takes power-of-two groups of up to 64 lanes, and matrices whose unit numbers and
// remainders the 32-bit arithmetic covers (row widths up to some 500 000 columns).
static bool quant_fam(const MatDev& m, int lanes, const void* w0, const void* w1, int interleave, QuantFam& f, uint32_t& blocks) {
  const uint64_t upr = (uint64_t)m.ng * lanes, units = upr * (uint64_t)m.N;
  if (upr * (upr + QF_UNITS) >= ((uint64_t)1 << 32) || units + QF_UNITS >= ((uint64_t)1 << 32)) return false;
  f.m = m; f.upr = (uint32_t)upr; f.interleave = interleave; f.w0 = w0; f.w1 = w1;
  f.magic = (uint32_t)((((uint64_t)1 << 32) + upr - 1) / upr);
  blocks = (uint32_t)((units + QF_UNITS - 1) / QF_UNITS);
  return true;
}

template <int WDT>
static void launch_flat(int bits, dim3 grid, hipStream_t st, const QuantArgs& q) {
  const dim3 blk(QF_WAVES * 64);
  if (bits == 4) quantize_flat_kernel<WDT, 4><<<grid, blk, 0, st>>>(q);
  else if (bits == 3) quantize_flat_kernel<WDT, 3><<<grid, blk, 0, st>>>(q);
  else quantize_flat_kernel<WDT, 2><<<grid, blk, 0, st>>>(q);
}

int smoe_launch_quantize(smoe_ctx* ctx, smoe_bank* bank, int e0, int n, const void* wg, const void* wu, const void* wd) {
  const BankDev& b = bank->dev;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  const int G = b.group;
  if (G <= 512 && (G & (G - 1)) == 0) {
    QuantArgs q{};
    q.e0 = e0; q.lanes = G / 8; q.sc_bf16 = b.sc_bf16; q.symmetric = bank->desc.symmetric;
    uint32_t nb_dn = 0;
    if (quant_fam(b.gu, q.lanes, wg, wu, 1, q.gu, q.nb_gu) && quant_fam(b.dn, q.lanes, wd, nullptr, 0, q.dn, nb_dn)) {
      const dim3 grid(q.nb_gu + nb_dn, n);
      if (bank->desc.w_dtype == SMOE_F32) launch_flat<SMOE_F32>(b.bits, grid, ctx->stream, q);
      else launch_flat<SMOE_BF16>(b.bits, grid, ctx->stream, q);
      HIPCHK(ctx, hipGetLastError());
      return SMOE_OK;
    }
  }
  dim3 blk(256);
  if (bank->desc.w_dtype == SMOE_F32) {
    quantize_rows_kernel<SMOE_F32><<<dim3(b.gu.N, n), blk, 0, ctx->stream>>>(wg, wu, b.gu, e0, b.group, b.sc_bf16, 1, bank->desc.symmetric);
    quantize_rows_kernel<SMOE_F32><<<dim3(b.dn.N, n), blk, 0, ctx->stream>>>(wd, nullptr, b.dn, e0, b.group, b.sc_bf16, 0, bank->desc.symmetric);
  } else {
    quantize_rows_kernel<SMOE_BF16><<<dim3(b.gu.N, n), blk, 0, ctx->stream>>>(wg, wu, b.gu, e0, b.group, b.sc_bf16, 1, bank->desc.symmetric);
    quantize_rows_kernel<SMOE_BF16><<<dim3(b.dn.N, n), blk, 0, ctx->stream>>>(wd, nullptr, b.dn, e0, b.group, b.sc_bf16, 0, bank->desc.symmetric);
  }
  HIPCHK(ctx, hipGetLastError());
  return SMOE_OK;
}
