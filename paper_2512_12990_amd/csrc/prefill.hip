// Prefill (paper Section 4.3: token-parallel, every expert high-bit, per-expert access counts):
//   route        router mat-vec, top-k (route.hip)
//   group        one work-group per expert: histogram, stable list of the expert's (token, slot) pairs; gate
//                weights of the shared experts
//   gemm<0>      grouped GEMM  H = silu(X Wg^T) * (X Wu^T)     (bf16 MFMA, fp32 accumulate)
//   gemm<1>      grouped GEMM  O = w * (H Wd^T)
//   combine      Y[t] = sum over slots (slot order) O[(t, slot)]  (+ x)
// Weights are read from the same nibble planes the decode path uses and expanded to
// bf16 s*(16 msb + lsb - zp) in the registers of the wave that multiplies them.
#include "route_device.hpp"
#include <type_traits>
#include <algorithm>
#include <math.h>

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define PF_BK 64
// waves of a GEMM work-group (32 weight rows each) by the fragments of its tile
static constexpr int pf_waves(int nf) { return nf > 5 ? 8 : 4; }

// ------------------------------------------------------------------------------- small kernels
#define GR_THREADS 1024
// gamma[t] = sigmoid(w_sg . x[t]), or 1 without a gate vector: the weight of the shared experts' output for
// token t.  One wave per token.
__device__ __forceinline__ void shared_gate_token(const uint16_t* x, const uint16_t* w_sg, int t, int d, float* gamma, int lane) {
  float g = 1.0f;
  if (w_sg) {
    // 32 columns per lane are fetched into raw registers before the first is used (arithmetic on a
    // loaded value at the load site would make the wave wait for every load in turn)
    const uint16_t* xr = x + (size_t)t * d;
    float s = 0.0f;
    for (int i0 = 0; i0 < d; i0 += 2048) {
      uint32_t wv[32], xv[32];
#pragma unroll
      for (int u = 0; u < 32; u++) {
        const int i = min(i0 + u * 64 + lane, d - 1);
        wv[u] = w_sg[i];
        xv[u] = xr[i];
      }
#pragma unroll
      for (int u = 0; u < 32; u++) {
        const float q = fmaf(__uint_as_float(wv[u] << 16), __uint_as_float(xv[u] << 16), s);
        s = (i0 + u * 64 + lane) < d ? q : s;
      }
    }
    s = wave_sum(s);
    g = 1.0f / (1.0f + __expf(-s));
  }
  if (lane == 0) gamma[t] = g;
}

// Work-groups below E, one per expert e, group the (token, slot) pairs by expert; no atomics and no ordering between
// work-groups: each thread counts, over a contiguous run of pairs, those of e and those of the experts before e.
//   hist[e]    number of pairs routed to e (the per-expert access count of the layer)
//   rows[p]    flat (token*k + slot) index of the p-th row of the grouped layout (expert after expert), ascending
//              inside an expert; pos = inverse of rows.
// The work-groups from E on make the weights of the shared experts, 16 tokens each (nothing connects the two; one launch
// less).  16384 pairs, 60 experts and the gates of 4096 tokens: 8 us, against 17 + 6 for two launches, the pairs counted by
// LDS atomics; 8192 pairs alone: 7.5 -> 5 us.
__global__ __launch_bounds__(GR_THREADS) void group_kernel(const int32_t* idx, int n, int E, uint32_t* hist, int32_t* rows, int32_t* pos,
                                                           const uint16_t* x, const uint16_t* w_sg, int T, int d, float* gamma) {
  __shared__ int wtot[GR_THREADS / 64], wbef[GR_THREADS / 64];
  const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (e >= E) {
    const int t = (e - E) * (GR_THREADS / 64) + wave;
    if (t < T) shared_gate_token(x, w_sg, t, d, gamma, lane);
    return;
  }
  // every thread owns a contiguous run of c pairs, c a multiple of four (16-byte loads: idx is 16-byte aligned); runs of up to GR_RUN pairs
  // are fetched into registers before the first is used (all loads in flight at once) and serve both passes
  const int c = ((n + GR_THREADS - 1) / GR_THREADS + 3) & ~3;
  const int i0 = min(n, tid * c), i1 = min(n, i0 + c);
  constexpr int GR_RUN = 16;
  int v[GR_RUN];
  const bool in_regs = c <= GR_RUN;
  int mine = 0, before = 0;
  if (in_regs) {
#pragma unroll
    for (int u = 0; u < GR_RUN; u += 4) {
      int4 q = make_int4(-1, -1, -1, -1);
      if (i0 + u + 4 <= i1) q = *(const int4*)(idx + i0 + u);
      else {
        if (i0 + u < i1) q.x = idx[i0 + u];
        if (i0 + u + 1 < i1) q.y = idx[i0 + u + 1];
        if (i0 + u + 2 < i1) q.z = idx[i0 + u + 2];
      }
      v[u] = q.x; v[u + 1] = q.y; v[u + 2] = q.z; v[u + 3] = q.w;
    }
#pragma unroll
    for (int u = 0; u < GR_RUN; u++) { mine += v[u] == e; before += (unsigned)v[u] < (unsigned)e; }
  } else {
    for (int i = i0; i < i1; i++) { const int w = idx[i]; mine += w == e; before += (unsigned)w < (unsigned)e; }
  }
  int incl = mine;
  for (int s = 1; s < 64; s <<= 1) { const int o = __shfl_up(incl, s); if (lane >= s) incl += o; }
  for (int m = 32; m >= 1; m >>= 1) before += __shfl_xor(before, m);
  if (lane == 63) { wtot[wave] = incl; wbef[wave] = before; }
  __syncthreads();
  int p = incl - mine, ne = 0;
#pragma unroll
  for (int w = 0; w < GR_THREADS / 64; w++) {
    const int t = wtot[w];
    p += wbef[w] + (w < wave ? t : 0);
    ne += t;
  }
  if (in_regs) {
#pragma unroll
    for (int u = 0; u < GR_RUN; u++)
      if (v[u] == e) { rows[p] = i0 + u; pos[i0 + u] = p; p++; }
  } else {
    for (int i = i0; i < i1; i++)
      if (idx[i] == e) { rows[p] = i; pos[i] = p; p++; }
  }
  if (tid == 0) hist[e] = (uint32_t)ne;
}

// Inclusive prefix sum over the lanes of a wave.
template <int CTRL, int ROWM> __device__ __forceinline__ int dpp_add_i32(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWM, 0xF, true);
}
__device__ __forceinline__ int wave_scan(int v) {
  v = dpp_add_i32<0x111, 0xF>(v);      // row_shr 1
  v = dpp_add_i32<0x112, 0xF>(v);      // row_shr 2
  v = dpp_add_i32<0x114, 0xF>(v);      // row_shr 4
  v = dpp_add_i32<0x118, 0xF>(v);      // row_shr 8: every row of 16 lanes scanned
  v = dpp_add_i32<0x142, 0xA>(v);      // row_bcast 15 into rows 1 and 3
  v = dpp_add_i32<0x143, 0xC>(v);      // row_bcast 31 into rows 2 and 3
  return v;
}

// ------------------------------------------------------------------------------- grouped GEMM
struct GemmArgs {
  MatDev w;                 // gu (MODE 0) or dn (MODE 1) family of the bank
  int group_shift;          // quantisation group = 1 << group_shift columns
  int E, k, d_model, d_ff;
  int n_col_tiles;          // column tiles of this GEMM
  int super;                // row tiles that share a column tile before the next column tile starts (see smoe_prefill_histogram)
  const uint32_t* hist;     // [E] rows of an expert (written by group_kernel, like rows)
  const int32_t* rows;      // [T*k]
  const uint16_t* x;        // MODE 0: X [T, d_model] bf16
  uint16_t* h;              // H [T*k, d_ff] bf16 (MODE 0 output, MODE 1 input)
  float* o;                 // MODE 1 output [T*k, d_model] fp32
  const float* wgt;         // [T*k] gate weights (flat token*k + slot)
  // dense_rows > 0: the n_dense experts from dense_expert on (shared experts) take every token: rows are
  // the tokens in their own order, no tile list, no row list; wgt[t] scales row t.  H of the first of
  // them is h, of the others h_more ([n_dense - 1, dense_rows, d_ff]); MODE 1 sums over the experts
  int dense_rows, dense_expert, n_dense;
  uint16_t* h_more;
  uint32_t a_bytes;         // bytes of X (MODE 0) / of one H buffer (MODE 1)
  int accumulate;           // MODE 1: add to O instead of overwriting it
};
// one launch serves two sets of experts: work-groups below nb0 belong to g[0] (nb0 is a multiple of 8)
// (zp_at, wave_lds: where a wave's zero-points start in its LDS area, and the area's size, by the smallest group of the two)
struct GemmPair { GemmArgs g[2]; int nb0, zp_at, wave_lds; };

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);
  return *(uint32_t*)&r;
}

__device__ __forceinline__ u32x4 pf_rsrc(const void* base, uint32_t bytes) {
  const uint64_t v = (uint64_t)base;
  return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v), (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) & 0xFFFFu,
               (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}
// 64 lanes x 16 bytes from memory straight into LDS: lane i's bytes land at lds + 16 i.  The LDS address is an operand in M0, so
// the compiler writes that register and knows its contents (one wait state between the write and the load).  It does not count
// these loads: see the K loop for what orders them.
__device__ __forceinline__ void dma16(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds)
               : "memory");
}

// the same by the wave's first 32 lanes (all 64 are active around it)
__device__ __forceinline__ void dma16_half(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 exec_hi, 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds\n\ts_mov_b32 exec_hi, -1" ::"v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds)
               : "memory");
}

// the same for one dword / one byte (zero-extended) per lane: lane i's dword lands at lds + 4 i
__device__ __forceinline__ void dma4(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_nop 0\n\tbuffer_load_dword %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds)
               : "memory");
}
__device__ __forceinline__ void dma1(u32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_nop 0\n\tbuffer_load_ubyte %0, %1, %2 offen lds" ::"v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds)
               : "memory");
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// LDS of a GEMM work-group: row buffers (one 64-column step each), the waves' weight areas.  A step of a short tile is over before its token
// rows have come from L2, so those are sent for up to four steps ahead: as many buffers as fit beside two work-groups per CU (one with
// eight waves, where a tile of fewer fragments has more buffers).  32 and 64 rows with two, later four buffers: 173 tokens through 64
// experts 173.5 -> 166.6 us per layer.  (There the waves' areas are also cut to the groups at hand; elsewhere their size is fixed.)
// 96 rows of the 4/2 nest, whose planes are small: two buffers, which leave room for a third work-group.  70 experts of d_model 2048, d_ff 384, groups
// of 32, 1718 tokens, popularity even / 1/rank^1.1: 101.6 / 127.6 -> 97.0 / 116.6 us; 45 layers of 55 - 95 rows per expert 2 - 3 % faster.
template <int SCB, int FMT, int NF> struct PfLds {
  static constexpr int NW = pf_waves(NF), ROWS = NF == 8 ? 81920 : NF == 5 ? 40960 : NF == 3 ? (FMT == 1 ? 24576 : 36864) : NF * 16384, PLANE = FMT == 0 ? 4096 : FMT == 1 ? 2048 : 3072;
  static constexpr int nbuf(int f) { return ROWS / (f * 4096) < 4 ? ROWS / (f * 4096) : 4; }      // buffers of a tile of f fragments
  static constexpr bool FIT = NF <= 2;
  static constexpr int ZP_AT = 2 * PLANE + (SCB ? 4 : 8) * 128, WAVE = ZP_AT + 8 * 128;      // two planes, scale dwords, zero-points of 32 rows and 256 columns in groups of 32
};

// One expert's 32 * NF token rows times 32 weight rows per wave, four or (NF = 8) eight waves.  A wave owns all the token rows and 32 of
// the weight rows; it expands its weights to bf16 in registers -- lane (n, h) holds columns 32 h .. 32 h + 31 of one
// row of a K step (64 columns), and MFMA s of the step contracts columns {8 s ..} and {32 + 8 s ..} on both operands --
// so every weight is expanded once per tile and LDS carries bf16 only for the token rows.  All memory reaches LDS
// by direct loads: token rows into a ring of step buffers; planes, scales and zero-points 256 columns (a
// whole 128-byte line of a nibble plane) at a time into an area of the wave's own, fetched while the previous 256
// columns, by then in registers, are multiplied.
// Bound: with few rows per expert the weights' bytes.  With many, a step is a stream of 200 - 260 instructions per wave (4 F products of 32
// cycles, 107 vector instructions of expansion, 4 F LDS reads of 1 KB), two waves per SIMD.  Time stamps in the kernel (60 experts of
// d_model 2048, d_ff 1408, 137 rows) showed what a step cost beyond that, and the loop is built around it: 28 % of it went into sending
// direct loads and fetching planes in one go at the head of a step (now one load behind a product, 35 - 70 cycles each), 22 % into waiting for
// rows, the rest into products and expansion running one after the other in both waves that left a barrier together (now a fifth of the
// expansion and a read behind every product, pinned there: the compiler sinks the work otherwise).  No load depends on a condition: past the
// last step the range is empty, the load counts all the same, and every wait is a constant.  Cycles per step, two work-groups of four
// waves: 1865 before, 1708 now (mean of 3 to 5 fragments); eight waves: 1785 at 4 fragments, 2657 at 8, i.e. 446 and 332 per fragment -- a weight is
// expanded for more rows.  Of those 2657 the products are 2048, the barrier 400.  Taller tiles take more of a CU at
// once; where that leaves the chip unfilled the shorter ones are faster (pick_nf).  A layer of 2048 / 4096 tokens (60 experts of d_ff 1408,
// the longer one with a shared expert of 5632): 291 -> 250 - 268 / 806 -> 697 - 714 us.  Registers: the tall gate/up kernel of the 8/4 nest with bf16
// scales is at 256 and keeps five in scratch, stored before the loops and fetched after them; the down kernels keep up to 109 scalars in vector lanes.  Not kept: eight waves and 160 rows (287 / 786 us), eight-wave
// work-groups that stay and take a list of tiles, the next one's weights sent for before the epilogue (286 / 798 us against 270 / 747).
// Earlier shapes, gate/up GEMM of 60 experts at 137 rows each / of 64 such experts at 16 rows: planes loaded straight into the lanes that use
// them, every lane of a load in another cache line, 215 / 183 us; 128 columns at a time through LDS, half a line, 165 / 123 us; a whole line
// and 32 instead of 64 weight rows per wave 149 / 94 us.
template <int MODE, int SCB, int FMT, int NF>      // FMT 0: 8/4 nest, nibble planes; 1: 4/2 nest, 2-bit planes; 2: 6/3 nest, 3-bit planes
__global__ __launch_bounds__(64 * pf_waves(NF), NF == 1 ? 3 : 2) void grouped_gemm_kernel(GemmPair pair) {
  constexpr int BM = 32 * NF;
  constexpr int PB32 = FMT == 0 ? 16 : FMT == 1 ? 8 : 12;      // plane bytes of 32 columns
  constexpr int PROW = 8 * PB32, PPR = PROW / 16, NPL = 32 * PROW / 1024;      // of a row and 256 columns; 16-byte pieces of that; loads per plane
  constexpr int PLANE = 32 * PROW;                             // bytes of one plane in a wave's area: MSB plane, LSB plane, scales, zero-points
  typedef PfLds<SCB, FMT, NF> Lds;
  constexpr int NW = Lds::NW, BN = 32 * NW;
  extern __shared__ __align__(1024) uint8_t As[];              // NBUF K steps of the token rows, 128 bytes per row; the waves' areas
  const int ZP_AT = Lds::FIT ? pair.zp_at : Lds::ZP_AT;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const bool second = (int)blockIdx.x >= pair.nb0;
  const GemmArgs& a = pair.g[second ? 1 : 0];
  const int bid = (int)blockIdx.x - (second ? pair.nb0 : 0);

  // ---- which tile.  The (row tile, column tile) items are listed in bands of a.super row tiles, column by
  // column inside a band, and the list is cut into eight equal runs, one per XCD (work-groups go to the
  // XCDs round-robin), so that the work-groups that share weight rows or token rows run side by side on one L2.
  int e_base = 0, e_cnt = 0, e_first = 0, e = 0, n_tiles;
  const int rt = a.dense_rows ? (a.dense_rows + BM - 1) / BM : 0;
  int tstart[4], toff[4], tcnt[4];      // experts lane, lane + 64, ...: first tile, first row, rows
  if (!a.dense_rows) {
    int tbase = 0, rbase = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int x = lane + 64 * j;
      tcnt[j] = x < a.E ? (int)a.hist[x] : 0;
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int x = lane + 64 * j;
      tstart[j] = 0x7FFFFFFF; toff[j] = 0;
      if (64 * j < a.E) {                               // (wave-uniform)
        const int tl = (tcnt[j] + BM - 1) / BM, ts = wave_scan(tl), rs = wave_scan(tcnt[j]);
        if (x < a.E) tstart[j] = tbase + ts - tl;
        toff[j] = rbase + rs - tcnt[j];
        tbase += __builtin_amdgcn_readlane(ts, 63);
        rbase += __builtin_amdgcn_readlane(rs, 63);
      }
    }
    n_tiles = tbase;
  } else {
    n_tiles = MODE == 0 ? rt * a.n_dense : rt;
  }
  const int n_items = n_tiles * a.n_col_tiles, run = (n_items + 7) >> 3;
  const int slot = bid >> 3, item = (bid & 7) * run + slot;
  if (slot >= run || item >= n_items) return;
  const int band = uni(item / (a.super * a.n_col_tiles)), in_band = item - band * a.super * a.n_col_tiles;
  const int band_rows = min(a.super, n_tiles - band * a.super);
  const int nt = uni(in_band / band_rows), ti = band * a.super + in_band - nt * band_rows;
  int row0;                                             // first row of the expert in the grouped layout
  uint16_t* h = a.h;
  if (a.dense_rows) {
    const int ex = MODE == 0 ? uni(ti / rt) : 0;
    e = a.dense_expert + ex; e_first = ex * rt; e_cnt = a.dense_rows; row0 = 0;
    if (ex > 0) h = a.h_more + (size_t)(ex - 1) * a.dense_rows * a.d_ff;
  } else {
    // the last expert whose first tile is not past ti
    int c = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) c += (int)__builtin_popcountll(__ballot(tstart[j] <= ti));
    e = uni(c - 1);
    const int jl = e >> 6, l = e & 63;
#pragma unroll
    for (int j = 0; j < 4; j++)
      if (j == jl) {
        e_first = __builtin_amdgcn_readlane(tstart[j], l);
        e_base = __builtin_amdgcn_readlane(toff[j], l);
        e_cnt = __builtin_amdgcn_readlane(tcnt[j], l);
      }
    row0 = e_base;
  }
  // an expert's rows are dealt to its tiles in whole fragments, as evenly as those go
  const int e_tiles = (e_cnt + BM - 1) / BM, tile_rows = 32 * uni(((e_cnt + 31) / 32 + e_tiles - 1) / e_tiles);
  const int m0 = uni((ti - e_first) * tile_rows), m_cnt = uni(min(tile_rows, e_cnt - m0));
  if (m_cnt <= 0) return;                               // (fewer fragments than tiles cannot be: kept as a guard)

  const int K = MODE == 0 ? a.d_model : a.d_ff;
  const int N = MODE == 0 ? a.d_ff : a.d_model;         // output columns of this GEMM
  const int nk = K / PF_BK;
  const int nf = (m_cnt + 31) >> 5;
  const int n = lane & 31, hh = lane >> 5;

  // ---- the wave's 32 weight rows.  MODE 0: gate and up rows alternate in the bank, so they are the gate and up rows
  // of 16 output columns; lanes 0 .. 15 take the gate rows, lanes 16 .. 31 the up rows.  Rows past the matrix read
  // out of the section's range.
  const uint32_t wrow = (uint32_t)(nt * BN + wave * 32);
  const uint32_t rowb = (uint32_t)(K >> 5) * PB32;
  const int sh = a.group_shift;
  const int n_grp = sh >= 8 ? 1 : 256 >> sh;                   // groups of 256 columns
  // plane loads: lane i's 16 bytes land at 16 i, row after row of PROW bytes; the nibble planes' eight pieces of a row
  // are stored permuted (piece p at p ^ (row / 2 % 8)), so that the operand reads hit all banks
  constexpr int NPO = FMT == 0 ? 2 : FMT == 1 ? 1 : NPL;       // load q: p_off[q % NPO], PSTEP rows further down for every NPO loads
  constexpr int PSTEP = NPO * 64 / PPR;
  uint32_t p_off[NPO];
#pragma unroll
  for (int q = 0; q < NPO; q++) {
    const uint32_t i = q * 64 + lane, r = i / PPR, c = i % PPR;
    p_off[q] = (wrow + r) * rowb + (FMT == 0 ? c ^ ((r >> 1) & 7u) : c) * 16;
  }
  // scales and zero-points: lanes 0 .. 31 fetch the first of two dwords / groups of their row, lanes 32 .. 63 the second
  // (a row holds an even number of scales, so a pair of bf16 scales is one aligned dword)
  const uint32_t s_off = (wrow + n) * (uint32_t)a.w.sng * (SCB ? 2u : 4u) + hh * 4u, z_off = (wrow + n) * (uint32_t)a.w.ng + hh;
  const uint32_t as_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)As;
  const uint32_t wofs = Lds::ROWS + (uint32_t)wave * (uint32_t)(Lds::FIT ? pair.wave_lds : Lds::WAVE);
  const uint8_t* warea = As + wofs;
  const uint32_t wr = MODE == 0 ? 2 * (n & 15) + (n >> 4) : n;                 // the lane's row of the 32
  const uint32_t p_rd = wr * PROW + (FMT == 0 ? ((uint32_t)hh ^ ((wr >> 1) & 7u)) * 16 : (uint32_t)hh * PB32);
  typedef typename std::conditional<FMT == 0, u32x4, typename std::conditional<FMT == 1, u32x2, u32x3>::type>::type PlaneV;
  struct Planes { PlaneV m, l; };
  struct Meta { uint32_t s, z; };
  const uint32_t hb = sh == 5 ? hh : 0, odd_group = sh == 5 ? 0u : 1u;
  const uint32_t s_rd = 2 * PLANE + wr * 4 + (SCB ? 0u : hb * 128u), z_rd = ZP_AT + wr * 4 + hb * 128u;

  f32x16 acc[NF];
#pragma unroll
  for (int i = 0; i < NF; i++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[i][r] = 0.0f;

  // where an expert's planes, scales and zero-points are, in scalar registers (fetched from the arguments in the K loop they would make
  // the wave wait for its LDS reads too)
  struct Bases { const uint8_t *m, *l, *s, *z; uint32_t p_bytes, s_bytes, z_bytes; };
  auto bases_of = [&](int ex) __attribute__((always_inline)) {
    const size_t ee = (size_t)uni(e + ex);
    Bases q{a.w.msb + ee * a.w.plane_stride, a.w.lsb + ee * a.w.plane_stride, a.w.sc + ee * a.w.sc_stride, a.w.zp + ee * a.w.zp_stride,
            (uint32_t)a.w.plane_stride, (uint32_t)a.w.sc_stride, (uint32_t)a.w.zp_stride};
    asm volatile("" : "+s"(q.m), "+s"(q.l), "+s"(q.s), "+s"(q.z), "+s"(q.p_bytes), "+s"(q.s_bytes), "+s"(q.z_bytes));
    return q;
  };
  // planes, scales and zero-points of columns 256 i .. 256 i + 255 (past the row's end: bytes of the next row, not used)
  auto load_meta = [&](const Bases& w, int i) __attribute__((always_inline)) {
    const u32x4 rs = pf_rsrc(w.s, w.s_bytes), rz = pf_rsrc(w.z, w.z_bytes);
    const uint32_t g0 = (uint32_t)(i * 256) >> sh, lds = as_base + wofs;
    const int nsd = SCB ? (n_grp + 1) >> 1 : n_grp;
    for (int j = 0; j < nsd; j += 2) dma4(rs, s_off, (SCB ? (g0 >> 1) : g0) * 4u + j * 4u, lds + 2 * PLANE + j * 128u);
    for (int j = 0; j < n_grp; j += 2) dma1(rz, z_off, g0 + j, lds + ZP_AT + j * 128u);
  };
  // (direct loads u0 .. u1 - 1 of the 2 NPL that fetch both planes; range 0: nothing is fetched)
  auto load_plane = [&](const Bases& w, int i, int u0, int u1, uint32_t range) __attribute__((always_inline)) {
    const uint32_t lds = as_base + wofs;
#pragma unroll
    for (int u = u0; u < u1; u++) {
      const int q = u >> 1;
      const u32x4 r = pf_rsrc((u & 1) ? w.l : w.m, range);
      dma16(r, p_off[q % NPO], (uint32_t)i * PROW + (uint32_t)(q / NPO) * PSTEP * rowb, lds + (u & 1) * PLANE + q * 1024u);
    }
  };
  Bases wb = bases_of(0);
  load_meta(wb, 0);                                      // on their way while the token rows are looked up
  load_plane(wb, 0, 0, 2 * NPL, wb.p_bytes);

  // ---- token rows: a wave's direct load q moves rows 8 (NW q + wave) .. + 7 of the tile, lane i the 16-byte
  // piece (i % 8) ^ (r / 2 % 8) of row r = i / 8 (of these eight): sixteen lanes of an operand read, sixteen rows of one piece, then fall into
  // the sixteen 16-byte slots of the LDS's 64 banks (with r % 8 rows r and r + 8 collide: half of all LDS
  // cycles were conflicts; 2048 / 4096 tokens 270 -> 267 / 721 -> 716 us per layer).
  // MODE 0 gathers the rows of X (a row past the tile's last one repeats that row); MODE 1 reads consecutive
  // rows of H (past the last one: another tile's, or zeros from out of range).  Rows of the product are
  // independent and the epilogue stores none of the surplus ones.
  // (eight waves and an odd number of fragments: the last load is half a load of every wave, rows 4 wave .. of the last fragment)
  constexpr int NA = MODE == 0 ? 4 * NF / NW : 1;
  uint32_t a_off[NA], a_half = 0;
  auto row_at = [&](int r) __attribute__((always_inline)) {
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    uint32_t src;
    if (MODE == 0) {
      const int rc = m0 + min(r, m_cnt - 1);
      src = (uint32_t)(a.dense_rows ? rc : a.rows[row0 + rc] / a.k) * (uint32_t)a.d_model;
    } else {
      src = (uint32_t)(row0 + m0 + r) * (uint32_t)a.d_ff;
    }
    return src * 2u + c * 16;
  };
#pragma unroll
  for (int q = 0; q < NA; q++) a_off[q] = row_at((NW * q + wave) * 8 + (lane >> 3));
  if (NW == 8 && (nf & 1)) a_half = row_at(32 * (nf - 1) + 4 * wave + ((lane >> 3) & 3));
  // operand reads: lane (n, hh) takes columns 32 hh + 8 s .. + 7 of row n: piece (4 hh + s) ^ (n / 2 % 8)
  const uint32_t a_rd = n * 128 + (((4 * hh) ^ ((n >> 1) & 7)) * 16);
  // MODE 1: the weight of row tid of the tile, for the epilogue
  float my_wt = 0.0f;
  if (MODE == 1 && tid < m_cnt) my_wt = a.wgt[a.dense_rows ? m0 + tid : a.rows[row0 + m0 + tid]];

  // codes of columns 8 s .. 8 s + 7 of the lane's 32 -> bf16 scale (q - zp).  With bf16 scales the K loop takes the codes as 1024 + q
  // (BIASED) and c0 = -(1024 + zp) scale; otherwise c0 = -zp scale.
  constexpr bool BIASED = SCB != 0;
  // codes of the even / odd columns, one per byte
  auto codes = [&](const PlaneV& m, const PlaneV& l, int s, uint32_t& qe, uint32_t& qo) __attribute__((always_inline)) {
    if constexpr (FMT == 0) {
      // (the planes hold n ^ 8 per nibble: taken back below)
      const uint32_t wm = m[s], wl = l[s];
      qe = ((wm << 4) & 0xF0F0F0F0u) | (wl & 0x0F0F0F0Fu);
      qo = (wm & 0xF0F0F0F0u) | ((wl >> 4) & 0x0F0F0F0Fu);
    } else if constexpr (FMT == 2) {
      // column 8s + i: two low bits in word s >> 1 at bits 4i + 2(s & 1), third bit in word 2 at bit
      // 4i + s; one value per nibble first, then code = 8 msb + lsb, one per byte
      auto nib = [&](const PlaneV& w) {
        const uint32_t lo = (w[s >> 1] >> (2 * (s & 1))) & 0x33333333u;
        const uint32_t hi = w[2] & (0x11111111u << s);
        return lo | (s < 2 ? hi << (2 - s) : hi >> (s - 2));
      };
      const uint32_t nm = nib(m), nl = nib(l);
      qe = ((nm & 0x0F0F0F0Fu) << 3) | (nl & 0x0F0F0F0Fu);
      qo = (((nm >> 4) & 0x0F0F0F0Fu) << 3) | ((nl >> 4) & 0x0F0F0F0Fu);
    } else {
      // sixteen 2-bit codes per plane word, column c in bits 2c, 2c+1: spread half a word to one
      // code per nibble, then code = 4 msb + lsb
      auto spread = [](uint32_t v) {
        v = (v | (v << 8)) & 0x00FF00FFu;
        v = (v | (v << 4)) & 0x0F0F0F0Fu;
        return (v | (v << 2)) & 0x33333333u;
      };
      const uint32_t hm = (m[s >> 1] >> (16 * (s & 1))) & 0xFFFFu, hl = (l[s >> 1] >> (16 * (s & 1))) & 0xFFFFu;
      const uint32_t qn = (spread(hm) << 2) | spread(hl);
      qe = qn & 0x0F0F0F0Fu;
      qo = (qn >> 4) & 0x0F0F0F0Fu;
    }
  };
  // weights of columns 2 b and 2 b + 1 of the eight
  auto weights = [&](auto biased_c, uint32_t qe, uint32_t qo, int b, float scale, float c0) __attribute__((always_inline)) {
    if constexpr (decltype(biased_c)::value) {
      // the codes of two columns as the halves 1024 + q (exact in fp16), which one mixed-precision FMA each turns
      // into s (1024 + q) - s (1024 + zp); a bf16 scale times 11 bits is exact in fp32, so this is s (q - zp) rounded once
      const f16x2 q2 = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(qo, qe, 0x0C000C00u | ((4u + b) << 16) | b) ^ (FMT == 0 ? 0x64886488u : 0x64006400u));
      return pack_bf16(fmaf((float)q2[0], scale, c0), fmaf((float)q2[1], scale, c0));
    } else {
      const uint32_t f = FMT == 0 ? 0x88888888u : 0u;
      const float we = fmaf((float)(((qe ^ f) >> (8 * b)) & 0xFF), scale, c0);
      const float wo = fmaf((float)(((qo ^ f) >> (8 * b)) & 0xFF), scale, c0);
      return pack_bf16(we, wo);
    }
  };
  auto expand = [&](auto biased_c, const PlaneV& m, const PlaneV& l, int s, float scale, float c0) __attribute__((always_inline)) {
    uint32_t qe, qo;
    codes(m, l, s, qe, qo);
    u32x4 out;
#pragma unroll
    for (int b = 0; b < 4; b++) out[b] = weights(biased_c, qe, qo, b, scale, c0);
    return __builtin_bit_cast(bf16x8, out);
  };
  const int n_pass = MODE == 1 && a.dense_rows ? a.n_dense : 1;
  const std::integral_constant<bool, BIASED> biased{};
  auto kloop = [&](auto nf_c) __attribute__((always_inline)) {
    constexpr int F = decltype(nf_c)::value;
    constexpr int NBUF = Lds::nbuf(F), STEP = F * 4096;      // row buffers, bytes of one
    constexpr int RF = 4 * F / NW, RQ = RF + ((4 * F) % NW != 0);      // row loads of a step and wave (the last may be half a load)
    for (int ex = 0; ex < n_pass; ex++) {
      if (ex) __syncthreads();                          // every wave is done with the LDS rows of the last pass
      const u32x4 ra = pf_rsrc(MODE == 0 ? a.x : ex == 0 ? h : a.h_more + (size_t)(ex - 1) * a.dense_rows * a.d_ff, a.a_bytes);
      auto load_rows = [&](int t, uint32_t buf, int q0, int q1) __attribute__((always_inline)) {
        u32x4 r = ra;
        r[2] = t < nk ? ra[2] : 0u;                     // past the last step nothing is fetched, but the load counts
#pragma unroll
        for (int q = q0; q < q1; q++) {
          const uint32_t lds = as_base + buf + (uint32_t)wave * 1024u + q * (NW * 1024u);
          if (q < RF) dma16(r, a_off[MODE == 0 ? q < NA ? q : 0 : 0], (uint32_t)t * (PF_BK * 2) + (MODE == 0 ? 0u : (uint32_t)q * (NW * 16u) * (uint32_t)a.d_ff), lds);
          else dma16_half(r, a_half, (uint32_t)t * (PF_BK * 2), lds - (uint32_t)wave * 512u);
        }
      };
      auto read_planes = [&](int b, Planes& p) __attribute__((always_inline)) {
        const uint8_t* q = warea + (FMT == 0 ? p_rd ^ (b * 32u) : p_rd + b * 2u * PB32);
        if constexpr (FMT == 2) {                       // (twelve bytes on a 4-byte boundary)
          const uint32_t *qm = (const uint32_t*)q, *ql = (const uint32_t*)(q + PLANE);
          p.m = u32x3{qm[0], qm[1], qm[2]};
          p.l = u32x3{ql[0], ql[1], ql[2]};
        } else {
          p.m = *(const PlaneV*)q;
          p.l = *(const PlaneV*)(q + PLANE);
        }
      };
      // scale and zero-point of the lane's row in a step, as they lie in LDS; scale_of: scale and offset (weight = scale * code + offset).
      // Groups of 32: the two halves of a wave are in different groups (hb).
      auto read_meta = [&](int b, Meta& m) __attribute__((always_inline)) {
        const uint32_t gl = (uint32_t)(b * PF_BK) >> sh;      // group inside the 256 columns
        m.s = *(const uint32_t*)(warea + s_rd + (SCB ? gl >> 1 : gl) * 128u);
        m.z = *(const uint32_t*)(warea + z_rd + gl * 128u);
      };
      auto scale_of = [&](int t, const Meta& m, float& sc, float& c0) __attribute__((always_inline)) {
        if (SCB) {                                      // (two bf16 scales share a dword)
          const uint32_t left = (16u - 16u * (((uint32_t)(t * PF_BK) >> sh) & odd_group)) - 16u * hb;
          sc = __uint_as_float((m.s << left) & 0xFFFF0000u);
        } else {
          sc = __uint_as_float(m.s);
        }
        c0 = -(float)((BIASED ? 1024u : 0u) + (m.z & 0xFFu)) * sc;
      };
      // A direct load keeps the texture path busy for 13 cycles or more and a wave for several issue slots, so they are dealt out to the products: a
      // step's rows to those of Q3 behind the barrier; the next 256 columns' weights, once the present ones have left LDS for the registers, to Q1
      // and Q2 of a chunk's first step and Q0 .. Q2 of its second (WS: loads sent before each of these quarters, metadata first).  Tall tiles
      // (two row buffers) take the planes of steps 2 and 3 to registers one step later, which saves eight, and send for the next in step 1.
      constexpr int WB = NBUF == 2 ? 1 : 0;
      constexpr int WS[6] = {0, NBUF > 2 ? NPL / 2 : NPL, NBUF > 2 ? NPL : 2 * NPL, NBUF > 2 ? (4 * NPL + 2) / 3 : 2 * NPL, NBUF > 2 ? (5 * NPL + 2) / 3 : 2 * NPL, 2 * NPL};
      bf16x8 af[F], bf;
      Planes p[4];
      Meta mt[4];
      float sc, c0;                                     // of the step whose weights are being expanded
      // One quarter: the F products of 16 columns.  Behind every product come the read of the token rows of its fragment for the next
      // quarter (at `next`) and a share of the expansion of that quarter's weights: a wave issues in order, and two waves that
      // leave a barrier together would otherwise both multiply and then both expand.  `extra` adds the direct loads.  In the last quarter of
      // a step (ARRIVE >= 0: what may be outstanding) the next rows are those of another step: a barrier comes first, behind the second
      // product, when the last reads of this step are back.
      auto quarter = [&](auto arrive_c, const uint8_t* next, const Planes& pn, int sn, auto extra) __attribute__((always_inline)) {
        constexpr int ARRIVE = decltype(arrive_c)::value, BI = ARRIVE < 0 ? -1 : F > 1 ? 1 : 0;
        uint32_t qe, qo;
        u32x4 bn;
#pragma unroll
        for (int i = 0; i < F; i++) {
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf, acc[i], 0, 0, 0);
          if (i == BI) {
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(ARRIVE < 0 ? 0 : ARRIVE) : "memory");
#pragma unroll
            for (int j = 0; j <= BI; j++) af[j] = *(const bf16x8*)(next + j * 4096);
          } else if (i > BI) {
            af[i] = *(const bf16x8*)(next + i * 4096);
          }
          extra(i);
#pragma unroll
          for (int j = 0; j < 5; j++)
            if (j * F / 5 == i) {
              if (j == 0) {
                codes(pn.m, pn.l, sn, qe, qo);
                asm volatile("" : "+v"(qe), "+v"(qo));  // (pinned here: without it the work sinks to where it is used)
              } else {
                uint32_t w = weights(biased, qe, qo, j - 1, sc, c0);
                asm volatile("" : "+v"(w));
                bn[j - 1] = w;
              }
            }
          __builtin_amdgcn_sched_barrier(0);
        }
        bf = __builtin_bit_cast(bf16x8, bn);
      };
      const std::integral_constant<int, -1> inside{};
      if (ex) { wb = bases_of(ex); load_meta(wb, 0); load_plane(wb, 0, 0, 2 * NPL, wb.p_bytes); }
      uint32_t cur = 0;                                 // buffer of the present step
#pragma unroll
      for (int t = 0; t < NBUF; t++) load_rows(t, t * STEP, 0, RQ);
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NBUF - 1) * RQ) : "memory");
#pragma unroll
      for (int b = 0; b < 4; b++) { read_planes(b, p[b]); read_meta(b, mt[b]); }
      scale_of(0, mt[0], sc, c0);
#pragma unroll
      for (int i = 0; i < F; i++) af[i] = *(const bf16x8*)(As + a_rd + i * 4096);
      bf = expand(biased, p[0].m, p[0].l, 0, sc, c0);
      for (int t0 = 0; t0 < nk; t0 += 4) {
        const int c1 = (t0 >> 2) + 1;
        const uint32_t wrange = t0 + 4 < nk ? wb.p_bytes : 0u;      // (the last 256 columns: nothing more to fetch)
        auto step = [&](auto b_c) __attribute__((always_inline)) {
          constexpr int b = decltype(b_c)::value, n1 = (b + 1) & 3;
          const int t = t0 + b;
          uint32_t at = cur + a_rd;                     // (buffers are multiples of 128 bytes: the quarters differ by an exclusive or)
          asm volatile("" : "+v"(at));
          const uint32_t nxt = cur == (NBUF - 1) * STEP ? 0 : cur + STEP;
          // the quarter's share w of the weights, dealt to its products
          auto deal = [&](int w, int i) __attribute__((always_inline)) {
            const int n_w = WS[w + 1] - WS[w];
            load_plane(wb, c1, WS[w] + n_w * i / F, WS[w] + n_w * (i + 1) / F, wrange);
          };
          quarter(inside, As + (at ^ 16u), p[b], 1, [&](int i) __attribute__((always_inline)) {
            if (NBUF > 2 && b == 1) deal(2, i);
            if (NBUF == 2 && b == 1) {
              if (i == 0) { read_planes(2, p[2]); read_meta(2, mt[2]); }
              if (i == 1) { read_planes(3, p[3]); read_meta(3, mt[3]); }
            }
          });
          if (b == WB) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the weights have left LDS for the registers: the next ones may come
          quarter(inside, As + (at ^ 32u), p[b], 2, [&](int i) __attribute__((always_inline)) {
            if (b == WB && i == 0) load_meta(wb, c1);
            if (b == WB) deal(0, i);
            if (b == WB + 1 && NBUF > 2) deal(3, i);
          });
          if (b == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * RQ) : "memory");      // the next weights are there
          quarter(inside, As + (at ^ 48u), p[b], 3, [&](int i) __attribute__((always_inline)) {
            if (b == WB) deal(1, i);
            if (b == WB + 1 && NBUF > 2) deal(4, i);
            if (b == 3 && i == 0) { read_planes(0, p[0]); read_meta(0, mt[0]); }
          });
          // younger than the rows of step t + 1: those of NBUF - 2 steps, and of the next weights what was sent after those rows
          constexpr int YW = NBUF == 2 ? (b == WB ? 2 + WS[5] : 0)
                                       : b == 0 ? 2 + WS[2] : b < NBUF - 1 ? 2 + WS[5] : b == NBUF - 1 ? WS[5] - WS[2] : 0;
          scale_of(t + 1, mt[n1], sc, c0);
          quarter(std::integral_constant<int, (NBUF - 2) * RQ + YW>(), As + nxt + a_rd, p[n1], 0, [&](int i) __attribute__((always_inline)) {
            constexpr int G0 = F > 2 ? 1 : F - 1;       // (behind the barrier)
            if (i >= G0) load_rows(t + NBUF, cur, RQ * (i - G0) / (F - G0), RQ * (i - G0 + 1) / (F - G0));
            if (b == 3)
#pragma unroll
              for (int j = 1; j < (NBUF == 2 ? 2 : 4); j++)
                if ((j - 1) * F / 3 == i) { read_planes(j, p[j]); read_meta(j, mt[j]); }
          });
          cur = nxt;
        };
        step(std::integral_constant<int, 0>());
        if (t0 + 1 < nk) step(std::integral_constant<int, 1>());
        if (t0 + 2 < nk) step(std::integral_constant<int, 2>());
        if (t0 + 3 < nk) step(std::integral_constant<int, 3>());
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (no load is on its way to LDS any more)
    }
  };
  if constexpr (NF == 8) {
    if (nf == 8) kloop(std::integral_constant<int, 8>());
    else if (nf == 7) kloop(std::integral_constant<int, 7>());
    else if (nf == 6) kloop(std::integral_constant<int, 6>());
    else if (nf == 5) kloop(std::integral_constant<int, 5>());
    else if (nf == 4) kloop(std::integral_constant<int, 4>());
    else if (nf == 3) kloop(std::integral_constant<int, 3>());
    else if (nf == 2) kloop(std::integral_constant<int, 2>());
    else kloop(std::integral_constant<int, 1>());
  } else {
    if (NF >= 5 && nf == 5) kloop(std::integral_constant<int, (NF >= 5 ? 5 : 1)>());
    else if (NF >= 4 && nf == 4) kloop(std::integral_constant<int, (NF >= 4 ? 4 : 1)>());
    else if (NF >= 3 && nf == 3) kloop(std::integral_constant<int, (NF >= 3 ? 3 : 1)>());
    else if (NF >= 2 && nf == 2) kloop(std::integral_constant<int, (NF >= 2 ? 2 : 1)>());
    else kloop(std::integral_constant<int, 1>());
  }

  // Scales from 2^128 / 1279 on overflow c0 of the biased form: such a weight is -inf, and any product with it leaves the sums of
  // its row not finite.  So a wave that finds its first sums not finite looks for such scales among its rows and, if there
  // are any, forms all its sums again from the unbiased form, straight from memory: slow, but only ever for such weights.
  // (The arguments are fetched anew there: kept in scalar registers over the K loop they would spill others.)
  if constexpr (BIASED) {
    if (__any(!(fabsf(acc[0][0]) < INFINITY))) {
      typedef __attribute__((address_space(4))) const GemmPair ArgsInMemory;
      ArgsInMemory* args = (ArgsInMemory*)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(args));
      const auto* b = &args->g[second ? 1 : 0];
      const int Kb = MODE == 0 ? b->d_model : b->d_ff, shb = b->group_shift, passes = MODE == 1 && b->dense_rows ? b->n_dense : 1;
      const uint32_t row = (uint32_t)(nt * BN + wave * 32) + wr;
      const bool inside = nt * BN + wave * 32 < (MODE == 0 ? 2 * b->d_ff : b->d_model);      // (all 32 rows of a wave or none)
      auto scale_at = [&](size_t ee, uint32_t g) { return bf16_bits_to_f32(((const uint16_t*)(b->w.sc + ee * b->w.sc_stride))[row * (uint32_t)b->w.sng + g]); };
      float top = 0.0f;
      if (inside)
        for (int ex = 0; ex < passes; ex++)
          for (int g = 0; g < b->w.ng; g++) top = fmaxf(top, scale_at((size_t)(e + ex), g));
      if (__any(!(top * 1279.0f < INFINITY))) {
        uint32_t src[NF];                               // token rows (past the tile's last one: that row again)
#pragma unroll
        for (int i = 0; i < NF; i++) {
          const int r = m0 + min(32 * i + n, m_cnt - 1);
          src[i] = (MODE == 0 ? (uint32_t)(b->dense_rows ? r : b->rows[row0 + r] / b->k) : (uint32_t)(row0 + r)) * (uint32_t)Kb;
#pragma unroll
          for (int q = 0; q < 16; q++) acc[i][q] = 0.0f;
        }
        for (int ex = 0; ex < passes; ex++) {
          const size_t ee = (size_t)(e + ex), plane_row = (size_t)row * ((uint32_t)(Kb >> 5) * PB32);
          const uint16_t* av = MODE == 0 ? b->x : ex == 0 ? b->h : b->h_more + (size_t)(ex - 1) * b->dense_rows * b->d_ff;
          const uint8_t* pm = b->w.msb + ee * b->w.plane_stride + plane_row;
          const uint8_t* pl = b->w.lsb + ee * b->w.plane_stride + plane_row;
          const uint8_t* pz = b->w.zp + ee * b->w.zp_stride + (size_t)row * b->w.ng;
          for (int t = 0; t < Kb / PF_BK; t++) {
            const uint32_t g = (uint32_t)(t * PF_BK + 32 * hh) >> shb;
            const float scale = scale_at(ee, g), c0 = -(float)pz[g] * scale;
            PlaneV m, l;
#pragma unroll
            for (int j = 0; j < PB32 / 4; j++) {
              m[j] = ((const uint32_t*)(pm + (2 * t + hh) * PB32))[j];
              l[j] = ((const uint32_t*)(pl + (2 * t + hh) * PB32))[j];
            }
#pragma unroll
            for (int s = 0; s < 4; s++) {
              const bf16x8 bf = expand(std::false_type(), m, l, s, scale, c0);
#pragma unroll
              for (int i = 0; i < NF; i++)
                if (i < nf) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)(av + src[i] + t * PF_BK + 32 * hh + 8 * s), bf, acc[i], 0, 0, 0);
            }
          }
        }
      }
    }
  }

  // ---- epilogue.  D layout: register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32.  Stores go through a
  // buffer resource that ends with the tile's last row, so surplus rows are dropped without a branch.
  __syncthreads();
  const size_t row_first = (size_t)(row0 + m0);
  if constexpr (MODE == 0) {
    // registers r and r + 8 of lanes 0 .. 15 (gate) and 16 .. 31 (up) are exchanged so that a lane holds gate and up of one
    // element; the bf16 tile is then turned in LDS, so that a row of it, 64 columns, leaves as one 128-byte line
    constexpr int HLD = NW * 32 + 16, HP = NW * 2;      // bytes of a row in LDS, 16-byte pieces of its columns
    const uint32_t col = (uint32_t)wave * 16 + (n & 15), rb = 4 * hh + 16 * (n >> 4);
#pragma unroll
    for (int i = 0; i < NF; i++) {
      if (i >= nf) continue;
      float lo = 0.0f, hi = 0.0f;
#pragma unroll
      for (int r = 0; r < 8; r++) {
        const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[i][r]), __float_as_uint(acc[i][r + 8]), false, false);
        acc[i][r] = __uint_as_float(sw[0]);             // gate
        acc[i][r + 8] = __uint_as_float(sw[1]);         // up
        lo = fminf(lo, acc[i][r]);
        hi = fmaxf(hi, acc[i][r]);
      }
      auto put = [&](int r, float hv) __attribute__((always_inline)) {
        *(uint16_t*)(As + (i * 32 + 8 * (r >> 2) + (r & 3) + rb) * HLD + col * 2) = (uint16_t)pack_bf16(hv, hv);
      };
      // u g / (1 + e^-g).  The quotient by the reciprocal unit's result, one Newton step and one correction from the remainder, 10
      // instructions instead of a division's 18 (this is half of the epilogue): the division's bits for every gate from -80 up to the largest
      // finite one (all 3.25e9 of them compared; only -0 gives +0).  Below, the reciprocal leaves the normal numbers (from -87.4 down), and an
      // infinite gate has no remainder: a wave that holds such a gate divides.  A row's result thus depends on nothing but the row.
      // (Without the correction 3 % of the gates differ in the last bit, and a row changed with its neighbours' gates; it costs 0.1 / 0.5 / 0.6 %
      // of a layer: 173 / 2048 / 4096 tokens, 165.0 -> 165.3, 262.9 -> 264.2, 707 -> 711 us.)
      if (__any(lo < -80.0f || hi == INFINITY)) {
#pragma unroll
        for (int r = 0; r < 8; r++) put(r, acc[i][r] / (1.0f + __expf(-acc[i][r])) * acc[i][r + 8]);
      } else {
#pragma unroll
        for (int r = 0; r < 8; r++) {
          const float g = acc[i][r], d = 1.0f + __expf(-g), r0 = __builtin_amdgcn_rcpf(d);
          const float r1 = fmaf(fmaf(-d, r0, 1.0f), r0, r0), q = g * r1;
          put(r, fmaf(fmaf(-d, q, g), r1, q) * acc[i][r + 8]);
        }
      }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(h + row_first * a.d_ff, 0, (int)((uint32_t)m_cnt * (uint32_t)a.d_ff * 2u), 0x00020000);
    for (int q = 0; q < nf; q++) {
      const uint32_t r = q * 32 + tid / HP, c = tid % HP;
      // (a tile of 128 columns may reach past the matrix)
      const uint32_t at = nt * (BN / 2) + c * 8 < (uint32_t)a.d_ff ? (r * (uint32_t)a.d_ff + nt * (BN / 2) + c * 8) * 2u : 0xFFFFFFF0u;
      __builtin_amdgcn_raw_buffer_store_b128(*(const u32x4*)(As + r * HLD + c * 16), ro, (int)at, 0, 0);
    }
  } else {
    float* row_wt = (float*)As;
    if (tid < BM) row_wt[tid] = my_wt;
    __syncthreads();
    if ((int)wrow < N) {                                // (a wave's 32 columns are inside or outside as a whole)
      const uint32_t ldo = (uint32_t)a.d_model * 4u;
      const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(a.o + row_first * a.d_model, 0, (int)((uint32_t)m_cnt * ldo), 0x00020000);
      const uint32_t vo = 4 * hh * ldo + (wrow + n) * 4u;
#pragma unroll
      for (int i = 0; i < NF; i++) {
        if (i >= nf) continue;
#pragma unroll
        for (int rq = 0; rq < 4; rq++) {
          const float4 w4 = *(const float4*)(row_wt + i * 32 + 8 * rq + 4 * hh);
          const float wt[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int so = (int)((uint32_t)(i * 32 + 8 * rq + r) * ldo);
            float v = wt[r] * acc[i][4 * rq + r];
            if (a.accumulate) v += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ro, (int)vo, so, 0));
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), ro, (int)vo, so, 0);
          }
        }
      }
    }
  }
}

// Y[t, c] = sum_j O[pos[t*k + j], c]  (+ OS[t, c], the shared experts' sum)  (+ x[t, c]); 4 columns per thread.
// Bound: HBM (k + 1 fp32 rows read per token).  The rows are fetched four at a time, all of them and OS and x before the
// first sum; the sums run in slot order.  173 tokens, top-6: 8.3 -> 5.8 us; 4096 tokens, top-4: 35 -> 32 us (201 MB, 6.3 TB/s).
__global__ __launch_bounds__(256) void combine_kernel(const float* o, const int32_t* pos, const float* o_s, const uint16_t* x,
                                                      uint16_t* y, int k, int d_model, int add_residual) {
  const int t = blockIdx.x;
  const int32_t* pt = pos + (size_t)t * k;
  for (int c = threadIdx.x * 4; c < d_model; c += 256 * 4) {
    float4 os = make_float4(0, 0, 0, 0);
    uint2 xv = make_uint2(0, 0);
    if (o_s) os = *(const float4*)(o_s + (size_t)t * d_model + c);
    if (add_residual) xv = *(const uint2*)(x + (size_t)t * d_model + c);
    float4 s = make_float4(0, 0, 0, 0);
    for (int j = 0; j < k; j += 4) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; u++) v[u] = *(const float4*)(o + (size_t)pt[min(j + u, k - 1)] * d_model + c);
#pragma unroll
      for (int u = 0; u < 4; u++)
        if (j + u < k) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
    }
    if (o_s) { s.x += os.x; s.y += os.y; s.z += os.z; s.w += os.w; }
    if (add_residual) {
      s.x += bf16_bits_to_f32(xv.x & 0xFFFF); s.y += bf16_bits_to_f32(xv.x >> 16);
      s.z += bf16_bits_to_f32(xv.y & 0xFFFF); s.w += bf16_bits_to_f32(xv.y >> 16);
    }
    uint2 r;
    r.x = f32_to_bf16_bits(s.x) | (f32_to_bf16_bits(s.y) << 16);
    r.y = f32_to_bf16_bits(s.z) | (f32_to_bf16_bits(s.w) << 16);
    *(uint2*)(y + (size_t)t * d_model + c) = r;
  }
}

// ------------------------------------------------------------------------------- host entry
static inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

template <int MODE, int SCB, int FMT, int NF>
static int launch_gemm_t(smoe_ctx* ctx, GemmPair& g, int grid) {
  // groups of 256 columns of the set with the smallest groups: two scale dwords / zero-points of 32 rows per 256 bytes
  int sh = 8;
  if (g.nb0) sh = std::min(sh, g.g[0].group_shift);
  if (grid > g.nb0) sh = std::min(sh, g.g[1].group_shift);
  const int n_grp = 256 >> sh, nsd = SCB ? (n_grp + 1) / 2 : n_grp;
  typedef PfLds<SCB, FMT, NF> Lds;
  g.zp_at = 2 * Lds::PLANE + (nsd + 1) / 2 * 256;
  g.wave_lds = g.zp_at + (n_grp + 1) / 2 * 256;
  const size_t lds = (size_t)Lds::ROWS + Lds::NW * (size_t)(Lds::FIT ? g.wave_lds : Lds::WAVE);
  static_assert((NF == 3 && FMT == 1 ? 3 : pf_waves(NF) == 4 ? 2 : 1) * (Lds::ROWS + Lds::NW * Lds::WAVE) <= 160 * 1024, "work-groups per CU");
  if (lds > 64u * 1024u) {       // beyond the default per-work-group limit: granted once per device
    size_t& granted = ctx->gemm_lds_granted[((MODE * 2 + SCB) * 3 + FMT) * 5 + (NF == 8 ? 4 : NF == 5 ? 3 : NF - 1)];
    if (lds > granted) {
      HIPCHK(ctx, hipFuncSetAttribute((const void*)grouped_gemm_kernel<MODE, SCB, FMT, NF>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      granted = lds;
    }
  }
  grouped_gemm_kernel<MODE, SCB, FMT, NF><<<grid, 64 * Lds::NW, lds, ctx->stream>>>(g);
  return SMOE_OK;
}
template <int MODE, int NF>
static int launch_gemm_nf(smoe_ctx* ctx, GemmPair& g, int sc_bf16, int bits, int grid) {
  if (bits == 2) return sc_bf16 ? launch_gemm_t<MODE, 1, 1, NF>(ctx, g, grid) : launch_gemm_t<MODE, 0, 1, NF>(ctx, g, grid);
  if (bits == 3) return sc_bf16 ? launch_gemm_t<MODE, 1, 2, NF>(ctx, g, grid) : launch_gemm_t<MODE, 0, 2, NF>(ctx, g, grid);
  return sc_bf16 ? launch_gemm_t<MODE, 1, 0, NF>(ctx, g, grid) : launch_gemm_t<MODE, 0, 0, NF>(ctx, g, grid);
}
// bits = plane bits per code of the bank (4: 8/4 nest, 3: 6/3 nest, 2: 4/2 nest); nf = fragments of the tallest tile
template <int MODE>
static int launch_gemm(smoe_ctx* ctx, GemmPair& g, int sc_bf16, int bits, int nf, int grid) {
  if (nf == 1) return launch_gemm_nf<MODE, 1>(ctx, g, sc_bf16, bits, grid);
  if (nf == 2) return launch_gemm_nf<MODE, 2>(ctx, g, sc_bf16, bits, grid);
  if (nf == 3) return launch_gemm_nf<MODE, 3>(ctx, g, sc_bf16, bits, grid);
  if (nf == 5) return launch_gemm_nf<MODE, 5>(ctx, g, sc_bf16, bits, grid);
  return launch_gemm_nf<MODE, 8>(ctx, g, sc_bf16, bits, grid);
}
// Tile height, in fragments of 32 rows.  Experts of few rows (up to 64 with one and a half standard deviations of even routing) take one
// tile of 32 or 64: their weights' bytes bound them.  Above that three heights compete: 96 and 160 rows with four waves, two work-groups
// per CU, and 256 with eight, one per CU, which expands a weight once for more rows but fills the chip in larger pieces, and in which the short tiles
// of unpopular experts are alone on a CU.  (There is no tile of 128 rows with four waves: it gains nothing or loses, because more experts need a second one.)
// Which is fastest hangs on how many tiles there are and how they fill the chip, so a layer's time is estimated.  The numbers are not those of the K loop
// but a fit, in arbitrary units, to the measured ratios of 148 layers of all three nests (d_model 256 - 2560, d_ff 128 - 2048, 8 - 96 experts; cold weights,
// calls back to back for 30 ms; popularity even to 1/rank^2): 256 against 160 rows with an error of 6 %, 96 against 160 rows of 5 %.
struct GemmSize { double experts, rows; int N, K; bool even; };      // even: every expert has just these rows
struct Tiles { double n, frags, deviation; };           // tiles per expert, mean fragments of one, relative deviation of the number of tiles
static Tiles tiles_around(int nf, const GemmSize& g, double deviation) {
  const double h = 32.0 * nf;
  double tiles = ceil(g.rows / h), var = 0.0;
  if (deviation > 0.0 && g.rows <= 64.0 * h) {
    tiles = 1.0;
    for (int j = 1; j * h < g.rows + 3.0 * deviation + 1.0; j++) {
      const double p = 1.0 / (1.0 + exp(1.7 * (j * h - g.rows) / deviation));
      tiles += p;
      var += p * (1.0 - p);
    }
  }
  return {tiles, std::min((double)nf, g.rows / (32.0 * tiles) + 0.5), sqrt(var / g.experts) / tiles};
}
// Rows per expert when popularity falls as 1 / rank^1.1 and a token takes k different experts: T (1 - e^(-c w)), c such that they add up.
struct SkewedRows {
  int n = 0;
  float rows[SMOE_MAX_EXPERTS];
  void fill(float T, float k, int E) {
    n = std::min(E, SMOE_MAX_EXPERTS);
    float w[SMOE_MAX_EXPERTS], c = 0.0f;
    for (int r = 0; r < n; r++) w[r] = exp2f(-1.1f * log2f(r + 1.0f));
    for (int it = 0; it < 6; it++) {                    // Newton's method from below: the sum is concave in c
      float sum = 0.0f, slope = 1e-6f;
      for (int r = 0; r < n; r++) { const float q = expf(-c * w[r]); sum += 1.0f - q; slope += q * w[r]; }
      c += std::max(0.0f, k - sum) / slope;
    }
    for (int r = 0; r < n; r++) rows[r] = T * (1.0f - expf(-c * w[r]));
  }
};
static Tiles tiles_skewed(int nf, const SkewedRows& s) {
  int tiles = 0, frags = 0;
  for (int r = 0; r < s.n; r++) {
    const int f = std::max(1, (int)ceilf(s.rows[r] / 32.0f));
    tiles += (f + nf - 1) / nf;
    frags += f;
  }
  return {(double)tiles / s.n, (double)frags / tiles, 0.0};
}
static double gemm_cost(int nf, const GemmSize* g, const Tiles* t, int n, int n_cu) {
  const bool tall = nf > 5;
  double items = 0, work = 0, longest = 0;
  for (int i = 0; i < n; i++) {
    const double steps = g[i].K / 64.0, it = g[i].experts * t[i].n * ((g[i].N + 32 * pf_waves(nf) - 1) / (32 * pf_waves(nf)));
    const double c = tall ? steps * (1040.0 + 227.0 * t[i].frags) + 6000.0 : steps * (810.0 + 304.0 * t[i].frags) + 900.0;
    items += it;
    work += it * c;
    longest = std::max(longest, c);
  }
  // rounds: how often the chip is filled; the mean over a deviation of the number of tiles either way
  const double fill = items / (tall ? n_cu : 2 * n_cu), wide = sqrt(1.7e-4 + t[0].deviation * t[0].deviation);
  double rounds = 0;
  for (double q : {(1.0 - wide) * fill, fill, (1.0 + wide) * fill}) {
    const double whole = floor(q), part = q - whole;
    rounds += tall ? (q <= 8.5 ? ceil(q) : q + 0.75) : whole + (part <= 0.0 ? 0.0 : part <= 0.5 ? 0.66 : 1.0);
  }
  return std::max(work / items * rounds / 3.0, longest * (tall || fill > 1.0 ? 1.0 : 0.66));
}
// Height of up to two sets of experts in common launches, {gate/up, down} of each: 96 rows up to a mean plus one and a half deviations of 96, else
// 160; the other one of these two where it is estimated to be no slower with even, with mildly uneven (a fifth of the mean) and with skewed popularity;
// 256 where it is no slower with mildly uneven routing, within 5 % with even and within bounds with skewed popularity: the host knows the mean alone.
// There the estimate of the tall tiles is too high, by most for the 8/4 nest (1.13 against 1.05 measured for the first line below; 1.11 and 1.13 in
// the other nests).  Microseconds per layer, popularity even / router over hidden states / 1/rank^1.1 / 1/rank^2, 160 rows, then 256:
//   60 experts of d_model 2048, d_ff 1408, top-4, 2048 tokens   243 / 261 / 277 / 313, 237 / 241 / 292 / 317   -> 256
//   the same, 6/3 nest, groups of 32                            299 / 321 / 331 / 371, 303 / 303 / 374 / 391   -> 160
//   8/4, 1500 tokens                                            219 / 221 / 239 / 266, 213 / 216 / 259 / 274   -> 160
//   3000 tokens                                                 360 / 367 / 361 / 386, 299 / 330 / 345 / 413   -> 256
//   with a shared expert of 5632, 4096 tokens                   709 / 736 / 737 / 756, 697 / 679 / 668 / 718   -> 256
//   36 experts of 896, 1024, top-3, 4/2 nest, 3692 tokens       136 / 143 / 145 / 143, 165 / 131 / 127 / 184   -> 160
static int pick_nf(const GemmSize (*g)[2], int n, int n_cu, int bits, SkewedRows& skewed, double T, double k) {
  const double rows = g[0][0].rows, want = rows + 1.5 * sqrt(rows);
  if (want <= 64.0) return want <= 32.0 ? 1 : 2;
  enum { EVEN, MILD, SKEWED };
  auto cost = [&](int nf, int routing) {
    Tiles t[2];
    for (int i = 0; i < n; i++)
      t[i] = g[i][0].even ? tiles_around(nf, g[i][0], 0.0) : routing == SKEWED ? tiles_skewed(nf, skewed)
             : tiles_around(nf, g[i][0], routing == EVEN ? sqrt(rows) : 0.2 * rows + 1.0);
    double c = 93e3;                                    // (routing, grouping, sums)
    for (int m = 0; m < 2; m++) {
      const GemmSize s[2] = {g[0][m], g[n - 1][m]};
      c += gemm_cost(nf, s, t, n, n_cu);
    }
    return c;
  };
  auto better = [&](int nf, int than, double even, double mild, double skew) {
    if (g[0][0].even) return cost(nf, EVEN) <= cost(than, EVEN);
    if (cost(nf, EVEN) > even * cost(than, EVEN) || cost(nf, MILD) > mild * cost(than, MILD)) return false;
    if (!skewed.n) skewed.fill((float)T, (float)k, (int)g[0][0].experts);
    return cost(nf, SKEWED) <= skew * cost(than, SKEWED);
  };
  int best = want <= 96.0 ? 3 : 5;
  // (beside shared experts the estimate of 96 rows is 7 % too low once their tiles fill the chip a few times)
  double items = 0;
  for (int i = 0; i < n; i++) items += g[i][0].experts * ceil(g[i][0].rows / 96.0) * ((g[i][0].N + 127) / 128);
  const double sure = n > 1 && best == 5 && items > 3.0 * n_cu ? 0.93 : 1.0;
  if (better(8 - best, best, sure, sure, sure)) best = 8 - best;
  return better(8, best, 1.05, 1.0, bits == 4 ? 1.2 : 1.06) ? 8 : best;
}

// Tile heights (in fragments) of the routed and the shared experts, and whether the shared experts' tiles ride in the routed experts' launches
// (then at the routed experts' height).
struct PrefillPlan { int nf, nfs; bool join; };
static PrefillPlan plan_prefill(int T, int k, int E, int d, int f, int bits, int ns, int f_s, int s_bits, bool same, int n_cu) {
  const GemmSize sizes[2][2] = {{{(double)E, (double)T * k / E, 2 * f, d, false}, {(double)E, (double)T * k / E, d, f, false}},
                                {{(double)ns, (double)T, 2 * f_s, d, true}, {1.0, (double)T, d, f_s * ns, true}}};
  SkewedRows skewed;
  PrefillPlan p{pick_nf(sizes, 1, n_cu, bits, skewed, T, k), ns ? pick_nf(sizes + 1, 1, n_cu, s_bits, skewed, T, k) : 0, false};
  if (!ns || !same) return p;      // (same: both banks have one nest and one scale type)
  if (p.nf >= 3 && p.nfs >= 3) {
    // taller tiles: one height for both sets, in common launches (of 48 layers none was faster with launches of their own at the better of both
    // choices: 64 experts and two shared of d_ff 1408, d_model 2048, 2048 tokens 420 / 387 us)
    p.nf = pick_nf(sizes, 2, n_cu, bits, skewed, T, k);
    p.join = true;
  } else {
    // The shared experts' tiles ride in the routed experts' launches, where they fill the chip's idle end (and, with few
    // tokens, most of a launch of their own: 173 tokens, two shared experts of d_ff 1408: 200 us of 422 were theirs), if both
    // want the same tile height, or if at the routed experts' (lower) height there is little to expand: a dense tile
    // expands its weights again, 600 million of them in about 55 us over the chip, which is what launches of their own lose to
    // their empty ends.  64 experts of d_ff 512, one shared of 1024, d_model 1024, 500 tokens: 101 -> 72 us; 96 experts, two
    // shared of 3840, d_model 2560, 500 tokens, all joined, would be 482 -> 515.
    const int bm = 32 * p.nf;
    const double again = 3.0 * d * f_s * ns * ((T + bm - 1) / bm);
    p.join = p.nf == p.nfs || T <= 8 * bm || (T <= 24 * bm && again <= 600e6);
  }
  return p;
}

struct PrefillLayout { size_t rows, pos, h, o, gamma, h_s, o_s, total; };

static inline int max_tiles(int T, int E, int k, int bm) { return E + (T * k) / bm; }

static PrefillLayout prefill_layout(int T, int E, int k, int d_model, int d_ff, int shared_d_ff) {
  PrefillLayout L;
  size_t off = 0;
  L.rows = off;    off = up256(off + (size_t)T * k * 4);
  L.pos = off;     off = up256(off + (size_t)T * k * 4);
  // (two areas that nothing uses: they keep what smoe_prefill_bytes returns, and with it which scratch sizes are refused, as it was)
  off = up256(off + (size_t)(E + 1) * 4);
  off = up256(off + (size_t)(4 + 4 * (E + (T * k) / 192 + 8)) * 4);
  L.h = off;       off = up256(off + (size_t)T * k * d_ff * 2);
  L.o = off;       off = up256(off + (size_t)T * k * d_model * 4);
  L.gamma = L.h_s = L.o_s = off;
  if (shared_d_ff > 0) {       // one shared expert at a time: its H rows, and the running sum of their outputs
    L.gamma = off; off = up256(off + (size_t)T * 4);
    L.h_s = off;   off = up256(off + (size_t)T * shared_d_ff * 2);
    L.o_s = off;   off = up256(off + (size_t)T * d_model * 4);
  }
  L.total = off;
  return L;
}

extern "C" int smoe_prefill_bytes(int T, int E, int k, int d_model, int d_ff, int shared_d_ff, size_t* scratch_bytes) {
  if (!scratch_bytes) return SMOE_EINVAL;
  if (T <= 0 || E <= 0 || k <= 0 || k > E || d_model <= 0 || d_ff <= 0 || shared_d_ff < 0) return SMOE_ESHAPE;
  *scratch_bytes = prefill_layout(T, E, k, d_model, d_ff, shared_d_ff).total;
  return SMOE_OK;
}

extern "C" int smoe_prefill_tiles(const smoe_bank_desc* routed, const smoe_bank_desc* shared, int T, int k, int n_cu, int* routed_rows,
                                  int* shared_rows, int* joined) {
  if (!routed || !routed_rows || !shared_rows || !joined) return SMOE_EINVAL;
  if (T <= 0 || k <= 0 || k > routed->n_experts || routed->d_model <= 0 || routed->d_ff <= 0 || n_cu <= 0) return SMOE_ESHAPE;
  if (shared && (shared->n_experts <= 0 || shared->d_model != routed->d_model || shared->d_ff <= 0)) return SMOE_ESHAPE;
  const PrefillPlan p = plan_prefill(T, k, routed->n_experts, routed->d_model, routed->d_ff, routed->b_low, shared ? shared->n_experts : 0,
                                     shared ? shared->d_ff : 0, shared ? shared->b_low : 0,
                                     shared && shared->scale_dtype == routed->scale_dtype && shared->b_low == routed->b_low, n_cu);
  *routed_rows = 32 * p.nf;
  *shared_rows = 32 * (p.join ? p.nf : p.nfs);
  *joined = p.join;
  return SMOE_OK;
}

extern "C" int smoe_prefill_histogram(smoe_ctx* ctx, const smoe_bank* routed, const smoe_bank* shared, int T,
                                      const void* x_dev, int act_dtype, int k, const float* logits_dev,
                                      const float* w_router_dev, int norm_topk, float routed_scale,
                                      const void* shared_gate_w_dev, int add_residual, void* scratch_dev,
                                      size_t scratch_bytes, void* y_dev, int32_t* idx_dev, float* w_dev,
                                      uint32_t* hist_dev) {
  if (!ctx || !routed || !x_dev || !scratch_dev || !y_dev || !idx_dev || !w_dev || !hist_dev) return SMOE_EINVAL;
  if (!logits_dev && !w_router_dev) return SMOE_EINVAL;
  if (shared_gate_w_dev && !shared) return SMOE_EINVAL;
  if (act_dtype != SMOE_BF16) return SMOE_ENOTIMPL;
  if (routed->device != ctx->device || (shared && shared->device != ctx->device)) return SMOE_EINVAL;
  const int E = routed->desc.n_experts, d = routed->desc.d_model, f = routed->desc.d_ff;
  if (T <= 0 || k <= 0 || k > E || k > SMOE_MAX_TOPK || E > SMOE_MAX_EXPERTS) return SMOE_ESHAPE;
  if (f % PF_BK || d % PF_BK || routed->desc.group < 32 || (routed->desc.group & (routed->desc.group - 1))) return SMOE_ESHAPE;
  if ((size_t)T * d >= 0x7FFFFFFFu || (size_t)T * k * f >= 0x7FFFFFFFu) return SMOE_ESHAPE;   // 32-bit element offsets
  const int f_s = shared ? shared->desc.d_ff : 0;
  if (shared) {
    const int gs = shared->desc.group;
    if (shared->desc.d_model != d || f_s % PF_BK || gs < 32 || (gs & (gs - 1))) return SMOE_ESHAPE;
    if ((size_t)T * f_s >= 0x7FFFFFFFu) return SMOE_ESHAPE;
  }
  if (!aligned16(x_dev) || !aligned16(y_dev) || !aligned16(idx_dev) || !aligned16(w_dev) || !aligned16(hist_dev) ||
      !aligned16(logits_dev) || !aligned16(w_router_dev) || !aligned16(shared_gate_w_dev) || (((uintptr_t)scratch_dev) & 255u))
    return SMOE_EALIGN;
  const PrefillLayout L = prefill_layout(T, E, k, d, f, f_s);
  if (scratch_bytes < L.total) return SMOE_ESIZE;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  uint8_t* s = (uint8_t*)scratch_dev;
  int32_t* rows = (int32_t*)(s + L.rows);
  int32_t* pos = (int32_t*)(s + L.pos);
  uint16_t* h = (uint16_t*)(s + L.h);
  float* o = (float*)(s + L.o);
  hipStream_t st = ctx->stream;

  RouteArgs ra{E, k, d, logits_dev, x_dev, w_router_dev, nullptr, norm_topk, routed_scale, nullptr, idx_dev, w_dev};
  { const int rc = smoe_launch_route(ctx, ra, T, SMOE_BF16); if (rc) return rc; }
  const PrefillPlan plan = plan_prefill(T, k, E, d, f, routed->dev.bits, shared ? shared->desc.n_experts : 0, f_s, shared ? shared->dev.bits : 0,
                                        shared && shared->dev.sc_bf16 == routed->dev.sc_bf16 && shared->dev.bits == routed->dev.bits, ctx->n_cu);
  const int nf = plan.nf, nfs = plan.nfs;
  const bool join = plan.join;
  const int bm = 32 * nf;
  float* gamma = shared ? (float*)(s + L.gamma) : nullptr;
  group_kernel<<<E + (shared ? (T + GR_THREADS / 64 - 1) / (GR_THREADS / 64) : 0), GR_THREADS, 0, st>>>(
      idx_dev, T * k, E, hist_dev, rows, pos, (const uint16_t*)x_dev, (const uint16_t*)shared_gate_w_dev, T, d, gamma);

  GemmArgs g{};
  g.group_shift = __builtin_ctz((unsigned)routed->dev.group); g.rows = rows; g.hist = hist_dev;
  g.x = (const uint16_t*)x_dev; g.h = h; g.o = o; g.wgt = w_dev; g.E = E; g.k = k; g.d_model = d; g.d_ff = f;
  // Row tiles side by side on a column tile's weights: four where an expert has several tiles, eight of the dense ones.  Between 1 and
  // 16 it matters little: 1 / 4 / 8 give 430 / 435 / 430 us (60 experts, 273 rows each), 802 / 809 / 816 (546 rows), 565 / 553 / 541 (16 experts
  // of d_model 4096, 500 rows); dense tiles 1 / 8 / 32: 163.7 / 158.8 / 159.2 us (173 tokens), 189 / 180 / 181 (300), 727 / 732 / 750 (4096).
  g.super = (double)T * k / E > bm ? 4 : 1;
  const int mt = max_tiles(T, E, k, bm);         // upper bound of the tile count; surplus work-groups return at once
  const int scb = routed->dev.sc_bf16, bits = routed->dev.bits;
  auto grid_of = [](int n_tiles, int n_col) { return (n_tiles * n_col + 7) / 8 * 8; };
  GemmPair gu{}, dn{};
  gu.g[1] = dn.g[1] = g;
  gu.g[1].a_bytes = (uint32_t)((size_t)T * d * 2); dn.g[1].a_bytes = (uint32_t)((size_t)T * k * f * 2);      // (below 4 GiB: checked above)
  gu.g[1].w = routed->dev.gu; const int bn = 32 * pf_waves(nf);
  gu.g[1].n_col_tiles = (2 * f + bn - 1) / bn;
  dn.g[1].w = routed->dev.dn; dn.g[1].n_col_tiles = (d + bn - 1) / bn;
  const int gu_grid = grid_of(mt, gu.g[1].n_col_tiles), dn_grid = grid_of(mt, dn.g[1].n_col_tiles);
  float* o_s = nullptr;
  if (!shared) {
    { const int rc = launch_gemm<0>(ctx, gu, scb, bits, nf, gu_grid); if (rc) return rc; }
    { const int rc = launch_gemm<1>(ctx, dn, scb, bits, nf, dn_grid); if (rc) return rc; }
  } else {
    // the shared experts see every token: dense GEMMs over the token rows in their own order, their
    // gate-weighted outputs summed in O_s
    o_s = (float*)(s + L.o_s);
    GemmArgs q{};
    q.group_shift = __builtin_ctz((unsigned)shared->dev.group);
    q.x = (const uint16_t*)x_dev; q.h = (uint16_t*)(s + L.h_s); q.o = o_s; q.wgt = gamma; q.E = shared->desc.n_experts; q.k = 1; q.d_model = d; q.d_ff = f_s;
    q.dense_rows = T; q.super = 8;
    const int ns = shared->desc.n_experts;
    // H of one shared expert has its own place.  That of others waits in Y, which nothing else writes before the last
    // kernel, if Y is not X and they fit there; else in the rows of O until the routed experts' down GEMM
    // writes those: then the shared experts' down GEMM comes before it, and as many experts as fit are worked out together.
    const uint8_t *x0 = (const uint8_t*)x_dev, *y0 = (const uint8_t*)y_dev;
    const size_t td2 = (size_t)T * d * 2;
    const bool in_y = (size_t)(ns - 1) * f_s <= (size_t)d && (y0 + td2 <= x0 || x0 + td2 <= y0);
    q.h_more = in_y ? (uint16_t*)y_dev : (uint16_t*)o;
    const int at_once = in_y ? ns : (int)std::min<size_t>((size_t)ns, 1 + ((size_t)T * k * d * 4) / ((size_t)T * f_s * 2));
    for (int e0 = 0; e0 < ns; e0 += at_once) {
      q.dense_expert = e0; q.n_dense = std::min(at_once, ns - e0); q.accumulate = e0 > 0;
      const bool j0 = join && e0 == 0, j1 = j0 && (in_y || ns == 1);
      const int nq = j0 ? nf : nfs, bq = 32 * pf_waves(nq), rt = (T + 32 * nq - 1) / (32 * nq);
      GemmArgs qg = q, qd = q;
      qg.a_bytes = (uint32_t)((size_t)T * d * 2); qd.a_bytes = (uint32_t)((size_t)T * f_s * 2);
      qg.w = shared->dev.gu; qg.n_col_tiles = (2 * f_s + bq - 1) / bq;
      qd.w = shared->dev.dn; qd.n_col_tiles = (d + bq - 1) / bq;
      const int gg = grid_of(rt * q.n_dense, qg.n_col_tiles), gd = grid_of(rt, qd.n_col_tiles);
      if (j0) {
        gu.g[0] = qg; gu.nb0 = gg;
        { const int rc = launch_gemm<0>(ctx, gu, scb, bits, nf, gg + gu_grid); if (rc) return rc; }
      } else {
        GemmPair one{};
        one.g[0] = qg; one.nb0 = gg;
        { const int rc = launch_gemm<0>(ctx, one, shared->dev.sc_bf16, shared->dev.bits, nq, gg); if (rc) return rc; }
      }
      if (j1) {
        dn.g[0] = qd; dn.nb0 = gd;
      } else {
        GemmPair one{};
        one.g[0] = qd; one.nb0 = gd;
        { const int rc = launch_gemm<1>(ctx, one, shared->dev.sc_bf16, shared->dev.bits, nq, gd); if (rc) return rc; }
      }
    }
    if (!join) { const int rc = launch_gemm<0>(ctx, gu, scb, bits, nf, gu_grid); if (rc) return rc; }
    { const int rc = launch_gemm<1>(ctx, dn, scb, bits, nf, dn.nb0 + dn_grid); if (rc) return rc; }
  }
  combine_kernel<<<T, 256, 0, st>>>(o, pos, o_s, (const uint16_t*)x_dev, (uint16_t*)y_dev, k, d, add_residual);
  HIPCHK(ctx, hipGetLastError());
  return SMOE_OK;
}
