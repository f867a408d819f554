// FP8 expert layer on CDNA4's MX-scaled matrix cores: OCP MX FP8 operands
// (E4M3 codes, one E8M0 scale per 32 consecutive values along K), float32
// accumulation.  The paper runs BF16 and FP8 checkpoints of its model
// (Section 7.1) without describing the FP8 format; MX FP8 is the format the
// gfx950 matrix cores scale natively.
//
//  * permute_mx: the dispatch data movement of an FP8 context quantizes each
//    token's bf16 row once (per 32 values: shared exponent E = floor(log2
//    amax) - 8, codes = RNE(clamp(v / 2^E, +-448))) and writes the codes and
//    scale bytes to every row the token occupies;
//  * GEMM1 / GEMM2: v_mfma_scale_f32_32x32x64_f8f6f4 over 64-deep K steps.
//    Lane l of an operand holds row l % 32: its bytes 0-15 are K [16h, 16h+16)
//    and bytes 16-31 are K [32 + 16h, +16) of the step (h = l / 32), and its
//    scale register carries the scale of K block h of the step (32 values)
//    for that row.  GEMM1's epilogue applies the SwiGLU and quantizes h per
//    32 columns of a row (the two lanes holding a row's 32 columns exchange
//    their maxima), GEMM2 writes float32 y.
//
// Two tile shapes, as in the bf16 layer: the weight-streaming tile for small
// batches (up to 64 rows x 32 or 64 columns, one wave per workgroup, operands
// through the wave's LDS ring) and, for large batches, tiles of up to 256 rows by
// 128 (gate + up) / 256 columns, cut to the 32-row blocks that they hold and
// staged through LDS rings of 128-deep K slices (128 bytes per row, the byte
// layout of the bf16 ring's 64-deep slices), with the scale bytes staged
// alongside.
#include <math.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "pipeline.h"
#include "tiles.h"

namespace moepd {

typedef int32_t v8i32 __attribute__((ext_vector_type(8)));
typedef float f32x16_mx __attribute__((ext_vector_type(16)));
typedef float f32x4_mx __attribute__((ext_vector_type(4)));

constexpr float kE4M3Max = 448.f;

// Shared exponent of a block from its largest magnitude: floor(log2 amax) - 8
// from the float's exponent field (amax = 0 or subnormal gives -127; a
// normal amax never gives more than 119).
__device__ __forceinline__ int mx_exponent(float amax) {
  const int ef = (int)((__float_as_uint(amax) >> 23) & 0xffu);
  const int e = ef - 127 - 8;
  return ef == 0 ? -127 : (e < -127 ? -127 : e);
}

// 2^-e as a float for e in [-127, 119]: exact powers of two (2^127 at most).
__device__ __forceinline__ float pow2_neg(int e) { return ldexpf(1.f, -e); }

// Two values (already scaled) to two E4M3 codes, packed into the low half
// of the result (RNE; the clamp makes |v| <= 448 so nothing overflows).
__device__ __forceinline__ uint32_t e4m3_pair(float a, float b) {
  a = fminf(fmaxf(a, -kE4M3Max), kE4M3Max);
  b = fminf(fmaxf(b, -kE4M3Max), kE4M3Max);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false) & 0xffffu;
}

// ------------------------------------------------------------------ permute + quantize

// One wave per token (per part of its row for small batches, see
// waves_per_row).  Lane l takes 16-byte vector v = v0 + l of the bf16 row
// (8 values); four consecutive lanes hold one 32-value block.
__global__ __launch_bounds__(256) void permute_mx_kernel(const u32x4* __restrict__ x, int T, int k, int H,
                                                         int parts, const int32_t* __restrict__ row_of_slot,
                                                         uint8_t* __restrict__ codes, uint8_t* __restrict__ scales) {
  const int wi = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int t = wi / parts, part = wi - t * parts;
  if (t >= T) return;  // whole wave leaves together
  const int lane = threadIdx.x & 63;
  const int r_l = lane < k ? row_of_slot[(size_t)t * k + lane] : -1;
  const uint64_t resident = __ballot(r_l >= 0);
  if (!resident) return;
  const int nv = H / 8, nb = H / 32;
  const u32x4* xt = x + (size_t)t * nv;
  for (int v0 = part * kWave; v0 < nv; v0 += parts * kWave) {
    const int v = v0 + lane;
    const bool on = v < nv;  // nv is a multiple of 4: a block is all on or all off
    float f[8];
    float amax = 0.f;
    if (on) {
      const u32x4 u = xt[v];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(u[i] << 16);
        f[2 * i + 1] = __uint_as_float(u[i] & 0xffff0000u);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(f[i]));
    }
    amax = fmaxf(amax, __shfl_xor(amax, 1, kWave));
    amax = fmaxf(amax, __shfl_xor(amax, 2, kWave));
    const int e = mx_exponent(amax);
    const float inv = pow2_neg(e);
    uint32_t lo = 0, hi = 0;
    if (on) {
      lo = e4m3_pair(f[0] * inv, f[1] * inv) | (e4m3_pair(f[2] * inv, f[3] * inv) << 16);
      hi = e4m3_pair(f[4] * inv, f[5] * inv) | (e4m3_pair(f[6] * inv, f[7] * inv) << 16);
    }
    uint64_t m = resident;
    while (m) {
      const int j = __builtin_ctzll(m);
      m &= m - 1;
      const int row = __builtin_amdgcn_readlane(r_l, j);
      if (on) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<u32x2*>(codes + (size_t)row * H + (size_t)v * 8) = u32x2{lo, hi};
        if ((lane & 3) == 0) scales[(size_t)row * nb + v / 4] = (uint8_t)(e + 127);
      }
    }
  }
}

hipError_t launch_permute_mx(const void* x, int T, int k, int H, const int32_t* row_of_slot, uint8_t* codes,
                             uint8_t* scales, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  const int parts = waves_per_row(T, H / 8, 1);
  const long long waves = (long long)T * parts;
  permute_mx_kernel<<<dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s>>>((const u32x4*)x, T, k, H, parts,
                                                                             row_of_slot, codes, scales);
  return hipGetLastError();
}

// ------------------------------------------------------------------ grouped GEMM

struct GemmArgsMX {
  const uint8_t* A;   // [R, K] codes, expert-contiguous rows
  const uint8_t* As;  // [R, K / 32] scales
  const uint8_t* B;   // expert e at B + e * b_stride: [N rows (x2 for gate/up), K] codes
  const uint8_t* Bs;  // expert e at Bs + e * bs_stride: [rows, K / 32] scales
  void* C;            // GATED: h codes [R, N]; else float32 y [R, N]
  uint8_t* Cs;        // GATED: h scales [R, N / 32]
  const int32_t* offsets;
  const int32_t* tile_base;
  long long b_stride, bs_stride;
  int e_loc, N, K, n_tiles, up_row;
  int n_group, m_super, xcd_local;
  YieldTo yield;
};

__device__ __forceinline__ v8i32 join(const u32x4& a, const u32x4& b) {
  return v8i32{(int32_t)a[0], (int32_t)a[1], (int32_t)a[2], (int32_t)a[3],
               (int32_t)b[0], (int32_t)b[1], (int32_t)b[2], (int32_t)b[3]};
}

// silu(g) * u (the hardware reciprocal, about 1 ulp, is far inside E4M3's
// rounding of h).
__device__ __forceinline__ float silu_mul_mx(float gt, float up) {
  return gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up;
}

// Small batches: one wave (32 output columns) per workgroup, so that the
// tiles spread evenly over the CUs whatever their count (with four-wave
// workgroups, 1.5 tiles per CU left half the CUs with two).
constexpr int kMxDecodeWaves = 1;

// One wave: up to 32 MB rows of one expert and two blocks of 32 weight rows (gate
// and up, or columns of y), over all of K.  As the bf16 decode tile: a 128-deep
// K block of a panel (32 rows) is 4 KB, moved HBM -> LDS by four 1 KB DMA
// instructions of eight whole 128-byte row pieces each (lane l: row 8i + l/8,
// 16-byte unit l%8; unit c of row r at slot 8r + (c ^ stage_swz(r)), no bank
// conflicts when the fragments are read), SLOTS blocks in the wave's ring, a
// slot refilled once its fragments are in registers.  SC4 (K a multiple of
// 512, scale arrays 16-byte aligned): a 16-byte gather brings a row's scales of
// four blocks into one buffer, read into registers at the first of them;
// otherwise each block's four bytes per row are gathered into its slot.  A
// gather touches a line per row whatever its width.  The MFMAs take the weight
// rows as their first operand, so lane l ends with token row l % 32 of each
// block and the 16 columns 8q + 4h + (0..3), q = 0..3.
//
// DeepSeek-V3-shaped FP8 share, GEMM1 / GEMM2 in us, against 32-row tiles with
// two blocks in flight in registers and scales loaded there: 4 tokens 43 / 16
// -> 28 / 13, 40 tokens 134 / 65 -> 127 / 68, 128 tokens 188 / 90 -> 178 / 94,
// 256 skewed tokens 287 / 153 -> 239 / 120 (the weights alone: 162 / 81).
constexpr int mx_decode_gathers(int mb) { return (mb + 3) / 2; }  // of 64 rows each: mb + 2 panels
constexpr int mx_decode_slot(int mb, bool sc4) {                  // 16-byte chunks
  return (mb + 2) * 256 + (sc4 ? 0 : 16 * mx_decode_gathers(mb));
}
template <int MB, int SLOTS, bool GATED, bool SC4>
__device__ __forceinline__ void gemm_mx_skinny_tile(const GemmArgsMX& g, const TileCoord& tc, u32x4* lds) {
  static_assert(kMxDecodeWaves == 1, "the LDS ring below is private to the workgroup's one wave");
  static_assert(SLOTS >= 1 && SLOTS <= 4, "a group's gathers are older than the block that first needs them");
  constexpr int NB = 2;  // 32 columns of gate and of up, or two blocks of 32 columns
  constexpr int NP = MB + NB, PANEL = 256;
  constexpr int NG = mx_decode_gathers(MB);
  constexpr int SLOT = mx_decode_slot(MB, SC4);
  constexpr int NPS = 4 * NP + (SC4 ? 0 : NG);  // DMA instructions of a block
  u32x4* const scales = lds + SLOTS * SLOT;      // SC4
  const int lane = threadIdx.x & 63;
  const int r = lane & 31, h = lane >> 5;
  const int lr = lane >> 3, lc = lane & 7;
  const int m0 = __builtin_amdgcn_readfirstlane(tc.m0), m_end = __builtin_amdgcn_readfirstlane(tc.m_end);
  const int n0 = __builtin_amdgcn_readfirstlane(tc.n0), e = __builtin_amdgcn_readfirstlane(tc.e);
  const int KS = g.K / 32, KB = g.K / 128;
  const int b_step = GATED ? g.up_row : 32;  // weight rows from one block of 32 to the next
  auto rsrc = [](const uint8_t* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, bytes, kBufferRsrcWord3);
  };
  const __amdgpu_buffer_rsrc_t a_rsrc = rsrc(g.A + (size_t)m0 * g.K, min(m_end - m0, 32 * MB) * g.K);
  const __amdgpu_buffer_rsrc_t b_rsrc = rsrc(g.B + (size_t)e * g.b_stride, (int)g.b_stride);
  int off[2];  // stage_swz repeats every 16 rows
#pragma unroll
  for (int i = 0; i < 2; ++i) off[i] = (8 * i + lr) * g.K + (lc ^ stage_swz(8 * i + lr)) * 16;
  const int row16 = 16 * g.K;
  // Gather q: panel 2q + h, row r of it (the last panel again where they run
  // out); rows past the expert's end repeat its last (never stored).
  const uint8_t* sc_src[NG];
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    const int p = min(2 * q + h, NP - 1);
    sc_src[q] = p < MB ? g.As + (size_t)min(m0 + 32 * p + r, m_end - 1) * KS
                       : g.Bs + (size_t)e * g.bs_stride + (size_t)((p - MB) * b_step + n0 + r) * KS;
  }
  auto issue = [&](int kb, int slot) {
    u32x4* dst = lds + slot * SLOT;
    if constexpr (!SC4) {
#pragma unroll
      for (int q = 0; q < NG; ++q)
        __builtin_amdgcn_global_load_lds(MOEPD_GPTR(sc_src[q] + kb * 4), MOEPD_LPTR(dst + NP * PANEL + q * 16), 4, 0, 0);
    }
#pragma unroll
    for (int p = 0; p < MB; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        // rows past the expert's end lie past the resource: the row part stays in the lane offset, which is checked
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, MOEPD_LPTR(dst + p * PANEL + i * 64), 16,
                                                 off[i & 1] + (2 * p + (i >> 1)) * row16, kb * 128, 0, 0);
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, MOEPD_LPTR(dst + (MB + p) * PANEL + i * 64), 16, off[i & 1],
                                                 kb * 128 + (p * b_step + n0) * g.K + (i >> 1) * row16, 0, 0);
  };
  auto issue_group = [&](int kb) {
#pragma unroll
    for (int q = 0; q < NG; ++q)
      __builtin_amdgcn_global_load_lds(MOEPD_GPTR(sc_src[q] + kb * 4), MOEPD_LPTR(scales + q * 64), 16, 0, 0);
  };
  // Step s (64 deep) of a block: lane (r, h) holds units 4s + h and 4s + 2 + h
  // of its row and the scale of 32-value block 2s + h.
  int rslot[2][2];
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int u = 0; u < 2; ++u) rslot[st][u] = r * 8 + ((4 * st + 2 * u + h) ^ stage_swz(r));

  f32x16_mx acc[MB][NB];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[m][j][q] = 0.f;

  u32x4 raw[NP];  // SC4: the panels' scale words of four blocks; else the 16 bytes that hold this block's
  if constexpr (SC4) issue_group(0);
#pragma unroll
  for (int q = 0; q < SLOTS; ++q)
    if (q < KB) issue(q, q);
  int slot = 0;
  for (int kb = 0; kb < KB; ++kb) {
    // block kb has landed once at most the newer blocks remain (a group's
    // gathers among them make the wait stricter)
    wait_rings_lgkm0<NPS, 0, SLOTS - 1, 0>(KB - 1 - kb);
    const u32x4* src = lds + slot * SLOT;
    v8i32 f[2][NP];
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int p = 0; p < NP; ++p) f[st][p] = join(src[p * PANEL + rslot[st][0]], src[p * PANEL + rslot[st][1]]);
    if constexpr (SC4) {
      if ((kb & 3) == 0)
#pragma unroll
        for (int p = 0; p < NP; ++p) raw[p] = scales[32 * p + r];
    } else {
#pragma unroll
      for (int p = 0; p < NP; ++p) raw[p] = src[NP * PANEL + (32 * p + r) / 4];
    }
    wait_vmcnt_lgkm0<63>();  // the block is in registers: its slot is free
    if constexpr (SC4) {
      if ((kb & 3) == 0 && kb + 4 < KB) issue_group(kb + 4);
    }
    if (kb + SLOTS < KB) issue(kb + SLOTS, slot);
    uint32_t scl[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int c = SC4 ? kb & 3 : lane & 3;
      scl[p] = (c == 0 ? raw[p][0] : c == 1 ? raw[p][1] : c == 2 ? raw[p][2] : raw[p][3]) >> (8 * h);
    }
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[m][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f[st][MB + j], f[st][m], acc[m][j], 0, 0, 0,
                                                                      (int)(scl[MB + j] >> (16 * st)), 0,
                                                                      (int)(scl[m] >> (16 * st)));
    if (++slot == SLOTS) slot = 0;
  }

#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int row = m0 + 32 * m + r;
    const bool live = row < m_end;
    if (GATED) {
      float v[16];
      float amax = 0.f;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        v[q] = silu_mul_mx(acc[m][0][q], acc[m][NB - 1][q]);
        amax = fmaxf(amax, fabsf(v[q]));
      }
      amax = fmaxf(amax, __shfl_xor(amax, 32, kWave));  // the row's other 16 columns
      if (!live) continue;
      const int ex = mx_exponent(amax);
      const float inv = pow2_neg(ex);
      uint8_t* hrow = static_cast<uint8_t*>(g.C) + (size_t)row * g.N + n0 + 4 * h;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t w = e4m3_pair(v[4 * q] * inv, v[4 * q + 1] * inv) |
                           (e4m3_pair(v[4 * q + 2] * inv, v[4 * q + 3] * inv) << 16);
        *reinterpret_cast<uint32_t*>(hrow + 8 * q) = w;
      }
      if (h == 0) g.Cs[(size_t)row * (g.N / 32) + n0 / 32] = (uint8_t)(ex + 127);
    } else {
      if (!live) continue;
      float* yrow = static_cast<float*>(g.C) + (size_t)row * g.N + n0 + 4 * h;
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4_mx*>(yrow + 32 * j + 8 * q) =
              f32x4_mx{acc[m][j][4 * q], acc[m][j][4 * q + 1], acc[m][j][4 * q + 2], acc[m][j][4 * q + 3]};
    }
  }
}

// ------------------------------------------------------------------ LDS ring (prefill)

// One workgroup of 4 waves, a BM x BN output tile of one expert.  Per
// 128-deep K slice, A (BM rows) and B (BR = NB x BN weight rows) travel HBM ->
// LDS by 16-byte DMA (swizzled like the bf16 ring) into a ring of SA slots
// for A and one of SB >= SA slots for B: the weights, whose first touch goes
// to HBM, run one slice further ahead where the LDS has room for it.  A slice
// is two 64-deep MFMA steps; fragments of the next step are read from LDS
// while the current step's MFMAs run, and the slice's barrier sits between
// its steps, when every wave holds step 1's fragments.  After the barrier of
// slice kt its slots are free: A(kt + SA) goes out beside the MFMAs of step 1
// and B(kt + SB) beside those of the next slice's step 0, so the queue holds
// ..., A(kt + SA), B(kt + SB), A(kt + 1 + SA), ... in this order.
//
// Scale bytes (one per 32 values, four per row and slice) are gathered by
// DMA from one line per row.  SC4 (K a multiple of 512, the scale arrays
// 16-byte aligned): one 16-byte gather brings a row's scales of four slices
// into a single buffer, read into registers at the group's first slice and
// refilled after that slice's barrier; otherwise each slice gathers four bytes
// per row into a slot that goes with A's.  A gather touches 64 lines whatever
// its width, as many as the codes of 64 rows: with a gather per slice the
// scales cost 12 % of the 8192-token layer's GEMM1 (368 us with every lane
// reading one row's scales, 420 in full).
//
// Each wave counts its own DMA instructions: loads complete in order, every
// wave issues the same ones (a gather is repeated where rows run out), so a
// counted wait at a slice's barrier retires exactly what the next slice needs
// (with a group's gathers in flight, two instructions more).
constexpr int mx_scale_rows(int bm) { return (bm + 63) / 64 * 64; }  // A rows in whole gathers
constexpr int kMxB = 256;                                             // weight rows of a ring tile
constexpr int kMxTallRows = 256;                                      // rows of the tallest ring tile
constexpr int kMxRingRows = 192;                                      // and of the others
// 16-byte chunks of LDS: the rings, and the scale area in its larger form.
constexpr int mx_ring_chunks(int bm, int sa, int sb) {
  return sa * bm * 8 + sb * kMxB * 8 + (sa > 4 ? sa : 4) * (mx_scale_rows(bm) + kMxB) / 4;
}

// TALL names the kernel that the body is part of (gemm_mx_ring): each has its own,
// since the host pass cannot use one body from two kernels.
template <int BM, int WM, int WN, int SA, int SB, bool GATED, bool SC4, bool TALL>
__device__ __forceinline__ void gemm_mx_ring_body(const GemmArgsMX& g, const TileCoord& tc, u32x4* lds) {
  constexpr int BR = kMxB;
  constexpr int NB = GATED ? 2 : 1;
  constexpr int BN = BR / NB;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int FM = WTM / 32, FN = WTN / 32, FB = FN * NB;
  constexpr int BK = 128;                           // K values (bytes) per slice
  constexpr int CPR = 8;                            // 16-byte chunks per staged row
  constexpr int RPI = 8;                            // rows per 16-byte DMA instruction
  constexpr int A_INS = BM / RPI / 4, B_INS = BR / RPI / 4;
  constexpr int SC_A = mx_scale_rows(BM), SC_W = SC_A + BR;  // scale rows of a slot
  constexpr int SC_INS = 2;                         // gathers per wave: one of A's rows, one of B's
  constexpr int NA = A_INS + (SC4 ? 0 : SC_INS);    // DMA instructions per wave of an A and a B group
  constexpr int A_CH = BM * CPR, B_CH = BR * CPR;
  constexpr int NRD = FM + FB, NMF = FM * FB;
  static_assert(WM * WN == 4, "four waves");
  static_assert(A_INS * RPI * 4 == BM && B_INS * RPI * 4 == BR, "slices split into whole DMA instructions");
  static_assert(BR == 4 * 64 && SC_A <= 4 * 64, "one gather of 64 rows per wave");
  static_assert(FM * 32 == WTM && FN * 32 == WTN, "wave tile must be a multiple of 32x32");
  static_assert(SA >= 2 && (SB == SA || SB == SA + 1) && NA * (SA - 1) + B_INS * (SB - 1) < 64, "pipeline depth");
  constexpr bool BNOW = SB == 2;                    // B goes out with A
  static_assert(SA <= 4, "a group's gathers, issued at its first slice, are older than the next group's A");
  u32x4(*const ring_a)[A_CH] = reinterpret_cast<u32x4(*)[A_CH]>(lds);
  u32x4(*const ring_b)[B_CH] = reinterpret_cast<u32x4(*)[B_CH]>(lds + SA * A_CH);
  u32x4* const scales = lds + SA * A_CH + SB * B_CH;

  const int lane = threadIdx.x & 63;
  const int h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int KT = g.K / BK;
  const int KS = g.K / 32;  // scale bytes per row
  const int lrow = lane / CPR, lphys = lane % CPR;

  // All operands are read through buffer resources with 32-bit lane offsets:
  // per-lane row and chunk in a vector register, the K offset (and B's row
  // group) in the scalar one, so an issue takes no vector instruction.
  // A's resource covers exactly the tile's rows of its expert: rows past the
  // end lie outside it, so their loads return zeros and make no memory
  // request.  Groups of eight weight rows past N (a multiple of 128) and scale
  // rows past the end read the last ones; their outputs are never stored.
  const int m0 = __builtin_amdgcn_readfirstlane(tc.m0);
  const int m_end = __builtin_amdgcn_readfirstlane(tc.m_end);
  const int n0 = __builtin_amdgcn_readfirstlane(tc.n0);
  const int e = __builtin_amdgcn_readfirstlane(tc.e);
  auto rsrc = [](const uint8_t* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, bytes, kBufferRsrcWord3);
  };
  const __amdgpu_buffer_rsrc_t a_rsrc = rsrc(g.A + (size_t)m0 * g.K, min(m_end - m0, BM) * g.K);
  const __amdgpu_buffer_rsrc_t b_rsrc = rsrc(g.B + (size_t)e * g.b_stride, (int)g.b_stride);
  const __amdgpu_buffer_rsrc_t as_rsrc = rsrc(g.As + (size_t)m0 * KS, (m_end - m0) * KS);
  const __amdgpu_buffer_rsrc_t bs_rsrc = rsrc(g.Bs + (size_t)e * g.bs_stride, (int)g.bs_stride);
  auto brow_of = [&](int r) {  // weight row of staged row r (a multiple of 8, or any row of such a group)
    if (GATED) return r < BN ? n0 + r : g.up_row + n0 + r - BN;
    return n0 + r < g.N ? n0 + r : g.N - 8 + (r & 7);
  };
  // Staged row r = 8 (wave INS + i) + lrow holds chunk c of its row at slot
  // c ^ swz(r), and swz(r) depends on r modulo 16 alone.
  int a_off[A_INS], b_off[2], b_row[B_INS];
#pragma unroll
  for (int i = 0; i < A_INS; ++i) {
    const int r = (wave * A_INS + i) * RPI + lrow;
    a_off[i] = r * g.K + (lphys ^ swz<64>(r)) * 16;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) b_off[i] = lrow * g.K + (lphys ^ swz<64>((wave * B_INS + i) * RPI + lrow)) * 16;
#pragma unroll
  for (int i = 0; i < B_INS; ++i) b_row[i] = __builtin_amdgcn_readfirstlane(brow_of((wave * B_INS + i) * RPI)) * g.K;
  const int sc_a = wave % (SC_A / 64) * 64;  // first A row of this wave's gather
  const int sa_off = min(sc_a + lane, m_end - m0 - 1) * KS;
  const int sb_off = brow_of(wave * 64 + lane) * KS;

  // Scales of slice kt into slot `slot`, or (SC4) of the group that starts at
  // slice kt into the one buffer.
  auto issue_scales = [&](int kt, int slot) {
    if constexpr (SC4) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(as_rsrc, MOEPD_LPTR(scales + sc_a), 16, sa_off, kt * 4, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(bs_rsrc, MOEPD_LPTR(scales + SC_A + wave * 64), 16, sb_off, kt * 4, 0,
                                               0);
    } else {
      u32x4* s = scales + slot * (SC_W / 4);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(as_rsrc, MOEPD_LPTR(s + sc_a / 4), 4, sa_off, kt * 4, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(bs_rsrc, MOEPD_LPTR(s + (SC_A + wave * 64) / 4), 4, sb_off, kt * 4, 0,
                                               0);
    }
  };
  // Instruction i of A(kt): the scale gathers first where they go with A.
  auto issue_a = [&](int i, int kt, int slot) {
    if (!SC4 && i < SC_INS) {
      if (i == 0) issue_scales(kt, slot);
      return;
    }
    i -= SC4 ? 0 : SC_INS;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, MOEPD_LPTR(&ring_a[slot][(wave * A_INS + i) * 64]), 16, a_off[i],
                                             kt * BK, 0, 0);
  };
  auto issue_b = [&](int i, int kt, int slot) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, MOEPD_LPTR(&ring_b[slot][(wave * B_INS + i) * 64]), 16,
                                             b_off[i & 1], b_row[i] + kt * BK, 0, 0);
  };

  // step s of a slice: lane half h takes chunks 4s + h and 4s + 2 + h of its
  // row (K [64s + 16h, +16) and [64s + 32 + 16h, +16)); its scale word holds
  // the slice's four block scales, of which step s uses byte 2s + h.
  v8i32 fa[2][FM], fb[2][FB];
  u32x4 sa_raw[FM], sb_raw[FB];
  uint32_t sa[FM], sb[FB];
  // Fragment i of step `sub`: A's FM row blocks, then B's FB column blocks
  // (gate, up).
  auto read_frag = [&](int i, int aslot, int bslot, int sub, v8i32 (&a)[FM], v8i32 (&b)[FB]) {
    const int c0 = 4 * sub + h, c1 = 4 * sub + 2 + h;
    if (i < FM) {
      const int r = wm * WTM + i * 32 + (lane & 31);
      a[i] = join(ring_a[aslot][r * CPR + (c0 ^ swz<64>(r))], ring_a[aslot][r * CPR + (c1 ^ swz<64>(r))]);
    } else {
      const int j = i - FM, r = j / FN * BN + wn * WTN + j % FN * 32 + (lane & 31);
      b[j] = join(ring_b[bslot][r * CPR + (c0 ^ swz<64>(r))], ring_b[bslot][r * CPR + (c1 ^ swz<64>(r))]);
    }
  };
  // SC4: a row's 16 bytes, the words of four slices.  Otherwise the 16 bytes
  // that hold the row's word among four rows' (4-byte LDS reads right after
  // the DMA issue made the compiler wait for every outstanding DMA, vmcnt(0),
  // in the K loop).
  auto read_scales = [&](int slot) {
    const u32x4* S = SC4 ? scales : scales + slot * (SC_W / 4);
    constexpr int SH = SC4 ? 0 : 2;
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) sa_raw[fm] = S[(wm * WTM + fm * 32 + (lane & 31)) >> SH];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        sb_raw[nb * FN + fn] = S[(SC_A + nb * BN + wn * WTN + fn * 32 + (lane & 31)) >> SH];
  };
  // the lane's word of slice kt, shifted to block h
  auto pick = [&](const u32x4& v, int kt) {
    const int c = SC4 ? kt & 3 : lane & 3;
    const uint32_t w = c == 0 ? v[0] : c == 1 ? v[1] : c == 2 ? v[2] : v[3];
    return w >> (8 * h);
  };

  f32x16_mx acc[FM][FB];
  auto mfma = [&](int i, int sub, const v8i32 (&a)[FM], const v8i32 (&b)[FB]) {
    const int fm = i / FB, j = i % FB;
    acc[fm][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b[j], a[fm], acc[fm][j], 0, 0, 0,
                                                                 (int)(sb[j] >> (16 * sub)), 0,
                                                                 (int)(sa[fm] >> (16 * sub)));
  };
  auto no_op = [](auto) {};

  if constexpr (SC4) issue_scales(0, 0);
#pragma unroll
  for (int st = 0; st < SB; ++st) {
    if (st >= KT) break;
    if (st < SA)
#pragma unroll
      for (int i = 0; i < NA; ++i) issue_a(i, st, st);
#pragma unroll
    for (int i = 0; i < B_INS; ++i) issue_b(i, st, st);
  }

#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  wait_rings_lgkm0<NA, B_INS, SA - 1, SB - 1>(KT - 1);
  bare_barrier();
#pragma unroll
  for (int i = 0; i < FM + FB; ++i) read_frag(i, 0, 0, 0, fa[0], fb[0]);
  read_scales(0);

  // One K slice.  LAST: the tile's last slice (no barrier, nothing to read
  // ahead).  FILL: A(kt + SA) exists.  PEND: B(kt - 1 + SB) exists and is still
  // to go out, into the slot that slice kt - 1 freed.
  auto slice = [&](auto last, auto fill, auto pend, int kt, int aslot, int bslot) {
    constexpr bool LAST = decltype(last)::value, FILL = decltype(fill)::value, PEND = decltype(pend)::value;
#pragma unroll
    for (int i = 0; i < FM; ++i) sa[i] = pick(sa_raw[i], kt);
#pragma unroll
    for (int j = 0; j < FB; ++j) sb[j] = pick(sb_raw[j], kt);
    // step 0: read step 1's fragments, multiply step 0
    weave<NMF, NRD, PEND && !BNOW ? B_INS : 0>([&](auto i) { mfma(i, 0, fa[0], fb[0]); },
                                               [&](auto i) { read_frag(i, aslot, bslot, 1, fa[1], fb[1]); },
                                               [&](auto i) { issue_b(i, kt - 1 + SB, bslot == 0 ? SB - 1 : bslot - 1); });
    auto mul1 = [&](auto i) { mfma(i, 1, fa[1], fb[1]); };
    if constexpr (!LAST) {
      if constexpr (FILL || PEND) wait_vmcnt_lgkm0<NA*(SA - 2) + B_INS * (SB - 2)>();
      else wait_rings_lgkm0<NA, B_INS, SA - 2, SB - 2>(KT - 2 - kt);
      bare_barrier();
      const int na = aslot + 1 == SA ? 0 : aslot + 1, nb = bslot + 1 == SB ? 0 : bslot + 1;
      if constexpr (SC4) {
        if ((kt & 3) == 0 && kt + 4 < KT) issue_scales(kt + 4, 0);
        if ((kt & 3) == 3) read_scales(0);
      }
      if constexpr (!SC4) read_scales(na);
      weave<NMF, NRD, FILL ? NA + (BNOW ? B_INS : 0) : 0>(
          mul1, [&](auto i) { read_frag(i, na, nb, 0, fa[0], fb[0]); },
          [&](auto i) {
            if constexpr (i < NA) issue_a(i, kt + SA, aslot);
            else issue_b(i - NA, kt + SB, bslot);
          });
    } else {
      weave<NMF, 0, 0>(mul1, no_op, no_op);
    }
  };
  int kt = 0, aslot = 0, bslot = 0;
  auto advance = [&] {
    ++kt;
    if (++aslot == SA) aslot = 0;
    if (++bslot == SB) bslot = 0;
  };
  using T = std::true_type;
  using F = std::false_type;
  if (KT > SA) {
    slice(F{}, T{}, F{}, kt, aslot, bslot);  // the prologue's groups went out whole
    advance();
    while (kt < KT - SA) {
      slice(F{}, T{}, T{}, kt, aslot, bslot);
      advance();
    }
    if constexpr (SB == SA && !BNOW) {  // B(KT - 1)
      slice(F{}, F{}, T{}, kt, aslot, bslot);
      advance();
    }
  }
  while (kt < KT - 1) {
    slice(F{}, F{}, F{}, kt, aslot, bslot);
    advance();
  }
  slice(T{}, F{}, F{}, kt, aslot, bslot);
  // The last MFMAs, and the vector code that picks their scales, stay above
  // the epilogue's per-row branches: under a partial EXEC mask the picks would
  // leave the scales of weight rows on masked lanes unset.
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j) asm volatile("" : "+a"(acc[i][j]));

  // epilogue (lane l: row l & 31 of each 32-row block, columns 8q + 4h + t)
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    const int row = tc.m0 + wm * WTM + fm * 32 + (lane & 31);
    const bool live = row < tc.m_end;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const int col0 = tc.n0 + wn * WTN + fn * 32;  // a 32-column block: all in range or all out
      if (GATED) {
        float v[16];
        float amax = 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          v[q] = silu_mul_mx(acc[fm][fn][q], acc[fm][FN + fn][q]);
          amax = fmaxf(amax, fabsf(v[q]));
        }
        amax = fmaxf(amax, __shfl_xor(amax, 32, kWave));
        if (!live || col0 >= g.N) continue;
        const int e = mx_exponent(amax);
        const float inv = pow2_neg(e);
        uint8_t* hrow = static_cast<uint8_t*>(g.C) + (size_t)row * g.N + col0 + 4 * h;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t w = e4m3_pair(v[4 * q] * inv, v[4 * q + 1] * inv) |
                             (e4m3_pair(v[4 * q + 2] * inv, v[4 * q + 3] * inv) << 16);
          *reinterpret_cast<uint32_t*>(hrow + 8 * q) = w;
        }
        if (h == 0) g.Cs[(size_t)row * (g.N / 32) + col0 / 32] = (uint8_t)(e + 127);
      } else {
        if (!live || col0 >= g.N) continue;
        float* yrow = static_cast<float*>(g.C) + (size_t)row * g.N + col0 + 4 * h;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4_mx*>(yrow + 8 * q) =
              f32x4_mx{acc[fm][fn][4 * q], acc[fm][fn][4 * q + 1], acc[fm][fn][4 * q + 2], acc[fm][fn][4 * q + 3]};
      }
    }
  }
}

// A ring tile, cut to the 32-row blocks it holds: an expert's rows are shared
// evenly among its m-tiles, and a tile's MFMAs, A transfers and fragment reads
// all go with the rows it is built for.  Up to 160 rows the four waves stand
// side by side along N (each reads every A fragment and its own weights'); the
// taller tiles take a 2 x 2 grid, whose fragment reads per MFMA are fewer.  The
// LDS that shorter tiles leave goes to more slots.  What bounds these tiles is
// the LDS (fragment reads and DMA writes, about as many cycles as the MFMAs at
// 160 rows) and, with few rows, the weight stream.  The DeepSeek-V3-shaped
// share (H 7168, I 2048, 32 experts), P alone, GEMM1 / GEMM2 in us, one tile
// of 256 rows for any number of rows -> cut to the rows:
//   32 rows per expert   237 / 128 -> 184 / 101 (5.3 TB/s of weights in GEMM1)
//   128                  263 / 155 -> 208 / 135
//   256                  444 / 236 -> 317 / 204
//   512                  616 / 365 -> 521 / 353
// and with 47 rows per expert at H 2560, I 768 (64 experts) 90 / 50 -> 65 / 43.
//
// TALL: the batch's m-tiles hold up to 256 rows (ffn_mx_bm), else up to 192.
// Without the 256-row body a kernel takes 440 registers and 151 KB of LDS instead of
// 512 and 160, spills nothing, and leaves a CU room for the other phase's route,
// permute and combine waves: at 512 experts, H 2560, I 768, D's layer of 256 tokens
// under 8192-token prefills 199 -> 169 us, with the prefill alone as fast.
constexpr int mx_lds_chunks(bool tall) { return tall ? 160 * 1024 / 16 : mx_ring_chunks(kMxRingRows, 2, 3); }
template <bool GATED, bool SC4, bool TALL>
__device__ __forceinline__ void gemm_mx_ring(const GemmArgsMX& g) {
  __shared__ u32x4 lds[mx_lds_chunks(TALL)];
  const int L = block_tile(g);
  if (L < 0) return;
  yield_to_window(g.yield);
  TileCoord tc;
  tile_at(g, L, TALL ? kMxTallRows : kMxRingRows, GATED ? 128 : 256, tc);
  const int blocks = __builtin_amdgcn_readfirstlane((tc.m_end - tc.m0 + 31) / 32);
#define MOEPD_MX_RING(BM, WM, WN, SA, SB, SC4)                                           \
  do {                                                                                   \
    static_assert(mx_ring_chunks(BM, SA, SB) <= mx_lds_chunks(TALL), "ring exceeds the LDS"); \
    gemm_mx_ring_body<BM, WM, WN, SA, SB, GATED, SC4, TALL>(g, tc, lds);                     \
  } while (0)
  if (blocks <= 1) MOEPD_MX_RING(32, 1, 4, 3, 4, SC4);
  else if (blocks == 2) MOEPD_MX_RING(64, 1, 4, 3, 3, SC4);
  else if (blocks == 3) MOEPD_MX_RING(96, 1, 4, 3, 3, SC4);
  else if (blocks == 4) MOEPD_MX_RING(128, 1, 4, 3, 3, SC4);
  else if (blocks == 5) MOEPD_MX_RING(160, 1, 4, 2, 3, SC4);
  else if (!TALL || blocks == 6) MOEPD_MX_RING(192, 2, 2, 2, 3, SC4);
  else if constexpr (TALL) MOEPD_MX_RING(256, 2, 2, 2, 2, SC4);
#undef MOEPD_MX_RING
}
// With the 256-row body and the four-slice scale gathers the registers are all
// 512, and five (GEMM1) and four (GEMM2) values are spilled around the K loops, none
// inside them.
template <bool SC4, bool TALL>
__global__ __launch_bounds__(256) void gemm1_mx_prefill(GemmArgsMX g) { gemm_mx_ring<true, SC4, TALL>(g); }
template <bool SC4, bool TALL>
__global__ __launch_bounds__(256) void gemm2_mx_prefill(GemmArgsMX g) { gemm_mx_ring<false, SC4, TALL>(g); }

// Small-batch tiles of up to kMxDecodeRows rows, cut to their 32-row blocks (64 is
// what one slot and the scales of the eight-per-CU form take; with 96 rows and
// six per CU instead, 40 tokens at H 7168 took 145 us for GEMM1 against 127,
// 256 skewed ones 225 against 239).  GEMM1's are 32 columns of gate and up,
// GEMM2's 64 columns.
constexpr int kMxDecodeRows = 64;
constexpr int mx_decode_chunks(int form) { return decode_lds(form, true) / 16; }
constexpr int mx_decode_slots(int mb, int form, bool sc4) {
  const int n = (mx_decode_chunks(form) - (sc4 ? 64 * mx_decode_gathers(mb) : 0)) / mx_decode_slot(mb, sc4);
  return n > 4 ? 4 : n;
}
template <bool GATED, bool SC4, int FORM>
__global__ __launch_bounds__(64 * kMxDecodeWaves) void gemm_mx_skinny(GemmArgsMX g) {
  __shared__ u32x4 lds[mx_decode_chunks(FORM)];
  const int L = block_tile(g);
  if (L < 0) return;
  yield_to_window(g.yield);
  TileCoord tc;
  tile_at(g, L, kMxDecodeRows, GATED ? 32 : 64, tc);
  const int blocks = __builtin_amdgcn_readfirstlane((tc.m_end - tc.m0 + 31) / 32);
  if (blocks <= 1) gemm_mx_skinny_tile<1, mx_decode_slots(1, FORM, SC4), GATED, SC4>(g, tc, lds);
  else gemm_mx_skinny_tile<2, mx_decode_slots(2, FORM, SC4), GATED, SC4>(g, tc, lds);
}

static inline int round8_mx(long long v) { return (int)((v + 7) / 8 * 8); }

hipError_t launch_ffn_mx(int regime, int gemm, const PhaseBuffers& b, const MxBuffers& mx, const MxWeights& w,
                         int e_loc, int H, int I, int bm, int max_m_tiles, double m_tiles_hint, Beside beside,
                         YieldTo yield, hipStream_t s) {
  GemmArgsMX g{};
  g.offsets = b.offsets;
  g.tile_base = b.tile_base;
  g.e_loc = e_loc;
  g.yield = yield;
  g.n_group = 1;
  g.xcd_local = 1;
  if (gemm == 1) {
    g.A = mx.x_codes;
    g.As = mx.x_scales;
    g.B = (const uint8_t*)w.gu;
    g.Bs = (const uint8_t*)w.gu_scales;
    g.C = mx.h_codes;
    g.Cs = mx.h_scales;
    g.b_stride = 2LL * I * H;
    g.bs_stride = 2LL * I * (H / 32);
    g.N = I;
    g.K = H;
    g.up_row = I;
  } else {
    g.A = mx.h_codes;
    g.As = mx.h_scales;
    g.B = (const uint8_t*)w.dn;
    g.Bs = (const uint8_t*)w.dn_scales;
    g.C = b.y;
    g.Cs = nullptr;
    g.b_stride = (long long)H * I;
    g.bs_stride = (long long)H * (I / 32);
    g.N = H;
    g.K = I;
    g.up_row = 0;
  }
  if (regime == 0) {
    g.n_tiles = gemm == 1 ? (g.N + 127) / 128 : (g.N + 255) / 256;
    const dim3 grid(round8_mx((long long)max_m_tiles * g.n_tiles));
    // a row's scales of four slices in one aligned 16-byte gather
    const bool sc4 = g.K % 512 == 0 && ((uintptr_t)g.As | (uintptr_t)g.Bs) % 16 == 0;
    auto go = [&](auto k) { k<<<grid, 256, 0, s>>>(g); };
    if (bm == kMxTallRows) {
      if (gemm == 1) sc4 ? go(gemm1_mx_prefill<true, true>) : go(gemm1_mx_prefill<false, true>);
      else sc4 ? go(gemm2_mx_prefill<true, true>) : go(gemm2_mx_prefill<false, true>);
    } else {
      if (gemm == 1) sc4 ? go(gemm1_mx_prefill<true, false>) : go(gemm1_mx_prefill<false, false>);
      else sc4 ? go(gemm2_mx_prefill<true, false>) : go(gemm2_mx_prefill<false, false>);
    }
  } else {
    g.n_tiles = g.N / (gemm == 1 ? 32 : 64);
    g.xcd_local = g.n_tiles % 8 == 0 ? 2 : 1;
    const dim3 grid(round8_mx((long long)max_m_tiles * g.n_tiles));
    const bool sc4 = g.K % 512 == 0 && ((uintptr_t)g.As | (uintptr_t)g.Bs) % 16 == 0;
    auto go = [&](auto k) { k<<<grid, 64 * kMxDecodeWaves, 0, s>>>(g); };
    auto form = [&](auto f) {
      constexpr int F = decltype(f)::value;
      if (gemm == 1) sc4 ? go(gemm_mx_skinny<true, true, F>) : go(gemm_mx_skinny<true, false, F>);
      else sc4 ? go(gemm_mx_skinny<false, true, F>) : go(gemm_mx_skinny<false, false, F>);
    };
    switch (decode_form(m_tiles_hint * g.n_tiles, beside)) {
      case kDecodeRoom: form(std::integral_constant<int, kDecodeRoom>{}); break;
      case kDecodeSix: form(std::integral_constant<int, kDecodeSix>{}); break;
      case kDecodeEight: form(std::integral_constant<int, kDecodeEight>{}); break;
      default: form(std::integral_constant<int, kDecodeFour>{});
    }
  }
  return hipGetLastError();
}

// Rows per m-tile of the ring: an expert of r rows takes ceil(r / this) tiles.
// 192, unless taller tiles save most experts one: an expert's rows scatter
// about the expected count by its square root, so that is asked at one such
// deviation above it.  A 256-row tile has room for two slots of each ring only,
// and two tiles of half its rows take about its time, so it pays where the
// number of tiles (and of rounds over the CUs) falls.  The share above, whole
// layer in us, 192 / 256:  192 rows 621 / 558,  224 rows 627 / 589,
// 256 rows 669 / 727,  320 rows 774 / 776,  384 rows 938 / 932,
// 512 rows 1127 / 1175;  skewed 16384-token batch 5680 / 5882.
int ffn_mx_bm(int regime, long long avg_rows) {
  if (regime != 0) return kMxDecodeRows;
  long long dev = 0;
  while ((dev + 1) * (dev + 1) <= avg_rows) ++dev;
  const long long r = avg_rows + dev;
  return (r + kMxTallRows - 1) / kMxTallRows < (r + kMxRingRows - 1) / kMxRingRows ? kMxTallRows : kMxRingRows;
}

}  // namespace moepd
