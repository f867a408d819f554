// Building blocks of the LDS-ring GEMMs (bf16 and MX FP8): counted waits on
// this wave's vector-memory operations, the fence-free workgroup barrier,
// the LDS row swizzle, the order of a step's instructions, and the raw
// buffer-resource word used for bounds-checked DMA.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace moepd {

// Word 3 of a raw (unstructured) buffer resource on gfx9: 32-bit data
// format, no swizzle; out-of-range loads return zero without a memory access.
constexpr int kBufferRsrcWord3 = 0x00020000;

#define MOEPD_GPTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define MOEPD_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

// The swizzle depends on the row length.
// A staged row is BK bf16 = 2 BK bytes = CPR 16-byte chunks, and 256 / (2 BK)
// rows share one 256-byte sweep of the 64 LDS banks.  Chunk c of row r is
// stored at c ^ swz(r), swz(r) = (r / rows_per_sweep) % CPR, so the 16 lanes
// that a ds_read_b128 serves together (16 consecutive rows, one chunk each)
// cover all 64 banks once.
template <int BK>
__device__ __forceinline__ int swz(int row) {
  constexpr int CPR = BK / 8, RPS = 256 / (2 * BK);
  return (row / RPS) & (CPR - 1);
}

// Swizzle of the small-batch tiles' per-wave LDS stage: a 64-deep K block of
// 32 rows, chunk c (16 bytes) of row r at slot 8 r + (c ^ stage_swz(r)).  A
// 16-lane group of the whole-line writes covers two rows, which share the
// swizzle, so it writes 256 consecutive bytes; a 16-lane group of the MFMA
// reads takes one chunk of 16 consecutive rows, whose slots then fall on
// (r % 2, stage_swz(r)) = 16 different 16-byte bank groups.  (Swizzling by
// r % 8 put rows r and r + 8 on the same banks: two-way conflicts.)
__device__ __forceinline__ int stage_swz(int row) { return (row >> 1) & 7; }

// Workgroup barrier without a memory fence; the signal fences keep the
// compiler from moving LDS accesses across it.  Visibility of the DMA'd
// stages is established by wait_vmcnt before the barrier.
__device__ __forceinline__ void bare_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// s_waitcnt vmcnt(n) lgkmcnt(0): this wave's LDS reads are done and at most
// n of its vector-memory operations are outstanding (gfx9 encoding: vmcnt[3:0],
// expcnt[6:4], lgkmcnt[11:8], vmcnt[5:4] in bits [15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x70);
}

// Wait until at most NA min(CA, n) + NB min(CB, n) DMA instructions (and no LDS
// operation) of this wave are in flight; n is wave-uniform, n >= 0.
template <int NA, int NB, int CA, int CB, int N = (CA > CB ? CA : CB)>
__device__ __forceinline__ void wait_rings_lgkm0(int n) {
  if constexpr (N > 0) {
    if (n < N) return wait_rings_lgkm0<NA, NB, CA, CB, N - 1>(n);
  }
  wait_vmcnt_lgkm0<NA*(CA < N ? CA : N) + NB * (CB < N ? CB : N)>();
}

// f(I), ..., f(N - 1), each index an integral constant.
template <int I, int N, class F>
__device__ __forceinline__ void weave_run(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    weave_run<I + 1, N>(f);
  }
}

// One step of a ring GEMM: NM MFMAs with NR LDS reads and ND DMA issues
// placed between them, in exactly this order (a scheduling barrier after each
// MFMA holds it): the reads go behind the first three quarters of the MFMAs, so
// they have the rest to land before the next step needs them, and the DMA
// issues are spread over all of them, so the texture path, which takes a 1 KB
// instruction in about 16 cycles, never makes a wave wait to issue.  m, r and d
// take the index of the MFMA, read or issue as an integral constant.  Left to
// scheduling-group hints the compiler put the slice end's issues before its
// MFMAs: the 16384-token skewed layer's 256-row GEMMs 4700 / 2545 us with
// scalar-offset transfers so, 4225 / 2490 as the hints fell with 64-bit
// addresses, 4070 / 2450 in this order.  Reads over half or a quarter of the
// MFMAs, and issues over their second half, measured within 1 %.
template <int NM, int NR, int ND, int I = 0, class M, class R, class D>
__device__ __forceinline__ void weave(M&& m, R&& r, D&& d) {
  if constexpr (I < NM) {
    constexpr int H = (3 * NM + 3) / 4;
    m(std::integral_constant<int, I>{});
    if constexpr (I < H) weave_run<NR * I / H, NR*(I + 1) / H>(r);
    weave_run<ND * I / NM, ND*(I + 1) / NM>(d);
    __builtin_amdgcn_sched_barrier(0);
    weave<NM, NR, ND, I + 1>(m, r, d);
  }
}

}  // namespace moepd
