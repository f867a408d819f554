// Grouped expert FFN in float32 (contexts created with MOE_DTYPE_F32).
//
// Same contraction and device-side tile schedule as the bf16 path (see
// ffn_bf16.hip): GEMM1 h = silu(x_perm W1^T) * (x_perm W3^T) with the SwiGLU
// in the epilogue, GEMM2 y = h W2^T, rows of expert e = [offsets[e],
// offsets[e+1]).  Products and sums are float32 (v_mfma_f32_32x32x2_f32: exact
// products, float32 accumulation).
//
// A float32 layer is small (it serves as the exact-arithmetic check of the
// layer), so what it costs is latency: a workgroup that walks K in steps of a
// barrier and a memory round trip each took 55 + 66 us for the two GEMMs of 64
// tokens at H 256, I 512, for 8 MB of operands.  Here a workgroup owns 32 rows
// x 32 columns (of gate and of up), its four waves take a run of K each, with
// operands loaded straight into the MFMA lane layout 32 K values at a time and
// the next 32 in flight, and the four partial sums are added in wave order
// through LDS: one memory round trip per 128 K values and two barriers in all.
// 64 tokens 57 + 68 -> 10 + 9 us, 1024 tokens 63 + 95 -> 31 + 20; at H 2048,
// I 1024 64 tokens 451 + 247 -> 130 + 73, 2048 tokens 1077 + 637 -> 937 + 570.
#include "common.h"
#include "kernels.h"
#include "tiles.h"

namespace moepd {

struct GemmArgsF {
  const float* A;
  const float* B;
  float* C;
  const int32_t* offsets;
  const int32_t* tile_base;
  long long b_stride;
  int e_loc, N, K, n_tiles, up_row;
};

// Tile of this workgroup (same schedule as the bf16 path); tile_base and
// offsets are copied to LDS first so the search costs one memory latency.
__device__ __forceinline__ bool tile_lookup_f(const GemmArgsF& g, int bm, int bn, int& e, int& m0, int& m_end,
                                              int& n0) {
  __shared__ int s_tb[kMaxLocalExperts + 1];
  __shared__ int s_off[kMaxLocalExperts + 1];
  for (int i = threadIdx.x; i <= g.e_loc; i += blockDim.x) {
    s_tb[i] = g.tile_base[i];
    s_off[i] = g.offsets[i];
  }
  __syncthreads();
  const int total = s_tb[g.e_loc] * g.n_tiles;
  const int per_xcd = (total + 7) >> 3;
  const int block = blockIdx.x + blockIdx.y * gridDim.x;
  const int xcd = block & 7, slot = block >> 3;
  if (slot >= per_xcd) return false;
  const int L = xcd * per_xcd + slot;
  if (L >= total) return false;
  int lo = 0, hi = g.e_loc - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_tb[mid] * g.n_tiles <= L) lo = mid;
    else hi = mid - 1;
  }
  e = lo;
  const int mt_e = s_tb[e + 1] - s_tb[e];
  const int local = L - s_tb[e] * g.n_tiles;
  const int nt = local / mt_e, mt = local - nt * mt_e;
  m0 = s_off[e] + mt * bm;
  m_end = s_off[e + 1];
  n0 = nt * bn;
  return true;
}

typedef float f32x16_f __attribute__((ext_vector_type(16)));
// The caller's weights need no more than a float's alignment.
typedef float f32x4_f __attribute__((ext_vector_type(4), aligned(4)));

template <bool GATED>
__global__ __launch_bounds__(256) void gemm_f32(GemmArgsF g) {
  constexpr int BM = 32, BN = 32;
  constexpr int NB = GATED ? 2 : 1;
  __shared__ float part[4][NB][BM][BN + 1];
  int e, m0, m_end, n0;
  if (!tile_lookup_f(g, BM, BN, e, m0, m_end, n0)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, kg = lane >> 5;
  const float* Be = g.B + (size_t)e * g.b_stride;
  // Block b holds K [32 b, 32 b + 32); of it, lane group kg loads the 16 values
  // from 32 b + 16 kg on as four vectors, and MFMA (i, j) takes element j of
  // vector i of both groups (the same K order for A and B).  Rows past the
  // expert's end repeat its last row (never stored); N is a multiple of 32.
  const f32x4_f* pa = reinterpret_cast<const f32x4_f*>(g.A + (size_t)min(m0 + r, m_end - 1) * g.K) + kg * 4;
  const f32x4_f* pb[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n)
    pb[n] = reinterpret_cast<const f32x4_f*>(Be + (size_t)(n * g.up_row + n0 + r) * g.K) + kg * 4;

  f32x16_f acc[NB];
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[n][q] = 0.f;
  const int KB = g.K / 32, per = (KB + 3) / 4;
  const int b0 = wave * per, b1 = min(KB, b0 + per);
  f32x4_f va[2][4], vb[2][NB][4];
  auto load = [&](int b, f32x4_f (&a)[4], f32x4_f (&w)[NB][4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = pa[b * 8 + i];
#pragma unroll
      for (int n = 0; n < NB; ++n) w[n][i] = pb[n][b * 8 + i];
    }
  };
  auto multiply = [&](const f32x4_f (&a)[4], const f32x4_f (&w)[NB][4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][j], w[n][i][j], acc[n], 0, 0, 0);
  };
  if (b0 < b1) load(b0, va[0], vb[0]);
  for (int b = b0; b < b1; b += 2) {
    if (b + 1 < b1) load(b + 1, va[1], vb[1]);
    multiply(va[0], vb[0]);
    if (b + 2 < b1) load(b + 2, va[0], vb[0]);
    if (b + 1 < b1) multiply(va[1], vb[1]);
  }
  // accumulator element q of lane (r, kg): row 8 (q / 4) + 4 kg + q % 4, column r
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int q = 0; q < 16; ++q) part[wave][n][8 * (q >> 2) + 4 * kg + (q & 3)][r] = acc[n][q];
  __syncthreads();
  const int col = threadIdx.x & 31;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rr = (threadIdx.x >> 5) + 8 * i, row = m0 + rr;
    if (row >= m_end) continue;
    float v[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      v[n] = part[0][n][rr][col];
#pragma unroll
      for (int w = 1; w < 4; ++w) v[n] += part[w][n][rr][col];
    }
    if (GATED) v[0] = v[0] / (1.f + expf(-v[0])) * v[NB - 1];
    g.C[(size_t)row * g.N + n0 + col] = v[0];
  }
}

int ffn_f32_bm() { return 32; }

hipError_t launch_ffn_f32(int gemm, const PhaseBuffers& b, const void* w_gu, const void* w_dn, int e_loc, int H,
                          int I, int max_m_tiles, hipStream_t s) {
  GemmArgsF g;
  g.offsets = b.offsets;
  g.tile_base = b.tile_base;
  g.e_loc = e_loc;
  if (gemm == 1) {
    g.A = (const float*)b.x_perm;
    g.B = (const float*)w_gu;
    g.C = (float*)b.h;
    g.b_stride = 2LL * I * H;
    g.N = I;
    g.K = H;
    g.up_row = I;
  } else {
    g.A = (const float*)b.h;
    g.B = (const float*)w_dn;
    g.C = b.y;
    g.b_stride = (long long)H * I;
    g.N = H;
    g.K = I;
    g.up_row = 0;
  }
  g.n_tiles = g.N / 32;
  const long long blocks = ((long long)max_m_tiles * g.n_tiles + 7) / 8 * 8;
  if (gemm == 1)
    gemm_f32<true><<<grid_of(blocks, 256), dim3(256), 0, s>>>(g);
  else
    gemm_f32<false><<<grid_of(blocks, 256), dim3(256), 0, s>>>(g);
  return hipGetLastError();
}

// Router GEMM of float32 contexts: one wave per token, lane l computes the
// logits of experts l, l + 64, ... as a sequential float32 FMA chain over h
// (x[t][h] is the same address for every lane of the wave).
__global__ __launch_bounds__(256) void router_f32(const float* __restrict__ x, const float* __restrict__ w, int T,
                                                  int E, int H, float* __restrict__ out) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const int lane = threadIdx.x & 63;
  const float* xr = x + (size_t)t * H;
  for (int e = lane; e < E; e += 64) {
    const float* wr = w + (size_t)e * H;
    float acc = 0.f;
    for (int h = 0; h < H; ++h) acc = fmaf(xr[h], wr[h], acc);
    out[(size_t)t * E + e] = acc;
  }
}

hipError_t launch_router_f32(const float* x, const float* w, int T, int E, int H, float* out, hipStream_t s) {
  if (T <= 0) return hipSuccess;
  router_f32<<<dim3((T + 3) / 4), dim3(256), 0, s>>>(x, w, T, E, H, out);
  return hipGetLastError();
}

}  // namespace moepd
