// fp32 projections (fp32 compute path).
#include "gemm_tile.h"

#include <algorithm>

namespace fd {
namespace {

// ---------------------------------------------------------------------------
// fp32 GEMM (fp32 compute path) on the 16x16x4 fp32 MFMA (fp32 products and
// sums). A workgroup computes a 16 F x 16 F tile; its 4 waves split K: wave w
// takes the 16-column chunks w, w + 4, .., and the four partial sums meet in LDS
// as (p0 + p2) + (p1 + p3). Operands go from memory straight to registers: lane
// (g, r) reads the 16 bytes at row r, columns 16 c + 4 g .. + 3 of a chunk, and
// component j of them is its operand of MFMA step j. Every output is the same
// sum whatever F, so a call's rows do not depend on how many rows it has.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

// VEC: K, lda and ldw multiples of 4 and 16-byte aligned operands (16-byte
// loads); otherwise single floats. EPI_SWIGLU: W holds the gate rows 0 .. N/2 - 1
// and the up rows N/2 .. N - 1; the tile covers 16 F columns of both.
template <int EPI, int F, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A,
                                                       const float* __restrict__ W, int M, int N,
                                                       int K, int lda, int ldw, EpiParams ep,
                                                       int tiles_m, int tiles_n, int tile0) {
  constexpr bool SW = EPI == EPI_SWIGLU;
  constexpr int NB = SW ? 2 : 1;          // W row sets
  constexpr int PD = F == 1 ? 6 : (F == 2 ? 3 : 2);  // chunks in flight per wave
  constexpr int T = 16 * F, LS = T + 4;   // LDS row stride
  __shared__ float red[4][NB][T * LS];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  int tm, tn;
  tile_of(blockIdx.x + tile0, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * T, n0 = tn * T;
  const int NO = SW ? N / 2 : N;  // output columns
  const float* pa[F];
  const float* pw[NB][F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    pa[i] = A + (int64_t)min(m0 + 16 * i + lr, M - 1) * lda;
#pragma unroll
    for (int h = 0; h < NB; ++h) pw[h][i] = W + (int64_t)(h * NO + min(n0 + 16 * i + lr, NO - 1)) * ldw;
  }
  f32x4 fa[PD][F], fw[PD][NB][F];
  // 4 columns from k on; a vector past the end of the row reads its last four
  // columns instead (masked to zero before use)
  auto ld4 = [&](const float* p, int k) {
    if constexpr (VEC) {
      return *reinterpret_cast<const f32x4*>(p + min(k, K - 4));
    } else {
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = p[min(k + j, K - 1)];
      return v;
    }
  };
  auto load = [&](int slot, int c) {
    const int k = 16 * c + 4 * lg;
#pragma unroll
    for (int i = 0; i < F; ++i) fa[slot][i] = ld4(pa[i], k);
#pragma unroll
    for (int h = 0; h < NB; ++h)
#pragma unroll
      for (int i = 0; i < F; ++i) fw[slot][h][i] = ld4(pw[h][i], k);
  };
  f32x4 acc[NB][F][F];
#pragma unroll
  for (int h = 0; h < NB; ++h)
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) acc[h][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int nch = (K + 15) / 16;
  const bool ragged = (K & 15) != 0;
  auto mul = [&](int slot, int c) {
    if (ragged && c == nch - 1) {  // the row's end inside the chunk
      const int k = 16 * c + 4 * lg;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j >= K) {
#pragma unroll
          for (int i = 0; i < F; ++i) {
            fa[slot][i][j] = 0.f;
#pragma unroll
            for (int h = 0; h < NB; ++h) fw[slot][h][i][j] = 0.f;
          }
        }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int h = 0; h < NB; ++h)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j)
            acc[h][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[slot][i][s], fw[slot][h][j][s], acc[h][i][j], 0, 0, 0);
  };
  // this wave's chunks: wave, wave + 4, ..; PD of them are in flight (past the
  // last one the loads read in bounds and are not used)
  const int n_my = nch > wave ? (nch - wave + 3) / 4 : 0;
#pragma unroll
  for (int p = 0; p < PD; ++p) load(p, wave + 4 * p);
  int base = 0;
  for (; base + PD < n_my; base += PD)
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      mul(p, wave + 4 * (base + p));
      load(p, wave + 4 * (base + PD + p));
    }
#pragma unroll
  for (int p = 0; p < PD; ++p)
    if (base + p < n_my) mul(p, wave + 4 * (base + p));
  // lane (g, r) holds rows 4 g .. 4 g + 3 of column r of each 16 x 16 block
#pragma unroll
  for (int h = 0; h < NB; ++h)
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][h][(16 * i + 4 * lg + r) * LS + 16 * j + lr] = acc[h][i][j][r];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < F * F; ++e) {
    const int x = tid + 256 * e, rr = x / T, cc = x % T;
    const int row = m0 + rr, col = n0 + cc;
    if (row >= M || col >= NO) continue;
    const int o = rr * LS + cc;
    const float c = (red[0][0][o] + red[2][0][o]) + (red[1][0][o] + red[3][0][o]);
    if constexpr (SW) {
      const float u = (red[0][NB - 1][o] + red[2][NB - 1][o]) + (red[1][NB - 1][o] + red[3][NB - 1][o]) + ep.bias[NO + col];
      const float g = c + ep.bias[col];
      ((float*)ep.out_a)[(int64_t)row * ep.ld_out + col] = g / (1.f + expf(-g)) * u;
    } else {
      epi_one<EPI, float>(ep, row, col, c);
    }
  }
}

template <int EPI, int F, bool VEC>
hipError_t launch_f32_tile(const GemmArgs& g, hipStream_t s) {
  const int no = EPI == EPI_SWIGLU ? g.N / 2 : g.N;
  const int tm = (g.M + 16 * F - 1) / (16 * F), tn = (no + 16 * F - 1) / (16 * F);
  hipError_t e = hipSuccess;
  for (int t0 = 0; t0 < tm * tn && e == hipSuccess; t0 += kMaxLaunch) {
    hipLaunchKernelGGL((gemm_f32_kernel<EPI, F, VEC>), dim3(std::min(tm * tn - t0, kMaxLaunch)), dim3(256), 0, s,
                       (const float*)g.A, (const float*)g.W, g.M, g.N, g.K, g.lda, g.ldw, g.ep, tm, tn, t0);
    e = hipGetLastError();
  }
  return e;
}

template <int EPI>
hipError_t launch_f32(const GemmArgs& g, hipStream_t s) {
  const bool vec = g.K % 4 == 0 && g.lda % 4 == 0 && g.ldw % 4 == 0 && (uintptr_t)g.A % 16 == 0 && (uintptr_t)g.W % 16 == 0;
  if (!vec) return launch_f32_tile<EPI, 2, false>(g, s);
  // The F whose rounds of one workgroup per CU take the least time; a round's time
  // for K = 1536 is 6, 13.4, 20 and 29 us for F = 1 to 4. Measured, us at F = 1 / 2 /
  // 3 / 4: 130 x 1536 x 6144 86 / 46 / 67 / 99, 520 x 1536 x 6144 272 / 171 / 134 /
  // 102, 1100 x 1536 x 1536 137 / 80 / 61 / 67, 512 x 128 x 512 5.2 / 6.6 / 10 / 13
  const int64_t no = EPI == EPI_SWIGLU ? g.N / 2 : g.N;
  auto rounds = [&](int t) { return (((g.M + t - 1) / t) * ((no + t - 1) / t) + 255) / 256; };
  const double us[4] = {6.0 * rounds(16), 13.4 * rounds(32), 20.0 * rounds(48),
                        EPI == EPI_SWIGLU ? 1e30 : 29.0 * rounds(64)};  // (SwiGLU's two weight sets: F <= 3)
  int f = 0;
  for (int i = 1; i < 4; ++i)
    if (us[i] < us[f]) f = i;
  if constexpr (EPI != EPI_SWIGLU)
    if (f == 3) return launch_f32_tile<EPI, 4, true>(g, s);
  if (f == 2) return launch_f32_tile<EPI, 3, true>(g, s);
  if (f == 1) return launch_f32_tile<EPI, 2, true>(g, s);
  return launch_f32_tile<EPI, 1, true>(g, s);
}

}  // namespace

hipError_t gemm_f32(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.a_packed || g.ep.out_packed) return hipErrorInvalidValue;  // row-major fp32 operands
  switch (g.epi) {
    case EPI_STORE_F32: return launch_f32<EPI_STORE_F32>(g, s);
    case EPI_RESID_ADD: return launch_f32<EPI_RESID_ADD>(g, s);
    case EPI_STORE_SILU: return launch_f32<EPI_STORE_SILU>(g, s);
    case EPI_STORE_GELU: return launch_f32<EPI_STORE_GELU>(g, s);
    case EPI_TUP: return launch_f32<EPI_TUP>(g, s);
    case EPI_PIXEL: return launch_f32<EPI_PIXEL>(g, s);
    case EPI_LINEAR_PIXEL: return launch_f32<EPI_LINEAR_PIXEL>(g, s);
    case EPI_SWIGLU: return g.N % 2 ? hipErrorInvalidValue : launch_f32<EPI_SWIGLU>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fd
