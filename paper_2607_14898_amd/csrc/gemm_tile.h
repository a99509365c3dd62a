// What the decoder's GEMM kernels share: the fused epilogues, the workgroup to
// tile mapping, the MFMA wrappers and the tile configurations.
#pragma once

#include "fd_kernels.h"

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include <type_traits>

namespace fd {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// SiLU with the hardware reciprocal (1 ulp) instead of an IEEE division; the
// limits hold: x -> -inf gives x * rcp(inf) = -0.
__device__ __forceinline__ float silu_f(float x) { return x * __builtin_amdgcn_rcpf(1.f + __expf(-x)); }
__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.f + erff(x * 0.70710678118654752f)); }

template <typename T> __device__ __forceinline__ T to_act(float v);
template <> __device__ __forceinline__ _Float16 to_act<_Float16>(float v) { return (_Float16)v; }
template <> __device__ __forceinline__ __hip_bfloat16 to_act<__hip_bfloat16>(float v) { return __float2bfloat16(v); }
// bit pattern of a 16-bit value (for packed stores without a stack array)
__device__ __forceinline__ uint32_t bits16(_Float16 x) { return __builtin_bit_cast(uint16_t, x); }
__device__ __forceinline__ uint32_t bits16(__hip_bfloat16 x) { return __bfloat16_as_ushort(x); }
template <> __device__ __forceinline__ float to_act<float>(float v) { return v; }

// A value bound for a 16-bit operand, clamped to the fp16 range when T is
// fp16 (+-65504; NaN passes unchanged), counting the clamped values in n.
template <typename T>
__device__ __forceinline__ float sat16(float v, int& n) {
  if constexpr (std::is_same<T, _Float16>::value) {
    const bool big = fabsf(v) > 65504.f;
    n += big;
    return big ? copysignf(65504.f, v) : v;
  } else {
    return v;
  }
}

// Adds this wave's count of clamped values to *sat (one atomic per wave that
// clamped anything).
__device__ __forceinline__ void count_sat(unsigned* sat, int n) {
  if (!sat || __builtin_amdgcn_ballot_w64(n != 0) == 0) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
  if ((threadIdx.x & 63) == 0) atomicAdd(sat, (unsigned)n);
}

// Every epilogue stores to out[row_off(row) + col_off(col)]: the destination
// offset splits into a part that depends only on the output row and a part
// that depends only on the column, so the per-element cost is one add. The
// reshapes of the temporal upsampling (Eq. temporal_upsample) and of the
// PixelShuffle store (Sec. 3.4 Step 3) are expressed this way, and so is the
// packed operand layout of 16-bit activations (blocks of 16 rows x 32
// columns: row part (row / 16) 16 ld + (row % 16) 8, column part
// (col / 32) 512 + (col % 32 / 8) 128 + col % 8).
template <int EPI>
constexpr bool kPackable = EPI == EPI_SWIGLU || EPI == EPI_STORE_SILU || EPI == EPI_STORE_GELU;
template <int EPI>
__device__ __forceinline__ int64_t row_off(const EpiParams& p, int row) {
  if constexpr (EPI == EPI_TUP) {
    // row = frame L + n  ->  refinement rows (frame r_t + j) L + n
    const int f = row / p.L, n = row - f * p.L;
    return ((int64_t)f * p.r_t * p.L + n) * p.ld_out;
  } else if constexpr (EPI == EPI_PIXEL || EPI == EPI_LINEAR_PIXEL) {
    const int bo = row / p.L, n = row - bo * p.L;
    const int h = n / p.grid_w, w = n - h * p.grid_w;
    const int OW = p.grid_w * p.s;
    const int64_t OHW = (int64_t)p.grid_h * p.s * OW;
    int b, fo;
    if constexpr (EPI == EPI_PIXEL) {      // row block bo = b frames_out + fo
      b = bo / p.frames_out;
      fo = bo - b * p.frames_out;
    } else {                               // row block bo = b frames_in + f; sub-frame in col
      b = bo / p.frames_in;
      fo = (bo - b * p.frames_in) * p.r_t;
    }
    return ((int64_t)b * p.C * p.frames_out + fo) * OHW + (int64_t)p.s * h * OW + p.s * w;
  } else {
    if constexpr (kPackable<EPI>)
      if (p.out_packed) return (int64_t)(row >> 4) * p.ld_out * 16 + (row & 15) * 8;
    return (int64_t)row * p.ld_out;
  }
}

template <int EPI>
__device__ __forceinline__ int64_t col_off(const EpiParams& p, int col) {
  if constexpr (EPI == EPI_TUP) {
    const int j = col / p.dim, d = col - j * p.dim;
    return (int64_t)j * p.L * p.ld_out + d;
  } else if constexpr (EPI == EPI_PIXEL || EPI == EPI_LINEAR_PIXEL) {
    const int OW = p.grid_w * p.s;
    const int64_t OHW = (int64_t)p.grid_h * p.s * OW;
    const int s2 = p.s * p.s;
    int j = 0, ch = col;
    if constexpr (EPI == EPI_LINEAR_PIXEL) {  // col = j C s^2 + c s^2 + i1 s + i2
      j = col / (p.C * s2);
      ch = col - j * p.C * s2;
    }
    const int c3 = ch / s2, rem = ch - c3 * s2;
    const int i1 = rem / p.s, i2 = rem - i1 * p.s;
    return ((int64_t)c3 * p.frames_out + j) * OHW + (int64_t)i1 * OW + i2;
  } else {
    if constexpr (kPackable<EPI>)
      if (p.out_packed) return (int64_t)(col >> 5) * 512 + ((col >> 3) & 3) * 128 + (col & 7);
    return col;
  }
}

// One output pixel: clamped to [-1, 1] if requested, then in the destination
// format (fp32; bf16 rounded to nearest even; uint8 = rint of the fp32 fma
// x 127.5 + 127.5, ties to even, limited to 0..255).
__device__ __forceinline__ float px_clamp(const EpiParams& p, float v) {
  return p.clamp ? fminf(1.f, fmaxf(-1.f, v)) : v;
}
__device__ __forceinline__ uint32_t px_u8(float v) {
  return (uint32_t)fminf(255.f, fmaxf(0.f, rintf(fmaf(v, 127.5f, 127.5f))));
}
// PXF: the format when known at compile time, -1 to read p.out_fmt
template <int PXF>
__device__ __forceinline__ void px_store(const EpiParams& p, int64_t off, float v) {
  const int f = PXF >= 0 ? PXF : p.out_fmt;
  v = px_clamp(p, v);
  if (f == 0) p.out_f[off] = v;
  else if (f == 1) reinterpret_cast<__hip_bfloat16*>(p.out_f)[off] = __float2bfloat16(v);
  else reinterpret_cast<uint8_t*>(p.out_f)[off] = (uint8_t)px_u8(v);
}

// Store one value (bias already added) at the precomputed offset.
template <int EPI, typename TA, int PXF = -1>
__device__ __forceinline__ void epi_store(const EpiParams& p, int64_t off, float c) {
  if constexpr (EPI == EPI_STORE_F32 || EPI == EPI_TUP) {
    p.out_f[off] = c;
  } else if constexpr (EPI == EPI_RESID_ADD) {
    p.out_f[off] += c;
  } else if constexpr (EPI == EPI_STORE_SILU) {
    ((TA*)p.out_a)[off] = to_act<TA>(silu_f(c));
  } else if constexpr (EPI == EPI_STORE_GELU) {
    ((TA*)p.out_a)[off] = to_act<TA>(gelu_f(c));
  } else if constexpr (EPI == EPI_PIXEL || EPI == EPI_LINEAR_PIXEL) {
    px_store<PXF>(p, off, c);
  }
}

template <int EPI, typename TA>
__device__ __forceinline__ void epi_one(const EpiParams& p, int row, int col, float c) {
  epi_store<EPI, TA>(p, row_off<EPI>(p, row) + col_off<EPI>(p, col), c + p.bias[col]);
}

// ---------------------------------------------------------------------------
// 16-bit MFMA GEMM
// ---------------------------------------------------------------------------

template <typename T> struct Mfma;
template <> struct Mfma<_Float16> {
  using V = f16x8;
  static __device__ __forceinline__ f32x16 run(V a, V b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma<__hip_bfloat16> {
  using V = bf16x8;
  static __device__ __forceinline__ f32x16 run(V a, V b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};

// Raw buffer resource over `bytes` bytes at `base`: loads at offsets past the
// end return zeros, which covers the ragged M / N edges of a tile.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, 0x00020000);
}

// Workgroup -> output tile. The hardware deals workgroups round-robin to the 8
// XCDs (workgroup i runs on XCD i % 8), each with its own L2. Give every XCD a
// contiguous range of tiles, and order tiles in groups of GROUP_M row blocks so
// that the tiles an XCD runs at once cover a compact 2D region: their A row
// blocks and W column blocks are then shared through that XCD's L2.
constexpr int GROUP_M = 8;
__device__ __forceinline__ void tile_of(int bid, int n_tiles, int tiles_m, int tiles_n, int& tm,
                                        int& tn) {
  const int q = n_tiles / 8, r = n_tiles % 8, x = bid % 8, i = bid / 8;
  const int t = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + i;
  const int per_group = GROUP_M * tiles_n;
  const int grp = t / per_group, first_m = grp * GROUP_M;
  const int gm = min(GROUP_M, tiles_m - first_m);
  const int in = t - grp * per_group;
  tm = first_m + in % gm;
  tn = in / gm;
}

// x / d for 0 <= x < 2^23 and 0 < d < 2^23, given inv = 1.0f / d (float product,
// then one exact integer correction; the products fit 24 bits)
__device__ __forceinline__ int div_small(int x, int d, float inv) {
  int q = (int)((float)x * inv);
  const int r = x - __mul24(q, d);
  return q + (r >= d) - (r < 0);
}

// Epilogues with 16-bit destinations take the accumulators transposed: four
// consecutive columns per lane make one 8-byte store and one bias / SiLU pass
// per four values. fp32 destinations keep the direct layout, where the 32 lanes
// of a half-wave write one full 128-byte row segment per store.
template <int EPI> constexpr bool kTransposed = EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_E4M3 ||
    EPI == EPI_STORE_SILU || EPI == EPI_STORE_GELU;

// Epilogue of one wave's FM x FN blocks of 32 x 32 accumulators whose first
// output row / column are r0 / c0. MFMA accumulator layout: lane (lk, lr) holds
// column lr of each block and rows 8 (r / 4) + 4 lk + r % 4 for r = 0..15.
// Loads of the destination (residual add) are issued for a whole 32-row block
// before any of its stores: interleaved, every load would wait for the store
// before it (the compiler cannot tell the addresses apart) and each element
// would cost a full memory round trip.
template <int EPI, typename T, int FM, int FN, bool FAST_RMW, int PXF = 0>
__device__ __forceinline__ void store_tile(const EpiParams& ep, const f32x16 (&acc)[FM][FN], int r0,
                                           int c0, int M, int N, int lr, int lk) {
  int64_t coff[FN];
  float cb[FN];
  bool cok[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int col = min(c0 + j * 32 + lr, N - 1);
    coff[j] = col_off<EPI>(ep, col);
    cb[j] = ep.bias[col];
    cok[j] = c0 + j * 32 + lr < N;
  }
  // interior blocks (the wave's rows and columns all in range) skip the
  // per-element checks; for the residual read-modify-write only where other
  // waves of the CU cover its load latency (measured: slower on a lone
  // 4-wave workgroup per CU)
  const bool interior = (EPI != EPI_RESID_ADD || FAST_RMW) && r0 + FM * 32 <= M && c0 + FN * 32 <= N;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    int64_t ro[16];
    bool rok[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = r0 + i * 32 + 8 * (r >> 2) + 4 * lk + (r & 3);
      rok[r] = row < M;
      ro[r] = row_off<EPI>(ep, min(row, M - 1));
    }
    if (interior) {
      if constexpr (EPI == EPI_RESID_ADD || EPI == EPI_STORE_F32) {
        // row-major destination: column blocks j are 32 floats apart, an
        // immediate offset from one row pointer
        float* rp[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)
          rp[r] = ep.out_f + (int64_t)(r0 + i * 32 + 8 * (r >> 2) + 4 * lk + (r & 3)) * ep.ld_out + c0 + lr;
        if constexpr (EPI == EPI_RESID_ADD) {
          float old[16][FN];
#pragma unroll
          for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int j = 0; j < FN; ++j) old[r][j] = rp[r][32 * j];
#pragma unroll
          for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int j = 0; j < FN; ++j) rp[r][32 * j] = old[r][j] + (acc[i][j][r] + cb[j]);
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int j = 0; j < FN; ++j) rp[r][32 * j] = acc[i][j][r] + cb[j];
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int j = 0; j < FN; ++j) epi_store<EPI, T, PXF>(ep, ro[r] + coff[j], acc[i][j][r] + cb[j]);
      }
      continue;
    }
    if constexpr (EPI == EPI_RESID_ADD) {
      float old[16][FN];
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < FN; ++j) old[r][j] = rok[r] && cok[j] ? ep.out_f[ro[r] + coff[j]] : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          if (rok[r] && cok[j]) ep.out_f[ro[r] + coff[j]] = old[r][j] + (acc[i][j][r] + cb[j]);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          if (rok[r] && cok[j]) epi_store<EPI, T, PXF>(ep, ro[r] + coff[j], acc[i][j][r] + cb[j]);
    }
  }
}

// The QKV projection's post step (Sec. 3.2, Eq. kv_cache) on transposed
// accumulators: a wave's 64 columns are one head vector (head slot c0 / 64:
// query heads, then key groups, then value groups), and a lane holds 32 of one
// row's 64 values in groups of 4 consecutive columns 32 j + 8 q + 4 lk (its other
// half, lane ^ 32, holds the rest). So the row's position is worked out once per
// lane, the 3D-RoPE pairs sit inside a lane, and the KV-norm's sum of squares
// takes one exchange per group (summed as a tree over the 16 groups). Queries
// go to the query buffer in 8-column chunks (chunk-major, then rows: 32 lanes
// write 512 bytes in a row, and the attention reads them so), normalised and
// rotated keys to their ring slot, normalised values to the V^T ring with
// neighbouring lanes' positions paired into 4-byte stores.
// (Through LDS, 16 lanes to a row, this step took about 4 us of a small call's
// launch: 11.3 us for 130 rows of the XL projection.)
template <typename T, int FM>
__device__ __forceinline__ void store_qkv(const EpiParams& ep, const f32x16 (&acc)[FM][2], int r0, int c0, int M, int N,
                                          int lr, int lk) {
  if (c0 >= N) return;
  const QkvPostArgs& a = ep.qkv;
  const int hs = c0 >> 6;
  const bool is_q = hs < a.N, is_v = hs >= a.N + a.G;
  const float* gn = is_q ? nullptr : (is_v ? a.vnorm_g : a.knorm_g);
  const int kvg = hs - a.N - (is_v ? a.G : 0);  // KV group
  const float inv_rpb = 1.f / a.rows_per_batch, inv_L = 1.f / a.L;
  const float inv_gw = 1.f / a.grid_w, inv_U = 1.f / a.U;
  const int slot0 = (int)(a.u0 % a.S);
  float4 bias[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) bias[j][q] = *reinterpret_cast<const float4*>(ep.bias + c0 + 32 * j + 8 * q + 4 * lk);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row_t = r0 + i * 32 + lr, row = min(row_t, M - 1);
    const bool ok = row_t < M;
    float4 v[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        v[j][q] = make_float4(acc[i][j][4 * q] + bias[j][q].x, acc[i][j][4 * q + 1] + bias[j][q].y,
                              acc[i][j][4 * q + 2] + bias[j][q].z, acc[i][j][4 * q + 3] + bias[j][q].w);
    if (gn) {
      float ss[2][4];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 x = v[j][q];
          ss[j][q] = x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
          ss[j][q] += __shfl_xor(ss[j][q], 32);
        }
      const float sum = ((ss[0][0] + ss[0][1]) + (ss[0][2] + ss[0][3])) + ((ss[1][0] + ss[1][1]) + (ss[1][2] + ss[1][3]));
      const float rn = rsqrtf(sum * (1.f / 64.f) + a.eps);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 g4 = *reinterpret_cast<const float4*>(gn + 32 * j + 8 * q + 4 * lk);
          const float4 x = v[j][q];
          v[j][q] = make_float4(x.x * rn * g4.x, x.y * rn * g4.y, x.z * rn * g4.z, x.w * rn * g4.w);
        }
    }
    // row of the call -> stream and row of the stream; (unit, position) and
    // (sub-frame, h, w) from that
    const int b = div_small(row, a.rows_per_batch, inv_rpb);
    const int rb = row - __mul24(b, a.rows_per_batch);
    if (a.rope && !is_v) {
      const int fs = div_small(rb, a.L, inv_L), tok = rb - __mul24(fs, a.L);
      const int hh = div_small(tok, a.grid_w, inv_gw), ww = tok - __mul24(hh, a.grid_w);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // RoPE pairs pa and pa + 1 of this group; an axis boundary may lie between them
          const int pa = 16 * j + 4 * q + 2 * lk;
          const int ax0 = a.rope_axis[pa], ax1 = a.rope_axis[pa + 1];
          const float2 c0v = ax0 == 0 ? a.rope_t[fs * 32 + pa] : a.rope_hw[(ax0 == 1 ? hh : ww) * 32 + pa];
          const float2 c1v = ax1 == 0 ? a.rope_t[fs * 32 + pa + 1] : a.rope_hw[(ax1 == 1 ? hh : ww) * 32 + pa + 1];
          const float4 x = v[j][q];
          v[j][q] = make_float4(x.x * c0v.x - x.y * c0v.y, x.x * c0v.y + x.y * c0v.x,
                                x.z * c1v.x - x.w * c1v.y, x.z * c1v.y + x.w * c1v.x);
        }
    }
    auto pack4 = [](float4 x) {
      return make_uint2(bits16(to_act<T>(x.x)) | (bits16(to_act<T>(x.y)) << 16),
                        bits16(to_act<T>(x.z)) | (bits16(to_act<T>(x.w)) << 16));
    };
    if (is_q) {
      if (!ok) continue;
      T* dst = (T*)a.q + ((int64_t)hs * 8 * M + row) * 8 + 4 * lk;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(dst + (int64_t)(4 * j + q) * M * 8) = pack4(v[j][q]);
      continue;
    }
    const int lu = div_small(rb, a.U, inv_U), pos = rb - __mul24(lu, a.U);
    const int sl = slot0 + lu;  // (below 2 S: a call has at most S units)
    const int64_t kv = (int64_t)(b * a.G + kvg) * a.S + (sl >= a.S ? sl - a.S : sl);  // ring slot
    if (!is_v) {
      if (!ok) continue;
      T* dst = (T*)a.k_ring + (kv * a.U_pad + pos) * 64 + 4 * lk;
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(dst + 32 * j + 8 * q) = pack4(v[j][q]);
      continue;
    }
    // V^T[dim][pos]: lanes 2 m and 2 m + 1 hold neighbouring rows; where these are
    // an aligned pair of positions of one slot (rows stay in order, so only a
    // unit's end or an odd start breaks a pair), the even lane stores both of
    // dimension d, the odd lane both of d + 1
    const int odd = lr & 1;
    const int pos_e = odd ? pos - 1 : pos;  // the pair's first position
    const bool pair = (row_t | 1) < M && (pos_e & 1) == 0 && pos_e >= 0 && pos_e + 1 < a.U;
    T* vt = (T*)a.vt_ring + kv * 64 * a.U_pad;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint2 w = pack4(v[j][q]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // dimensions d and d + 1
          const int d = 32 * j + 8 * q + 4 * lk + 2 * h;
          const uint32_t own = h ? w.y : w.x;
          const uint32_t oth = (uint32_t)__shfl_xor((int)own, 1);
          if (pair) {
            const uint32_t x = odd ? (oth >> 16) | (own & 0xFFFF0000u) : (own & 0xFFFFu) | (oth << 16);
            *reinterpret_cast<uint32_t*>(vt + (int64_t)(d + odd) * a.U_pad + pos_e) = x;
          } else if (ok) {
            vt[(int64_t)d * a.U_pad + pos] = __builtin_bit_cast(T, (uint16_t)(own & 0xFFFFu));
            vt[(int64_t)(d + 1) * a.U_pad + pos] = __builtin_bit_cast(T, (uint16_t)(own >> 16));
          }
        }
      }
  }
}

// Epilogue of one wave's blocks computed transposed (acc[i][j] = W block j
// times A block i): lane (lk, lr) holds output row r0 + 32 i + lr and, in
// registers 4 q .. 4 q + 3, the four consecutive columns c0 + 32 j + 8 q +
// 4 lk + 0..3. Every store covers those four columns at once (8 bytes, or 4 of
// E4M3 codes); vec == false (a ragged or unaligned SiLU / GELU destination) stores
// element by element.
template <int EPI, typename T, int FM, int FN, bool SCALED = false>
__device__ __forceinline__ void store_tile_t(const EpiParams& ep, const f32x16 (&acc)[FM][FN], int r0,
                                             int c0, int M, int N, int lr, int lk, bool vec) {
  // SCALED (FP8 GEMM, SwiGLU only): each accumulator is multiplied by its
  // column's then its row's dequantisation scale right before use
  static_assert(kTransposed<EPI> && (!SCALED || EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_E4M3),
                "epilogues with 16-bit or E4M3 destinations; scaled: SwiGLU only");
  if constexpr (EPI == EPI_QKV) {
    store_qkv<T, FM>(ep, acc, r0, c0, M, N, lr, lk);
    return;
  }
  int nsat = 0;  // fp16 values clamped to +-65504 by this lane
  int64_t ro[FM];
  bool rok[FM];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int row = r0 + i * 32 + lr;
    rok[i] = row < M;
    ro[i] = row_off<EPI>(ep, min(row, M - 1));
  }
  if constexpr (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_E4M3) {
    float rs[FM];
#pragma unroll
    for (int i = 0; i < FM; ++i)
      rs[i] = SCALED ? ep.row_scale[min(r0 + i * 32 + lr, M - 1) * ep.row_scale_stride] : 1.f;
    const float q_inv = EPI == EPI_SWIGLU_E4M3 ? ep.out_scale[1] : 1.f;
    // gate block j and up block j + 1 give output columns (c0 + 32 j) / 2 + 0..31
#pragma unroll
    for (int j = 0; j < FN; j += 2)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int lc = 8 * q + 4 * lk, pc = c0 + j * 32 + lc;
        if (pc >= N) continue;  // N % 64 == 0: a group is valid as a whole
        float bg[4], bu[4], sg[4], su[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bg[e] = ep.bias[pc + e];
          bu[e] = ep.bias[pc + 32 + e];
          sg[e] = SCALED ? ep.col_scale[pc + e] : 1.f;
          su[e] = SCALED ? ep.col_scale[pc + 32 + e] : 1.f;
        }
        const int oc = (c0 + j * 32) / 2 + lc;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          if (!rok[i]) continue;
          T o4[4];
          float h4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float g = acc[i][j][4 * q + e], u = acc[i][j + 1][4 * q + e];
            // (the row scale and the bias in one rounding, written out so that it
            // is the same in every tile shape)
            g = SCALED ? fmaf(g * sg[e], rs[i], bg[e]) : g + bg[e];
            u = SCALED ? fmaf(u * su[e], rs[i], bu[e]) : u + bu[e];
            o4[e] = to_act<T>(sat16<T>(silu_f(g) * u, nsat));
            h4[e] = (float)o4[e];
          }
          if constexpr (EPI == EPI_SWIGLU_E4M3) {
            // codes of the fp16-rounded hidden value at the static scale (saturating)
            auto cl = [&](float v) { return fminf(448.f, fmaxf(-448.f, v * q_inv)); };
            int w = __builtin_amdgcn_cvt_pk_fp8_f32(cl(h4[0]), cl(h4[1]), 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(cl(h4[2]), cl(h4[3]), w, true);
            // E4M3 codes: row-major, or the FP8 GEMM's packed operand layout
            // (blocks of 16 rows x 64 bytes)
            const int64_t rr = r0 + i * 32 + lr;
            const int64_t bo = ep.out_packed ? (rr >> 4) * ep.ld_out * 16 + (rr & 15) * 64 +
                                                   (int64_t)(oc >> 6) * 1024 + (oc & 63)
                                             : ro[i] + oc;
            *reinterpret_cast<int*>((uint8_t*)ep.out_a + bo) = w;
            continue;
          }
          *reinterpret_cast<uint2*>((T*)ep.out_a + ro[i] + col_off<EPI>(ep, oc)) =
              *reinterpret_cast<const uint2*>(o4);
        }
      }
  } else {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      int64_t co[4];
      float cb[4][4];
      bool cok[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = c0 + j * 32 + 8 * q + 4 * lk;
        cok[q] = n < N;
        co[q] = col_off<EPI>(ep, min(n, N - 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) cb[q][e] = ep.bias[min(n + e, N - 1)];
      }
      if (!vec) {  // element by element
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int n = c0 + j * 32 + 8 * q + 4 * lk + e;
              if (!(rok[i] && n < N)) continue;
              if constexpr (EPI == EPI_STORE_SILU)
                ((T*)ep.out_a)[ro[i] + col_off<EPI>(ep, n)] = to_act<T>(sat16<T>(silu_f(acc[i][j][4 * q + e] + cb[q][e]), nsat));
              else
                epi_store<EPI, T>(ep, ro[i] + col_off<EPI>(ep, n), acc[i][j][4 * q + e] + cb[q][e]);
            }
        continue;
      }
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (!(rok[i] && cok[q])) continue;
          T o4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = acc[i][j][4 * q + e] + cb[q][e];
            if constexpr (EPI == EPI_STORE_SILU) o4[e] = to_act<T>(sat16<T>(silu_f(v), nsat));
            else o4[e] = to_act<T>(gelu_f(v));
          }
          *reinterpret_cast<uint2*>((T*)ep.out_a + ro[i] + co[q]) = *reinterpret_cast<const uint2*>(o4);
        }
    }
  }
  if constexpr (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_E4M3 || EPI == EPI_STORE_SILU) count_sat(ep.sat, nsat);
}

// ---------------------------------------------------------------------------
// 16-bit MFMA GEMM. K tiles of 32 columns go from memory straight into LDS
// with buffer_load_dwordx4 ... lds (no register staging, no LDS store
// instructions), NS tiles deep: while tile t is multiplied, tiles t + 1 ..
// t + NS - 1 are in flight. A DMA instruction writes the 16 bytes of lane l to
// LDS slot l after a wave-uniform base; the operands are stored in fragment
// order, so a 1 KB block lands in LDS as it is read.
// ---------------------------------------------------------------------------
constexpr int BKD = 32;  // K-columns per stage: 4 chunks of 16 bytes per row

// Tile configuration: BM x BN output tile, WAVES_M x WAVES_N wave64s (each a
// (BM / WAVES_M) x (BN / WAVES_N) sub-tile of 32 x 32 MFMA blocks), NS stages.
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, int NS_, bool IL_ = false>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, NS = NS_;
  // IL: the stage refill DMAs are spread between the MFMAs instead of issued
  // as one burst between two k-steps
  static constexpr bool IL = IL_;
  static constexpr int NW = WAVES_M * WAVES_N, NT = 64 * NW;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, FM = WM / 32, FN = WN / 32;
  static constexpr int STAGE = (BM + BN) * 4;                 // 16-byte slots per stage
  static constexpr int QA = BM / 16 / NW, QB = BN / 16 / NW;  // DMAs per thread and stage
  static constexpr int LDS_BYTES = NS * STAGE * 16;
  static constexpr int MIN_BLOCKS = 163840 / LDS_BYTES >= 2 ? 2 : 1;
  static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0, "DMA rows split evenly over waves");
  static_assert(NS >= 3 && LDS_BYTES <= 163840, "at least 3 stages, within 160 KB of LDS");
  static_assert((NS - 2) * (QA + QB) < 64, "vmcnt range");
};

// s_waitcnt immediates (gfx9 encoding): vmcnt(n) with lgkmcnt and expcnt
// untouched, and lgkmcnt(0) alone.
#define FD_VMCNT(n) ((((n) & 0xF) | ((((n) >> 4) & 3) << 14) | (0x7 << 4) | (0xF << 8)))
#define FD_LGKMCNT0 (0xF | (0x3 << 14) | (0x7 << 4))

// The DMAs are issued from inline assembly (M0 = LDS destination of the wave),
// so the compiler neither sees nor orders them; every ordering they need is
// explicit: s_waitcnt on the wave's own DMAs, then s_barrier (with compiler
// memory barriers around it) before any wave reads the tile or refills a stage.

using TileL = TileCfg<256, 256, 2, 4, 4, true>;   // 8 waves of 128 x 64, 128 KB LDS
using TileD = TileCfg<128, 256, 1, 4, 3, true>;   // 4 waves of 128 x 64, 72 KB: two per CU
using TileE = TileCfg<128, 192, 2, 2, 3>;         // 4 waves of 64 x 96, 60 KB: two per CU
using TileW = TileCfg<256, 192, 2, 2, 5>;         // 4 waves of 128 x 96, 140 KB
using TileM = TileCfg<192, 128, 2, 2, 6>;         // 4 waves of 96 x 64, 120 KB
using TileM4 = TileCfg<192, 128, 2, 2, 4>;        // the same, 80 KB: two per CU
using TileS1 = TileCfg<128, 128, 2, 2, 6, true>;  // 4 waves of 64 x 64, 96 KB
using TileS8 = TileCfg<128, 128, 2, 4, 6, true>;  // 8 waves of 64 x 32, 96 KB
using TileH = TileCfg<128, 64, 2, 2, 6>;          // 4 waves of 64 x 32, 72 KB
using TileS = TileCfg<128, 128, 2, 2, 3, true>;   // 4 waves of 64 x 64, 48 KB

}  // namespace
}  // namespace fd
