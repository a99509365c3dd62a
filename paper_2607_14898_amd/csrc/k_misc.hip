// Bandwidth-bound passes of the decoder forward:
//  * norm_rows       pre-sublayer RMSNorm / LayerNorm of the fp32 residual
//                    stream (Sec. 3.2 "Base Architecture") into the operand
//                    format and packed block layout of the next projection;
//  * qkv_post        KV-norm and 3D-RoPE (Sec. 3.2), then the rolling-cache
//                    append of Sec. 3.3 / Algorithm 1 as a write into ring slot
//                    (unit mod S);
//  * prologue        PixelUnshuffle(p) + raster flatten of latent frames
//                    (Sec. 4.3 and Eq. projection) and the call's temporal
//                    RoPE tables;
//  * quant_rows_e4m3 per-row E4M3 codes and scales of the FP8 MLP (Sec. 4.6).
#include "fd_kernels.h"

#include <hip/hip_bf16.h>

#include <algorithm>
#include <type_traits>

namespace fd {
namespace {

__device__ __forceinline__ void store_kind(void* out, int64_t i, float v, int kind) {
  if (kind == 0) ((_Float16*)out)[i] = (_Float16)v;
  else if (kind == 1) ((__hip_bfloat16*)out)[i] = __float2bfloat16(v);
  else ((float*)out)[i] = v;
}

// Element (row, k) of a 16-bit [rows, K] activation in the packed operand
// layout of the MFMA GEMM (blocks of 16 rows x 32 columns, block-row major,
// inside a block 8-column chunks, then rows).
__device__ __forceinline__ int64_t pk16(int64_t row, int k, int K) {
  return ((row >> 4) * (K >> 5) + (k >> 5)) * 512 + ((k >> 3) & 3) * 128 + (row & 15) * 8 + (k & 7);
}
// Byte (row, k) of E4M3 codes [rows, K] in the packed operand layout of the
// FP8 GEMM (blocks of 16 rows x 64 bytes).
__device__ __forceinline__ int64_t pk8(int64_t row, int k, int K) {
  return ((row >> 4) * (K >> 6) + (k >> 6)) * 1024 + (row & 15) * 64 + (k & 63);
}

// Four consecutive values as one 8-byte (16-bit kinds) or 16-byte (fp32) store.
__device__ __forceinline__ void store4(void* out, int64_t i, float4 y, int kind) {
  if (kind == 0) {
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    const h4 h = {(_Float16)y.x, (_Float16)y.y, (_Float16)y.z, (_Float16)y.w};
    *reinterpret_cast<h4*>((_Float16*)out + i) = h;
  } else if (kind == 1) {
    __hip_bfloat16 h[4] = {__float2bfloat16(y.x), __float2bfloat16(y.y), __float2bfloat16(y.z),
                           __float2bfloat16(y.w)};
    *reinterpret_cast<uint2*>((__hip_bfloat16*)out + i) = *reinterpret_cast<uint2*>(h);
  } else {
    *reinterpret_cast<float4*>((float*)out + i) = y;
  }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// E4M3 quantisation of a row whose amplitude (max |v|) is m: inv = 448 / m,
// codes of fp32(v * inv) by the gfx950 conversion (round to nearest even),
// after clamping to +-448 so that the code saturates; scale m / 448. A zero
// row gets scale 1 (and codes 0).
struct E4m3Row {
  float inv, scale;
  __device__ __forceinline__ explicit E4m3Row(float m) {
    const float mm = m > 0.f ? m : 448.f;
    inv = 448.f / mm;
    scale = mm / 448.f;
  }
  // a static (calibrated) scale: {scale, inverse scale}
  __device__ __forceinline__ explicit E4m3Row(const float* sc) : inv(sc[1]), scale(sc[0]) {}
  // four values -> four codes, byte e = value e
  __device__ __forceinline__ uint32_t pack4(float a, float b, float c, float d) const {
    auto cl = [&](float v) { return fminf(448.f, fmaxf(-448.f, v * inv)); };
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(cl(a), cl(b), 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(cl(c), cl(d), w, true);
    return (uint32_t)w;
  }
};

// Sum of squares of a lane's four values of a row, written as the fused
// multiply-adds it is: the order that the compiler picks by itself differs
// between the norm's widths, and with it the last bit of a row's scale.
__device__ __forceinline__ float sum_sq4(float x, float y, float z, float w) {
  return fmaf(w, w, fmaf(z, z, fmaf(x, x, y * y)));
}

// One wave per row; rows of D floats (D % 4 == 0), NV = ceil(D / 256) float4 per
// lane, all valid when FULL (D % 256 == 0; NV = 8 and FULL = false take any D up
// to 2048). A row is one chain of load, wave reduction, store, so what a small
// pass costs is latency: the row and gain loads go out together, unbranched
// (60 rows of 1536: 6.6 -> 4.6 us).
template <int KIND, int OUT, int NV, bool FULL>
__global__ __launch_bounds__(256) void norm_kernel(const float* __restrict__ x, int M, int D,
                                                   const float* __restrict__ g,
                                                   const float* __restrict__ bta, float eps,
                                                   void* out, float* row_scale,
                                                   const float* __restrict__ static_sc,
                                                   unsigned* __restrict__ amax_out, int packed) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const float4* xr = reinterpret_cast<const float4*>(x + (int64_t)row * D);
  const int nv = D / 4;
  float4 v[NV], gv[NV], bv[KIND == 1 ? NV : 1];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = FULL ? lane + 64 * i : min(lane + 64 * i, nv - 1);
    v[i] = xr[c];
    gv[i] = reinterpret_cast<const float4*>(g)[c];
    if (KIND == 1) bv[i] = reinterpret_cast<const float4*>(bta)[c];
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const float t = KIND == 0 ? sum_sq4(v[i].x, v[i].y, v[i].z, v[i].w) : v[i].x + v[i].y + v[i].z + v[i].w;
    if (FULL || lane + 64 * i < nv) s += t;
  }
  s = wave_sum(s);
  float mu = 0.f, rs;
  if (KIND == 0) {
    rs = rsqrtf(s / D + eps);
  } else {
    mu = s / D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (FULL || lane + 64 * i < nv) q += sum_sq4(v[i].x - mu, v[i].y - mu, v[i].z - mu, v[i].w - mu);
    }
    q = wave_sum(q);
    rs = rsqrtf(q / D + eps);
  }
  float amax = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = lane + 64 * i;
    if (FULL || c < nv) {
      float4 y = make_float4((v[i].x - mu) * rs * gv[i].x, (v[i].y - mu) * rs * gv[i].y,
                             (v[i].z - mu) * rs * gv[i].z, (v[i].w - mu) * rs * gv[i].w);
      if (KIND == 1) {
        y.x += bv[i].x; y.y += bv[i].y; y.z += bv[i].z; y.w += bv[i].w;
      }
      if (OUT == 3) {  // E4M3: keep the row for its amplitude
        v[i] = y;
        amax = fmaxf(fmaxf(amax, fmaxf(fabsf(y.x), fabsf(y.y))), fmaxf(fabsf(y.z), fabsf(y.w)));
      } else {
        store4(out, packed ? pk16(row, 4 * c, D) : (int64_t)row * D + 4 * c, y, OUT);
      }
    }
  }
  if (OUT == 3) {
    const float m = wave_max(amax);
    if (amax_out && lane == 0) atomicMax(amax_out, __float_as_uint(m));  // non-negative: ordered as bits
    const E4m3Row q = static_sc ? E4m3Row(static_sc) : E4m3Row(m);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = lane + 64 * i;
      if (FULL || c < nv)
        *reinterpret_cast<uint32_t*>((uint8_t*)out + (packed ? pk8(row, 4 * c, D) : (int64_t)row * D + 4 * c)) =
            q.pack4(v[i].x, v[i].y, v[i].z, v[i].w);
    }
    if (!static_sc && lane == 0) row_scale[row] = q.scale;
  }
}

// Per-row E4M3 codes of in [M, K] (fp16 or fp32, K % 8 == 0): one wave per row,
// a first pass for the amplitude, a second (from cache) for the codes.
template <typename TIN>
__global__ __launch_bounds__(256) void quant_rows_kernel(const TIN* __restrict__ in, int64_t M, int K,
                                                         uint8_t* __restrict__ codes,
                                                         float* __restrict__ scale,
                                                         unsigned* __restrict__ amax_out, int packed) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const TIN* r = in + row * K;
  float amax = 0.f;
  for (int c = 8 * lane; c < K; c += 512) {
#pragma unroll
    for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf((float)r[c + e]));
  }
  const float m = wave_max(amax);
  if (amax_out && lane == 0) atomicMax(amax_out, __float_as_uint(m));
  const E4m3Row q(m);
  for (int c = 8 * lane; c < K; c += 512) {
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = (float)r[c + e];
    uint2 w;
    w.x = q.pack4(f[0], f[1], f[2], f[3]);
    w.y = q.pack4(f[4], f[5], f[6], f[7]);
    *reinterpret_cast<uint2*>(codes + (packed ? pk8(row, c, K) : row * K + c)) = w;
  }
  if (lane == 0) scale[row] = q.scale;
}

// The same for fp16 rows of 512 NV values held in registers: one pass over
// memory, all of a row's loads in flight (1560 rows of 6144: 27 us with the two
// passes above). Built for the hidden widths (4 D) of the named decoder sizes;
// other widths, for which nothing was measured, take the two passes.
template <int NV>
__global__ __launch_bounds__(256) void quant_rows16_kernel(const _Float16* __restrict__ in, int64_t M,
                                                           uint8_t* __restrict__ codes, float* __restrict__ scale,
                                                           unsigned* __restrict__ amax_out, int packed) {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  constexpr int K = 512 * NV;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const h8* r = reinterpret_cast<const h8*>(in + row * K);
  h8 v[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = r[lane + 64 * i];
  float amax = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf((float)v[i][e]));
  const float m = wave_max(amax);
  if (amax_out && lane == 0) atomicMax(amax_out, __float_as_uint(m));
  const E4m3Row q(m);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = 8 * (lane + 64 * i);
    uint2 w;
    w.x = q.pack4((float)v[i][0], (float)v[i][1], (float)v[i][2], (float)v[i][3]);
    w.y = q.pack4((float)v[i][4], (float)v[i][5], (float)v[i][6], (float)v[i][7]);
    *reinterpret_cast<uint2*>(codes + (packed ? pk8(row, c, K) : row * K + c)) = w;
  }
  if (lane == 0) scale[row] = q.scale;
}

// cos / sin of the RoPE angle of channel pair `pair` for the row (frame-or-
// sub-frame fs of the call, token tok): temporal pairs read the per-call table
// (fs), spatial pairs the table indexed by the token's row h or column w.
__device__ __forceinline__ float2 rope_cs(const QkvPostArgs& a, int pair, int fs, int tok) {
  const int axis = a.rope_axis[pair];
  const int np = a.Dh / 2;
  if (axis == 0) return a.rope_t[fs * np + pair];
  const int p = axis == 1 ? tok / a.grid_w : tok % a.grid_w;
  return a.rope_hw[p * np + pair];
}

// The fp32 path's QKV post step in one launch: workgroups below qk_blocks take
// queries and keys, one thread per 4 consecutive channels of a (row, head slot),
// slots 0..N-1 query heads and N..N+G-1 key groups, so a head vector is Dh / 4
// consecutive lanes; the others take values, one workgroup per 64 consecutive
// positions of one causal unit, one stream and one KV group, KV-normed by the
// same lane layout and written transposed ([D_h][U_pad] per slot) through LDS.
// (As two launches, the values with one 64-lane sum per row: 9 + 4 us at 130
// rows, where a launch's latency is all there is.)
constexpr int VP_ROWS = 64;
__global__ __launch_bounds__(256) void qkv_post_kernel(QkvPostArgs a, int rows, int qk_blocks, int blocks_per_unit,
                                                       int block0) {
  __shared__ float vt[64][VP_ROWS + 1];  // [dim][position]
  const int Dh = a.Dh, qpv = Dh / 4;  // threads per head vector
  const int width = a.N * Dh + 2 * a.G * Dh;
  // KV-norm: RMSNorm over D_h (the qpv lanes of the vector) with a learned gain
  auto kvnorm = [&](float4 x, const float* gain, int qd) {
    float ss = x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
    for (int o = qpv / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    const float r = rsqrtf(ss / Dh + a.eps);
    const float4 gv = reinterpret_cast<const float4*>(gain)[qd];
    return make_float4(x.x * r * gv.x, x.y * r * gv.y, x.z * r * gv.z, x.w * r * gv.w);
  };
  const int bid = blockIdx.x + block0;
  if (bid >= qk_blocks) {  // values
    const int vb = bid - qk_blocks;
    const int g = vb % a.G, blk = vb / a.G % blocks_per_unit, bu = vb / a.G / blocks_per_unit;
    const int units_per_batch = a.rows_per_batch / a.U;
    const int lu = bu % units_per_batch, b = bu / units_per_batch;
    const int pos0 = blk * VP_ROWS;
    const int npos = min(VP_ROWS, a.U - pos0);
    const int64_t row0 = (int64_t)b * a.rows_per_batch + (int64_t)lu * a.U + pos0;
    const int per = 256 / qpv, qd = threadIdx.x % qpv;
    for (int p = threadIdx.x / qpv; p < VP_ROWS; p += per) {
      float4 x = *reinterpret_cast<const float4*>(a.raw + (row0 + min(p, npos - 1)) * width + (a.N + a.G + g) * Dh + 4 * qd);
      if (a.vnorm_g) x = kvnorm(x, a.vnorm_g, qd);
      vt[4 * qd][p] = x.x;
      vt[4 * qd + 1][p] = x.y;
      vt[4 * qd + 2][p] = x.z;
      vt[4 * qd + 3][p] = x.w;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int slot = (int)((a.u0 + lu) % a.S);
    const int64_t vbase = ((int64_t)(b * a.G + g) * a.S + slot) * Dh * a.U_pad + pos0;
    for (int d = wave; d < Dh; d += 4)
      if (lane < npos) store_kind(a.vt_ring, vbase + (int64_t)d * a.U_pad + lane, vt[d][lane], a.out_kind);
    return;
  }
  const int slots = a.N + a.G;
  const int64_t t = (int64_t)bid * 256 + threadIdx.x;
  const int64_t per_row = (int64_t)slots * qpv;
  const bool valid = t < (int64_t)rows * per_row;
  const int row = valid ? (int)(t / per_row) : 0;
  const int rem = (int)(t - (int64_t)row * per_row);
  const int hs = valid ? rem / qpv : 0, qd = valid ? rem - hs * qpv : 0;
  float4 x = *reinterpret_cast<const float4*>(a.raw + (int64_t)row * width + hs * Dh + 4 * qd);
  const bool is_q = hs < a.N;
  if (!is_q && a.knorm_g) x = kvnorm(x, a.knorm_g, qd);
  if (!valid) return;
  const int b = row / a.rows_per_batch, rb = row - b * a.rows_per_batch;
  if (a.rope) {
    const int fs = rb / a.L, tok = rb - fs * a.L;
    const float2 c0 = rope_cs(a, 2 * qd, fs, tok), c1 = rope_cs(a, 2 * qd + 1, fs, tok);
    x = make_float4(x.x * c0.x - x.y * c0.y, x.x * c0.y + x.y * c0.x,
                    x.z * c1.x - x.w * c1.y, x.z * c1.y + x.w * c1.x);
  }
  if (is_q) {
    store4(a.q, (int64_t)row * a.N * Dh + hs * Dh + 4 * qd, x, a.out_kind);
    return;
  }
  const int lu = rb / a.U, pos = rb - lu * a.U;
  const int slot = (int)((a.u0 + lu) % a.S);
  const int64_t base = (((int64_t)(b * a.G + hs - a.N) * a.S + slot) * a.U_pad + pos) * Dh;
  store4(a.k_ring, base + 4 * qd, x, a.out_kind);
}

// Temporal RoPE cos / sin of a stack's (sub-)frames: entry (fs, pair) for
// position tau0 + fs; the angle is reduced modulo 2 pi in double precision so
// that long streams keep full accuracy.
__device__ __forceinline__ void rope_time_entry(const RopeTimeArgs& a, int np, int i) {
  const int fs = i / np, pair = i - fs * np;
  float2 r = make_float2(1.f, 0.f);
  if (a.axis[pair] == 0) {
    const double ph = (double)(a.tau0 + fs) * a.freq[pair];
    const double red = ph - 6.283185307179586 * floor(ph * 0.15915494309189535);
    float sn, cs;
    sincosf((float)red, &sn, &cs);
    r = make_float2(cs, sn);
  }
  a.out[i] = r;
}

// The call's prologue in one launch: workgroups below rope_blocks fill the
// temporal RoPE tables of both stacks, the others unshuffle the latents:
// u[(b F + f) L + h W_t + w, c p^2 + i p + j] = z[b, c, f, p h + i, p w + j]; zero padding to K_pad.
__global__ __launch_bounds__(256) void prologue_kernel(RopeTimeArgs r0, RopeTimeArgs r1, int np, int rope_blocks,
                                                       const void* z, int z_kind, int B, int C,
                                                       int F, int H, int W, int p, int K_pad,
                                                       void* u, int out_kind, int packed) {
  if ((int)blockIdx.x < rope_blocks) {
    const int i = blockIdx.x * 256 + threadIdx.x, n0 = r0.n_fs * np, n1 = r1.n_fs * np;
    if (i < n0) rope_time_entry(r0, np, i);
    else if (i - n0 < n1) rope_time_entry(r1, np, i - n0);
    return;
  }
  const int Ht = H / p, Wt = W / p, L = Ht * Wt;
  const int64_t total = (int64_t)B * F * L * K_pad;
  const int64_t nblk = gridDim.x - rope_blocks;
  for (int64_t e = (blockIdx.x - rope_blocks) * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += nblk * blockDim.x) {
    const int k = (int)(e % K_pad);
    const int64_t row = e / K_pad;
    float v = 0.f;
    if (k < C * p * p) {
      const int n = (int)(row % L);
      const int64_t bf = row / L;
      const int f = (int)(bf % F), b = (int)(bf / F);
      const int c = k / (p * p), rem = k % (p * p), i = rem / p, j = rem % p;
      const int h = n / Wt, w = n % Wt;
      const int64_t zi = ((((int64_t)b * C + c) * F + f) * H + (p * h + i)) * W + p * w + j;
      if (z_kind == 0) v = ((const float*)z)[zi];
      else if (z_kind == 1) v = __bfloat162float(((const __hip_bfloat16*)z)[zi]);
      else v = (float)((const _Float16*)z)[zi];
    }
    store_kind(u, packed ? pk16(row, k, K_pad) : e, v, out_kind);
  }
}

__global__ __launch_bounds__(256) void convert_kernel(const float* src, void* dst, int64_t n,
                                                      int out_kind) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x)
    store_kind(dst, e, src[e], out_kind);
}

int grid_for(int64_t total) {
  int64_t b = (total + 255) / 256;
  return (int)(b < 65536 ? (b > 0 ? b : 1) : 65536);
}

struct NormLaunch {
  const float* x;
  int M, D;
  const float *g, *b;
  float eps;
  void* out;
  float* row_scale;
  const float* static_sc;
  unsigned* amax_out;
  int packed;
};

template <int KIND, int OUT>
hipError_t norm_width(const NormLaunch& n, hipStream_t s) {
  auto launch = [&](auto nv, auto full) {
    hipLaunchKernelGGL((norm_kernel<KIND, OUT, decltype(nv)::value, decltype(full)::value>), dim3((n.M + 3) / 4),
                       dim3(256), 0, s, n.x, n.M, n.D, n.g, n.b, n.eps, n.out, n.row_scale, n.static_sc, n.amax_out,
                       n.packed);
    return hipGetLastError();
  };
  using std::integral_constant;
  const std::true_type full{};
  const std::false_type ragged{};
  // the decoder widths (multiples of 256) unbranched, narrow ones with one
  // vector per lane, any other with the general eight
  if (n.D <= 256) return n.D == 256 ? launch(integral_constant<int, 1>{}, full) : launch(integral_constant<int, 1>{}, ragged);
  switch (n.D) {
    case 512: return launch(integral_constant<int, 2>{}, full);
    case 768: return launch(integral_constant<int, 3>{}, full);
    case 1024: return launch(integral_constant<int, 4>{}, full);
    case 1280: return launch(integral_constant<int, 5>{}, full);
    case 1536: return launch(integral_constant<int, 6>{}, full);
    case 1792: return launch(integral_constant<int, 7>{}, full);
    case 2048: return launch(integral_constant<int, 8>{}, full);
    default: return launch(integral_constant<int, 8>{}, ragged);
  }
}

template <int KIND>
hipError_t norm_out(const NormLaunch& n, int out_kind, hipStream_t s) {
  switch (out_kind) {
    case 0: return norm_width<KIND, 0>(n, s);
    case 1: return norm_width<KIND, 1>(n, s);
    case 2: return norm_width<KIND, 2>(n, s);
    default: return norm_width<KIND, 3>(n, s);
  }
}

}  // namespace

hipError_t norm_rows(const float* x, int M, int D, const float* g, const float* b, int kind,
                     float eps, void* out, int out_kind, hipStream_t s, float* row_scale,
                     const float* static_sc, unsigned* amax_out, bool packed) {
  if (M <= 0) return hipSuccess;
  if (D % 4 || D > 2048 || (out_kind == 3 && !row_scale && !static_sc)) return hipErrorInvalidValue;
  if (packed && (out_kind == 3 ? D % 64 : (D % 32 || (out_kind != 0 && out_kind != 1))))
    return hipErrorInvalidValue;
  const NormLaunch n{x, M, D, g, b, eps, out, row_scale, static_sc, amax_out, packed ? 1 : 0};
  if (kind == 0) return norm_out<0>(n, out_kind, s);
  return norm_out<1>(n, out_kind, s);
}

hipError_t quant_rows_e4m3(const void* in, int in_kind, int64_t M, int K, uint8_t* codes,
                           float* scale, hipStream_t s, unsigned* amax_out, bool packed) {
  if (M <= 0) return hipSuccess;
  if (K <= 0 || K % 8 || (in_kind != 0 && in_kind != 2) || (packed && K % 64)) return hipErrorInvalidValue;
  constexpr int64_t most = (int64_t)4 * kMaxLaunch;  // rows of a launch (whole 16-row blocks)
  for (; M > most; M -= most) {
    const hipError_t e = quant_rows_e4m3(in, in_kind, most, K, codes, scale, s, amax_out, packed);
    if (e != hipSuccess) return e;
    in = (const char*)in + most * K * (in_kind == 0 ? 2 : 4);
    codes += most * K;
    scale += most;
  }
  const dim3 grid((unsigned)((M + 3) / 4));
  if (in_kind == 0 && (uintptr_t)in % 16 == 0 && (uintptr_t)codes % 8 == 0) {
    auto launch = [&](auto nv) {
      hipLaunchKernelGGL((quant_rows16_kernel<decltype(nv)::value>), grid, dim3(256), 0, s, (const _Float16*)in, M,
                         codes, scale, amax_out, packed ? 1 : 0);
      return hipGetLastError();
    };
    switch (K) {  // the hidden widths of the decoder sizes (4 D)
      case 1024: return launch(std::integral_constant<int, 2>{});
      case 2048: return launch(std::integral_constant<int, 4>{});
      case 3072: return launch(std::integral_constant<int, 6>{});
      case 4096: return launch(std::integral_constant<int, 8>{});
      case 6144: return launch(std::integral_constant<int, 12>{});
      default: break;
    }
  }
  if (in_kind == 0)
    hipLaunchKernelGGL(quant_rows_kernel<_Float16>, grid, dim3(256), 0, s, (const _Float16*)in, M,
                       K, codes, scale, amax_out, packed ? 1 : 0);
  else
    hipLaunchKernelGGL(quant_rows_kernel<float>, grid, dim3(256), 0, s, (const float*)in, M, K,
                       codes, scale, amax_out, packed ? 1 : 0);
  return hipGetLastError();
}

hipError_t qkv_post(const QkvPostArgs& a, hipStream_t s) {
  const int rows = a.B * a.rows_per_batch;
  if (rows <= 0) return hipSuccess;
  // (a head vector is Dh / 4 lanes of a workgroup, which the sums halve)
  if ((a.Dh != 16 && a.Dh != 32 && a.Dh != 64) || a.rows_per_batch % a.U) return hipErrorInvalidValue;
  const int64_t threads = (int64_t)rows * (a.N + a.G) * (a.Dh / 4);
  const int qk_blocks = (int)((threads + 255) / 256);
  const int blocks_per_unit = (a.U + VP_ROWS - 1) / VP_ROWS;
  const int blocks = qk_blocks + blocks_per_unit * a.B * (a.rows_per_batch / a.U) * a.G;
  hipError_t e = hipSuccess;
  for (int b0 = 0; b0 < blocks && e == hipSuccess; b0 += kMaxLaunch) {
    hipLaunchKernelGGL(qkv_post_kernel, dim3(std::min(blocks - b0, kMaxLaunch)), dim3(256), 0, s, a, rows, qk_blocks,
                       blocks_per_unit, b0);
    e = hipGetLastError();
  }
  return e;
}

hipError_t prologue(const void* z, int z_kind, int B, int C, int F, int H, int W, int p, int K_pad, void* u,
                    int out_kind, bool packed, const RopeTimeArgs& r0, const RopeTimeArgs& r1, int np, hipStream_t s) {
  if (packed && (K_pad % 32 || (out_kind != 0 && out_kind != 1))) return hipErrorInvalidValue;
  const int64_t total = (int64_t)B * F * (H / p) * (W / p) * K_pad;
  const int rope_blocks = ((r0.n_fs + r1.n_fs) * np + 255) / 256;
  hipLaunchKernelGGL(prologue_kernel, dim3(rope_blocks + grid_for(total)), dim3(256), 0, s, r0, r1, np, rope_blocks, z,
                     z_kind, B, C, F, H, W, p, K_pad, u, out_kind, packed ? 1 : 0);
  return hipGetLastError();
}

hipError_t convert_f32_to_16(const float* src, void* dst, int64_t n, int out_kind, hipStream_t s) {
  hipLaunchKernelGGL(convert_kernel, dim3(grid_for(n)), dim3(256), 0, s, src, dst, n, out_kind);
  return hipGetLastError();
}

}  // namespace fd
