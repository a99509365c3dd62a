// Dense projections of the decoder: C = A W^T + b with fused epilogues.
//
// Every Linear layer of the decoder goes through here: the latent projection
// (Eq. projection), the QKV / output / MLP projections of each block (Sec. 3.2),
// the temporal upsampling Linear D -> r_t D (Eq. temporal_upsample) and the
// 2-layer pixel head (Sec. 3.4 Step 3). The epilogues fuse what follows each
// projection: bias, residual add into the fp32 stream, SiLU / GELU / SwiGLU,
// the channel -> sub-frame reshape of Step 1 and the PixelShuffle store.
//
// 16-bit path: one workgroup of wave64s computes a BM x BN tile with the
// gfx950 32x32x16 MFMA (fp32 accumulate). A and W are both K-contiguous; K
// tiles of 32 columns are copied from memory straight into LDS by the buffer
// unit (buffer_load ... lds, no register staging) several tiles ahead of the
// MFMAs, and read back as MFMA fragments with 16-byte ds_read_b128 per lane.
// Both operands are stored in fragment order (pack_w16_index), so the 16 rows
// one ds_read_b128 serves at once are 256 contiguous bytes of LDS.
#pragma once

#include "gemm_small.h"
#include "gemm_tile.h"

namespace fd {
namespace {

template <typename T, class C, int EPI>
__global__ __launch_bounds__(C::NT, C::MIN_BLOCKS) void gemm_mfma_kernel(
    const T* __restrict__ A, const T* __restrict__ W, int M, int N, int K,
    EpiParams ep, int tiles_m, int tiles_n, int vec_store) {
  constexpr int BM = C::BM, BN = C::BN, FM = C::FM, FN = C::FN, NS = C::NS, NW = C::NW;
  constexpr int QA = C::QA, Q = C::QA + C::QB, STAGE = C::STAGE;
  using V = typename Mfma<T>::V;
  __shared__ uint4 lds[NS * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  tile_of(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int wm0 = (wave / C::WAVES_N) * C::WM, wn0 = (wave % C::WAVES_N) * C::WN;

  // A and W are packed K-tile-major: blocks of 16 rows x 32 K-columns (1 KB),
  // block (row / 16, k / 32) at ((row / 16) (K / 32) + k / 32) KB, in whole
  // 16-row blocks, so each DMA reads one contiguous 1 KB block.
  const int KB = K / BKD;  // K tiles
  const int nblk_a = min(BM / 16, (M + 15) / 16 - m0 / 16), nblk_w = min(BN / 16, (N + 15) / 16 - n0 / 16);
  const __amdgpu_buffer_rsrc_t rA = make_rsrc(A + (int64_t)(m0 / 16) * KB * 512, (uint32_t)nblk_a * KB * 1024u);
  const __amdgpu_buffer_rsrc_t rB = make_rsrc(W + (int64_t)(n0 / 16) * KB * 512, (uint32_t)nblk_w * KB * 1024u);
  // DMA j of this wave fills block q = j NW + wave of the stage (A blocks for
  // j < QA, W blocks after); lane l moves the block's 16 bytes at 16 l.
  uint32_t voff[Q];
#pragma unroll
  for (int j = 0; j < Q; ++j) {
    const int q = j * NW + wave;
    voff[j] = (uint32_t)(j >= QA ? q - BM / 16 : q) * KB * 1024u + (uint32_t)lane * 16u;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4*)lds;
  // DMA instruction j of the refill of stage st with K tile kt
  auto dma1 = [&](int st, int kt, int j) {
    const uint32_t soff = (uint32_t)kt * 1024u;
    const uint32_t m0addr = lds0 + (uint32_t)(st * STAGE + 64 * (j * NW + wave)) * 16u;
    // M0 is reserved by the compiler, but nothing else in this kernel reads it
    // (no LDS DMA builtins, interpolation, GWS or message sends).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(m0addr), "v"(voff[j]), "s"(j < QA ? rA : rB), "s"(soff)
                 : "m0");
#pragma clang diagnostic pop
  };
  auto dma = [&](int st, int kt) {
#pragma unroll
    for (int j = 0; j < Q; ++j) dma1(st, kt, j);
  };
  // Every wave waits for its own DMAs of the next tile (all but the (NS - 2) Q
  // youngest, or all of them near the end of K) and for its LDS reads; the
  // barrier then makes the tile visible and frees the stage read before it.
  auto sync = [&](bool drain) {
    if (drain) __builtin_amdgcn_s_waitcnt(FD_VMCNT(0));
    else __builtin_amdgcn_s_waitcnt(FD_VMCNT((NS - 2) * Q));
    __builtin_amdgcn_s_waitcnt(FD_LGKMCNT0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int lr = lane & 31, lk = lane >> 5;
  // slot of fragment row (A: wm0 + lr, W: BM + wn0 + lr) at k-step ks: chunk
  // 2 ks + lk of its block
  const int ia0 = (wm0 / 16 + (lr >> 4)) * 64 + lk * 16 + (lr & 15), ia1 = ia0 + 32;
  const int ib0 = ((BM + wn0) / 16 + (lr >> 4)) * 64 + lk * 16 + (lr & 15), ib1 = ib0 + 32;
  V fa[2][FM], fb[2][FN];
  auto load_frags = [&](int slot, int st, int ks) {
    const uint4* sb = lds + st * STAGE;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const uint4 v = sb[(ks ? ia1 : ia0) + i * 128];
      fa[slot][i] = *reinterpret_cast<const V*>(&v);
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const uint4 v = sb[(ks ? ib1 : ib0) + j * 128];
      fb[slot][j] = *reinterpret_cast<const V*>(&v);
    }
  };
  auto mfmas = [&](int slot) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = kTransposed<EPI> ? Mfma<T>::run(fb[slot][j], fa[slot][i], acc[i][j])
                                     : Mfma<T>::run(fa[slot][i], fb[slot][j], acc[i][j]);
  };
  // the MFMAs of a k-step with DMA instructions j0 .. j0 + Q / 2 - 1 of a
  // stage refill between them, evenly spaced, in this order
  auto mfmas_dma = [&](int slot, int st, int kt, int j0) {
    if constexpr (C::IL) {
      constexpr int NM = FM * FN, ND = Q / 2;
      static_assert(Q % 2 == 0 && ND <= NM, "DMA spacing");
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const int i = m / FN, j = m % FN;
        acc[i][j] = kTransposed<EPI> ? Mfma<T>::run(fb[slot][j], fa[slot][i], acc[i][j])
                                     : Mfma<T>::run(fa[slot][i], fb[slot][j], acc[i][j]);
        if ((m + 1) * ND / NM != m * ND / NM) {
          __builtin_amdgcn_sched_barrier(0);
          dma1(st, kt, j0 + m * ND / NM);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };

  // Tile t sits in stage t % NS. The loop starts at the barrier (whose
  // explicit lgkmcnt(0) leaves no LDS read pending at the loop header), then
  // reads k-step 0 of tile t + 1, multiplies k-step 1 of tile t, reads k-step 1
  // of tile t + 1, refills the stage of tile t (read by everyone before the
  // barrier) with tile t + NS, and multiplies k-step 0 of tile t + 1.
  const int KT = K / BKD;
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < KT) dma(p, p);
  sync(KT < NS - 1);
  load_frags(0, 0, 0);
  load_frags(1, 0, 1);
  if (NS - 1 < KT) dma(NS - 1, NS - 1);
  mfmas(0);
  int sc = 0;  // stage of tile t
  int t = 0;
  if constexpr (C::IL) {
    for (; t < KT - NS; ++t) {
      const int sn = sc + 1 == NS ? 0 : sc + 1;
      sync(false);
      load_frags(0, sn, 0);
      mfmas_dma(1, sc, t + NS, 0);
      load_frags(1, sn, 1);
      mfmas_dma(0, sc, t + NS, Q / 2);
      sc = sn;
    }
  }
  for (; t < KT - 1; ++t) {
    const int sn = sc + 1 == NS ? 0 : sc + 1;
    sync(t + NS - 1 >= KT);
    load_frags(0, sn, 0);
    mfmas(1);
    load_frags(1, sn, 1);
    if (t + NS < KT) dma(sc, t + NS);
    mfmas(0);
    sc = sn;
  }
  mfmas(1);
  if constexpr (kTransposed<EPI>)
    store_tile_t<EPI, T, FM, FN>(ep, acc, m0 + wm0, n0 + wn0, M, N, lr, lk, vec_store != 0);
  else if constexpr (EPI == EPI_PIXEL || EPI == EPI_LINEAR_PIXEL) {
    // one instantiation per pixel format, chosen once per tile (a format test
    // per store makes the epilogue loops too large to unroll, and the
    // accumulators would go to scratch memory)
    constexpr bool R = !(C::NW == 4 && C::MIN_BLOCKS == 1);
    if (ep.out_fmt == 0) store_tile<EPI, T, FM, FN, R, 0>(ep, acc, m0 + wm0, n0 + wn0, M, N, lr, lk);
    else if (ep.out_fmt == 1) store_tile<EPI, T, FM, FN, R, 1>(ep, acc, m0 + wm0, n0 + wn0, M, N, lr, lk);
    else store_tile<EPI, T, FM, FN, R, 2>(ep, acc, m0 + wm0, n0 + wn0, M, N, lr, lk);
  } else {
    store_tile<EPI, T, FM, FN, !(C::NW == 4 && C::MIN_BLOCKS == 1)>(ep, acc, m0 + wm0, n0 + wn0, M, N, lr, lk);
  }
}

// Four consecutive columns of a 16-bit output land contiguously and 8-byte aligned
// in the destination.
inline bool vec_stores(const GemmArgs& g) {
  return g.N % 4 == 0 && g.ep.ld_out % 4 == 0 && (uintptr_t)g.ep.out_a % 8 == 0;
}

template <typename T, int FN, int PD, int EPI>
hipError_t launch_direct(const GemmArgs& g, hipStream_t s) {
  const int tm = (g.M + 31) / 32, tn = (g.N + 32 * FN - 1) / (32 * FN);
  hipLaunchKernelGGL((gemm_direct_kernel<T, FN, PD, EPI>), dim3(tm * tn), dim3(64), 0, s, (const T*)g.A,
                     (const T*)g.W, g.M, g.N, g.K, g.ep, tm, tn, vec_stores(g) ? 1 : 0);
  return hipGetLastError();
}

template <typename T, class C, int EPI>
hipError_t launch_small(const GemmArgs& g, hipStream_t s) {
  const int tm = (g.M + C::BM - 1) / C::BM, tn = (g.N + C::BN - 1) / C::BN;
  hipLaunchKernelGGL((gemm_small_kernel<T, C, EPI>), dim3(tm * tn), dim3(C::NT), 0, s, (const T*)g.A, (const T*)g.W,
                     g.M, g.N, g.K, g.ep, tm, tn, vec_stores(g) ? 1 : 0);
  return hipGetLastError();
}

template <typename T, class C, int EPI>
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
  const int tm = (g.M + C::BM - 1) / C::BM, tn = (g.N + C::BN - 1) / C::BN;
  hipLaunchKernelGGL((gemm_mfma_kernel<T, C, EPI>), dim3(tm * tn), dim3(C::NT), 0, s,
                     (const T*)g.A, (const T*)g.W, g.M, g.N, g.K, g.ep, tm, tn, vec_stores(g) ? 1 : 0);
  return hipGetLastError();
}

// Tile choice, measured on the decoder's shapes at 480p, 720p and 1080p and the S,
// B, L and XL widths (random fp16 data). 128 x 256 tiles (TileD), two workgroups
// to a CU, let one workgroup's epilogue and pipeline fill run under the other's
// MFMAs, and win wherever they come to at least two rounds of 512 or to one
// nearly full round. us, 128 x 256 / what else serves that shape best:
//   SwiGLU 14400 x 12288 x 1536 459 / 471 (256 x 256), 6400 x 8192 x 1024 103 /
//   120, 1040 x 12288 x 1536 46 / 51; but 1560 x 12288 x 1536 (1.2 rounds) 65 / 64
//   SiLU 14400 x 6144 x 1536 259 / 282, 6240 x 6144 x 1536 116 / 133
//   residual add 14400 x 1536 x 6144 250 / 280, 32640 x 1536 x 1536 174 / 192
template <typename T, int EPI>
hipError_t dispatch_tiles(const GemmArgs& g, hipStream_t s) {
  auto tiles = [&](int bm, int bn) { return ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn); };
  // Few output tiles: a wave per 32-row tile, then 2 x 2 waves through LDS (see
  // gemm_small.h). Each line lies where the next kernel is as fast (us, this /
  // next): residual adds of K = 6144 at 384 tiles of 32 x 32 21 / 28, at 624 28 /
  // 24 (small), at 816 24 / 41, at 1584 48 / 42 (large); QKV (32 x 64 tiles, K =
  // 1536) at 240 11 / 17, at 510 16 / 18, at 990 19 / 24, at 1470 21 / 24, at 2220
  // 35 / 31; SwiGLU at 384 13 / 16, at 960 20 / 15.
  if constexpr (EPI == EPI_QKV) {
    if (tiles(32, 64) <= 640) return launch_direct<T, 2, 6, EPI>(g, s);
    if (tiles(32, 64) <= 1600) return launch_small<T, SmallCfg<2, 2, 1, 2, 2, 3>, EPI>(g, s);
  } else if constexpr (EPI == EPI_SWIGLU) {
    if (tiles(32, 64) <= 400) return launch_direct<T, 2, 6, EPI>(g, s);
  } else {
    if (tiles(32, 32) <= 500) return launch_direct<T, 1, 12, EPI>(g, s);
    if (tiles(32, 32) <= 1000) return launch_small<T, SmallCfg<2, 2, 1, 1, 4, 4>, EPI>(g, s);
  }
  const int tl = tiles(256, 256), td = tiles(128, 256), tm = tiles(192, 128);
  const bool d_round = td > 400 && td <= 512;  // one nearly full round, two per CU
  if constexpr (EPI == EPI_STORE_F32) {
    // the embedding's K loop is two stages: nothing but the store (3600 rows: 7.4
    // us against 9.7 with 192 x 128 tiles, 8160 rows 10.8 / 19.0 with 256 x 192)
    if (g.K <= 128) return launch_gemm<T, TileS, EPI>(g, s);
  } else if constexpr (EPI == EPI_SWIGLU || EPI == EPI_QKV) {
    // (QKV, 32640 / 8160 x 1920 x 1536: 196 / 204 us, 54 / 57)
    if (td >= 1024 || d_round) return launch_gemm<T, TileD, EPI>(g, s);
    if (tl >= 160) return launch_gemm<T, TileS, EPI>(g, s);
  } else {
    // one workgroup of 128 x 64 per CU (us, this / 128 x 128): residual adds 1040
    // x 1536 x 6144 37 / 42, 1600 x 1024 x 4096 25 / 32; 1560 x 1536 x 6144, 312
    // tiles, 53 / 44
    if (tiles(128, 64) <= 256) return launch_gemm<T, TileH, EPI>(g, s);
    // 128 x 192 tiles that make one nearly full round, two per CU: the pixel store
    // of 14400 x 768 x 6144 134 / 142 us (a residual add would spill registers)
    if constexpr (EPI == EPI_PIXEL || EPI == EPI_LINEAR_PIXEL)
      if (const int te = tiles(128, 192); te > 400 && te <= 512) return launch_gemm<T, TileE, EPI>(g, s);
    if ((EPI == EPI_STORE_SILU || EPI == EPI_STORE_GELU) && td >= 300)
      return launch_gemm<T, TileD, EPI>(g, s);
    // temporal upsampling of 3600 rows (696 tiles): 75 / 81 us; of 8160 rows 167 /
    // 162 with the 256-row tiles below
    if (EPI == EPI_TUP && td >= 512 && tl < 512) return launch_gemm<T, TileD, EPI>(g, s);
    if constexpr (EPI == EPI_RESID_ADD) {
      if (g.K <= 2048) {
        if (td >= 1024) return launch_gemm<T, TileD, EPI>(g, s);
      } else if (td >= 600 && tl * 10 < (tl + 255) / 256 * 256 * 9) {
        // (256 x 256 tiles where their last round is nearly full: 21000 x 1536 x
        // 6144, 498 tiles, 351 / 361 us)
        return launch_gemm<T, TileD, EPI>(g, s);
      }
    }
    if (tl >= 160 && !(EPI == EPI_RESID_ADD && g.K <= 2048)) {
      // 256 x 192 tiles where their rounds of 256 CUs, weighted by tile area, are
      // fewer than those of 256 x 256 tiles (the GELU epilogue's erf needs more
      // registers than a 4-wave 256 x 192 tile leaves)
      if constexpr (EPI != EPI_STORE_GELU) {
        const int rounds_l = (tl + 255) / 256, rounds_w = (tiles(256, 192) + 255) / 256;
        if (4 * rounds_w * 3 < 4 * rounds_l * 4) return launch_gemm<T, TileW, EPI>(g, s);
      }
      return launch_gemm<T, TileL, EPI>(g, s);
    }
    if constexpr (EPI == EPI_RESID_ADD) {
      // residual adds: 192 x 128 tiles with 4 stages (two workgroups per CU)
      // behind a long K loop in one round, and wherever they fill most of one
      // round of two per CU (396 tiles, the 480p refinement's: 37 / 43 us; at 272,
      // 6400 x 1024 x 4096, 76 / 57)
      if ((tm >= 200 && tm <= 256 && g.K > 2048) || (tm >= 340 && tm <= 512))
        return launch_gemm<T, TileM4, EPI>(g, s);
    }
  }
  // 192 x 128 tiles in one nearly full round of one workgroup per CU (the 720p
  // backbone's residual adds); where even 128 x 128 tiles leave CUs idle, each CU
  // runs one workgroup, with 6 stages in flight (residual adds with 8 waves: 1560 x
  // 1536 x 1536 15.1 / 16.2 us); otherwise 128 x 128 tiles, several per CU
  if (tm >= 200 && tm <= 256) return launch_gemm<T, TileM, EPI>(g, s);
  if (tiles(128, 128) <= 256) {
    if constexpr (EPI == EPI_RESID_ADD) return launch_gemm<T, TileS8, EPI>(g, s);
    else return launch_gemm<T, TileS1, EPI>(g, s);
  }
  return launch_gemm<T, TileS, EPI>(g, s);
}

template <typename T>
hipError_t dispatch_epi(const GemmArgs& g, hipStream_t s) {
  switch (g.epi) {
    case EPI_STORE_F32: return dispatch_tiles<T, EPI_STORE_F32>(g, s);
    case EPI_RESID_ADD: return dispatch_tiles<T, EPI_RESID_ADD>(g, s);
    case EPI_STORE_SILU: return dispatch_tiles<T, EPI_STORE_SILU>(g, s);
    case EPI_STORE_GELU: return dispatch_tiles<T, EPI_STORE_GELU>(g, s);
    case EPI_SWIGLU: return dispatch_tiles<T, EPI_SWIGLU>(g, s);
    case EPI_TUP: return dispatch_tiles<T, EPI_TUP>(g, s);
    case EPI_PIXEL: return dispatch_tiles<T, EPI_PIXEL>(g, s);
    case EPI_LINEAR_PIXEL: return dispatch_tiles<T, EPI_LINEAR_PIXEL>(g, s);
    case EPI_QKV: return dispatch_tiles<T, EPI_QKV>(g, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
}  // namespace fd
