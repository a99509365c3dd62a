// 16-bit projections of few rows: calls whose 128 x 128 tiles would leave most
// CUs without a workgroup, and whose time is the K loop's latency chain (one
// 32-column stage per barrier: 375 cycles, 40 us for K = 6144, whatever M is).
// Two kernels, by how many 32 x 32 output tiles there are:
//
// gemm_direct_kernel (fewest tiles): one wave per workgroup and 32 x 32 FN tile,
// operands straight from memory to registers, PD K tiles ahead. There is nothing
// to wait for but the loads: at one wave per CU a 1 KB load takes 30 to 40 cycles
// (weights from memory, 1 us away, 48 KB in flight), 13 us for K = 6144, where the
// MFMA chain itself would take 6 (33 cycles an MFMA, dependent or not).
//
// gemm_small_kernel (more tiles than CUs can each run alone): 2 x 2 waves share
// the operands through LDS, KS K tiles to a barrier, and read the fragments of
// the next stage into a second register set while the current one is
// multiplied. Per-CU load traffic halves against the direct kernel.
//
// Measured, fp16, weights from memory, residual add, this / the 128 x 128 tiles:
// 130 x 1536 x 6144: 13.1 / 39.8 us, 130 x 1536 x 1536: 5.6 / 14.1 (direct);
// 520 x 1536 x 6144: 24.2 / 40.6, 520 x 1536 x 1536: 8.9 / 14.4 (small).
//
// The MFMA sequence of an output element is the one of the large tiles, so
// results do not depend on the tile choice (a call of several frames equals the
// calls of one frame).
#pragma once

#include "gemm_tile.h"

namespace fd {
namespace {

// Epilogue of one wave's 32 FM x 32 FN block.
template <int EPI, typename T, int FM, int FN>
__device__ __forceinline__ void store_small(const EpiParams& ep, const f32x16 (&acc)[FM][FN], int r0, int c0, int M,
                                            int N, int lr, int lk, bool vec) {
  if constexpr (kTransposed<EPI>)
    store_tile_t<EPI, T, FM, FN>(ep, acc, r0, c0, M, N, lr, lk, vec);
  else if constexpr (EPI == EPI_PIXEL || EPI == EPI_LINEAR_PIXEL) {
    if (ep.out_fmt == 0) store_tile<EPI, T, FM, FN, true, 0>(ep, acc, r0, c0, M, N, lr, lk);
    else if (ep.out_fmt == 1) store_tile<EPI, T, FM, FN, true, 1>(ep, acc, r0, c0, M, N, lr, lk);
    else store_tile<EPI, T, FM, FN, true, 2>(ep, acc, r0, c0, M, N, lr, lk);
  } else {
    store_tile<EPI, T, FM, FN, true>(ep, acc, r0, c0, M, N, lr, lk);
  }
}

// One wave per workgroup, 32 x 32 FN outputs, PD K tiles of 32 columns in flight.
// A packed (whole 16-row blocks readable), W packed, as for gemm_mfma_kernel.
template <typename T, int FN, int PD, int EPI>
__global__ __launch_bounds__(64, 1) void gemm_direct_kernel(const T* __restrict__ A, const T* __restrict__ W, int M,
                                                            int N, int K, EpiParams ep, int tiles_m, int tiles_n,
                                                            int vec_store) {
  using V = typename Mfma<T>::V;
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x;
  int tm, tn;
  tile_of(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 32, n0 = tn * 32 * FN;
  const int KB = K / BKD;  // K tiles
  const int lr = lane & 31, lk = lane >> 5;
  // 16-row blocks of this tile in A and W; the ragged edge of a tile rereads the
  // last one (such rows only reach outputs that are not stored)
  const int a_blk = min(2, (M + 15) / 16 - m0 / 16), w_blk = min(2 * FN, (N + 15) / 16 - n0 / 16);
  const __amdgpu_buffer_rsrc_t rA = make_rsrc(A + (int64_t)m0 * K, (uint32_t)a_blk * KB * 1024u);
  const __amdgpu_buffer_rsrc_t rB = make_rsrc(W + (int64_t)n0 * K, (uint32_t)w_blk * KB * 1024u);
  // lane (lk, lr): row lr, K-chunk 2 ks + lk of a K tile at step ks
  const uint32_t lo = (uint32_t)((lr & 15) * 16 + lk * 256);
  const uint32_t va = (uint32_t)min(lr >> 4, a_blk - 1) * KB * 1024u + lo;
  uint32_t vb[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) vb[j] = (uint32_t)min(2 * j + (lr >> 4), w_blk - 1) * KB * 1024u + lo;
  u4 fa[PD][2], fb[PD][2][FN];
  auto load = [&](int p, int kt) {  // past the last K tile the loads reread it
    const uint32_t so = (uint32_t)min(kt, KB - 1) * 1024u;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      fa[p][ks] = __builtin_amdgcn_raw_buffer_load_b128(rA, va + ks * 512, so, 0);
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[p][ks][j] = __builtin_amdgcn_raw_buffer_load_b128(rB, vb[j] + ks * 512, so, 0);
    }
  };
  f32x16 acc[1][FN];
#pragma unroll
  for (int j = 0; j < FN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][j][r] = 0.f;
  auto mul = [&](int p) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const V a = __builtin_bit_cast(V, fa[p][ks]), b = __builtin_bit_cast(V, fb[p][ks][j]);
        acc[0][j] = kTransposed<EPI> ? Mfma<T>::run(b, a, acc[0][j]) : Mfma<T>::run(a, b, acc[0][j]);
      }
  };
#pragma unroll
  for (int p = 0; p < PD; ++p) load(p, p);
  int base = 0;
  for (; base + PD < KB; base += PD)
#pragma unroll
    for (int p = 0; p < PD; ++p) {
      mul(p);
      load(p, base + PD + p);
      __builtin_amdgcn_sched_barrier(0);  // (the loads stay where they are issued)
    }
#pragma unroll
  for (int p = 0; p < PD; ++p)
    if (base + p < KB) mul(p);
  store_small<EPI, T, 1, FN>(ep, acc, m0, n0, M, N, lr, lk, vec_store != 0);
}

// WAVES_M x WAVES_N waves of 32 FM x 32 FN; NS stages of KS 32-column K tiles.
template <int WAVES_M_, int WAVES_N_, int FM_, int FN_, int KS_, int NS_>
struct SmallCfg {
  static constexpr int WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, FM = FM_, FN = FN_, KS = KS_, NS = NS_;
  static constexpr int NW = WAVES_M * WAVES_N, NT = 64 * NW;
  static constexpr int WM = 32 * FM, WN = 32 * FN, BM = WM * WAVES_M, BN = WN * WAVES_N;
  static constexpr int SUB = (BM + BN) * 4;   // 16-byte slots of a 32-column K tile
  static constexpr int STAGE = KS * SUB;
  static constexpr int QB16 = (BM + BN) / 16;            // 16-row blocks of a K tile
  static constexpr int Q = KS * QB16 / NW;               // DMAs per wave and stage
  static constexpr int LDS_BYTES = NS * STAGE * 16;
  static_assert(KS * QB16 % NW == 0, "DMA blocks split evenly over waves");
  static_assert(NS >= 2 && LDS_BYTES <= 163840, "at least 2 stages, within 160 KB of LDS");
  static_assert((NS - 2) * Q < 64, "vmcnt range");
};

// A packed (whole 16-row blocks readable), W packed, as for gemm_mfma_kernel.
template <typename T, class C, int EPI>
__global__ __launch_bounds__(C::NT, 1) void gemm_small_kernel(const T* __restrict__ A, const T* __restrict__ W, int M,
                                                              int N, int K, EpiParams ep, int tiles_m, int tiles_n,
                                                              int vec_store) {
  constexpr int BM = C::BM, BN = C::BN, FM = C::FM, FN = C::FN, KS = C::KS, NS = C::NS, NW = C::NW, Q = C::Q;
  constexpr int NK = 2 * KS;  // MFMA k-steps of a stage
  using V = typename Mfma<T>::V;
  __shared__ uint4 lds[NS * C::STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  tile_of(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int wm0 = (wave / C::WAVES_N) * C::WM, wn0 = (wave % C::WAVES_N) * C::WN;

  const int KB = K / BKD;  // K tiles
  // 16-row blocks of this tile in A and W; the ragged edge of a tile rereads the
  // last one (such rows only reach outputs that are not stored)
  const int a_blk = min(BM / 16, (M + 15) / 16 - m0 / 16), w_blk = min(BN / 16, (N + 15) / 16 - n0 / 16);
  const __amdgpu_buffer_rsrc_t rA = make_rsrc(A + (int64_t)m0 * K, (uint32_t)a_blk * KB * 1024u);
  const __amdgpu_buffer_rsrc_t rB = make_rsrc(W + (int64_t)n0 * K, (uint32_t)w_blk * KB * 1024u);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4*)lds;
  // DMA j of wave w moves block q = j NW + w of the stage: 16-row block q % QB16
  // (A rows, then W rows) of K tile q / QB16, as it lies in memory. K tiles past
  // the end reread the last one and are not multiplied.
  const uint32_t lvoff = (uint32_t)lane * 16u;
  auto dma = [&](int st, int t) {
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const int q = j * NW + wave, sub = q / C::QB16, blk = q - sub * C::QB16;
      const int kt = min(t * KS + sub, KB - 1);
      const bool isA = blk < BM / 16;
      const int rb = isA ? min(blk, a_blk - 1) : min(blk - BM / 16, w_blk - 1);
      const uint32_t soff = __builtin_amdgcn_readfirstlane((uint32_t)(rb * KB + kt) * 1024u);
      const uint32_t m0addr =
          __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(st * C::STAGE + sub * C::SUB + blk * 64) * 16u);
      const __amdgpu_buffer_rsrc_t r = isA ? rA : rB;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
      asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :
                   : "s"(m0addr), "v"(lvoff), "s"(r), "s"(soff)
                   : "m0");
#pragma clang diagnostic pop
    }
  };
  // this wave's DMAs but those of the NS - 2 youngest stages (drain: all), and its
  // LDS reads, are done; then the barrier publishes the stage and frees the one
  // read before
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
  const int ia = (wm0 / 16 + (lr >> 4)) * 64 + (lr & 15), ib = ((BM + wn0) / 16 + (lr >> 4)) * 64 + (lr & 15);
  V fa[2][NK][FM], fb[2][NK][FN];
  auto load_frags = [&](int slot, int st) {
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
      const uint4* sb = lds + st * C::STAGE + (ks >> 1) * C::SUB;
      const int ch = (2 * (ks & 1) + lk) * 16;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const uint4 v = sb[ia + ch + i * 128];
        fa[slot][ks][i] = *reinterpret_cast<const V*>(&v);
      }
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const uint4 w = sb[ib + ch + j * 128];
        fb[slot][ks][j] = *reinterpret_cast<const V*>(&w);
      }
    }
  };
  auto mfma1 = [&](int slot, int ks) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = kTransposed<EPI> ? Mfma<T>::run(fb[slot][ks][j], fa[slot][ks][i], acc[i][j])
                                     : Mfma<T>::run(fa[slot][ks][i], fb[slot][ks][j], acc[i][j]);
  };

  // Stage t sits in LDS stage t % NS and, while multiplied, in register set
  // t & 1. Step t: the barrier publishes stage t + 1 (and frees the LDS stage
  // of t, whose fragments everyone has read), its fragments are read, the stage of t
  // is refilled with t + NS, and stage t is multiplied.
  const int TS = (KB + KS - 1) / KS;
#pragma unroll
  for (int p = 0; p < NS - 1; ++p)
    if (p < TS) dma(p, p);
  // stage 0 only; up to NS - 2 younger ones may be in flight
  sync(TS < NS - 1);
  load_frags(0, 0);
  if (NS - 1 < TS) dma(NS - 1, NS - 1);
  int sc = 0;
  auto step = [&](int t, int slot) {
    const int sn = sc + 1 == NS ? 0 : sc + 1;
    sync(t + NS > TS);
    load_frags(slot ^ 1, sn);
    if (t + NS < TS) dma(sc, t + NS);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) mfma1(slot, ks);
    sc = sn;
  };
  int t = 0;
  for (; t + 2 <= TS - 1; t += 2) {
    step(t, 0);
    step(t + 1, 1);
  }
  if (t < TS - 1) {
    step(t, 0);
    ++t;
  }
  // the last stage, in set t & 1; its K tiles past the end are left out
  const int last = KB - t * KS;
  if (t & 1) {
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[0][ks][i] = fa[1][ks][i];
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[0][ks][j] = fb[1][ks][j];
    }
  }
#pragma unroll
  for (int sub = 0; sub < KS; ++sub)
    if (sub < last) {
      mfma1(0, 2 * sub);
      mfma1(0, 2 * sub + 1);
    }
  store_small<EPI, T, FM, FN>(ep, acc, m0 + wm0, n0 + wn0, M, N, lr, lk, vec_store != 0);
}

}  // namespace
}  // namespace fd
