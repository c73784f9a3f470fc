// bf16 GEMM main loop for small tiles, C = A W^T: a deep LDS ring.
//
// A product with about one tile per CU is a chain of tile loads: with two buffers every K
// tile costs a memory latency.  Here NS K tiles of 64 are in the ring and the loads of
// NS - 1 of them stay in flight across the barriers (counted waits).  Four waves (2 x 2)
// share the tile.  64 x 64 tiles, against the two-buffer loop of gemm_bf16_kernel on the same
// tiles (weights from HBM): 64 x 3 072 x 2 048 17.2 -> 12.2 us, 384 x 768 x 2 048 16.5 -> 12.1,
// 384 x 4 096 x 768 9.0 -> 8.3, 1 024 x 2 048 x 2 048 18.6 -> 15.8; with more than two tiles per
// CU the blocks hide each other's latency and the two-buffer loop is as fast or faster
// (launch_small).  Also measured: fragments loaded straight into registers, the waves splitting
// K (384 x 768 x 2 048 13.4 to 17.9 us: the loads touch 64 bytes a row), and eight waves splitting
// every K tile (10.8 us there, but 23.5 at 3 072 rows).
#pragma once
#include "gemm_kernel.h"

namespace tadm {
namespace {

// A K tile's fragments (both 32-deep halves), read and waited for in one block, so that no
// instruction can be placed between a read and its wait.
__device__ __forceinline__ void read_tile(uint32_t a, uint32_t w, bf16x8 (&fa)[2][2], bf16x8 (&fw)[2][2]) {
  asm volatile(
      "ds_read_b128 %0, %8\n\t"
      "ds_read_b128 %4, %9\n\t"
      "ds_read_b128 %1, %8 offset:2048\n\t"
      "ds_read_b128 %5, %9 offset:2048\n\t"
      "ds_read_b128 %2, %10\n\t"
      "ds_read_b128 %6, %11\n\t"
      "ds_read_b128 %3, %10 offset:2048\n\t"
      "ds_read_b128 %7, %11 offset:2048\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(fa[0][0]), "=&v"(fa[0][1]), "=&v"(fa[1][0]), "=&v"(fa[1][1]), "=&v"(fw[0][0]), "=&v"(fw[0][1]),
        "=&v"(fw[1][0]), "=&v"(fw[1][1])
      : "v"(a), "v"(w), "v"(a ^ 64), "v"(w ^ 64)
      : "memory");
}
__device__ __forceinline__ void read_tile(uint32_t a, uint32_t w, bf16x8 (&fa)[2][1], bf16x8 (&fw)[2][1]) {
  asm volatile(
      "ds_read_b128 %0, %4\n\t"
      "ds_read_b128 %2, %5\n\t"
      "ds_read_b128 %1, %6\n\t"
      "ds_read_b128 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(fa[0][0]), "=&v"(fa[1][0]), "=&v"(fw[0][0]), "=&v"(fw[1][0])
      : "v"(a), "v"(w), "v"(a ^ 64), "v"(w ^ 64)
      : "memory");
}
__device__ __forceinline__ void read_tile(uint32_t a, uint32_t w, bf16x8 (&fa)[2][2], bf16x8 (&fw)[2][3]) {
  asm volatile(
      "ds_read_b128 %0, %10\n\t"
      "ds_read_b128 %1, %10 offset:2048\n\t"
      "ds_read_b128 %4, %11\n\t"
      "ds_read_b128 %5, %11 offset:2048\n\t"
      "ds_read_b128 %6, %11 offset:4096\n\t"
      "ds_read_b128 %2, %12\n\t"
      "ds_read_b128 %3, %12 offset:2048\n\t"
      "ds_read_b128 %7, %13\n\t"
      "ds_read_b128 %8, %13 offset:2048\n\t"
      "ds_read_b128 %9, %13 offset:4096\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(fa[0][0]), "=&v"(fa[0][1]), "=&v"(fa[1][0]), "=&v"(fa[1][1]), "=&v"(fw[0][0]), "=&v"(fw[0][1]),
        "=&v"(fw[0][2]), "=&v"(fw[1][0]), "=&v"(fw[1][1]), "=&v"(fw[1][2])
      : "v"(a), "v"(w), "v"(a ^ 64), "v"(w ^ 64)
      : "memory");
}

template <int BM, int BN, int NS, int MINB, EpiKind KIND>
__global__ __launch_bounds__(256, MINB) void gemm_ring_kernel(GemmProblem p, EpiParams ep) {
#ifdef __HIP_DEVICE_COMPILE__  // buffer resources are a device type: the host pass only needs the stub
  using E = Epi<KIND, bf16>;
  constexpr int NW = 4, ROW = 128, STAGE = (BM + BN) * ROW;
  constexpr int LA = BM / 8 / NW, LW = BN / 8 / NW, LPT = LA + LW;
  static_assert(LA * 8 * NW == BM && LW * 8 * NW == BN, "tile rows must split evenly over waves");
  constexpr int WTM = BM / 2, WTN = BN / 2, TM = WTM / 16, TN = WTN / 16;
  __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  if (p.M_dev) p.M = min(*p.M_dev, p.M);  // rows present this call; the grid was sized for p.M
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  int tmi, tni;
  tile_of(p, blockIdx.x, tiles_m, tiles_n, tmi, tni);
  if (tmi >= tiles_m) return;  // padding of a banded grid, or no rows for this block
  const int m0 = __builtin_amdgcn_readfirstlane(tmi * BM), n0 = __builtin_amdgcn_readfirstlane(tni * BN);
  const int NKT = p.K / 64, kt_base = (int)((long)blockIdx.y * NKT / p.ksplit);
  const int nk = (int)((long)(blockIdx.y + 1) * NKT / p.ksplit) - kt_base;

  const int lrow = lane >> 3, lchunk = (lane & 7) ^ (lane >> 3);
  auto rsrc = [](const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, -1, 0x00027000);
  };
  const bf16* A1 = static_cast<const bf16*>(p.A1);
  const bf16* A2 = p.A2 ? static_cast<const bf16*>(p.A2) - p.K1 : A1;
  const auto ra1 = rsrc(A1 + (size_t)m0 * p.lda1), ra2 = rsrc(A2 + (size_t)m0 * (p.A2 ? p.lda2 : p.lda1));
  const auto rw = rsrc(static_cast<const bf16*>(p.W) + (size_t)n0 * p.ldw);
  uint32_t offA[LA], offA2[LA], offW[LW];
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const uint32_t r = (uint32_t)(min(m0 + (wave + NW * j) * 8 + lrow, p.M - 1) - m0);
    offA[j] = r * (uint32_t)(2 * p.lda1) + 16 * lchunk;
    offA2[j] = r * (uint32_t)(2 * (p.A2 ? p.lda2 : p.lda1)) + 16 * lchunk;
  }
#pragma unroll
  for (int j = 0; j < LW; ++j)
    offW[j] = (uint32_t)(min(n0 + (wave + NW * j) * 8 + lrow, p.N - 1) - n0) * (uint32_t)(2 * p.ldw) + 16 * lchunk;
  auto issue = [&](int kt, int slot) {
    const int k0 = (kt_base + kt) * 64;
    const bool second = k0 >= p.K1;
    const auto r = second ? ra2 : ra1;
    char* sb = smem + slot * STAGE;
#pragma unroll
    for (int j = 0; j < LA; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)(sb + (wave + NW * j) * 1024), 16, second ? offA2[j] : offA[j],
                                               k0 * 2, 0, 0);
#pragma unroll
    for (int j = 0; j < LW; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(sb + BM * ROW + (wave + NW * j) * 1024), 16, offW[j], k0 * 2,
                                               0, 0);
  };

  // epilogue operands first: the oldest vector-memory operations, which the counted waits
  // below only ever wait for
  constexpr int NPRE = PreCount<E>::value;
  constexpr bool PRE = NPRE > 0 && TN * TM * NPRE <= 18;
  float4 pre[PRE ? TN : 1][PRE ? TM : 1][PRE ? NPRE : 1];
  if constexpr (PRE) {
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
      for (int b = 0; b < TM; ++b) {
        const int m = m0 + wm * WTM + (lane & 15) + b * 16, n = n0 + wn * WTN + 4 * (lane >> 4) + a * 16;
        if (m < p.M && n < p.N) E::pre(ep, m, n, pre[a][b]);
      }
  }

#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) issue(s, s);

  f32x4 acc[TN][TM];
  const bf16x8 zero = mfma_zero_operand();
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) mfma_first(acc[a][b], zero, zero);

  const int fr = lane & 15, fq = lane >> 4, sw = lane & 7;
  const uint32_t lbase = (uint32_t)(uintptr_t)(lds_ptr)smem;
  const uint32_t la = lbase + (wm * WTM + fr) * ROW + ((fq ^ sw) * 16);
  const uint32_t lw = lbase + BM * ROW + (wn * WTN + fr) * ROW + ((fq ^ sw) * 16);

  int slot = 0;  // kt % NS
  for (int kt = 0; kt < nk; ++kt) {
    // K tile kt has landed for every wave, and every wave has read K tile kt - 1
    if (kt + NS - 2 < nk)
      asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 2) * LPT) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    if (kt + NS - 1 < nk) issue(kt + NS - 1, slot == 0 ? NS - 1 : slot - 1);
    const uint32_t o = slot * STAGE;
    bf16x8 fa[2][TM], fw[2][TN];
    read_tile(la + o, lw + o, fa, fw);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) mfma_acc(acc[a][b], fw[h][a], fa[h][b]);
    slot = slot + 1 == NS ? 0 : slot + 1;
  }
  // the last products must be written before any accumulator is read back (see
  // gemm_bf16_kernel)
  asm volatile("s_nop 15\n s_nop 15\n s_nop 15" ::: "memory");
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) asm volatile("" : "+a"(acc[a][b]));
  finish_tile<BM, BN, sizeof(smem), 2, 2, KIND, PRE>(p, ep, acc, pre, m0, n0, blockIdx.y, wave, lane, smem);
#endif
}

template <int BM, int BN, int NS, int MINB, EpiKind K>
hipError_t launch_ring(const GemmProblem& p0, const EpiParams& e, hipStream_t s) {
  GemmProblem p = p0;
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  if (!p.M_dev) xcd_regions(tiles_m, tiles_n, BM, BN, p.rm, p.rn);
  if (BN == 96 && p.rm > 0) {
    // two of these tiles per CU fill the chip: an XCD holds 64, and where its region is too long
    // (an odd number of tile rows leaves 1 x 8 regions) a band streams fewer rows per K step
    // (residual 3 500 x 768 x 768, regions of 55 x 1 tiles: 14.5 -> 12.2 us, x 2 048 24.0 -> 20.7; 3 072
    // rows, regions of 6 x 8: 11.4 against 11.8)
    const int wm = p.rm < 64 ? p.rm : 64, wn = (64 + wm - 1) / wm, h = xcd_band(tiles_m, BM, BN, 64);
    if (wm * BM + (wn < p.rn ? wn : p.rn) * BN > h * BM + (64 + h - 1) / h * BN) p.rm = p.rn = 0;
  }
  p.band = p.rm > 0 ? 0 : xcd_band(tiles_m, BM, BN, 32);
  const int blocks = p.band > 0 ? (tiles_m * tiles_n + 7) / 8 * 8 : tiles_m * tiles_n;
  launch_timed(gemm_ring_kernel<BM, BN, NS, MINB, K>, dim3(blocks, p.ksplit), dim3(256), 0, s, p, e);
  return hipGetLastError();
}

}  // namespace
}  // namespace tadm
