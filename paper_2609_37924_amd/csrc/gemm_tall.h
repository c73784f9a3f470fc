// The vocabulary head's main loop: 256 x 128 tiles at two blocks per CU, C = A W^T.
//
// Four wave64s (2 x 2, 128 x 64 outputs each), K tiles of 64, 80 KB of LDS: two blocks share a
// CU, so that one block's sampling epilogue (about as many vector cycles as the tile's
// products take matrix cycles at K = 2 048) runs beside the other's products.  The tile loads
// bound the products: 1.5 times those of 256 x 256 tiles (one block per CU, no overlap), 0.75
// times those of 128 x 128 ones.  Plain stores, 4 096 x 50 304 x 2 048: 128 x 128 tiles 866 us,
// this loop 726, 256 x 256 671; 512 x 262 144 x 4 608: 1 351, 1 054 and 933 us.
//
// A K tile is four phases as in the ping-pong kernel (quadrants (a0, b0), (a0, b1), (a1, b1),
// (a1, b0); reads a0 | b1 | a1 | the next b0), one barrier per phase.  LDS holds three
// activation halves (128 rows, 16 KB each) and four weight halves (64 rows, 8 KB each),
// each ring filled one half per second phase: an activation half four phases before it is
// read, a weight half six.  Reads of phase p are waited for after the barrier of phase p, so a
// slot read in phase p is free for loads issued in phase p + 2, past the next barrier.
// Counted waits: the halves read in even phases are followed by 8 younger loads per wave.
#pragma once
#include "gemm_pingpong.h"

namespace tadm {
namespace {

// The reads of one phase (see read4_sync): fragments at lds0 and lds1 (+ OFF, row subtiles 2048
// bytes apart), at most VM tile loads left in flight (VM < 0: no wait), barrier, fragments in.
template <int OFF, int VM>
__device__ __forceinline__ void read_phase(uint32_t lds0, uint32_t lds1, bf16x8 (&f)[4][2]) {
  asm volatile(
      "ds_read_b128 %0, %8 offset:%10\n\t"
      "ds_read_b128 %1, %9 offset:%10\n\t"
      "ds_read_b128 %2, %8 offset:%11\n\t"
      "ds_read_b128 %3, %9 offset:%11\n\t"
      "ds_read_b128 %4, %8 offset:%12\n\t"
      "ds_read_b128 %5, %9 offset:%12\n\t"
      "ds_read_b128 %6, %8 offset:%13\n\t"
      "ds_read_b128 %7, %9 offset:%13\n\t"
      "s_waitcnt vmcnt(%14)\n\t"
      "s_barrier\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[1][0]), "=&v"(f[1][1]), "=&v"(f[2][0]), "=&v"(f[2][1]),
        "=&v"(f[3][0]), "=&v"(f[3][1])
      : "v"(lds0), "v"(lds1), "n"(OFF), "n"(OFF + 2048), "n"(OFF + 4096), "n"(OFF + 6144), "n"(VM < 0 ? 63 : VM)
      : "memory");
}
template <int OFF, int VM>
__device__ __forceinline__ void read_phase(uint32_t lds0, uint32_t lds1, bf16x8 (&f)[2][2]) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%6\n\t"
      "ds_read_b128 %1, %5 offset:%6\n\t"
      "ds_read_b128 %2, %4 offset:%7\n\t"
      "ds_read_b128 %3, %5 offset:%7\n\t"
      "s_waitcnt vmcnt(%8)\n\t"
      "s_barrier\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[1][0]), "=&v"(f[1][1])
      : "v"(lds0), "v"(lds1), "n"(OFF), "n"(OFF + 2048), "n"(VM < 0 ? 63 : VM)
      : "memory");
}

// Epi<KIND>::tile<TN, TM, GAP> takes the wave's accumulators with GAP rows between its two
// activation halves.
template <EpiKind KIND>
__global__ __launch_bounds__(256, 2) void gemm_tall_kernel(GemmProblem p, EpiParams ep) {
#ifdef __HIP_DEVICE_COMPILE__  // buffer resources are a device type: the host pass only needs the stub
  using E = Epi<KIND, bf16>;
  constexpr int BM = 256, BN = 128, TM = 8, TN = 4;
  constexpr int AH = 128 * 128, WH = 64 * 128;  // bytes of an activation / weight half
  constexpr int WBASE = 3 * AH;
  __shared__ __attribute__((aligned(1024))) char smem[3 * AH + 4 * WH];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  if (p.M_dev) p.M = min(*p.M_dev, p.M);  // rows present this call; the grid was sized for p.M
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
  int tmi, tni;
  tile_of(p, blockIdx.x, tiles_m, tiles_n, tmi, tni);
  if (tmi >= tiles_m) return;  // padding of a banded grid, or no rows for this block
  const int m0 = __builtin_amdgcn_readfirstlane(tmi * BM), n0 = __builtin_amdgcn_readfirstlane(tni * BN);
  const int nk = p.K / 64;

  // a tile with at most 128 rows present leaves out the products and the epilogue of its
  // second activation half (its loads, all of the last row, keep the waits' counts)
  const bool whole = m0 + 128 < p.M;

  // tile loads.  Activation half h: rows 128 h + [0, 128), 64 of them for each wave row; weight
  // half h: rows 64 i + 32 h + [0, 32); in LDS the halves' rows are consecutive
  const int lrow = lane >> 3, lchunk = (lane & 7) ^ (lane >> 3);
  auto rsrc = [](const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, -1, 0x00027000);
  };
  const auto ra = rsrc(static_cast<const bf16*>(p.A1) + (size_t)m0 * p.lda1);
  const auto rw = rsrc(static_cast<const bf16*>(p.W) + (size_t)n0 * p.ldw);
  uint32_t offA[2][4], offW[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // 8-row group wave + 4 j of the half
      offA[h][j] = (uint32_t)(min(m0 + 128 * h + 8 * (wave + 4 * j) + lrow, p.M - 1) - m0) * (uint32_t)(2 * p.lda1) +
                   16 * lchunk;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      offW[h][j] = (uint32_t)(min(n0 + 64 * j + 32 * h + 8 * wave + lrow, p.N - 1) - n0) * (uint32_t)(2 * p.ldw) +
                   16 * lchunk;
  }
  auto issue_a = [&](int kt, int slot, int h) {  // half h of K tile kt into activation slot
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr)(smem + slot * AH + (wave + 4 * j) * 1024), 16, offA[h][j],
                                               kt * 128, 0, 0);
  };
  auto issue_w = [&](int kt, int h) {  // weight half h of K tile kt into its slot 2 (kt % 2) + h
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(smem + WBASE + (2 * (kt & 1) + h) * WH + (wave + 4 * j) * 1024),
                                               16, offW[h][j], kt * 128, 0, 0);
  };

  issue_w(0, 0);
  issue_a(0, 0, 0);
  issue_w(0, 1);
  issue_a(0, 1, 1);
  if (nk > 1) {
    issue_w(1, 0);
    issue_w(1, 1);
  }
  f32x4 acc[TN][TM];
  const bf16x8 zero = mfma_zero_operand();
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) mfma_first(acc[a][b], zero, zero);

  // fragment addresses of this lane in a half: activation rows 64 wm + 16 t + fr, weight rows
  // 32 wn + 16 t + fr
  const int fr = lane & 15, fq = lane >> 4, sw = lane & 7;
  const uint32_t lbase = (uint32_t)(uintptr_t)(lds_ptr)smem;
  const uint32_t la = lbase + (64 * wm + fr) * 128 + ((fq ^ sw) * 16);
  const uint32_t lw = lbase + WBASE + (32 * wn + fr) * 128 + ((fq ^ sw) * 16);

  bf16x8 fa[4][2], fb[2][2][2];  // activation half; two weight halves
  auto mul = [&](auto ha, auto hb, const bf16x8 (&w)[2][2]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) mfma_acc(acc[decltype(hb)::value * 2 + a][decltype(ha)::value * 4 + b], w[a][kk], fa[b][kk]);
    __builtin_amdgcn_s_setprio(0);
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  int slot = 0;  // activation slot of half 2 kt, (2 kt) % 3; its other half is in the next
  auto next = [](int s) { return s == 2 ? 0 : s + 1; };
  // K tile kt, kt % 2 == P; b0 is in fb[P].  The last K tiles issue less and wait for all
  // that is left; after the last one the b0 read is stale and unused.
  auto body = [&](auto par, int kt) {
    constexpr int P = decltype(par)::value;
    const int left = nk - 1 - kt, s1 = next(slot), s2 = next(s1);
    uint32_t a0 = la + slot * AH, a1 = la + s1 * AH;
    // a half s + 3 takes the slot of half s, two phases after its read: halves 2 kt + 2 and
    // 2 kt + 3 here
    if (left >= 1) issue_a(kt + 1, s2, 0);
    read_phase<0, -1>(a0, a0 ^ 64, fa);
    mul(H0{}, H0{}, fb[P]);
    if (left >= 2) {
      issue_w(kt + 2, 0);
      read_phase<P * 2 * WH + WH, 8>(lw, lw ^ 64, fb[P ^ 1]);
    } else if (left == 1) {
      read_phase<P * 2 * WH + WH, 6>(lw, lw ^ 64, fb[P ^ 1]);
    } else {
      read_phase<P * 2 * WH + WH, 0>(lw, lw ^ 64, fb[P ^ 1]);
    }
    mul(H0{}, H1{}, fb[P ^ 1]);
    if (left >= 1) issue_a(kt + 1, slot, 1);
    read_phase<0, -1>(a1, a1 ^ 64, fa);
    if (whole) mul(H1{}, H1{}, fb[P ^ 1]);
    if (left >= 2) {
      issue_w(kt + 2, 1);
      read_phase<(P ^ 1) * 2 * WH, 8>(lw, lw ^ 64, fb[P ^ 1]);
    } else {
      read_phase<(P ^ 1) * 2 * WH, 4>(lw, lw ^ 64, fb[P ^ 1]);
    }
    if (whole) mul(H1{}, H0{}, fb[P]);
    slot = s2;
  };
  // b0 and a0 of K tile 0: the younger loads are b1, a1 (and b0, b1 of K tile 1)
  if (nk > 1)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(10));
  else
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(6));
  block_barrier();
  read_phase<0, -1>(lw, lw ^ 64, fb[0]);
  // b1 of K tile 0, read in phase 1 without a wait of its own
  if (nk > 1)
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));
  else
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(4));
  for (int kt = 0;; kt += 2) {
    body(H0{}, kt);
    if (kt + 1 == nk) break;
    body(H1{}, kt + 1);
    if (kt + 2 == nk) break;
  }
  block_barrier();
  // the last products must be written before any accumulator is read back (see
  // gemm_bf16_kernel)
  asm volatile("s_nop 15\n s_nop 15\n s_nop 15" ::: "memory");
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) asm volatile("" : "+a"(acc[a][b]));
  // row subtiles 0-3 are rows 64 wm + [0, 64) of the tile, 4-7 the same of its second half
  E::template tile<TN, TM, 64>(ep, p, acc, m0 + wm * 64, n0 + wn * 64, lane);
#endif
}

// One activation operand.  The grid is walked in bands, also where the row count is known to the
// host: the head's is not (tile_of).
template <EpiKind K>
hipError_t launch_tall(const GemmProblem& p0, const EpiParams& e, hipStream_t s) {
  if (p0.K1 < p0.K) return hipErrorInvalidValue;
  GemmProblem p = p0;
  const int tiles_m = (p.M + 255) / 256, tiles_n = (p.N + 127) / 128;
  p.band = xcd_band(tiles_m, 256, 128, 64);
  const int blocks = (tiles_m * tiles_n + 7) / 8 * 8;
  launch_timed(gemm_tall_kernel<K>, dim3(blocks), dim3(256), 0, s, p, e);
  return hipGetLastError();
}

}  // namespace
}  // namespace tadm
