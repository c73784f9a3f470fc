// bf16 GEMM main loop for 256 x 256 tiles, C = A W^T: two groups of four waves take turns.
//
// 8 wave64s (2 x 4, 128 x 64 outputs each), K tiles of 64 in a two-buffer LDS ring.  On
// every SIMD one wave of each group is resident, the second group half a phase behind the
// first: while one group multiplies, the other reads its next fragments from LDS and
// issues tile loads, and a block barrier hands over.  A K tile is four phases, one per
// 64 x 32 quadrant of the wave's tile (16 MFMAs): quadrants (a0, b0), (a0, b1), (a1, b1),
// (a1, b0) of the activation halves a and the weight halves b, reading a0 | b1 | a1 | the
// next K tile's b0.
//
// Tile loads (global_load_lds_dwordx4) move in units of one operand half (128 rows, 16 KB
// per block, two loads per wave), one unit per phase, each into the slot of the unit of
// the previous K tile pair that every wave has read.  A unit is issued six phases before
// it is read, and a phase only waits for the unit that the next phase reads (at most ten
// younger loads stay in flight across the barriers): 64 to 96 KB per block are in flight
// at any time, where a loop that drains its loads at every K tile has 64 KB just after the
// barrier and none before it.
//
// A block (one per CU) walks several tiles; the next tile's first loads are issued before
// the epilogue of the present one, whose stores and arithmetic they hide behind.
//
// Measured (normal operands, plain bf16 store, against the loop of gemm_bf16_kernel on the
// same tiles, which drains at each K tile and starts a block per tile): 8 192^3 1 360 -> 1 495
// TFLOP/s, 32 768 x 8 192 x 2 048 1 161 -> 1 350 (of it 8 % from the 16-byte stores of
// store_rows, which both have), 1 024 x 73 728 x 4 608 1 115 -> 1 300.  What is left at K =
// 2 048 is the epilogue: without its stores 740 of 815 us.
//
// The order of a unit's refill after its last read.  Reads of phase p are issued in the
// group's slot before a barrier and waited for (lgkmcnt) right after that barrier, so
// the second group's reads of phase p are done when the barrier two slots later is
// passed; the refill is issued by either group in phase p + 2 or later, past it.
#pragma once
#include "gemm_kernel.h"

namespace tadm {
namespace {

// One phase's reads of fragments (row subtiles 2048 bytes apart, both 32-deep halves at
// lds0 and lds1), then: at most ten tile loads left in flight (near the end of K, where
// fewer are issued after the one awaited: V1 with one K tile left after this one, V0 with
// none), the barrier that hands over to the other group, and the wait for the fragments.
// One block, so that no instruction can be placed between a read and its wait.
#define TADM_PP_SYNC                \
  "s_cmp_gt_i32 %[left], 1\n\t"     \
  "s_cbranch_scc1 1f\n\t"           \
  "s_cmp_eq_i32 %[left], 1\n\t"     \
  "s_cbranch_scc1 0f\n\t"           \
  "s_waitcnt vmcnt(%[v0])\n\t"      \
  "0:\n\t"                          \
  "s_waitcnt vmcnt(%[v1])\n\t"      \
  "1:\n\t"                          \
  "s_waitcnt vmcnt(10)\n\t"         \
  "s_barrier\n\t"                   \
  "s_waitcnt lgkmcnt(0)"
template <int OFF, int V1, int V0>
__device__ __forceinline__ void read4_sync(uint32_t lds0, uint32_t lds1, int left, bf16x8 (&f)[4][2]) {
  static_assert(V0 <= V1 && V1 <= 10, "the waits follow one another");
  asm volatile(
      "ds_read_b128 %0, %8 offset:%[o0]\n\t"
      "ds_read_b128 %1, %9 offset:%[o0]\n\t"
      "ds_read_b128 %2, %8 offset:%[o1]\n\t"
      "ds_read_b128 %3, %9 offset:%[o1]\n\t"
      "ds_read_b128 %4, %8 offset:%[o2]\n\t"
      "ds_read_b128 %5, %9 offset:%[o2]\n\t"
      "ds_read_b128 %6, %8 offset:%[o3]\n\t"
      "ds_read_b128 %7, %9 offset:%[o3]\n\t" TADM_PP_SYNC
      : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[1][0]), "=&v"(f[1][1]), "=&v"(f[2][0]), "=&v"(f[2][1]),
        "=&v"(f[3][0]), "=&v"(f[3][1])
      : "v"(lds0), "v"(lds1), [left] "s"(left), [o0] "n"(OFF), [o1] "n"(OFF + 2048), [o2] "n"(OFF + 4096),
        [o3] "n"(OFF + 6144), [v1] "n"(V1), [v0] "n"(V0)
      : "memory", "scc");
}
template <int OFF, int V1, int V0>
__device__ __forceinline__ void read2_sync(uint32_t lds0, uint32_t lds1, int left, bf16x8 (&f)[2][2]) {
  static_assert(V0 <= V1 && V1 <= 10, "the waits follow one another");
  asm volatile(
      "ds_read_b128 %0, %4 offset:%[o0]\n\t"
      "ds_read_b128 %1, %5 offset:%[o0]\n\t"
      "ds_read_b128 %2, %4 offset:%[o1]\n\t"
      "ds_read_b128 %3, %5 offset:%[o1]\n\t" TADM_PP_SYNC
      : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[1][0]), "=&v"(f[1][1])
      : "v"(lds0), "v"(lds1), [left] "s"(left), [o0] "n"(OFF), [o1] "n"(OFF + 2048), [v1] "n"(V1), [v0] "n"(V0)
      : "memory", "scc");
}
#undef TADM_PP_SYNC
__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Whether the ping-pong kernel takes the product: at least two K tiles per slice, and one
// row stride for both activation operands (their rows share one offset per lane).
inline bool pingpong_ok(const GemmProblem& p) {
  return p.K / 64 / p.ksplit >= 2 && (p.K1 >= p.K || p.lda1 == p.lda2);
}

// Blocks of a launch: one per CU, each walking tiles b, b + kPpBlocks, ... of the grid.
constexpr int kPpBlocks = 256;

template <EpiKind KIND>
__global__ __launch_bounds__(512, 1) void gemm_pp_kernel(GemmProblem p, EpiParams ep, int grid_tiles) {
#ifdef __HIP_DEVICE_COMPILE__  // buffer resources are a device type: the host pass only needs the stub
  using E = Epi<KIND, bf16>;
  constexpr int BM = 256, BN = 256, WGM = 2, WGN = 4, TM = 8, TN = 4;
  constexpr int BUF = 256 * 128;       // one operand's K tile: 256 rows of 64 bf16
  constexpr int WBASE = 2 * BUF;       // activation buffers, then weight buffers
  __shared__ __attribute__((aligned(1024))) char smem[4 * BUF];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WGM, wn = wave / WGM;
  if (p.M_dev) p.M = min(*p.M_dev, p.M);  // rows present this call; the grid was sized for p.M
  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;

  // the tile at position t of this launch's walk (K slices one after the other): its
  // corner and its K tiles [kt_base, kt_base + nk)
  struct Tile {
    int m0, n0, slice, kt_base, nk;
  };
  const int NKT = p.K / 64, total = grid_tiles * p.ksplit;
  auto find = [&](int& t, Tile& o) {  // the first position >= t with rows to compute
    for (; t < total; t += gridDim.x) {
      int tm, tn;
      const int s = t / grid_tiles;
      tile_of(p, t - s * grid_tiles, tiles_m, tiles_n, tm, tn);
      if (tm >= tiles_m) continue;  // padding of a banded grid, or no rows here
      o.m0 = __builtin_amdgcn_readfirstlane(tm * BM);
      o.n0 = __builtin_amdgcn_readfirstlane(tn * BN);
      o.slice = s;
      o.kt_base = (int)((long)s * NKT / p.ksplit);
      o.nk = (int)((long)(s + 1) * NKT / p.ksplit) - o.kt_base;  // >= 2 (pingpong_ok)
      return true;
    }
    return false;
  };

  // tile loads: a buffer resource at the tile's first row of each operand, per lane the
  // byte offset of its row and swizzled chunk.  Unit h of A: rows 128 i + 64 h + [0, 64),
  // i = 0, 1; of W: rows 64 i + 32 h + [0, 32), i = 0..3; as 8-row groups, two per wave.
  const int lrow = lane >> 3, lchunk = (lane & 7) ^ (lane >> 3);
  auto rsrc = [](const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, -1, 0x00027000);
  };
  const bf16* A1 = static_cast<const bf16*>(p.A1);
  const bf16* A2 = p.A2 ? static_cast<const bf16*>(p.A2) - p.K1 : A1;
  const int lda2 = p.A2 ? p.lda2 : p.lda1;
  __amdgpu_buffer_rsrc_t ra1, ra2, rw;
  uint32_t offA[2][2], offW[2][2];
  int kt_base, nk;
  auto aim = [&](const Tile& o) {  // the loads at a tile
    ra1 = rsrc(A1 + (size_t)o.m0 * p.lda1);
    ra2 = rsrc(A2 + (size_t)o.m0 * lda2);
    rw = rsrc(static_cast<const bf16*>(p.W) + (size_t)o.n0 * p.ldw);
    kt_base = o.kt_base;
    nk = o.nk;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int row_a = min(o.m0 + 128 * j + 64 * h + 8 * wave + lrow, p.M - 1) - o.m0;
        const int row_w = min(o.n0 + 64 * ((wave >> 2) + 2 * j) + 32 * h + 8 * (wave & 3) + lrow, p.N - 1) - o.n0;
        offA[h][j] = (uint32_t)row_a * (uint32_t)(2 * p.lda1) + 16 * lchunk;
        offW[h][j] = (uint32_t)row_w * (uint32_t)(2 * p.ldw) + 16 * lchunk;
      }
  };
  auto issue_a = [&](int kt, int buf, int h) {
    const int k0 = (kt_base + kt) * 64;
    const auto r = k0 >= p.K1 ? ra2 : ra1;
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)(smem + buf * BUF + (128 * j + 64 * h + 8 * wave) * 128), 16,
                                               offA[h][j], k0 * 2, 0, 0);
  };
  auto issue_w = [&](int kt, int buf, int h) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rw, (lds_ptr)(smem + WBASE + buf * BUF + (64 * ((wave >> 2) + 2 * j) + 32 * h + 8 * (wave & 3)) * 128), 16,
          offW[h][j], (kt_base + kt) * 128, 0, 0);
  };
  auto issue_first = [&] {  // K tile 0
    issue_w(0, 0, 0);
    issue_a(0, 0, 0);
    issue_w(0, 0, 1);
    issue_a(0, 0, 1);
  };
  auto issue_second = [&] {  // K tile 1 but for its last unit, which the first phase issues
    issue_w(1, 1, 0);
    issue_a(1, 1, 0);
    issue_w(1, 1, 1);
  };

  f32x4 acc[TN][TM];

  // this lane's fragment addresses in LDS, both 32-deep halves
  const int fr = lane & 15, fq = lane >> 4, sw = lane & 7;
  const uint32_t lbase = (uint32_t)(uintptr_t)(lds_ptr)smem;
  const uint32_t la0 = lbase + (wm * 128 + fr) * 128 + ((fq ^ sw) * 16), la1 = la0 ^ 64;
  const uint32_t lw0 = lbase + WBASE + (wn * 64 + fr) * 128 + ((fq ^ sw) * 16), lw1 = lw0 ^ 64;

  bf16x8 fa[4][2], fb[2][2][2];  // activation half; two weight halves
  // the 16 products of activation half ha and weight half hb
  auto mul = [&](auto ha, auto hb, const bf16x8 (&w)[2][2]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) mfma_acc(acc[decltype(hb)::value * 2 + a][decltype(ha)::value * 4 + b], w[a][kk], fa[b][kk]);
    __builtin_amdgcn_s_setprio(0);
    block_barrier();
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
  // K tile kt in buffer P (kt % 2); b0 is in fb[P].  With no K tile after this one, the
  // last phase reads the b0 of a K tile that does not follow: stale, unused.
  auto body = [&](auto par, int kt) {
    constexpr int P = decltype(par)::value;
    const int left = nk - 1 - kt;
    if (left >= 1) issue_a(kt + 1, P ^ 1, 1);
    read4_sync<P * BUF, 10, 2>(la0, la1, left, fa);
    mul(H0{}, H0{}, fb[P]);
    if (left >= 2) issue_w(kt + 2, P, 0);
    read2_sync<P * BUF + 4096, 8, 0>(lw0, lw1, left, fb[P ^ 1]);
    mul(H0{}, H1{}, fb[P ^ 1]);
    if (left >= 2) issue_a(kt + 2, P, 0);
    read4_sync<P * BUF + 8192, 6, 0>(la0, la1, left, fa);
    mul(H1{}, H1{}, fb[P ^ 1]);
    if (left >= 2) issue_w(kt + 2, P, 1);
    read2_sync<(P ^ 1) * BUF, 4, 0>(lw0, lw1, left, fb[P ^ 1]);
    mul(H1{}, H0{}, fb[P]);
  };

  // an epilogue that stages through LDS does so in the buffers of odd K tiles, so that
  // the next tile's first K tile can land meanwhile
  constexpr bool kStaged = TileLdsEpi<E>::value;
  int t = blockIdx.x;
  Tile cur, nxt;
  bool more = find(t, cur);
  if (more) {
    aim(cur);
    issue_first();
    issue_second();
  }
  while (more) {
    // zero accumulators, written by the matrix unit: they are accumulator registers from
    // their first value on
    const bf16x8 zero = mfma_zero_operand();
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
      for (int b = 0; b < TM; ++b) mfma_first(acc[a][b], zero, zero);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(10));  // b0 and a0 of K tile 0
    block_barrier();
    // b0 of K tile 0 (this wait-and-barrier is the first group's first hand-over, which
    // the second group passes one barrier later)
    read2_sync<0, 10, 10>(lw0, lw1, 2, fb[0]);
    if (wave >= 4) block_barrier();
    for (int kt = 0;; kt += 2) {
      body(H0{}, kt);
      if (kt + 1 == nk) break;
      body(H1{}, kt + 1);
      if (kt + 2 == nk) break;
    }
    if (wave < 4) block_barrier();  // here every wave has read its last fragment
    // the next tile's first loads fly during this one's epilogue
    t += gridDim.x;
    more = find(t, nxt);
    if (more) {
      aim(nxt);
      issue_first();
      if (!kStaged) issue_second();
    }
    // the last products must be written before any accumulator is read back (see
    // gemm_bf16_kernel)
    asm volatile("s_nop 15\n s_nop 15\n s_nop 15" ::: "memory");
#pragma unroll
    for (int a = 0; a < TN; ++a)
#pragma unroll
      for (int b = 0; b < TM; ++b) asm volatile("" : "+a"(acc[a][b]));
    // the epilogue's per-lane addresses are formed here, not kept in registers over the
    // main loop
    int elane = lane;
    asm volatile("" : "+v"(elane));
    if constexpr (kStaged) {
      // 8 KB per wave, in two passes of 64 rows: waves 0-3 in the activations' odd
      // buffer, 4-7 in the weights'
      char* stage = smem + BUF + (wave >> 2) * WBASE + (wave & 3) * 8192;
      const int mb = cur.m0 + wm * 128, nb = cur.n0 + wn * 64;
      E::template tile_lds<TN, TM, 0, TM / 2>(ep, p, acc, mb, nb, elane, stage);
      __syncthreads();  // the staged rows are read before they are overwritten
      E::template tile_lds<TN, TM, TM / 2, TM / 2>(ep, p, acc, mb + 64, nb, elane, stage);
      __syncthreads();
      if (more) issue_second();
    } else {
      float4 pre[1][1][1];
      finish_tile<BM, BN, 4 * BUF, WGM, WGN, KIND, false>(p, ep, acc, pre, cur.m0, cur.n0, cur.slice, wave, elane, smem);
    }
    cur = nxt;
  }
#endif
}

template <EpiKind K>
hipError_t launch_pp(const GemmProblem& p0, const EpiParams& e, hipStream_t s) {
  GemmProblem p = p0;
  const int tiles_m = (p.M + 255) / 256, tiles_n = (p.N + 255) / 256;
  if (!p.M_dev) xcd_regions(tiles_m, tiles_n, 256, 256, p.rm, p.rn);
  xcd_patch(p.rm, p.rn, 256, 256, 32, p.gm, p.gn);
  p.band = p.rm > 0 ? 0 : xcd_band(tiles_m, 256, 256, 32);
  // a multiple of 8 either way, so that position b + kPpBlocks stays on b's XCD
  const int tiles = p.band > 0 ? (tiles_m * tiles_n + 7) / 8 * 8 : tiles_m * tiles_n;
  const long total = (long)tiles * p.ksplit;
  launch_timed(gemm_pp_kernel<K>, dim3((unsigned)(total < kPpBlocks ? total : kPpBlocks)), dim3(512), 0, s, p, e, tiles);
  return hipGetLastError();
}

}  // namespace
}  // namespace tadm
