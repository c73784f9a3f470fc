// Dense contractions of the TADM step: C = A W^T with fused epilogues.
//
// bf16 operands run on the MFMA kernel template of gemm_kernel.h with the epilogues
// below; the tile shape is picked per call from the number of blocks it yields.
// float32 operands (small fp32 models) run on the float32 matrix instructions with the
// same epilogues.
#include <algorithm>

#include "gemm_kernel.h"
#include "gemm_pingpong.h"
#include "gemm_ring.h"

namespace tadm {
namespace {

// ------------------------------------------------------------------ epilogues

template <class T>
struct Epi<EPI_STORE, T> {
  static constexpr bool kGlu = false;
  static constexpr bool kRow = true;
  __device__ static T* out_row(const EpiParams& e, int m) { return static_cast<T*>(e.out) + (size_t)m * e.ldo; }
  __device__ static f32x4 row_out(f32x4 v) { return v; }
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    store4(static_cast<T*>(e.out) + (size_t)m * e.ldo + n, v[0], v[1], v[2], v[3]);
  }
};
template <class T>
struct Epi<EPI_STORE_F32, T> {
  static constexpr bool kGlu = false;
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    store4(static_cast<float*>(e.out) + (size_t)m * e.ldo + n, v[0], v[1], v[2], v[3]);
  }
};
template <class T>
struct Epi<EPI_SCALE_F32, T> {
  static constexpr bool kGlu = false;
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const float r = e.row1[m];
    store4(static_cast<float*>(e.out) + (size_t)m * e.ldo + n, r * v[0], r * v[1], r * v[2], r * v[3]);
  }
};
template <class T>
struct Epi<EPI_RESID, T> {
  static constexpr bool kGlu = false;
  static constexpr int kPre = 1;
  __device__ static void pre(const EpiParams& e, int m, int n, float4* o) {
    o[0] = *reinterpret_cast<const float4*>(e.resid + (size_t)m * e.ldr + n);
  }
  __device__ static void apply_pre(const EpiParams& e, int m, int n, f32x4 v, const float4* o) {
    float4 x = o[0];
    x.x += v[0]; x.y += v[1]; x.z += v[2]; x.w += v[3];
    *reinterpret_cast<float4*>(e.resid + (size_t)m * e.ldr + n) = x;
  }
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    float4 o;
    pre(e, m, n, &o);
    apply_pre(e, m, n, v, &o);
  }
};
template <class T>
struct Epi<EPI_GELU, T> {
  static constexpr bool kGlu = false;
  static constexpr bool kRow = true;
  __device__ static T* out_row(const EpiParams& e, int m) { return static_cast<T*>(e.out) + (size_t)m * e.ldo; }
  __device__ static f32x4 row_out(f32x4 v) { return f32x4{gelu_act<T>(v[0]), gelu_act<T>(v[1]), gelu_act<T>(v[2]), gelu_act<T>(v[3])}; }
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    store4(static_cast<T*>(e.out) + (size_t)m * e.ldo + n, gelu_act<T>(v[0]), gelu_act<T>(v[1]),
           gelu_act<T>(v[2]), gelu_act<T>(v[3]));
  }
};
template <class T>
struct Epi<EPI_FUSION1, T> {
  static constexpr bool kGlu = false;
  static constexpr bool kTile = true;  // bf16 kernels; split is a multiple of every strip's width
  template <int TN, int TM>
  __device__ static void tile(const EpiParams& e, const GemmProblem& p, const f32x4 (&acc)[TN][TM], int mb, int nb,
                              int lane) {
    const int fr = lane & 15, fq = lane >> 4;
#pragma unroll
    for (int a = 0; a < TN; a += 2)
#pragma unroll
      for (int b = 0; b < TM; ++b) {
        const int m = mb + 16 * b + fr, n = nb + 16 * a;
        if (nb < e.split) {
          bf16x4 h[2];
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const float4 c = *reinterpret_cast<const float4*>(e.bias + min(n + 16 * i, p.N - 16) + 4 * fq);
            const f32x4 v = acc[a + i][b];
            h[i] = bf16x4{(bf16)gelu_act<T>(v[0] + c.x), (bf16)gelu_act<T>(v[1] + c.y), (bf16)gelu_act<T>(v[2] + c.z),
                          (bf16)gelu_act<T>(v[3] + c.w)};
          }
          store_rows(reinterpret_cast<bf16*>(e.out) + (size_t)m * e.ldo, n, e.split, m < p.M, h[0], h[1], fq);
        } else {
#pragma unroll
          for (int i = 0; i < 2; ++i)
            if (m < p.M && n + 16 * i + 4 * fq < p.N) apply(e, m, n + 16 * i + 4 * fq, acc[a + i][b]);
        }
      }
  }
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const float4 b = *reinterpret_cast<const float4*>(e.bias + n);
    if (n < e.split) {
      store4(static_cast<T*>(e.out) + (size_t)m * e.ldo + n, gelu_act<T>(v[0] + b.x),
             gelu_act<T>(v[1] + b.y), gelu_act<T>(v[2] + b.z), gelu_act<T>(v[3] + b.w));
    } else {
      store4(e.out2 + (size_t)m * e.ldo2 + (n - e.split), sigmoid_act<T>(v[0] + b.x),
             sigmoid_act<T>(v[1] + b.y), sigmoid_act<T>(v[2] + b.z), sigmoid_act<T>(v[3] + b.w));
    }
  }
};
template <class T>
struct Epi<EPI_FUSION2, T> {
  static constexpr bool kGlu = false;
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const float4 b = *reinterpret_cast<const float4*>(e.bias + n);
    const float4 h = *reinterpret_cast<const float4*>(e.aux + (size_t)m * e.ld_aux + n);
    const float4 g = *reinterpret_cast<const float4*>(e.gate + (size_t)m * e.ldg + n);
    store4(e.resid + (size_t)m * e.ldr + n, h.x + g.x * (v[0] + b.x), h.y + g.y * (v[1] + b.y),
           h.z + g.z * (v[2] + b.z), h.w + g.w * (v[3] + b.w));
  }
};
template <class T>
struct Epi<EPI_SILU, T> {
  static constexpr bool kGlu = false;
  static constexpr bool kRow = true;
  __device__ static T* out_row(const EpiParams& e, int m) { return static_cast<T*>(e.out) + (size_t)m * e.ldo; }
  __device__ static f32x4 row_out(f32x4 v) { return f32x4{silu_act<T>(v[0]), silu_act<T>(v[1]), silu_act<T>(v[2]), silu_act<T>(v[3])}; }
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    store4(static_cast<T*>(e.out) + (size_t)m * e.ldo + n, silu_act<T>(v[0]), silu_act<T>(v[1]),
           silu_act<T>(v[2]), silu_act<T>(v[3]));
  }
};
template <class T>
struct Epi<EPI_ADD_F32, T> {
  static constexpr bool kGlu = false;
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const float4 a = *reinterpret_cast<const float4*>(e.aux + (size_t)m * e.ld_aux + n);
    store4(static_cast<float*>(e.out) + (size_t)m * e.ldo + n, a.x + v[0], a.y + v[1], a.z + v[2],
           a.w + v[3]);
  }
};
template <class T>
struct Epi<EPI_ADD_BOTH, T> {
  static constexpr bool kGlu = false;
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const float4 a = *reinterpret_cast<const float4*>(e.aux + (size_t)m * e.ld_aux + n);
    const float r0 = a.x + v[0], r1 = a.y + v[1], r2 = a.z + v[2], r3 = a.w + v[3];
    store4(static_cast<float*>(e.out) + (size_t)m * e.ldo + n, r0, r1, r2, r3);
    store4(static_cast<T*>(e.out_t) + (size_t)m * e.ld_out_t + n, r0, r1, r2, r3);
  }
};
template <class T>
struct Epi<EPI_ADD_SUB, T> {
  static constexpr bool kGlu = false;
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const float4 a = *reinterpret_cast<const float4*>(e.aux + (size_t)m * e.ld_aux + n);
    const float4 b = *reinterpret_cast<const float4*>(e.aux2 + (size_t)m * e.ld_aux2 + n);
    store4(static_cast<T*>(e.out_t) + (size_t)m * e.ld_out_t + n, (a.x + v[0]) - b.x, (a.y + v[1]) - b.y,
           (a.z + v[2]) - b.z, (a.w + v[3]) - b.w);
  }
};
template <class T>
struct Epi<EPI_PAIRED, T> {
  static constexpr bool kGlu = false;
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const float4 h = *reinterpret_cast<const float4*>(e.aux + (size_t)m * e.ld_aux + n);
    const float f = e.row1[m] * e.row2[m];
    store4(static_cast<float*>(e.out) + (size_t)m * e.ldo + n, h.x + f * v[0], h.y + f * v[1],
           h.z + f * v[2], h.w + f * v[3]);
  }
};
template <class T>
struct Epi<EPI_QKV_ROPE, T> {
  static constexpr bool kGlu = false;
  static constexpr bool kTileLds = true;  // bf16 kernel: staged through LDS (tile_lds)
  __device__ static int fdiv(int n, uint32_t mul, int shift) {
    return (int)((__umulhi((uint32_t)n, mul) + (uint32_t)n) >> shift);
  }
  // one 4-feature fragment, stored directly (float32 kernel, and head widths whose
  // slots a wave strip does not tile)
  __device__ static void apply(const EpiParams& e, int m, int n, f32x4 v) {
    const int b = fdiv(m, e.l_mul, e.l_shift), l = m - b * e.L;
    const int slot = fdiv(n, e.dh_mul, e.dh_shift), c = n - slot * e.dh;  // c is a multiple of 4
    if (slot < e.H + e.Hkv) {
      // (v0, v1) = pair j, (v2, v3) = pair j + 1 with j = c / 2
      const int j = c >> 1, half = e.dh >> 1;
      // (cos j, sin j, cos j+1, sin j+1): j is even, so the load is 16-byte aligned
      const float4 r = *reinterpret_cast<const float4*>(e.rope + ((size_t)(e.pos0 + l) * half + j) * 2);
      const float a0 = v[0] * r.x - v[1] * r.y, b0 = v[1] * r.x + v[0] * r.y;
      const float a1 = v[2] * r.z - v[3] * r.w, b1 = v[3] * r.z + v[2] * r.w;
      T* row = slot < e.H
                   ? static_cast<T*>(e.q) + (((size_t)b * e.H + slot) * e.L + l) * e.dh
                   : static_cast<T*>(e.k) + (((size_t)b * e.Hkv + (slot - e.H)) * e.kv_cap + e.kv_off + l) * e.dh;
      store2(row + j, a0, a1);  // j is even: 4-byte (bf16) or 8-byte (float) aligned pairs
      store2(row + j + half, b0, b1);
    } else {
      T* col = static_cast<T*>(e.vt) + (((size_t)b * e.Hkv + (slot - e.H - e.Hkv)) * e.dh + c) * e.kv_cap +
               e.kv_off + l;
#pragma unroll
      for (int t = 0; t < 4; ++t) col[(size_t)t * e.kv_cap] = from_f32<T>(v[t]);
    }
  }

  // Byte offset of element (r, col) of a [rows][C] bf16 staging tile: the 16-byte chunks
  // of row r rotated by r + r / 8, so that the fragment writes (16 rows of one chunk)
  // and the chunk reads (whole rows) meet distinct LDS banks.
  template <int C>
  __device__ static int staged(int r, int col) {
    constexpr int NCH = C / 8;
    return r * (C * 2) + (((col >> 3) + r + (r >> 3)) % NCH) * 16 + (col & 7) * 2;
  }

  // The wave's WTM tokens x WTN features lie in one head slot (dh % WTN == 0).  Q and K
  // strips are rotated in registers and staged token-major, with the pair halves j and
  // j + dh/2 already apart, so that each token's run of the head row leaves as 16-byte
  // stores; V strips are staged feature-major and leave as 16-byte runs of 8 tokens of a
  // V^T row.  Two phases with a block barrier between them (every wave of the block runs
  // this function; the barrier orders each wave's LDS writes before its reads).
  // B0, NB: the row subtiles to store, [B0, B0 + NB) of the tile (mb is the first one's row).
  template <int TN, int TM, int B0 = 0, int NB = TM>
  __device__ static void tile_lds(const EpiParams& e, const GemmProblem& p, const f32x4 (&acc)[TN][TM], int mb,
                                  int nb, int lane, char* lds) {
    constexpr int WTN = TN * 16, WTM = NB * 16;
    const int fr = lane & 15, fq = lane >> 4;
    // the staging maps rows and chunks to lanes by powers of two: the 48-column strips of 64 x
    // 96 tiles are stored directly
    constexpr bool kStaged = (WTN & (WTN - 1)) == 0;
    if (!kStaged || e.dh % WTN != 0) {  // the same for every wave of the grid
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int m = mb + 16 * b + fr, n = nb + 16 * a + 4 * fq;
          if (m < p.M && n < p.N) apply(e, m, n, acc[a][B0 + b]);
        }
      return;
    }
    const bool live = nb < p.N;
    const int slot = fdiv(nb, e.dh_mul, e.dh_shift), c0 = nb - slot * e.dh;  // strip offset in the head
    const int half = e.dh >> 1, jbase = c0 >> 1;
    const bool is_v = slot >= e.H + e.Hkv;
    // phase 1: stage
    if (live && !is_v) {
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int r = 16 * b + fr;
        const int m = min(mb + r, p.M - 1);  // rows past M are staged but never stored
        const int bb = fdiv(m, e.l_mul, e.l_shift), l = m - bb * e.L;
        const float* rp = e.rope + ((size_t)(e.pos0 + l) * half + jbase) * 2;
#pragma unroll
        for (int a = 0; a < TN; ++a) {
          const int pl = 8 * a + 2 * fq;  // local pair index of (v0, v1); (v2, v3) is pl + 1
          const f32x4 v = acc[a][B0 + b];
          const float4 rr = *reinterpret_cast<const float4*>(rp + 2 * pl);  // cos, sin of pl and pl + 1
          const float a0 = v[0] * rr.x - v[1] * rr.y, b0 = v[1] * rr.x + v[0] * rr.y;
          const float a1 = v[2] * rr.z - v[3] * rr.w, b1 = v[3] * rr.z + v[2] * rr.w;
          store2(reinterpret_cast<bf16*>(lds + staged<WTN>(r, pl)), a0, a1);
          store2(reinterpret_cast<bf16*>(lds + staged<WTN>(r, WTN / 2 + pl)), b0, b1);
        }
      }
    } else if (live) {
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            *reinterpret_cast<bf16*>(lds + staged<WTM>(16 * a + 4 * fq + jj, 16 * b + fr)) = (bf16)acc[a][B0 + b][jj];
    }
    __syncthreads();
    // phase 2: 16-byte chunks to the attention layouts
    if (live && !is_v) {
      constexpr int NC = WTN / 8;
      T* base = slot < e.H ? static_cast<T*>(e.q) : static_cast<T*>(e.k);
#pragma unroll
      for (int idx = lane; idx < WTM * NC; idx += 64) {
        const int r = idx / NC, c = idx % NC, m = mb + r;
        if (m >= p.M) continue;
        const int bb = fdiv(m, e.l_mul, e.l_shift), l = m - bb * e.L;
        const size_t row = slot < e.H ? ((size_t)bb * e.H + slot) * e.L + l
                                      : ((size_t)bb * e.Hkv + (slot - e.H)) * e.kv_cap + e.kv_off + l;
        const int col = c < NC / 2 ? jbase + 8 * c : jbase + half + 8 * (c - NC / 2);
        *reinterpret_cast<bf16x8*>(base + row * e.dh + col) = *reinterpret_cast<const bf16x8*>(lds + staged<WTN>(r, 8 * c));
      }
    } else if (live) {
      constexpr int NC = WTM / 8;
      const int hv = slot - e.H - e.Hkv;
#pragma unroll
      for (int idx = lane; idx < WTN * NC; idx += 64) {
        const int f = idx / NC, c = idx % NC, m0 = mb + 8 * c;
        if (m0 >= p.M) continue;
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(lds + staged<WTM>(f, 8 * c));
        T* vrow = static_cast<T*>(e.vt) + (((size_t)0 * e.Hkv + hv) * e.dh + c0 + f) * e.kv_cap + e.kv_off;
        const int b0 = fdiv(m0, e.l_mul, e.l_shift), l0 = m0 - b0 * e.L;
        const size_t bstride = (size_t)e.Hkv * e.dh * e.kv_cap;  // one batch row of V^T
        if (m0 + 8 <= p.M && l0 + 8 <= e.L && ((e.kv_off + l0) & 7) == 0) {
          *reinterpret_cast<bf16x8*>(vrow + b0 * bstride + l0) = v;
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int m = m0 + u;
            if (m >= p.M) break;
            const int bb = fdiv(m, e.l_mul, e.l_shift), l = m - bb * e.L;
            vrow[bb * bstride + l] = v[u];
          }
        }
      }
    }
  }
};
template <class T>
struct Epi<EPI_GLU_SILU, T> {
  static constexpr bool kGlu = true;
  static constexpr bool kRow = true;
  __device__ static T* out_row(const EpiParams& e, int m) { return static_cast<T*>(e.out) + (size_t)m * e.ldo; }
  __device__ static f32x4 row_out(f32x4 g, f32x4 u) {
    return f32x4{silu_act<T>(g[0]) * u[0], silu_act<T>(g[1]) * u[1], silu_act<T>(g[2]) * u[2], silu_act<T>(g[3]) * u[3]};
  }
  __device__ static void glu(const EpiParams& e, int m, int f, f32x4 g, f32x4 u) {
    store4(static_cast<T*>(e.out) + (size_t)m * e.ldo + f, silu_act<T>(g[0]) * u[0],
           silu_act<T>(g[1]) * u[1], silu_act<T>(g[2]) * u[2], silu_act<T>(g[3]) * u[3]);
  }
};
template <class T>
struct Epi<EPI_GLU_GELU, T> {
  static constexpr bool kGlu = true;
  static constexpr bool kRow = true;
  __device__ static T* out_row(const EpiParams& e, int m) { return static_cast<T*>(e.out) + (size_t)m * e.ldo; }
  __device__ static f32x4 row_out(f32x4 g, f32x4 u) {
    return f32x4{gelu_act<T>(g[0]) * u[0], gelu_act<T>(g[1]) * u[1], gelu_act<T>(g[2]) * u[2], gelu_act<T>(g[3]) * u[3]};
  }
  __device__ static void glu(const EpiParams& e, int m, int f, f32x4 g, f32x4 u) {
    store4(static_cast<T*>(e.out) + (size_t)m * e.ldo + f, gelu_act<T>(g[0]) * u[0],
           gelu_act<T>(g[1]) * u[1], gelu_act<T>(g[2]) * u[2], gelu_act<T>(g[3]) * u[3]);
  }
};

// ------------------------------------------------------------ fp32 kernels
// float32 products on v_mfma_f32_16x16x4_f32 (a float32 multiply-add chain).  The order of
// every sum depends on K alone, so that a row has the same bits whatever the number of rows
// beside it: K in chunks of 16 (f32_chunk), the chunks in four quarters (f32_quarter), each
// quarter one chain from zero, the four sums added in order.  Two kernels share it: a quarter
// per wave for products too small to fill the chip otherwise, else a quarter after the other.
// The line lies where both take the same time, at 2 048 tiles of 16 x 16 (us, small against
// large, K = 64 / 256 / 512: 1 024 tiles 3.6 : 5.6, 6.5 : 10.5, 10.8 : 18.1; 2 048 tiles 4.7 : 5.8,
// 10.9 : 10.8, 18.1 : 18.4; 4 096 tiles 7.3 : 6.0, 18.6 : 11.9, 34.7 : 19.6).
constexpr long kF32SmallTiles = 2048;

// the first chunk of quarter q
__device__ __forceinline__ int f32_quarter(int K, int q) { return q * ((K + 15) / 16) / 4; }
// acc += a chunk's products: a lane holds four consecutive k of its activation row and of its
// weight row, product s takes element s of every lane's four (the same k on both sides)
__device__ __forceinline__ void f32_chunk(f32x4& acc, const float4& w, const float4& a) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, a.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, a.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, a.z, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, a.w, acc, 0, 0, 0);
}

// One 16 x 16 tile per block, the four waves a quarter of K each, four chunks' loads in flight.
// 32 rows, d = 64, d_ffn = 256, against 64 x 64 tiles that walk K in steps of 16, one memory
// latency each: 13.6 -> 4.6 us per residual product, 21.0 -> 5.0 for the second fusion product.
template <EpiKind KIND>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(GemmProblem p, EpiParams ep) {
  using E = Epi<KIND, float>;
  __shared__ float4 part[3][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, fr = lane & 15, fq = lane >> 4;
  if (p.M_dev) p.M = min(*p.M_dev, p.M);
  const int tiles_n = (p.N + 15) / 16;
  const int m0 = (blockIdx.x / tiles_n) * 16, n0 = (blockIdx.x % tiles_n) * 16;
  if (m0 >= p.M) return;
  const int gr = min(m0 + fr, p.M - 1), gn = min(n0 + fr, p.N - 1);
  const float* A1 = static_cast<const float*>(p.A1) + (size_t)gr * p.lda1;
  const float* A2 = static_cast<const float*>(p.A2) + (size_t)gr * p.lda2;
  const float* W = static_cast<const float*>(p.W) + (size_t)gn * p.ldw;
  const int c1 = f32_quarter(p.K, wave + 1);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;
  for (int c = f32_quarter(p.K, wave); c < c1; c += U) {
    float4 a[U], w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // K and K1 are multiples of 4
      const int k = 16 * (c + u) + 4 * fq;
      const bool in = c + u < c1 && k < p.K;
      a[u] = in ? *reinterpret_cast<const float4*>(k < p.K1 ? A1 + k : A2 + (k - p.K1)) : make_float4(0.f, 0.f, 0.f, 0.f);
      w[u] = in ? *reinterpret_cast<const float4*>(W + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c + u < c1) f32_chunk(acc, w[u], a[u]);
  }
  if (wave) part[wave - 1][lane] = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    const float4 x = part[w][lane];
    acc += f32x4{x.x, x.y, x.z, x.w};
  }
  // lane holds C[m0 + fr][n0 + 4 fq + j]
  const int m = m0 + fr, n = n0 + 4 * fq;
  if (m < p.M && n < p.N) E::apply(ep, m, n, acc);
}

// 64 x 64 tiles, a 32 x 32 part per wave (2 x 2); two chunks per step through two LDS buffers,
// the next step's loads in flight over the present one's products.  LDS rows of 36 floats: the
// 16-byte reads of 16 rows fall on different banks.  Bound by the matrix cores at depth (float32
// MFMA and VALU have the same peak): a head of 2 048 x 32 768 x 512 with its sampler, whose 64 x 64
// tiles were on the VALU before, 1 296 -> 903 us; 2 048 x 256 x 256 with its fusion 173 -> 95.
template <EpiKind KIND>
__global__ __launch_bounds__(256) void gemm_f32_large_kernel(GemmProblem p, EpiParams ep) {
  using E = Epi<KIND, float>;
  constexpr int TM = 2, TN = 2, CH = 2, LD = 16 * CH + 4;
  __shared__ __attribute__((aligned(16))) float sA[2][64 * LD], sW[2][64 * LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, fr = lane & 15, fq = lane >> 4;
  const int tiles_m = (p.M + 63) / 64;  // of the launch
  const int m0 = (blockIdx.x % tiles_m) * 64, n0 = (blockIdx.x / tiles_m) * 64;
  if (p.M_dev) p.M = min(*p.M_dev, p.M);
  if (m0 >= p.M) return;
  // this thread's part of a step: four k of one row of each operand, per chunk
  const int lr = tid >> 2, lk = 4 * (tid & 3);
  const int gr = min(m0 + lr, p.M - 1), gn = min(n0 + lr, p.N - 1);
  const float* A1 = static_cast<const float*>(p.A1) + (size_t)gr * p.lda1;
  const float* A2 = static_cast<const float*>(p.A2) + (size_t)gr * p.lda2;
  const float* W = static_cast<const float*>(p.W) + (size_t)gn * p.ldw;
  const int nc = (p.K + 15) / 16, steps = (nc + CH - 1) / CH;
  float4 ra[CH], rw[CH];
  auto load = [&](int st) {
#pragma unroll
    for (int h = 0; h < CH; ++h) {  // K and K1 are multiples of 4
      const int k = 16 * (CH * st + h) + lk;
      ra[h] = rw[h] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < p.K) {
        ra[h] = *reinterpret_cast<const float4*>(k < p.K1 ? A1 + k : A2 + (k - p.K1));
        rw[h] = *reinterpret_cast<const float4*>(W + k);
      }
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      *reinterpret_cast<float4*>(&sA[buf][lr * LD + 16 * h + lk]) = ra[h];
      *reinterpret_cast<float4*>(&sW[buf][lr * LD + 16 * h + lk]) = rw[h];
    }
  };
  f32x4 acc[TN][TM] = {}, sum[TN][TM] = {};
  int q = 0, end = f32_quarter(p.K, 1);  // the quarter of the next chunk, and where it ends
  auto close = [&] {                     // quarter q is summed
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        sum[i][j] = q ? sum[i][j] + acc[i][j] : acc[i][j];
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    ++q;
    end = f32_quarter(p.K, q + 1);
  };
  const int ao = ((wave & 1) * 32 + fr) * LD + 4 * fq, wo = ((wave >> 1) * 32 + fr) * LD + 4 * fq;
  load(0);
  stage(0);
  __syncthreads();
  for (int st = 0; st < steps; ++st) {
    const int buf = st & 1;
    if (st + 1 < steps) load(st + 1);
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const int c = CH * st + h;
      if (c >= nc) break;
      while (c == end) close();
      float4 a[TM], w[TN];
#pragma unroll
      for (int j = 0; j < TM; ++j) a[j] = *reinterpret_cast<const float4*>(&sA[buf][ao + 16 * j * LD + 16 * h]);
#pragma unroll
      for (int i = 0; i < TN; ++i) w[i] = *reinterpret_cast<const float4*>(&sW[buf][wo + 16 * i * LD + 16 * h]);
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) f32_chunk(acc[i][j], w[i], a[j]);
    }
    if (st + 1 < steps) stage(buf ^ 1);  // last read before the barrier of the step before
    __syncthreads();
  }
  while (q < 4) close();
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int m = m0 + 32 * (wave & 1) + 16 * j + fr, n = n0 + 32 * (wave >> 1) + 16 * i + 4 * fq;
      if (m < p.M && n < p.N) E::apply(ep, m, n, sum[i][j]);
    }
}

// Grids that leave CUs short of blocks.  Up to 512 tiles of 64 x 64, two per CU, run on the deep
// ring (gemm_ring.h); with at most 96 such tiles 32 x 32 ones, four times the blocks (64 x 3 072 x
// 2 048, 48 tiles: 12.2 -> 9.1 us; 384 x 768 x 2 048, 72 tiles: 12.1 -> 10.3; with 192 tiles, 1 024 x
// 768 x 512, 5.6 against 7.3).  Epilogues that pair weight blocks keep 64 columns.  Splitting K of
// the unsplit residual products over blocks would be faster still (384 x 768 x 2 048 in four: 6.8
// us), but the sums' other order moves tokens that nearly tie.
//
// More than 512 put three blocks on some CUs, which hide each other's latency:
//  - 64 x 96 tiles where they are at most 512 (residual, fusion 2 and float32 outputs, q/k/v of a
//    long K, whose strips then leave LDS out): no CU has more than two, which load 320 rows per
//    K step instead of 384.  us, 64 x 64 on the two-buffer loop against 64 x 96: 3 072 x 768 x 2 048
//    21.2 : 19.9, 3 500 x 768 x 3 072 30.5 : 28.9, 1 272 x 2 048 x 2 048 21.3 : 20.3, 640 x 4 608 x
//    4 096 52.7 : 44.8, 2 625 x 1 024 x 1 024 14.5 : 13.5, 3 000 x 768 x 768 11.8 : 11.9; q/k/v 1 024 x
//    2 304 x 768 10.7 : 11.8, 1 024 x 3 072 x 2 048 21.7 : 21.3 (a refresh step of three such layers
//    1 270 : 1 260).
//  - else the two-buffer loop (gemm_kernel.h); us, it against the ring: 768 x 3 840 x 1 536 15.9 :
//    17.5, 1 024 x 2 304 x 768 9.5 : 10.3, 300 x 10 240 x 4 096 55.2 : 61.4, fusion 1 900 x 3 840 x 1 536
//    22.5 : 24.9, 1 800 x 2 048 x 8 192 110.8 : 143.2.  Up to 768 tiles the ring stays for the up
//    projections (300 x 8 192 x 2 048 26.9 : 25.5, 768 x 3 072 x 768 10.6 : 10.2) and for at most 256
//    rows, whose weights stream from memory (200 x 10 240 x 4 096 50.8 : 46.7).
template <EpiKind K>
hipError_t launch_small(const GemmProblem& p, const EpiParams& e, hipStream_t s) {
  using E = Epi<K, bf16>;
  constexpr bool kFragments = !E::kGlu && !TileEpi<E>::value && !RowEpi<E>::value;
  constexpr bool kUp = K == EPI_GLU_SILU || K == EPI_GLU_GELU || K == EPI_GELU;
  const long t64 = (long)((p.M + 63) / 64) * ((p.N + 63) / 64);
  if constexpr (kFragments)
    if (t64 <= 96) return launch_ring<32, 32, 8, 2, K>(p, e, s);
  if (t64 > 512) {
    if constexpr (kFragments) {
      const long t96 = (long)((p.M + 63) / 64) * ((p.N + 95) / 96);
      if (t96 <= 512 && !(TileLdsEpi<E>::value && p.K < 2048)) return launch_ring<64, 96, 4, 2, K>(p, e, s);
    }
    if (t64 > 768 || !(kUp || p.M <= 256)) return launch_bf16<64, 64, 2, 2, 2, 3, K>(p, e, s);
  }
  return launch_ring<64, 64, 3, 3, K>(p, e, s);
}

template <EpiKind K>
hipError_t dispatch(DType dt, const GemmProblem& p, const EpiParams& e, hipStream_t s) {
  if (dt == F32) {
    // the kernels load four k at a time; float32 models run their gated units unfused (glu_f32)
    if constexpr (!Epi<K, float>::kGlu) {
      if (p.K % 4 || p.K1 % 4 || p.lda1 % 4 || p.lda2 % 4 || p.ldw % 4) return hipErrorInvalidValue;
      const long t16 = (long)((p.M + 15) / 16) * ((p.N + 15) / 16);
      const int t64 = ((p.M + 63) / 64) * ((p.N + 63) / 64);
      if (t16 <= kF32SmallTiles)
        launch_timed(gemm_f32_small_kernel<K>, dim3((unsigned)t16), dim3(256), 0, s, p, e);
      else
        launch_timed(gemm_f32_large_kernel<K>, dim3(t64), dim3(256), 0, s, p, e);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  // tile choice by how many blocks each shape yields (256 CUs) and the rounds they run in: 256 x
  // 256 tiles hold 256 blocks at once (gemm_pingpong.h), 192 x 128 and 128 x 128 ones 512
  const auto tiles = [&](int bm, int bn) { return (long)((p.M + bm - 1) / bm) * ((p.N + bn - 1) / bn); };
  const long t256 = tiles(256, 256), t128 = tiles(128, 128);
  const long r256 = (t256 + 255) / 256, r192 = (tiles(192, 128) + 511) / 512, r128 = (t128 + 511) / 512;
  if ((p.M >= 4096 || p.N >= 16384) && t256 >= 128) {
    // rounds times the time of one, 80 : 75 : 57 over K = 512 to 8 192 (by 256 x 256 / 192 x 128 / 128 x
    // 128 tiles, us: GLU 4 600 x 4 096 x 768 40.3 / 28.3 / 34.2, 8 192 x 4 096 x 768 46.2 / 64.4 /
    // 53.9; 6 144 x 3 072 x 2 048 110 / 75 / 88; residual 4 096 x 2 048 x 2 048 53 / 50 / 42, 32 768 x
    // 2 048 x 8 192 818 / 1 272 / 1 083).  Two exceptions: where one round of 256 x 256 tiles holds a
    // long K, 192 x 128 ones lose (5 000 x 2 048 x 8 192 162 : 189); and the staged q/k/v epilogue
    // stands between two tiles of a block, too long beside a short K (12 288 x 2 304 x 768 63.9 / 55.1
    // / 56.5, 16 384 rows 89.0 / 75.5 / 73.7).
    constexpr long kNever = 1l << 40;
    const long c256 = pingpong_ok(p) && !(TileLdsEpi<Epi<K, bf16>>::value && p.K < 2048) ? 80 * r256 : kNever;
    const long c192 = r256 == 1 && p.K >= 4096 ? kNever : 75 * r192, c128 = 57 * r128;
    if (c256 <= c192 && c256 <= c128) {
      // float32 outputs of a short K and fewer than 4 096 rows: a block per tile, which leaves
      // its stores behind when it ends, where the walking one waits for them before its next
      // tile (1 280 x 32 768 x 768 111 -> 94 us, 2 048 rows 166 -> 147, 3 500 x 16 384 x 512 127 -> 110;
      // from 4 600 rows on the other way round, 6 144 x 8 192 x 1 024 112 against 119)
      if constexpr (K == EPI_STORE_F32)
        if (p.K <= 1024 && p.M < 4096) return launch_bf16<256, 256, 2, 2, 4, 1, K>(p, e, s);
      return launch_pp<K>(p, e, s);
    }
    if (c192 <= c128) return launch_bf16<192, 128, 2, 2, 2, 2, K>(p, e, s);
    return launch_bf16<128, 128, 2, 2, 2, 2, K>(p, e, s);
  }
  if (t128 >= 256) {
    // 192 x 128 tiles win when they need fewer rounds for the same rows (e.g. 768 tiles of 128 x
    // 128 = 1.5 rounds -> 512 of 192 x 128)
    if (r192 * 192 < r128 * 128) return launch_bf16<192, 128, 2, 2, 2, 2, K>(p, e, s);
    return launch_bf16<128, 128, 2, 2, 2, 2, K>(p, e, s);
  }
  return launch_small<K>(p, e, s);
}

// out[m, n] = row1[m] * sum_s part[s, m, n], s ascending (float4 granules, N % 4 == 0)
__global__ void splitk_reduce_kernel(const float* part, int S, int M, int N, const float* row1, float* out, int ldo) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x, n4 = N / 4;
  if (i >= (long)M * n4) return;
  const int m = (int)(i / n4), n = (int)(i % n4) * 4;
  const size_t MN = (size_t)M * N;
  float4 acc = *reinterpret_cast<const float4*>(part + (size_t)m * N + n);
  for (int k = 1; k < S; ++k) {
    const float4 v = *reinterpret_cast<const float4*>(part + k * MN + (size_t)m * N + n);
    acc.x += v.x;
    acc.y += v.y;
    acc.z += v.z;
    acc.w += v.w;
  }
  const float r = row1[m];
  store4(out + (size_t)m * ldo + n, r * acc.x, r * acc.y, r * acc.z, r * acc.w);
}

// Row-scaled product with a long K and few output tiles (the self-conditioning product:
// K = vocabulary, N = d_model): 128 x 128 tiles split over K so that the grid fills the
// chip, the slices' fp32 products go to part [S, M, N], then an ordered reduction.
// Returns false when the split does not apply.
// K slices: double while the grid has fewer than 512 blocks, each slice keeps >= 8 K
// tiles and the tiles divide evenly (at most 16)
int split_slices(int M, int N, int K) {
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
  const int nk = K / 64;
  int S = 1;
  while (S < 16 && tiles * S < 512 && nk % (2 * S) == 0 && nk / (2 * S) >= 8) S *= 2;
  return S;
}

bool splitk_scale(const GemmProblem& p, const EpiParams& e, hipStream_t s, hipError_t* err) {
  if (!e.part || p.M_dev || p.N % 4 || p.K1 != p.K) return false;
  const int S = split_slices(p.M, p.N, p.K);
  if (S == 1) return false;
  GemmProblem q = p;
  q.ksplit = S;
  EpiParams f;
  f.out = e.part;
  f.ldo = p.N;
  f.split_stride = (size_t)p.M * p.N;
  *err = launch_bf16<128, 128, 2, 2, 2, 2, EPI_STORE_F32>(q, f, s);
  if (*err != hipSuccess) return true;
  const long total = (long)p.M * (p.N / 4);
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                     static_cast<const float*>(e.part), S, p.M, p.N, e.row1, static_cast<float*>(e.out), e.ldo);
  *err = hipGetLastError();
  return true;
}

// resid[m, n] += sum_s part[s, m, n], s ascending (float4 granules, N % 4 == 0)
__global__ void resid_reduce_kernel(const float* part, int S, int M, int N, float* resid, int ldr) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x, n4 = N / 4;
  if (i >= (long)M * n4) return;
  const int m = (int)(i / n4), n = (int)(i % n4) * 4;
  const size_t MN = (size_t)M * N;
  float4 acc = *reinterpret_cast<const float4*>(part + (size_t)m * N + n);
  for (int k = 1; k < S; ++k) {
    const float4 v = *reinterpret_cast<const float4*>(part + k * MN + (size_t)m * N + n);
    acc.x += v.x;
    acc.y += v.y;
    acc.z += v.z;
    acc.w += v.w;
  }
  float4* r = reinterpret_cast<float4*>(resid + (size_t)m * ldr + n);
  float4 x = *r;
  x.x += acc.x;
  x.y += acc.y;
  x.z += acc.z;
  x.w += acc.w;
  *r = x;
}

// resid[m, :] += sum_s part[s, m, :] as above, then y[m, :] = bf16(resid[m, :] * rsqrt(
// mean(resid[m, :]^2) + eps) * g): the RMSNorm that follows a residual product, in the
// same pass over the row.  One block of 256 threads per row, NV float4 per thread
// (N <= 1024 NV): every slice load of the row is independent, so the row costs one
// round trip; the row's sum of squares is a block reduction.
template <int NV>
__global__ __launch_bounds__(256) void resid_reduce_rms_kernel(const float* part, int S, int M, int N, float* resid,
                                                               int ldr, const float* g, float eps, bf16* y) {
  __shared__ float red[4];
  const int m = blockIdx.x, t = threadIdx.x;
  const size_t MN = (size_t)M * N;
  float4 x[NV];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = (t + 256 * i) * 4;
    if (c < N) {
      float4 acc = *reinterpret_cast<const float4*>(part + (size_t)m * N + c);
#pragma unroll 4
      for (int k = 1; k < S; ++k) {
        const float4 v = *reinterpret_cast<const float4*>(part + k * MN + (size_t)m * N + c);
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
      }
      float4* r = reinterpret_cast<float4*>(resid + (size_t)m * ldr + c);
      float4 v = *r;
      v.x += acc.x;
      v.y += acc.y;
      v.z += acc.z;
      v.w += acc.w;
      *r = v;
      x[i] = v;
      ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
  }
  ss = block_sum(ss, red);
  const float rs = rsqrtf(ss / N + eps);
  bf16* yr = y + (size_t)m * N;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = (t + 256 * i) * 4;
    if (c < N) {
      const float4 w = *reinterpret_cast<const float4*>(g + c);
      store4(yr + c, x[i].x * rs * w.x, x[i].y * rs * w.y, x[i].z * rs * w.z, x[i].w * rs * w.w);
    }
  }
}

// K slices of a residual product, counted as for 256 x 256 tiles at one block per CU whatever
// tiles they run on (slice_tiles): the count is the order of the sums, which outputs keep.  The S in
// [2, 16] (each slice >= 8 K tiles, slices as even as the tile count allows) that
// minimises the modelled time, in K-step units: rounds of 256 blocks x (K tiles per
// slice + 2 for a block's prologue and epilogue), plus 1.5 per slice for the ordered
// reduction's read of the slice's [M, N] partial; 1 when no split beats the unsplit
// grid.  Products with fewer than 128 K tiles are split only from 64 output tiles on:
// smaller ones run sooner on the 64 x 64 or 128 x 128 tiles at two or three blocks per CU
// (block workload's attention output, 1024 x 2048 x 2048, and the small workload's FFN
// down, 3072 x 768 x 2048: 2.5 % and 6.6 % slower per generation when split).  26B-class
// FFN down (1024 x 4608 x 36864): S = 7, 504 blocks in two rounds (468 -> 354 us against
// 128 x 128 tiles in 8 slices); its attention output (1024 x 4608 x 4096): S = 3.
int resid_slices256(int M, int N, int K) {
  const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
  const int nk = K / 64;
  if (N % 4 || nk < 32 || (nk < 128 && tiles < 64)) return 1;
  int best = 1;
  double best_t = (double)((tiles + 255) / 256) * (nk + 2);
  for (int S = 2; S <= 16 && nk / S >= 8; ++S) {
    const double t = (double)((tiles * S + 255) / 256) * ((double)nk / S + 2) + 1.5 * S;
    if (t < best_t - 1e-9) {
      best = S;
      best_t = t;
    }
  }
  return best;
}

// K slices of a residual product with a long K and fewer than two 128 x 128 tiles per
// CU (512 resident blocks): the S in {2, 4, 8} (each slice >= 16 K tiles) whose grid
// best fills whole rounds of 512 blocks, the smaller S on ties
int resid_slices(int M, int N, int K) {
  const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
  const int nk = K / 64;
  if (tiles >= 512 || nk < 64 || N % 4) return 1;
  int best = 1;
  double best_fill = 0.0;
  for (int S = 2; S <= 8; S *= 2) {
    if (nk % S || nk / S < 16) break;
    const long blocks = tiles * S, rounds = (blocks + 511) / 512;
    const double fill = (double)blocks / (512.0 * rounds);
    if (fill > best_fill + 1e-9) {
      best = S;
      best_fill = fill;
    }
  }
  return best;
}

// The tiles a residual product's K slices run on.  Their number is given by the two rules
// above whatever the tiles, so the sums have one order per shape.  64 x 64 tiles while their
// blocks fit the chip at once (512, two per CU) or nearly so (64 x 2 048 x 8 192, nine slices: 25 us
// on 256 x 256 tiles -> 11).  us, 64 x 64 against 128 x 128 tiles, by the number of the former: 416
// blocks 16.2 : 22.7 and 19.3 : 25.0, 512 10.2 : 14.4, 28.7 : 40.6 and 35.3 : 44.0; 576 17.9 : 18.8 and
// 15.8 : 15.3, 624 21.0 : 22.8 and 22.8 : 24.9, 640 15.5 : 16.3 and 15.9 : 15.4; 832 28.4 : 26.7, 864 17.3 :
// 16.4, 1 024 54.9 : 46.6.  Then 128 x 128 (256 rows 37.7 -> 27.2 against 256 x 256), else 256 x 256
// (1 024 rows, eight slices: 55.0 against 64.3 and 83.9).
enum SliceTiles { SLICE_64, SLICE_128, SLICE_256 };
SliceTiles slice_tiles(int M, int N, int S, bool on256) {
  const long t64 = (long)((M + 63) / 64) * ((N + 63) / 64), t128 = (long)((M + 127) / 128) * ((N + 127) / 128);
  if (t64 * S <= 640) return SLICE_64;
  return !on256 || t128 * S <= 512 ? SLICE_128 : SLICE_256;
}

// The slices' products of q (ksplit set) to f.out [S, M, N].
hipError_t launch_slices(SliceTiles t, const GemmProblem& q, const EpiParams& f, hipStream_t s) {
  switch (t) {
    case SLICE_64: return launch_ring<64, 64, 4, 2, EPI_STORE_F32>(q, f, s);
    case SLICE_256: return launch_pp<EPI_STORE_F32>(q, f, s);  // slices of >= 8 K tiles, one operand
    default: return launch_bf16<128, 128, 2, 2, 2, 2, EPI_STORE_F32>(q, f, s);
  }
}

}  // namespace

int gemm_split_slices(int M, int N, int K) { return split_slices(M, N, K); }
int gemm_resid_slices(int M, int N, int K) {
  const int S256 = resid_slices256(M, N, K);
  return S256 > 1 ? S256 : resid_slices(M, N, K);
}
bool gemm_resid_norms(int M, int N, int K) { return gemm_resid_slices(M, N, K) > 1 && N % 4 == 0 && N <= 8192; }

hipError_t gemm(DType dt, const GemmProblem& p, EpiKind kind, const EpiParams& e, hipStream_t s) {
  if (p.M <= 0 || p.N <= 0) return hipSuccess;
  if (kind == EPI_SCALE_F32 && dt == BF16) {
    hipError_t err = hipSuccess;
    if (splitk_scale(p, e, s, &err)) return err;
  }
  if (kind == EPI_RESID && dt == BF16 && e.part && !p.M_dev && p.K1 == p.K) {
    const int S256 = resid_slices256(p.M, p.N, p.K);
    const int S = S256 > 1 ? S256 : resid_slices(p.M, p.N, p.K);
    if (S > 1) {  // the slices' products to part [S, M, N], then an ordered sum into resid
      GemmProblem q = p;
      q.ksplit = S;
      EpiParams f;
      f.out = e.part;
      f.ldo = p.N;
      f.split_stride = (size_t)p.M * p.N;
      hipError_t err = launch_slices(slice_tiles(p.M, p.N, S, S256 > 1), q, f, s);
      if (err != hipSuccess) return err;
      if (e.norm_out) {  // the ordered sum and the RMSNorm of the updated rows in one pass
        if (!gemm_resid_norms(p.M, p.N, p.K) || !e.norm_g) return hipErrorInvalidValue;
        const float* part = static_cast<const float*>(e.part);
        bf16* y = static_cast<bf16*>(e.norm_out);
        const int nv = (p.N + 1023) / 1024;
        if (nv <= 1)
          hipLaunchKernelGGL(resid_reduce_rms_kernel<1>, dim3(p.M), dim3(256), 0, s, part, S, p.M, p.N, e.resid, e.ldr,
                             e.norm_g, e.norm_eps, y);
        else if (nv <= 2)
          hipLaunchKernelGGL(resid_reduce_rms_kernel<2>, dim3(p.M), dim3(256), 0, s, part, S, p.M, p.N, e.resid, e.ldr,
                             e.norm_g, e.norm_eps, y);
        else if (nv <= 5)
          hipLaunchKernelGGL(resid_reduce_rms_kernel<5>, dim3(p.M), dim3(256), 0, s, part, S, p.M, p.N, e.resid, e.ldr,
                             e.norm_g, e.norm_eps, y);
        else
          hipLaunchKernelGGL(resid_reduce_rms_kernel<8>, dim3(p.M), dim3(256), 0, s, part, S, p.M, p.N, e.resid, e.ldr,
                             e.norm_g, e.norm_eps, y);
        return hipGetLastError();
      }
      const long total = (long)p.M * (p.N / 4);
      hipLaunchKernelGGL(resid_reduce_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                         static_cast<const float*>(e.part), S, p.M, p.N, e.resid, e.ldr);
      return hipGetLastError();
    }
  }
  switch (kind) {
    case EPI_STORE: return dispatch<EPI_STORE>(dt, p, e, s);
    case EPI_STORE_F32: return dispatch<EPI_STORE_F32>(dt, p, e, s);
    case EPI_SCALE_F32: return dispatch<EPI_SCALE_F32>(dt, p, e, s);
    case EPI_RESID: return dispatch<EPI_RESID>(dt, p, e, s);
    case EPI_GELU: return dispatch<EPI_GELU>(dt, p, e, s);
    case EPI_GLU_SILU: return dispatch<EPI_GLU_SILU>(dt, p, e, s);
    case EPI_GLU_GELU: return dispatch<EPI_GLU_GELU>(dt, p, e, s);
    case EPI_FUSION1: return dispatch<EPI_FUSION1>(dt, p, e, s);
    case EPI_FUSION2: return dispatch<EPI_FUSION2>(dt, p, e, s);
    case EPI_SILU: return dispatch<EPI_SILU>(dt, p, e, s);
    case EPI_ADD_F32: return dispatch<EPI_ADD_F32>(dt, p, e, s);
    case EPI_ADD_BOTH: return dispatch<EPI_ADD_BOTH>(dt, p, e, s);
    case EPI_ADD_SUB: return dispatch<EPI_ADD_SUB>(dt, p, e, s);
    case EPI_PAIRED: return dispatch<EPI_PAIRED>(dt, p, e, s);
    case EPI_QKV_ROPE: {
      EpiParams f = e;
      fast_divider((uint32_t)e.L, f.l_mul, f.l_shift);
      fast_divider((uint32_t)e.dh, f.dh_mul, f.dh_shift);
      return dispatch<EPI_QKV_ROPE>(dt, p, f, s);
    }
    case EPI_SAMPLE: break;  // head_sample
  }
  return hipErrorInvalidValue;
}

}  // namespace tadm
