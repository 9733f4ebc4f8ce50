// Warm-start MLP for families of LPs: v = W3 relu(W2 relu(W1 u + b1) + b2) + b3.
//
// BF16 weights and activations feed the matrix cores (v_mfma_f32_32x32x16_bf16
// on gfx950) with FP32 accumulation; an FP32 master copy of the weights takes
// the Adam updates.  Every GEMM is C = op(A) op(B) with row-major operands,
// tiled 128 x 128 (four wavefronts of 64 x 64) or 64 x 64 (of 32 x 32) per
// workgroup, split along K when M x N alone cannot fill the chip; split partials are summed in a fixed
// order, so results are deterministic.  The products' epilogues do the rest of
// a training step where the data already sits in registers: bias and ReLU in
// the forward pass, the loss and its gradient in the output layer, the ReLU
// mask in the backward pass, and Adam in the weight-gradient products, so FP32
// weight gradients never travel through HBM during training.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <random>
#include <vector>

#include "../../include/pdcs.h"
#include "pdcs_engine.h"

using namespace pdcs;

namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Sides of a workgroup's output tile.  A K-split is chosen on tiles of kTileWide, so
// that a product's sums have the same order with either tile.
constexpr int kTileWide = 128, kTileNarrow = 64;

__device__ __forceinline__ bf16 to_bf16(float v) { return (bf16)v; }

// One operand tile (TT rows of op(X) x KT) staged through registers.  op(X)
// row r, column k lives at X[k * ld + r] when trans, else X[r * ld + k].  Each
// thread loads KQ = TT KT / 2048 8-element vectors, each along the source's
// contiguous direction:
//   not trans: vector e = tid + 256 q holds row e / (KT/8), k-block e % (KT/8);
//   trans    : thread t holds rows 8 (t % (TT/8)) .. +7 for the KQ consecutive
//              k = (t / (TT/8)) KQ + q, one vector per k; the TT/8 lanes of a k
//              read 2 TT contiguous bytes.  The store transposes these in registers
//              so that each row goes to LDS as one run of KQ k-values.
// vec: the launch guarantees 16-byte alignment of the source and ld % 8 == 0,
// so whole vectors inside the bounds load with one 16-byte access; anything
// else loads element by element.
//
// LDS holds TT rows of KT + 8 elements.  The 16-byte blocks of a row are
// swizzled by the row's group of eight (block b of row r sits at block
// b ^ ((r / 8) mod KT/8)): the transposed stores of 16 lanes (rows eight apart)
// and the MFMA reads of 32 lanes (32 consecutive rows) then fall on different
// banks.
template <int TT, int KT>
struct TileRegs {
  bf16x8 v[TT * KT / 2048];
};

template <int KT>
__device__ __forceinline__ int swz(int row, int blk) {
  return blk ^ ((row >> 3) & (KT / 8 - 1));
}

template <int TT, int KT>
__device__ __forceinline__ void tile_load(const bf16* __restrict__ X, int ld, int trans, int vec, int r0, int R,
                                          int k0, int kend, TileRegs<TT, KT>& t) {
  const int tid = threadIdx.x;
  constexpr int KQ = TT * KT / 2048;
#pragma unroll
  for (int q = 0; q < KQ; ++q) {
    bf16x8 v;
    if (!trans) {
      const int e = tid + q * 256;
      const int gr = r0 + e / (KT / 8), gk = k0 + (e % (KT / 8)) * 8;
      if (vec && gr < R && gk + 8 <= kend) {
        v = *reinterpret_cast<const bf16x8*>(X + (size_t)gr * ld + gk);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (gr < R && gk + i < kend) ? X[(size_t)gr * ld + gk + i] : to_bf16(0.0f);
      }
    } else {
      const int gr = r0 + (tid % (TT / 8)) * 8, gk = k0 + (tid / (TT / 8)) * KQ + q;
      if (vec && gk < kend && gr + 8 <= R) {
        v = *reinterpret_cast<const bf16x8*>(X + (size_t)gk * ld + gr);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (gk < kend && gr + i < R) ? X[(size_t)gk * ld + gr + i] : to_bf16(0.0f);
      }
    }
    t.v[q] = v;
  }
}

template <int TT, int KT>
__device__ __forceinline__ void tile_store(bf16 (*S)[KT + 8], int trans, const TileRegs<TT, KT>& t) {
  const int tid = threadIdx.x;
  constexpr int KQ = TT * KT / 2048;
  if (!trans) {
#pragma unroll
    for (int q = 0; q < KQ; ++q) {
      const int e = tid + q * 256;
      const int rr = e / (KT / 8), blk = e % (KT / 8);
      *reinterpret_cast<bf16x8*>(&S[rr][swz<KT>(rr, blk) * 8]) = t.v[q];
    }
  } else if constexpr (KQ == 1) {
    const int rb = (tid % (TT / 8)) * 8, kq = tid / (TT / 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) S[rb + i][swz<KT>(rb + i, kq >> 3) * 8 + (kq & 7)] = t.v[0][i];
  } else {
    typedef __bf16 bf16xq __attribute__((ext_vector_type(KQ)));
    const int rb = (tid % (TT / 8)) * 8, kq = (tid / (TT / 8)) * KQ;  // k-run kq .. kq + KQ - 1: within one 8-block
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      bf16xq w;
#pragma unroll
      for (int q = 0; q < KQ; ++q) w[q] = t.v[q][i];
      const int row = rb + i;
      *reinterpret_cast<bf16xq*>(&S[row][swz<KT>(row, kq >> 3) * 8 + (kq & 7)]) = w;
    }
  }
}

// How a GEMM output element is used once its FP32 sum s is known.
//   EPI_STORE: C[z][row][col] = s (split partials, or a plain FP32 product)
//   EPI_ACT  : s (+ bias[col]), ReLU, times (mask[idx] > 0) -- the derivative of
//              ReLU read from the BF16 activation it produced -- then times
//              osc[col] plus omu[col] (the network output in the caller's units),
//              stored as FP32 and/or BF16
//   EPI_ADAM : s is the gradient of weight idx: Adam on the FP32 master weight
//              and its moments, and the BF16 copy the next products read, so the
//              gradient itself never reaches memory
//   EPI_MSE  : s + bias[col] is the network output; with the target t
//              (standardized per column when tmu is set) the loss gradient
//              g = 2 (v - t) * gscale goes out as BF16, and each workgroup leaves
//              one loss partial (FP64) and per-column sums of g for each 64 rows
enum { EPI_STORE = 0, EPI_ACT = 1, EPI_ADAM = 2, EPI_MSE = 3 };

struct Epi {
  const float* bias = nullptr;
  int relu = 0;
  const bf16* mask = nullptr;
  const float* osc = nullptr;
  const float* omu = nullptr;
  float* out32 = nullptr;
  bf16* out16 = nullptr;
  float *p = nullptr, *m = nullptr, *v = nullptr;
  bf16* w16 = nullptr;
  float lr = 0, b1 = 0, b2 = 0, eps = 0, c1 = 1, c2 = 1;
  const float* t = nullptr;
  const float* tmu = nullptr;
  const float* tinv = nullptr;
  float gscale = 0;
  int vec4 = 0;  // EPI_ADAM: N % 4 == 0, p / m / v 16-byte and w16 8-byte aligned
  float* colpart = nullptr;
  double* lossp = nullptr;
};

__device__ __forceinline__ void epi_act(const Epi& e, size_t idx, int col, float s) {
  if (e.bias) s += e.bias[col];
  if (e.relu) s = fmaxf(s, 0.0f);
  if (e.mask) s = (float)e.mask[idx] > 0.0f ? s : 0.0f;
  if (e.osc) s = s * e.osc[col] + e.omu[col];
  if (e.out32) e.out32[idx] = s;
  if (e.out16) e.out16[idx] = to_bf16(s);
}

// Adam on one weight.  The multiply-adds are written out, so that a weight has the
// same bits whichever path its tile takes.
__device__ __forceinline__ void adam_update(const Epi& e, float g, float& p, float& m, float& v) {
  m = fmaf(e.b1, m, (1.0f - e.b1) * g);
  v = fmaf(e.b2, v, (1.0f - e.b2) * g * g);
  p = p - e.lr * (m / e.c1) / (sqrtf(v / e.c2) + e.eps);
}

// Raw buffer access (vector memory instructions with a uniform resource):
// 32-bit byte offsets, per lane plus uniform.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ float bload(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, float x) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, (int)voff, (int)soff, 0);
}
__device__ __forceinline__ float4 bload4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
  return make_float4(__int_as_float(v[0]), __int_as_float(v[1]), __int_as_float(v[2]), __int_as_float(v[3]));
}
// (The whole offset per lane: a 16-byte store still reads its data registers while
// the next instruction runs, and the compiler keeps that one from overwriting
// them only when the scalar offset is no register.  With one, stores followed
// at once by a write of their first register left that value in memory.)
__device__ __forceinline__ void bstore4(__amdgpu_buffer_rsrc_t r, uint32_t off, float4 x) {
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  const i32x4 v = {__float_as_int(x.x), __float_as_int(x.y), __float_as_int(x.z), __float_as_int(x.w)};
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)off, 0, 0);
}
__device__ __forceinline__ void bstore_2x32(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, uint32_t lo,
                                            uint32_t hi) {
  typedef int i32x2 __attribute__((ext_vector_type(2)));
  const i32x2 v = {(int)lo, (int)hi};
  __builtin_amdgcn_raw_buffer_store_b64(v, r, (int)voff, (int)soff, 0);
}
__device__ __forceinline__ void bstore16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff, bf16 x) {
  __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, x), r, (int)voff, (int)soff, 0);
}

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// C = op(A)[M x K] op(B)[K x N] by TT x TT output tiles, split S =
// gridDim.x / (gx * gy) ways along K (split z takes every S-th K-tile):
//   op(A)[m][k] = ta ? A[k * lda + m] : A[m * lda + k]
//   op(B)[k][n] = tb ? B[n * ldb + k] : B[k * ldb + n]
// (op(B) is staged as its transpose, rows n, so both tiles are row x k.)
// Workgroups are dispatched to the 8 XCDs round-robin by linear index; the
// index is remapped so that consecutive logical tiles share an XCD, and the
// tile order runs fastest along the shorter grid side, so the tiles that read
// the same operand panel (the same K-chunk of a split product, the same row or
// column panel otherwise) meet in one L2.
struct GemmArgs {
  const bf16* A;
  int lda, ta, veca;
  const bf16* B;
  int ldb, tb, vecb;
  float* C;
  int M, N, K, gx, gy;
  Epi e;
};

// Workgroup L of the total that the product takes.
template <int KIND, int KT, int TT>
__device__ __forceinline__ void gemm_block(const GemmArgs& q, int L, int total) {
  const bf16 *__restrict__ A = q.A, *__restrict__ B = q.B;
  float* __restrict__ C = q.C;
  const int lda = q.lda, ta = q.ta, veca = q.veca, ldb = q.ldb, tb = q.tb, vecb = q.vecb;
  const int M = q.M, N = q.N, K = q.K, gx = q.gx, gy = q.gy;
  const Epi& e = q.e;
  // operand tiles for the K-loop; the Adam epilogue reuses the same LDS to
  // stage the FP32 output tile (rows padded by 4 floats)
  // K-tiles staged together, the order of the sums staying: two narrow ones in the
  // loss layer, whose few workgroups (376 for 256 x 6000) each wait for every
  // K-tile's loads (25.4 us with one, 15.9 with two; the other kinds, one and two:
  // split products 7.9 and 8.9, 64 x 60000 outputs 19.7 and 20.5, Adam 19.1 and 19.0)
  constexpr int U = KIND == EPI_MSE && TT == kTileNarrow ? 2 : 1;
  constexpr int kTileBytes = U * 2 * TT * (KT + 8) * 2;
  constexpr int kStageBytes = KIND == EPI_ADAM ? TT * (TT + 4) * 4 : 0;
  constexpr int NF = TT / 64;  // 32 x 32 fragments of a wave along each side
  __shared__ __attribute__((aligned(16))) unsigned char smem[kTileBytes > kStageBytes ? kTileBytes : kStageBytes];
  bf16(*As)[TT][KT + 8] = reinterpret_cast<bf16(*)[TT][KT + 8]>(smem);
  bf16(*Bs)[TT][KT + 8] = reinterpret_cast<bf16(*)[TT][KT + 8]>(smem + U * TT * (KT + 8) * 2);
  const int full = total & ~7;
  const int Q = L < full ? (L & 7) * (full >> 3) + (L >> 3) : L;
  const int tiles = gx * gy;
  const int z = Q / tiles, tq = Q - z * tiles;
  int bx, by;
  if (gx <= gy) {
    bx = tq % gx;
    by = tq / gx;
  } else {
    by = tq % gy;
    bx = tq / gy;
  }
  const int m0 = by * TT, n0 = bx * TT;
  // K-tiles z, z + S, z + 2S, ... of the S-way split: the workgroups of one
  // output tile read adjacent K-tiles at about the same time, so each row of an
  // operand is fetched in long runs rather than one K-tile at a time
  const int S = total / tiles, kstep = S * KT;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave >> 1) * (TT / 2), wn = (wave & 1) * (TT / 2);
  f32x16 acc[NF][NF];
#pragma unroll
  for (int i = 0; i < NF; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
  TileRegs<TT, KT> ra[U], rb[U];
  const auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ku = k0 + u * kstep;
      if (ku < K) {
        tile_load<TT, KT>(A, lda, ta, veca, m0, M, ku, min(K, ku + KT), ra[u]);
        tile_load<TT, KT>(B, ldb, !tb, vecb, n0, N, ku, min(K, ku + KT), rb[u]);
      }
    }
  };
  load(z * KT);
  for (int k0 = z * KT; k0 < K; k0 += U * kstep) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k0 + u * kstep < K) {
        tile_store<TT, KT>(As[u], ta, ra[u]);
        tile_store<TT, KT>(Bs[u], !tb, rb[u]);
      }
    __syncthreads();
    load(k0 + U * kstep);  // prefetch the next tiles while the matrix cores work
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u * kstep >= K) break;
#pragma unroll
      for (int kk = 0; kk < KT; kk += 16) {
        bf16x8 a[NF], b[NF];
        const int kb = (kk >> 3) + (lane >> 5);  // 16-byte block of k-values kk + 8 (lane / 32) ..
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          const int row = wm + i * 32 + (lane & 31);
          a[i] = *reinterpret_cast<const bf16x8*>(&As[u][row][swz<KT>(row, kb) * 8]);
        }
#pragma unroll
        for (int j = 0; j < NF; ++j) {
          const int row = wn + j * 32 + (lane & 31);
          b[j] = *reinterpret_cast<const bf16x8*>(&Bs[u][row][swz<KT>(row, kb) * 8]);
        }
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
          for (int j = 0; j < NF; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
      }
    }
    __syncthreads();
  }
  // accumulator element r of acc[i][j] holds output (row0 + i*32 + (r/4)*8 + r%4, col0 + j*32)
  const int row0 = m0 + wm + (lane >> 5) * 4, col0 = n0 + wn + (lane & 31);
  if constexpr (KIND == EPI_STORE) {
    float* Cz = C + (size_t)z * M * N;
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + i * 32 + (r / 4) * 8 + (r % 4), col = col0 + j * 32;
          if (row < M && col < N) Cz[(size_t)row * N + col] = acc[i][j][r];
        }
  } else if constexpr (KIND == EPI_ACT) {
    // per 16-element group: the bias (one column) and the masks are loaded
    // before the first store, so the loads are all in flight together
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        const int col = col0 + j * 32;
        const float bv = (e.bias && col < N) ? e.bias[col] : 0.0f;
        const float sc = (e.osc && col < N) ? e.osc[col] : 1.0f, mu = (e.osc && col < N) ? e.omu[col] : 0.0f;
        float mk[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + i * 32 + (r / 4) * 8 + (r % 4);
          mk[r] = (e.mask && row < M && col < N) ? (float)e.mask[(size_t)row * N + col] : 1.0f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + i * 32 + (r / 4) * 8 + (r % 4);
          if (row < M && col < N) {
            float s = acc[i][j][r] + bv;
            if (e.relu) s = fmaxf(s, 0.0f);
            if (!(mk[r] > 0.0f)) s = 0.0f;
            if (e.osc) s = s * sc + mu;
            const size_t idx = (size_t)row * N + col;
            if (e.out32) e.out32[idx] = s;
            if (e.out16) e.out16[idx] = to_bf16(s);
          }
        }
      }
  } else if constexpr (KIND == EPI_ADAM) {
    // Element offsets are 32-bit (each weight matrix holds < 2^30 entries).
    // Interior tiles address the moments and weights through buffer resources:
    // one per-lane byte offset per column half plus a uniform row offset, so an
    // element costs no address registers.  The accumulators go in groups
    // of 8; the loads of group q+1 are issued before group q is updated and
    // stored, so they are in flight meanwhile.  Tiles that stick out of the
    // matrix take the guarded loop.
    if (e.vec4 && m0 + TT <= M && n0 + TT <= N) {
      // The tile goes through LDS so that each thread updates whole 16-byte
      // runs of a row: thread t takes columns 4 (t % LPR) .. +3 of rows
      // t / LPR + RP q, q < TT / RP, in groups of 4; the first group's
      // weights and moments are requested before the tile is staged, and each
      // next group's before the current one is updated.
      constexpr int LPR = TT / 4, RP = 256 / LPR, NG = TT / RP / 4;
      float(*S)[TT + 4] = reinterpret_cast<float(*)[TT + 4]>(smem);
      const int lr = threadIdx.x / LPR, lc = (threadIdx.x % LPR) * 4;
      // buffer resources: one per-lane offset, the row step as a uniform offset
      const uint32_t bytes = (uint32_t)M * (uint32_t)N * 4u;
      const __amdgpu_buffer_rsrc_t rp = make_rsrc(e.p, bytes), rm = make_rsrc(e.m, bytes),
                                   rv = make_rsrc(e.v, bytes), rw = make_rsrc(e.w16, bytes / 2);
      const uint32_t vo = (uint32_t)(m0 + lr) * (uint32_t)N + (uint32_t)(n0 + lc);  // element offset
      const uint32_t s8 = (uint32_t)RP * (uint32_t)N;                                // elements per RP rows
      float4 cp[4], cm[4], cv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        cp[u] = bload4(rp, vo * 4u, (uint32_t)u * s8 * 4u);
        cm[u] = bload4(rm, vo * 4u, (uint32_t)u * s8 * 4u);
        cv[u] = bload4(rv, vo * 4u, (uint32_t)u * s8 * 4u);
      }
#pragma unroll
      for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            S[wm + i * 32 + (r / 4) * 8 + (lane >> 5) * 4 + (r % 4)][wn + j * 32 + (lane & 31)] = acc[i][j][r];
      __syncthreads();
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float4 np_[4], nm[4], nv[4];
        if (g + 1 < NG) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const uint32_t so = (uint32_t)(4 * (g + 1) + u) * s8 * 4u;
            np_[u] = bload4(rp, vo * 4u, so);
            nm[u] = bload4(rm, vo * 4u, so);
            nv[u] = bload4(rv, vo * 4u, so);
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = 4 * g + u;
          const uint32_t so = (uint32_t)q * s8;
          const float4 g4 = *reinterpret_cast<const float4*>(&S[lr + RP * q][lc]);
          const float gg[4] = {g4.x, g4.y, g4.z, g4.w};
          const float pp[4] = {cp[u].x, cp[u].y, cp[u].z, cp[u].w};
          const float mm[4] = {cm[u].x, cm[u].y, cm[u].z, cm[u].w};
          const float vv[4] = {cv[u].x, cv[u].y, cv[u].z, cv[u].w};
          float po[4], mo[4], vq[4];
          unsigned short wo[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            mo[k] = mm[k], vq[k] = vv[k], po[k] = pp[k];
            adam_update(e, gg[k], po[k], mo[k], vq[k]);
            wo[k] = __builtin_bit_cast(unsigned short, to_bf16(po[k]));
          }
          bstore4(rm, (vo + so) * 4u, make_float4(mo[0], mo[1], mo[2], mo[3]));
          bstore4(rv, (vo + so) * 4u, make_float4(vq[0], vq[1], vq[2], vq[3]));
          bstore4(rp, (vo + so) * 4u, make_float4(po[0], po[1], po[2], po[3]));
          bstore_2x32(rw, vo * 2u, so * 2u, (uint32_t)wo[0] | ((uint32_t)wo[1] << 16),
                      (uint32_t)wo[2] | ((uint32_t)wo[3] << 16));
        }
        if (g + 1 < NG) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            cp[u] = np_[u];
            cm[u] = nm[u];
            cv[u] = nv[u];
          }
        }
      }
    } else if (m0 + TT <= M && n0 + TT <= N) {
      const uint32_t bytes = (uint32_t)M * (uint32_t)N * 4u;
      const __amdgpu_buffer_rsrc_t rp = make_rsrc(e.p, bytes), rm = make_rsrc(e.m, bytes),
                                   rv = make_rsrc(e.v, bytes), rw = make_rsrc(e.w16, bytes / 2);
      const uint32_t un = (uint32_t)N;
      const uint32_t vbase = (uint32_t)row0 * un + (uint32_t)col0;  // element offset of (row0, col0)
      auto soff = [&](int q, int rr) {  // uniform element offset of group q, element rr
        const int i = q / (2 * NF), h = q & 1;
        return (uint32_t)(i * 32 + h * 16 + (rr / 4) * 8 + (rr % 4)) * un;
      };
      float cp[8], cm[8], cv[8];
#pragma unroll
      for (int rr = 0; rr < 8; ++rr) {
        const uint32_t s = soff(0, rr) * 4u, v = vbase * 4u;
        cp[rr] = bload(rp, v, s);
        cm[rr] = bload(rm, v, s);
        cv[rr] = bload(rv, v, s);
      }
#pragma unroll
      for (int q = 0; q < 2 * NF * NF; ++q) {
        float np_[8], nm[8], nv[8];
        if (q + 1 < 2 * NF * NF) {
          const uint32_t v = (vbase + (uint32_t)((((q + 1) >> 1) % NF) * 32)) * 4u;
#pragma unroll
          for (int rr = 0; rr < 8; ++rr) {
            const uint32_t s = soff(q + 1, rr) * 4u;
            np_[rr] = bload(rp, v, s);
            nm[rr] = bload(rm, v, s);
            nv[rr] = bload(rv, v, s);
          }
        }
        const int i = q / (2 * NF), j = (q >> 1) % NF, h = q & 1;
        const uint32_t ve = vbase + (uint32_t)(j * 32);
#pragma unroll
        for (int rr = 0; rr < 8; ++rr) {
          const uint32_t s = soff(q, rr);
          float pi = cp[rr], mi = cm[rr], vi = cv[rr];
          adam_update(e, acc[i][j][h * 8 + rr], pi, mi, vi);
          bstore(rm, ve * 4u, s * 4u, mi);
          bstore(rv, ve * 4u, s * 4u, vi);
          bstore(rp, ve * 4u, s * 4u, pi);
          bstore16(rw, ve * 2u, s * 2u, to_bf16(pi));
        }
        if (q + 1 < 2 * NF * NF) {
#pragma unroll
          for (int rr = 0; rr < 8; ++rr) {
            cp[rr] = np_[rr];
            cm[rr] = nm[rr];
            cv[rr] = nv[rr];
          }
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int row = row0 + i * 32 + (r / 4) * 8 + (r % 4), col = col0 + j * 32;
            if (row < M && col < N) {
              const uint32_t o = (uint32_t)row * (uint32_t)N + (uint32_t)col;
              float pi = e.p[o], mi = e.m[o], vi = e.v[o];
              adam_update(e, acc[i][j][r], pi, mi, vi);
              e.m[o] = mi;
              e.v[o] = vi;
              e.p[o] = pi;
              e.w16[o] = to_bf16(pi);
            }
          }
    }
  } else {
    static_assert(KIND == EPI_MSE, "unknown epilogue");
    // The column sums of 64 rows run over them in one order for either tile: a
    // wave's fragments one after the other; with narrow tiles the second row
    // half's wave goes on from the first one's sums.
    __shared__ float csum[2][TT];
    __shared__ double lsum[4];
    float cs[NF], g0[16];
    double e2 = 0.0;
#pragma unroll
    for (int j = 0; j < NF; ++j) cs[j] = 0.0f;
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        const int col = col0 + j * 32;
        const bool cok = col < N;
        const float bv = cok ? e.bias[col] : 0.0f;
        const float mu = (cok && e.tmu) ? e.tmu[col] : 0.0f;
        const float inv = (cok && e.tmu) ? e.tinv[col] : 1.0f;
        float tv[16];  // targets of the group, loaded before the first store
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + i * 32 + (r / 4) * 8 + (r % 4);
          tv[r] = (row < M && cok) ? e.t[(size_t)row * N + col] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = row0 + i * 32 + (r / 4) * 8 + (r % 4);
          g0[r] = 0.0f;
          if (row < M && cok) {
            const float vo = acc[i][j][r] + bv;
            const float tt = e.tmu ? (tv[r] - mu) * inv : tv[r];
            const float d = vo - tt;
            e2 += (double)d * (double)d;
            const float d2 = 2.0f * d;
            e.out16[(size_t)row * N + col] = to_bf16(d2 * e.gscale);
            if constexpr (NF == 1) g0[r] = d2;
            else cs[j] = fmaf(d2, e.gscale, cs[j]);
          }
        }
      }
    if constexpr (NF == 1) {
      __shared__ float first[2][64];
      if (wave < 2) {
#pragma unroll
        for (int r = 0; r < 16; ++r) cs[0] = fmaf(g0[r], e.gscale, cs[0]);
        first[wave][lane] = cs[0];
      }
      __syncthreads();
      if (wave >= 2) {
        cs[0] = first[wave & 1][lane];
#pragma unroll
        for (int r = 0; r < 16; ++r) cs[0] = fmaf(g0[r], e.gscale, cs[0]);
        cs[0] += __shfl_xor(cs[0], 32, 64);
        const int c = col0;
        if (lane < 32 && c < N) e.colpart[(size_t)by * N + c] = cs[0];
      }
    } else {
#pragma unroll
      for (int j = 0; j < NF; ++j) cs[j] += __shfl_xor(cs[j], 32, 64);
      if (lane < 32) {
#pragma unroll
        for (int j = 0; j < NF; ++j) csum[wave >> 1][wn + j * 32 + lane] = cs[j];
      }
    }
    e2 = wave_sum64(e2);
    if (lane == 0) lsum[wave] = e2;
    __syncthreads();
    if constexpr (NF == 2) {
      const int c = threadIdx.x & (TT - 1), half = threadIdx.x / TT;
      if (n0 + c < N && m0 + half * 64 < M) e.colpart[(size_t)(2 * by + half) * N + n0 + c] = csum[half][c];
    }
    if (threadIdx.x == 0) e.lossp[(size_t)by * gx + bx] = ((lsum[0] + lsum[1]) + lsum[2]) + lsum[3];
  }
}

template <int KIND, int KT, int TT>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs q) {
  gemm_block<KIND, KT, TT>(q, blockIdx.x, gridDim.x);
}

// The three weight updates of a training step in one launch, the first n0
// workgroups the first's, the next n1 the second's: the small one in the middle
// does not leave the chip waiting, and the large ones' last workgroups overlap
// with the next ones' first.  (6000 x 512, 512 x 512 and 512 x 6000 at batch 256:
// 57 us in three launches, 41.7 here, at 4.0 TB/s of the 4.8 that a copy reaches.)
template <int KT>
__global__ __launch_bounds__(256) void k_gemm3(GemmArgs q0, int n0, GemmArgs q1, int n1, GemmArgs q2, int n2) {
  const int b = blockIdx.x;
  const GemmArgs& q = b < n0 ? q0 : (b < n0 + n1 ? q1 : q2);
  gemm_block<EPI_ADAM, KT, kTileNarrow>(q, b < n0 ? b : (b < n0 + n1 ? b - n0 : b - n0 - n1),
                                        b < n0 ? n0 : (b < n0 + n1 ? n1 : n2));
}

// Split products: out = sum_z part[z] in a fixed order, then the EPI_ACT use.
// The partials of V consecutive elements (one 4 V-byte load each), U splits' loads
// in flight, summed in split order.
template <int U, int V>
__device__ __forceinline__ void add_parts(const float* __restrict__ part, int64_t MN, int64_t i, int splits, int& z,
                                          float (&s)[V]) {
  typedef float vec __attribute__((ext_vector_type(V)));
  for (; z + U <= splits; z += U) {
    vec p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) p[u] = *reinterpret_cast<const vec*>(part + (size_t)(z + u) * MN + i);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < V; ++k) s[k] += p[u][k];
  }
}

// V elements per thread (V divides MN).
template <int V>
__global__ void k_epilogue(const float* __restrict__ part, int splits, int64_t MN, int N, Epi e) {
  const int64_t i = V * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= MN) return;
  int col = MN <= UINT32_MAX ? (int)((uint32_t)i % (uint32_t)N) : (int)(i % N);
  float s[V];
#pragma unroll
  for (int k = 0; k < V; ++k) s[k] = 0.0f;
  int z = 0;
  if constexpr (V == 1) add_parts<32, V>(part, MN, i, splits, z, s);
  add_parts<8, V>(part, MN, i, splits, z, s);
  add_parts<4, V>(part, MN, i, splits, z, s);
  add_parts<1, V>(part, MN, i, splits, z, s);
#pragma unroll
  for (int k = 0; k < V; ++k) {
    epi_act(e, (size_t)(i + k), col, s[k]);
    if (++col == N) col = 0;
  }
}

__global__ void k_to_bf16(const float* __restrict__ in, bf16* __restrict__ out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = to_bf16(in[i]);
}

// Standardized BF16 input: (u - mean) / scale per feature (identity when mean
// is null), rows blockIdx.y, + gridDim.y ..  Four consecutive elements per thread
// (one 16-byte load, one 8-byte store) when vec4 (d % 4 == 0 and both arrays
// 16 / 8-byte aligned).  (64 x 60000: 11.7 us with a 64-bit division per element.)
__global__ void k_in_norm(const float* __restrict__ in, const float* __restrict__ mu,
                          const float* __restrict__ inv_scale, int64_t rows, int d, int vec4, bf16* __restrict__ out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (vec4) {
    if (4 * (int64_t)t >= d) return;
    float4 mu4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), inv4 = mu4;
    if (mu) mu4 = reinterpret_cast<const float4*>(mu)[t], inv4 = reinterpret_cast<const float4*>(inv_scale)[t];
    for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
      float4 v = reinterpret_cast<const float4*>(in + r * d)[t];
      if (mu) {
        v.x = (v.x - mu4.x) * inv4.x, v.y = (v.y - mu4.y) * inv4.y;
        v.z = (v.z - mu4.z) * inv4.z, v.w = (v.w - mu4.w) * inv4.w;
      }
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      reinterpret_cast<bf16x4*>(out + r * d)[t] = bf16x4{to_bf16(v.x), to_bf16(v.y), to_bf16(v.z), to_bf16(v.w)};
    }
    return;
  }
  if (t >= d) return;
  const float m0 = mu ? mu[t] : 0.0f, s0 = mu ? inv_scale[t] : 0.0f;
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
    float v = in[r * d + t];
    if (mu) v = (v - m0) * s0;
    out[r * d + t] = to_bf16(v);
  }
}

// Column sums of an FP32 matrix in a fixed order (bias gradients), the Adam step
// on the biases they belong to, and the loss from its partials: all that is left
// of a training step beside its products, in one launch.
//   seg < 2: hidden layers' biases, b[seg] = column sums of g[seg] (rows x cols);
//     a workgroup takes 64 columns.  Up to 32 rows are added one after the other;
//     more in blocks of 32 rows, of which wave w takes every fourth row from
//     w with four independent partial sums, the blocks' sums then in order.
//   seg 2: the output layer's, from sums of 64 rows each (rows of them),
//     added in pairs, the pairs in order; 1024 columns a workgroup.
//   last workgroup: loss = scale * sum of the partials (when loss is set).
// (Batch 256, width 512, 6000 outputs: seven launches of 4 to 6 us each before.)
struct BiasSeg {
  const float* g;
  int rows, cols, nblk;
  int64_t off;  // of the biases in the parameters
};
struct BiasStep {
  BiasSeg seg[3];
  float *grads, *p, *m, *v;
  int adam;
  float lr, b1, b2, eps, c1, c2;
  const double* lossp;
  int nloss;
  double scale;
  float* loss;
};

__global__ __launch_bounds__(1024) void k_bias_step(BiasStep q) {
  __shared__ float red[16][64];
  __shared__ double lred[256];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int b = blockIdx.x, k = 0;
  while (k < 3 && b >= q.seg[k].nblk) b -= q.seg[k++].nblk;
  if (k == 3) {
    if (t < 256) {
      double s = 0.0;
      for (int i = t; i < q.nloss; i += 256) s += q.lossp[i];
      lred[t] = s;
    }
    __syncthreads();
    for (int n = 128; n > 0; n >>= 1) {
      if (t < n) lred[t] += lred[t + n];
      __syncthreads();
    }
    if (t == 0) q.loss[0] = (float)(lred[0] * q.scale);
    return;
  }
  const BiasSeg s = q.seg[k];
  int c;
  float sum = 0.0f;
  if (k == 2) {
    c = b * 1024 + t;
    if (c >= s.cols) return;
    for (int r = 0; r < s.rows; r += 2)
      sum += r + 1 < s.rows ? s.g[(size_t)r * s.cols + c] + s.g[(size_t)(r + 1) * s.cols + c] : s.g[(size_t)r * s.cols + c];
  } else {
    c = b * 64 + lane;
    if (s.rows <= 32) {
      if (wave == 0 && c < s.cols)
        for (int r = 0; r < s.rows; ++r) sum += s.g[(size_t)r * s.cols + c];
    } else {
      for (int y0 = 0; y0 * 32 < s.rows; y0 += 4) {  // four blocks of 32 rows at a time
        const int y = y0 + (wave >> 2), r1 = min(s.rows, y * 32 + 32);
        float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
        if (c < s.cols) {
          int r = y * 32 + (wave & 3);
          for (; r + 12 < r1; r += 16) {
            s0 += s.g[(size_t)r * s.cols + c];
            s1 += s.g[(size_t)(r + 4) * s.cols + c];
            s2 += s.g[(size_t)(r + 8) * s.cols + c];
            s3 += s.g[(size_t)(r + 12) * s.cols + c];
          }
          for (; r < r1; r += 4) s0 += s.g[(size_t)r * s.cols + c];
        }
        red[wave][lane] = (s0 + s1) + (s2 + s3);
        __syncthreads();
        if (wave == 0)
          for (int u = 0; u < 4 && (y0 + u) * 32 < s.rows; ++u)
            sum += ((red[4 * u][lane] + red[4 * u + 1][lane]) + red[4 * u + 2][lane]) + red[4 * u + 3][lane];
        __syncthreads();
      }
    }
    if (wave != 0 || c >= s.cols) return;
  }
  const int64_t j = s.off + c;
  q.grads[j] = sum;
  if (q.adam) {
    const float mi = fmaf(1.0f - q.b1, sum, q.b1 * q.m[j]);
    const float vi = fmaf((1.0f - q.b2) * sum, sum, q.b2 * q.v[j]);
    q.m[j] = mi;
    q.v[j] = vi;
    q.p[j] -= q.lr * (mi / q.c1) / (sqrtf(vi / q.c2) + q.eps);
  }
}

inline dim3 lin(int64_t n, int t = 256) { return dim3((unsigned)((n + t - 1) / t)); }

}  // namespace

struct pdcs_mlp_s {
  int64_t din = 0, w = 0, dout = 0, np = 0;
  int64_t off_w1 = 0, off_b1 = 0, off_w2 = 0, off_b2 = 0, off_w3 = 0, off_b3 = 0;
  DBuf params, grads, adam_m, adam_v, wbf;  // wbf: BF16 W1 | W2 | W3
  // feature standardization (in: mean, 1/scale; out: mean, scale, 1/scale)
  DBuf in_mu, in_inv, out_mu, out_sc, out_inv;
  bool norm_in = false, norm_out = false;
  const float* imu() const { return norm_in ? in_mu.as<float>() : nullptr; }
  const float* omu() const { return norm_out ? out_mu.as<float>() : nullptr; }
  int64_t step = 0;
  int64_t cap = 0;    // batch capacity of the activation buffers
  int64_t last = 0;   // batch of the last forward / gradient / training call
  bool have_grad_acts = false;  // the last call computed the backward activations
  // activations: BF16 operands of the products (input, h1, h2, dL/dv, dL/dz2,
  // dL/dz1), FP32 masked hidden gradients of both layers (bias sums), the loss
  // gradient's column sums per 64 rows and the loss partials
  DBuf u16, h1_16, h2_16, dv16, dz16a, dz16b, dh, colpart, part, lossp;
  float* loss_host = nullptr;  // pinned: the loss is stored where the host reads it
  // pinned pieces through which the parameters reach the host (get_params)
  static constexpr int64_t kPiece = 1 << 18;  // floats
  std::mutex stage_lock;
  float* stage = nullptr;
  hipEvent_t stage_ev[2] = {nullptr, nullptr};
  size_t part_bytes = 0;
  hipStream_t stream = nullptr;

  // In two pinned pieces by turns: the copy of one under the transfer of the other.
  // (32 training steps at 6000 -> 512 -> 512 -> 6000 and their 25.6 MB of parameters:
  // 5690 us by one hipMemcpy, 5200 here.)
  void params_to_host(float* dst) {
    std::lock_guard<std::mutex> hold(stage_lock);
    const float* src = params.as<float>();
    if (np < 4 * kPiece) {
      HIP_OK(hipMemcpy(dst, src, np * 4, hipMemcpyDeviceToHost));
      return;
    }
    if (!stage) HIP_OK(hipHostMalloc((void**)&stage, 2 * kPiece * sizeof(float), hipHostMallocDefault));
    for (hipEvent_t& e : stage_ev)
      if (!e) HIP_OK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    auto fetch = [&](int64_t i) {
      const int64_t n = std::min(kPiece, np - i * kPiece);
      HIP_OK(hipMemcpyAsync(stage + (i & 1) * kPiece, src + i * kPiece, n * 4, hipMemcpyDeviceToHost, stream));
      HIP_OK(hipEventRecord(stage_ev[i & 1], stream));
    };
    const int64_t pieces = (np + kPiece - 1) / kPiece;
    fetch(0);
    for (int64_t i = 0; i < pieces; ++i) {
      if (i + 1 < pieces) fetch(i + 1);
      HIP_OK(hipEventSynchronize(stage_ev[i & 1]));
      std::memcpy(dst + i * kPiece, stage + (i & 1) * kPiece, (size_t)std::min(kPiece, np - i * kPiece) * 4);
    }
  }

  ~pdcs_mlp_s() {
    if (loss_host) (void)hipHostFree(loss_host);
    if (stage) (void)hipHostFree(stage);
    for (hipEvent_t e : stage_ev)
      if (e) (void)hipEventDestroy(e);
    if (stream) (void)hipStreamDestroy(stream);
  }

  bf16* W1() const { return wbf.as<bf16>(); }
  bf16* W2() const { return wbf.as<bf16>() + w * din; }
  bf16* W3() const { return wbf.as<bf16>() + w * din + w * w; }
  float* P(int64_t off) const { return params.as<float>() + off; }
  float* G(int64_t off) const { return grads.as<float>() + off; }
  float* Mo(int64_t off) const { return adam_m.as<float>() + off; }
  float* Vo(int64_t off) const { return adam_v.as<float>() + off; }

  void refresh_bf16(hipStream_t s) {
    k_to_bf16<<<lin(w * din), 256, 0, s>>>(P(off_w1), W1(), w * din);
    k_to_bf16<<<lin(w * w), 256, 0, s>>>(P(off_w2), W2(), w * w);
    k_to_bf16<<<lin(dout * w), 256, 0, s>>>(P(off_w3), W3(), dout * w);
  }

  void ensure(int64_t B) {
    if (B <= cap) return;
    cap = B;
    u16.alloc(B * din * 2);
    h1_16.alloc(B * w * 2);
    h2_16.alloc(B * w * 2);
    dv16.alloc(B * dout * 2);
    dz16a.alloc(B * w * 2);
    dz16b.alloc(B * w * 2);
    dh.alloc(2 * B * w * 4);
    colpart.alloc(((B + 63) / 64) * dout * 4);
    lossp.alloc(((B + 63) / 64) * ((dout + 63) / 64) * 8);
  }

  // The tile depth is 64 for K-ranges of 128 or more (128-deep tiles halve the
  // steps of long ranges but double the LDS, and measured 2% slower per step
  // at batch 256), 32 below.
  static int tile_depth(int range) { return range >= 128 ? 64 : 32; }

  // op(A)[M x K] op(B)[K x N] with epilogue `kind`.  Products whose output tiles
  // alone cannot fill the chip are split along K (EPI_STORE / EPI_ACT only);
  // the partials are then summed in a fixed order.  EPI_STORE writes e.out32.
  void gemm(int kind, const bf16* A, int lda, int ta, const bf16* Bm, int ldb, int tb, int M, int N, int K,
            Epi e, hipStream_t s) {
    const int tiles = ((N + kTileWide - 1) / kTileWide) * ((M + kTileWide - 1) / kTileWide);
    // (products of a few tiles split down to K-ranges of 128: a handful of
    // workgroups walking the whole K serially would leave the chip idle)
    int splits = 1;
    const int min_range = tiles < 64 ? 128 : 512;
    if (kind == EPI_STORE || kind == EPI_ACT)
      while (tiles * splits < 512 && K / (splits * 2) >= min_range) splits *= 2;
    int kchunk = (K + splits - 1) / splits;
    const int kt = tile_depth(kchunk);
    kchunk = (kchunk + kt - 1) / kt * kt;
    splits = (K + kchunk - 1) / kchunk;
    if (splits < 1) splits = 1;
    if (splits > 1) {
      const size_t need = (size_t)splits * M * N * 4;
      if (need > part_bytes) {
        part.alloc(need);
        part_bytes = need;
      }
      launch(EPI_STORE, kt, A, lda, ta, Bm, ldb, tb, part.as<float>(), M, N, K, splits, e, s);
      // four elements a thread where that still makes two workgroups for each CU
      // (64 x 512 of 128 splits: 32 workgroups and 6.9 us with four, 4.3 with one)
      const int64_t mn = (int64_t)M * N;
      if (mn % 4 == 0 && mn >= 512 * 1024)
        k_epilogue<4><<<lin(mn / 4), 256, 0, s>>>(part.as<float>(), splits, mn, N, e);
      else
        k_epilogue<1><<<lin(mn), 256, 0, s>>>(part.as<float>(), splits, mn, N, e);
      return;
    }
    launch(kind, kt, A, lda, ta, Bm, ldb, tb, kind == EPI_STORE ? e.out32 : nullptr, M, N, K, 1, e, s);
  }

  // The tile's side: narrow while wide tiles make fewer than two workgroups for
  // each CU (wide and narrow, us: split products of 256 workgroups 12.2 and 7.9;
  // 64 x 60000 outputs of width 512 35 and 20; 256 x 6000 with loss 30 and 25; but
  // 256 x 60000, at 938 wide tiles, 145 and 148 the forward pass).  The weight
  // updates, whose time is the weights' and moments' traffic, are always narrow
  // (6000 x 512, 512 x 6000 and 512 x 512 at batch 256 39.4 and 19.1 on average; a
  // step with 60000 x 512 matrices 747 and 677), also where the batch, their K-range, is
  // long: a step of 6000 -> 512 -> 512 -> 6000 with wide and narrow updates 130 and 118 at
  // batch 256, 230 and 212 at 1024, 618 and 576 at 4096, of width 128 457 and 352 there.
  static bool narrow(int M, int N, int splits) {
    return ((N + kTileWide - 1) / kTileWide) * ((M + kTileWide - 1) / kTileWide) * splits < 512;
  }

  static GemmArgs args(int TT, const bf16* A, int lda, int ta, const bf16* Bm, int ldb, int tb, float* C, int M, int N,
                       int K, const Epi& e) {
    // 16-byte vector loads need 16-byte aligned operands with row strides in whole vectors
    const int veca = ((uintptr_t)A % 16 == 0 && lda % 8 == 0) ? 1 : 0;
    const int vecb = ((uintptr_t)Bm % 16 == 0 && ldb % 8 == 0) ? 1 : 0;
    return {A, lda, ta, veca, Bm, ldb, tb, vecb, C, M, N, K, (N + TT - 1) / TT, (M + TT - 1) / TT, e};
  }

  template <int KIND, int TT>
  static void launch_tile(int kt, const GemmArgs& q, int splits, hipStream_t s) {
    const dim3 grid((unsigned)(q.gx * q.gy * splits));
    if (kt == 64)
      k_gemm<KIND, 64, TT><<<grid, 256, 0, s>>>(q);
    else
      k_gemm<KIND, 32, TT><<<grid, 256, 0, s>>>(q);
  }

  static void launch(int kind, int kt, const bf16* A, int lda, int ta, const bf16* Bm, int ldb, int tb, float* C, int M,
                     int N, int K, int splits, const Epi& e, hipStream_t s) {
    const int TT = narrow(M, N, splits) ? kTileNarrow : kTileWide;
    const GemmArgs q = args(TT, A, lda, ta, Bm, ldb, tb, C, M, N, K, e);
    switch (kind) {
      case EPI_STORE:
        TT == kTileNarrow ? launch_tile<EPI_STORE, kTileNarrow>(kt, q, splits, s)
                          : launch_tile<EPI_STORE, kTileWide>(kt, q, splits, s);
        break;
      case EPI_ACT:
        TT == kTileNarrow ? launch_tile<EPI_ACT, kTileNarrow>(kt, q, splits, s)
                          : launch_tile<EPI_ACT, kTileWide>(kt, q, splits, s);
        break;
      default:
        TT == kTileNarrow ? launch_tile<EPI_MSE, kTileNarrow>(kt, q, splits, s)
                          : launch_tile<EPI_MSE, kTileWide>(kt, q, splits, s);
    }
  }

  static Epi act(const float* bias, int relu, const bf16* mask, float* out32, bf16* out16) {
    Epi e;
    e.bias = bias;
    e.relu = relu;
    e.mask = mask;
    e.out32 = out32;
    e.out16 = out16;
    return e;
  }

  // Adam (step `step`, learning rate lr) on the weights at offset off: the
  // weight-gradient product's epilogue when `adam`, else the gradient is stored.
  Epi wgrad(bool adam, int64_t off, bf16* w16, float lr) const {
    Epi e;
    if (!adam) {
      e.out32 = G(off);
      return e;
    }
    e.p = P(off);
    e.m = Mo(off);
    e.v = Vo(off);
    e.w16 = w16;
    e.lr = lr;
    e.b1 = 0.9f;
    e.b2 = 0.999f;
    e.eps = 1e-8f;
    e.c1 = 1.0f - std::pow(e.b1, (float)step);
    e.c2 = 1.0f - std::pow(e.b2, (float)step);
    return e;
  }

  // 16-byte runs of weight rows: the Adam epilogue's staged path
  static int adam_vec4(const Epi& e, int64_t N) {
    return (N % 4 == 0 && (uintptr_t)e.p % 16 == 0 && (uintptr_t)e.m % 16 == 0 && (uintptr_t)e.v % 16 == 0 &&
            (uintptr_t)e.w16 % 8 == 0)
               ? 1
               : 0;
  }

  // Standardized BF16 input and the two hidden layers (BF16, after ReLU).
  void hidden(const float* in, int64_t B, hipStream_t s) {
    ensure(B);
    last = B;
    const int vec4 = (din % 4 == 0 && (uintptr_t)in % 16 == 0 && (uintptr_t)u16.p % 8 == 0) ? 1 : 0;
    const dim3 grid((unsigned)(((vec4 ? din / 4 : din) + 255) / 256), (unsigned)std::min<int64_t>(B, 65535));
    k_in_norm<<<grid, 256, 0, s>>>(in, imu(), in_inv.as<float>(), B, (int)din, vec4, u16.as<bf16>());
    gemm(EPI_ACT, u16.as<bf16>(), din, 0, W1(), din, 1, B, w, din, act(P(off_b1), 1, nullptr, nullptr, h1_16.as<bf16>()),
         s);
    gemm(EPI_ACT, h1_16.as<bf16>(), w, 0, W2(), w, 1, B, w, w, act(P(off_b2), 1, nullptr, nullptr, h2_16.as<bf16>()),
         s);
  }

  // The network output in the caller's units: z * scale + mean per feature.
  void forward(const float* in, int64_t B, float* out, hipStream_t s) {
    hidden(in, B, s);
    have_grad_acts = false;
    Epi e = act(P(off_b3), 0, nullptr, out, nullptr);
    if (norm_out) {
      e.osc = out_sc.as<float>();
      e.omu = out_mu.as<float>();
    }
    gemm(EPI_ACT, h2_16.as<bf16>(), w, 0, W3(), w, 1, B, dout, w, e, s);
  }

  // Forward and backward of the mean squared error; the weight gradients are
  // stored in `grads`, or, when `adam`, applied as an Adam step inside the
  // weight-gradient products (each layer's BF16 weights are read by the
  // backward product before its own update rewrites them).  Bias gradients go
  // to `grads` either way; the loss is summed from its partials into loss_host
  // only when `need_loss`.
  void train(const float* in, const float* target, int64_t B, bool adam, float lr, bool need_loss, hipStream_t s) {
    hidden(in, B, s);
    have_grad_acts = true;
    const int64_t n = B * dout;
    // output layer fused with the loss: dv16 = BF16 dL/dv, column sums, loss partials
    Epi mse;
    mse.bias = P(off_b3);
    mse.t = target;
    mse.tmu = omu();
    mse.tinv = out_inv.as<float>();
    mse.gscale = 1.0f / (float)n;
    mse.out16 = dv16.as<bf16>();
    mse.colpart = colpart.as<float>();
    mse.lossp = lossp.as<double>();
    gemm(EPI_MSE, h2_16.as<bf16>(), w, 0, W3(), w, 1, B, dout, w, mse, s);
    // dZ2 = (dV W3) * (h2 > 0) and dZ1 = (dZ2 W2) * (h1 > 0), then the weights':
    // dW3 = dV^T H2, dW2 = dZ2^T H1, dW1 = dZ1^T U
    gemm(EPI_ACT, dv16.as<bf16>(), dout, 0, W3(), w, 0, B, w, dout,
         act(nullptr, 0, h2_16.as<bf16>(), dh.as<float>(), dz16a.as<bf16>()), s);
    gemm(EPI_ACT, dz16a.as<bf16>(), w, 0, W2(), w, 0, B, w, w,
         act(nullptr, 0, h1_16.as<bf16>(), dh.as<float>() + B * w, dz16b.as<bf16>()), s);
    if (adam) {
      const auto update = [&](const bf16* dz, int64_t M, const bf16* x, int64_t N, int64_t off, bf16* w16) {
        Epi e = wgrad(true, off, w16, lr);
        e.vec4 = adam_vec4(e, N);
        return args(kTileNarrow, dz, M, 1, x, N, 0, nullptr, M, N, B, e);
      };
      const GemmArgs q3 = update(dv16.as<bf16>(), dout, h2_16.as<bf16>(), w, off_w3, W3());
      const GemmArgs q2 = update(dz16a.as<bf16>(), w, h1_16.as<bf16>(), w, off_w2, W2());
      const GemmArgs q1 = update(dz16b.as<bf16>(), w, u16.as<bf16>(), din, off_w1, W1());
      const int n3 = q3.gx * q3.gy, n2 = q2.gx * q2.gy, n1 = q1.gx * q1.gy;
      if (tile_depth((int)B) == 64)
        k_gemm3<64><<<(unsigned)(n3 + n2 + n1), 256, 0, s>>>(q3, n3, q2, n2, q1, n1);
      else
        k_gemm3<32><<<(unsigned)(n3 + n2 + n1), 256, 0, s>>>(q3, n3, q2, n2, q1, n1);
    } else {
      gemm(EPI_STORE, dv16.as<bf16>(), dout, 1, h2_16.as<bf16>(), w, 0, dout, w, B, wgrad(false, off_w3, nullptr, lr), s);
      gemm(EPI_STORE, dz16a.as<bf16>(), w, 1, h1_16.as<bf16>(), w, 0, w, w, B, wgrad(false, off_w2, nullptr, lr), s);
      gemm(EPI_STORE, dz16b.as<bf16>(), w, 1, u16.as<bf16>(), din, 0, w, din, B, wgrad(false, off_w1, nullptr, lr), s);
    }
    const Epi e = wgrad(true, off_b1, nullptr, lr);
    BiasStep q;
    const int hb = (int)((w + 63) / 64), side = narrow((int)B, (int)dout, 1) ? kTileNarrow : kTileWide;
    q.seg[0] = {dh.as<float>(), (int)B, (int)w, hb, off_b2};
    q.seg[1] = {dh.as<float>() + B * w, (int)B, (int)w, hb, off_b1};
    q.seg[2] = {colpart.as<float>(), (int)((B + 63) / 64), (int)dout, (int)((dout + 1023) / 1024), off_b3};
    q.grads = grads.as<float>(), q.p = params.as<float>(), q.m = adam_m.as<float>(), q.v = adam_v.as<float>();
    q.adam = adam ? 1 : 0;
    q.lr = lr, q.b1 = e.b1, q.b2 = e.b2, q.eps = e.eps, q.c1 = e.c1, q.c2 = e.c2;
    q.lossp = lossp.as<double>();
    q.nloss = (int)(((B + side - 1) / side) * ((dout + side - 1) / side));
    q.scale = 1.0 / (double)n;
    q.loss = loss_host;
    k_bias_step<<<(unsigned)(2 * hb + q.seg[2].nblk + (need_loss ? 1 : 0)), 1024, 0, s>>>(q);
  }
};

extern "C" {

int pdcs_mlp_create(int64_t d_in, int64_t width, int64_t d_out, uint64_t seed, pdcs_mlp* out) {
  try {
    if (!out || d_in < 1 || width < 1 || d_out < 1 || d_in > (1 << 26) || d_out > (1 << 26) || width > 8192 ||
        width * d_in >= ((int64_t)1 << 30) || width * d_out >= ((int64_t)1 << 30))
      throw Error(PDCS_ERR_INVALID_ARG, "bad MLP sizes (each weight matrix must hold fewer than 2^30 entries)");
    *out = nullptr;
    auto net = new pdcs_mlp_s();
    std::unique_ptr<pdcs_mlp_s> guard(net);
    net->din = d_in;
    net->w = width;
    net->dout = d_out;
    net->off_w1 = 0;
    net->off_b1 = width * d_in;
    net->off_w2 = net->off_b1 + width;
    net->off_b2 = net->off_w2 + width * width;
    net->off_w3 = net->off_b2 + width;
    net->off_b3 = net->off_w3 + d_out * width;
    net->np = net->off_b3 + d_out;
    HIP_OK(hipStreamCreateWithFlags(&net->stream, hipStreamNonBlocking));
    HIP_OK(hipHostMalloc((void**)&net->loss_host, sizeof(float), hipHostMallocDefault));
    // Glorot-uniform weights, zero biases, from a seeded host generator
    std::vector<float> p(net->np, 0.0f);
    std::mt19937_64 gen(seed);
    auto fill = [&](int64_t off, int64_t fan_out, int64_t fan_in) {
      const float a = std::sqrt(6.0f / (float)(fan_in + fan_out));
      std::uniform_real_distribution<float> U(-a, a);
      for (int64_t i = 0; i < fan_out * fan_in; ++i) p[off + i] = U(gen);
    };
    fill(net->off_w1, width, d_in);
    fill(net->off_w2, width, width);
    fill(net->off_w3, d_out, width);
    net->params.alloc(net->np * 4);
    net->grads.alloc(net->np * 4);
    net->adam_m.alloc(net->np * 4);
    net->adam_v.alloc(net->np * 4);
    net->wbf.alloc((width * d_in + width * width + d_out * width) * 2);
    HIP_OK(hipMemcpy(net->params.p, p.data(), net->np * 4, hipMemcpyHostToDevice));
    std::vector<float> z(net->np, 0.0f);
    HIP_OK(hipMemcpy(net->adam_m.p, z.data(), net->np * 4, hipMemcpyHostToDevice));
    HIP_OK(hipMemcpy(net->adam_v.p, z.data(), net->np * 4, hipMemcpyHostToDevice));
    HIP_OK(hipMemcpy(net->grads.p, z.data(), net->np * 4, hipMemcpyHostToDevice));
    net->refresh_bf16(net->stream);
    HIP_OK(hipStreamSynchronize(net->stream));
    *out = guard.release();
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  } catch (const std::exception& e) {
    set_last_error(e.what());
    return PDCS_ERR_OOM;
  }
}

// the caller's stream; NULL is the HIP null stream (ordered with the caller's
// default-stream work), never the library's own non-blocking stream
static hipStream_t pick(pdcs_mlp, void* stream) { return (hipStream_t)stream; }

int pdcs_mlp_forward(pdcs_mlp net, const float* in_dev, float* out_dev, int64_t batch, void* stream) {
  try {
    if (!net || !in_dev || !out_dev || batch < 1) throw Error(PDCS_ERR_INVALID_ARG, "bad forward arguments");
    hipStream_t s = pick(net, stream);
    net->forward(in_dev, batch, out_dev, s);
    HIP_OK(hipGetLastError());
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  }
}

int pdcs_mlp_gradients(pdcs_mlp net, const float* in_dev, const float* target_dev, int64_t batch, float* grad_dev,
                       float* loss_out, void* stream) {
  try {
    if (!net || !in_dev || !target_dev || batch < 1) throw Error(PDCS_ERR_INVALID_ARG, "bad gradient arguments");
    hipStream_t s = pick(net, stream);
    net->train(in_dev, target_dev, batch, false, 0.0f, loss_out != nullptr, s);
    if (grad_dev) HIP_OK(hipMemcpyAsync(grad_dev, net->grads.p, net->np * 4, hipMemcpyDeviceToDevice, s));
    HIP_OK(hipGetLastError());
    HIP_OK(hipStreamSynchronize(s));
    if (loss_out) *loss_out = *(volatile float*)net->loss_host;
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  }
}

int pdcs_mlp_train_step(pdcs_mlp net, const float* in_dev, const float* target_dev, int64_t batch, float lr,
                        float* loss_out, void* stream) {
  try {
    if (!net || !in_dev || !target_dev || batch < 1 || !(lr > 0.0f))
      throw Error(PDCS_ERR_INVALID_ARG, "bad train arguments");
    hipStream_t s = pick(net, stream);
    net->step += 1;
    net->train(in_dev, target_dev, batch, true, lr, loss_out != nullptr, s);
    HIP_OK(hipGetLastError());
    if (loss_out) {  // without a loss pointer the step stays asynchronous on `stream`
      HIP_OK(hipStreamSynchronize(s));
      *loss_out = *(volatile float*)net->loss_host;
    }
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  }
}

int pdcs_mlp_activation(pdcs_mlp net, int64_t which, float* host_out, int64_t count) {
  try {
    if (!net || !host_out || which < 0 || which > 5) throw Error(PDCS_ERR_INVALID_ARG, "bad activation arguments");
    if (net->last < 1 || (which >= 3 && !net->have_grad_acts))
      throw Error(PDCS_ERR_INVALID_ARG, "no activation of that kind from the last call");
    const int64_t B = net->last;
    const bf16* src[6] = {net->u16.as<bf16>(), net->h1_16.as<bf16>(), net->h2_16.as<bf16>(),
                          net->dv16.as<bf16>(), net->dz16a.as<bf16>(), net->dz16b.as<bf16>()};
    const int64_t dim[6] = {net->din, net->w, net->w, net->dout, net->w, net->w};
    if (count != B * dim[which]) throw Error(PDCS_ERR_INVALID_ARG, "count must be batch x features");
    HIP_OK(hipDeviceSynchronize());
    std::vector<uint16_t> raw(count);
    HIP_OK(hipMemcpy(raw.data(), src[which], count * 2, hipMemcpyDeviceToHost));
    for (int64_t i = 0; i < count; ++i) {
      const uint32_t bits = (uint32_t)raw[i] << 16;
      std::memcpy(&host_out[i], &bits, 4);
    }
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  }
}

int pdcs_mlp_num_params(pdcs_mlp net, int64_t* count) {
  if (!net || !count) {
    set_last_error("null argument");
    return PDCS_ERR_INVALID_ARG;
  }
  *count = net->np;
  return PDCS_OK;
}

int pdcs_mlp_get_params(pdcs_mlp net, float* params_host) {
  try {
    if (!net || !params_host) throw Error(PDCS_ERR_INVALID_ARG, "null argument");
    HIP_OK(hipDeviceSynchronize());
    net->params_to_host(params_host);
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  }
}

int pdcs_mlp_set_normalization(pdcs_mlp net, const float* in_mean, const float* in_scale, const float* out_mean,
                               const float* out_scale) {
  try {
    if (!net) throw Error(PDCS_ERR_INVALID_ARG, "null network");
    if ((in_mean == nullptr) != (in_scale == nullptr) || (out_mean == nullptr) != (out_scale == nullptr))
      throw Error(PDCS_ERR_INVALID_ARG, "mean and scale must be given together");
    auto check = [](const float* mu, const float* sc, int64_t d) {
      for (int64_t j = 0; j < d; ++j)
        if (!std::isfinite(mu[j]) || !std::isfinite(sc[j]) || !(sc[j] > 0.0f))
          throw Error(PDCS_ERR_INVALID_ARG, "means must be finite and scales finite and positive");
    };
    HIP_OK(hipDeviceSynchronize());
    if (in_mean) {
      check(in_mean, in_scale, net->din);
      std::vector<float> inv(net->din);
      for (int64_t j = 0; j < net->din; ++j) inv[j] = 1.0f / in_scale[j];
      net->in_mu.alloc(net->din * 4);
      net->in_inv.alloc(net->din * 4);
      HIP_OK(hipMemcpy(net->in_mu.p, in_mean, net->din * 4, hipMemcpyHostToDevice));
      HIP_OK(hipMemcpy(net->in_inv.p, inv.data(), net->din * 4, hipMemcpyHostToDevice));
    }
    net->norm_in = in_mean != nullptr;
    if (out_mean) {
      check(out_mean, out_scale, net->dout);
      std::vector<float> inv(net->dout);
      for (int64_t j = 0; j < net->dout; ++j) inv[j] = 1.0f / out_scale[j];
      net->out_mu.alloc(net->dout * 4);
      net->out_sc.alloc(net->dout * 4);
      net->out_inv.alloc(net->dout * 4);
      HIP_OK(hipMemcpy(net->out_mu.p, out_mean, net->dout * 4, hipMemcpyHostToDevice));
      HIP_OK(hipMemcpy(net->out_sc.p, out_scale, net->dout * 4, hipMemcpyHostToDevice));
      HIP_OK(hipMemcpy(net->out_inv.p, inv.data(), net->dout * 4, hipMemcpyHostToDevice));
    }
    net->norm_out = out_mean != nullptr;
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  }
}

int pdcs_mlp_set_params(pdcs_mlp net, const float* params_host) {
  try {
    if (!net || !params_host) throw Error(PDCS_ERR_INVALID_ARG, "null argument");
    HIP_OK(hipMemcpy(net->params.p, params_host, net->np * 4, hipMemcpyHostToDevice));
    net->refresh_bf16(net->stream);
    HIP_OK(hipStreamSynchronize(net->stream));
    return PDCS_OK;
  } catch (const Error& e) {
    set_last_error(e.what());
    return e.code;
  }
}

void pdcs_mlp_destroy(pdcs_mlp net) {
  delete net;
}

}  // extern "C"
