// Small MLP for the learned MPC warm start: y = W3 relu(W2 relu(W1 x + b1) +
// b2) + b3, mean-squared-error loss, Adam.  Every matrix product runs on the
// gfx950 matrix cores (v_mfma_f32_16x16x32_bf16): operands rounded to
// bf16 (round to nearest even) on their way into registers, products
// accumulated in fp32.  Master weights, activations and gradients are fp32
// in device memory.  Bias, ReLU, the loss and its gradient, the ReLU mask of
// the backward pass and the Adam step are fused into the products; a
// training step is seven launches.  Reductions (split products, loss, bias
// gradients) use a fixed order, so results are deterministic.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <memory>
#include <mutex>
#include <vector>

#include "internal.h"

namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v8f __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));

// Products C = A B^T by groups of four wavefronts, a 64 x BN tile of C
// each (BN = 64: 2 x 2 wavefronts of 32 x 32; BN = 32: 4 wavefronts of
// 16 x 32), K in chunks of KC through LDS.
constexpr int BM = 64, KC = 128, GT = 256;
constexpr int LROW = KC + 8;   // LDS row: 16-byte aligned, rows four banks apart
constexpr int BSPLIT = 4;      // groups of a backward workgroup, which share K

__host__ __device__ constexpr int tiles(int n, int t) { return n / t + (n % t != 0); }

// A matrix operand in memory: element (i, k) at p[i ld + k], or, K-strided,
// at p[k ld + i].  vec: rows of k are 16-byte aligned.
struct Operand {
  const float* p;
  int ld;
  bool vec;
};
Operand operand(const float* p, int ld) {
  return Operand{p, ld, (reinterpret_cast<uintptr_t>(p) & 15) == 0 && ld % 4 == 0};
}

// One group's part of a chunk of R rows in flight: thread t holds R / 8
// groups of four k.  K in memory order: of the rows t / 32 + 8 j at
// k = 4 (t % 32), so that 32 lanes read 512 bytes in a row.  K-strided: of
// row t % R at the k of its GT / R-th of the chunk, a row of R elements per k.
template <int R>
struct Chunk {
  v4f v[R / 8];
};

// Rows past the end repeat the last one (they only make results that nobody
// stores); k past k1 (at least 1) read in range and become zero.
template <bool KS, int R>
__device__ __forceinline__ void load_chunk(Chunk<R>& c, const Operand& o, int rows, int r0, int kb,
                                           int k1, int t) {
  if constexpr (KS) {
    const int i = min(r0 + t % R, rows - 1), k = kb + t / R * (R / 2);
    if (kb + KC <= k1) {   // uniform
      const float* q = o.p + (int64_t)k * o.ld + i;
#pragma unroll
      for (int j = 0; j < R / 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e, q += o.ld) c.v[j][e] = *q;
    } else {
#pragma unroll
      for (int j = 0; j < R / 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int kk = k + 4 * j + e;
          const float x = o.p[(int64_t)min(kk, k1 - 1) * o.ld + i];
          c.v[j][e] = kk < k1 ? x : 0.f;
        }
    }
  } else {
    const int k = kb + 4 * (t % 32);
    if (o.vec && kb + KC <= k1) {   // uniform
#pragma unroll
      for (int j = 0; j < R / 8; ++j)
        c.v[j] = *(const v4f*)(o.p + (int64_t)min(r0 + t / 32 + 8 * j, rows - 1) * o.ld + k);
    } else if (o.vec && k1 % 4 == 0) {
#pragma unroll
      for (int j = 0; j < R / 8; ++j) {
        const int64_t row = (int64_t)min(r0 + t / 32 + 8 * j, rows - 1) * o.ld;
        const v4f x = *(const v4f*)(o.p + row + min(k, k1 - 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) c.v[j][e] = k < k1 ? x[e] : 0.f;
      }
    } else {
#pragma unroll
      for (int j = 0; j < R / 8; ++j) {
        const int64_t row = (int64_t)min(r0 + t / 32 + 8 * j, rows - 1) * o.ld;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = o.p[row + min(k + e, k1 - 1)];
          c.v[j][e] = k + e < k1 ? x : 0.f;
        }
      }
    }
  }
}

// Rounded to bf16 (to nearest even) into the rows [row][k] of LDS.
template <bool KS, int R>
__device__ __forceinline__ void store_chunk(const Chunk<R>& c, __bf16 (*s)[LROW], int t) {
  if constexpr (KS) {
#pragma unroll
    for (int j = 0; j < R / 16; ++j) {
      v8f v;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = c.v[2 * j + e / 4][e % 4];
      *(v8bf*)&s[t % R][t / R * (R / 2) + 8 * j] = __builtin_convertvector(v, v8bf);
    }
  } else {
#pragma unroll
    for (int j = 0; j < R / 8; ++j)
      *(v4bf*)&s[t / 32 + 8 * j][4 * (t % 32)] = __builtin_convertvector(c.v[j], v4bf);
  }
}

// (rows are written and read as vectors of 8 and 16 bytes)
template <int BN>
struct GroupSmem {
  alignas(16) __bf16 a[BM][LROW];
  alignas(16) __bf16 b[BN][LROW];
};
static_assert(LROW * sizeof(__bf16) % 16 == 0 && alignof(GroupSmem<32>) % 16 == 0,
              "rows of operands are 16-byte aligned");

template <int BN>
struct Tile {
  static constexpr int MI = BN / 32;   // MFMA tiles of a wavefront: MI x 2
  v4f acc[MI][2];
  // row and column in the 64 x BN tile of element q of MFMA tile (i, j)
  static __device__ __forceinline__ int row0() {
    const int w = (threadIdx.x >> 6) & 3;
    return BN == 64 ? (w >> 1) * 32 : w * 16;
  }
  static __device__ __forceinline__ int col0() {
    const int w = (threadIdx.x >> 6) & 3;
    return BN == 64 ? (w & 1) * 32 : 0;
  }
  static __device__ __forceinline__ int row(int i, int q) {
    return row0() + 16 * i + ((threadIdx.x >> 4) & 3) * 4 + q;
  }
  static __device__ __forceinline__ int col(int j) { return col0() + 16 * j + (threadIdx.x & 15); }
};

// The group's tile over k in [k0, k1), k ascending in steps of 32 (one
// v_mfma_f32_16x16x32_bf16 per 16 x 16 tile and step, fp32 accumulation).
// Every group of the workgroup calls this with the same number of chunks.
// The next chunk is on its way while the current one is multiplied.  asum
// (if SUM, A K-strided): this thread's part of its row's sum over k of A
// before rounding.
template <bool AKS, bool BKS, bool SUM, int BN>
__device__ __forceinline__ void group_product(const Operand& A, int M, const Operand& B, int N,
                                              int m0, int n0, int k0, int k1, int chunks,
                                              GroupSmem<BN>& sm, Tile<BN>& tile, float& asum) {
  const int t = threadIdx.x % GT, lane = t & 63;
#pragma unroll
  for (int i = 0; i < Tile<BN>::MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) tile.acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  asum = 0.f;
  Chunk<BM> ca;
  Chunk<BN> cb;
  load_chunk<AKS>(ca, A, M, m0, k0, k1, t);
  load_chunk<BKS>(cb, B, N, n0, k0, k1, t);
  for (int c = 0; c < chunks; ++c) {
    const int kb = k0 + c * KC;
    if (c > 0) __syncthreads();
    if constexpr (SUM) {
#pragma unroll
      for (int j = 0; j < BM / 8; ++j) asum += (ca.v[j][0] + ca.v[j][1]) + (ca.v[j][2] + ca.v[j][3]);
    }
    store_chunk<AKS>(ca, sm.a, t);
    store_chunk<BKS>(cb, sm.b, t);
    __syncthreads();
    if (c + 1 < chunks) {
      load_chunk<AKS>(ca, A, M, m0, kb + KC, k1, t);
      load_chunk<BKS>(cb, B, N, n0, kb + KC, k1, t);
    }
    const int steps = min(KC, k1 - kb);
#pragma unroll
    for (int kk = 0; kk < KC; kk += 32) {
      if (kk >= steps) break;   // uniform over the group
      v8bf fa[Tile<BN>::MI], fb[2];
#pragma unroll
      for (int i = 0; i < Tile<BN>::MI; ++i)
        fa[i] = *(const v8bf*)&sm.a[Tile<BN>::row0() + 16 * i + (lane & 15)][kk + 8 * (lane >> 4)];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        fb[j] = *(const v8bf*)&sm.b[Tile<BN>::col0() + 16 * j + (lane & 15)][kk + 8 * (lane >> 4)];
#pragma unroll
      for (int i = 0; i < Tile<BN>::MI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          tile.acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], tile.acc[i][j], 0, 0, 0);
    }
  }
}

// Layers of the forward pass: C = A B^T + bias, A [M][K], B [N][K], then
//   RELU    C = max(C, 0)
//   AFFINE  C = mu + sd C
//   LOSS    on normalised outputs: with th = (target - mu) / sd per column,
//           C = 2 (yh - th) scale, and per workgroup the sum of (yh - th)^2
// One group per tile (LN columns: layer_tile, loss_tile) with all of K (the order of its sums decides how the
// next layer's operands round).  What bounds it: a chunk's memory round trip
// (the operands are what other XCDs have just written) and the launch; a
// 64-wide tile, with half as many wavefronts, took 16.2 us for the loss
// layer.  Batch 2048: 256 -> 256 5.1 us (10.7 with 16-bit LDS accesses and
// the same tile in one wavefront each), 256 -> 1100 with the loss 13.4 us
// (31.9 in three launches).
enum Epi : int { EPI_RELU = 0, EPI_AFFINE = 1, EPI_LOSS = 2 };

template <int EPI, int LN>
__global__ __launch_bounds__(GT) void layer_kernel(int M, int N, int K, Operand A, Operand B,
                                                   const float* __restrict__ bias,
                                                   float* __restrict__ C,
                                                   const float* __restrict__ mu,
                                                   const float* __restrict__ sd,
                                                   const float* __restrict__ target, float scale,
                                                   float* __restrict__ part) {
  __shared__ GroupSmem<LN> sm;
  using TL = Tile<LN>;
  const int gm = tiles(M, BM);
  const int m0 = (int)blockIdx.x % gm * BM, n0 = (int)blockIdx.x / gm * LN;
  v4f tg[TL::MI][2];
  if constexpr (EPI == EPI_LOSS) {
    // read ahead of the product (clamped; what lies outside is not used)
#pragma unroll
    for (int i = 0; i < TL::MI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          tg[i][j][q] = target[(int64_t)min(m0 + TL::row(i, q), M - 1) * N + min(n0 + TL::col(j), N - 1)];
  }
  TL tile;
  float asum, loss = 0.f;
  group_product<false, false, false>(A, M, B, N, m0, n0, 0, K, tiles(K, KC), sm, tile, asum);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = n0 + TL::col(j);
    if (col >= N) continue;
    const float bc = bias[col];
    float mc = 0.f, sc = 1.f;
    if (EPI != EPI_RELU) {
      mc = mu[col];
      sc = sd[col];
    }
#pragma unroll
    for (int i = 0; i < TL::MI; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = m0 + TL::row(i, q);
        if (row >= M) continue;
        const int64_t at = (int64_t)row * N + col;
        float v = tile.acc[i][j][q] + bc;
        if (EPI == EPI_RELU) v = v > 0.f ? v : 0.f;
        if (EPI == EPI_AFFINE) v = mc + sc * v;
        if (EPI == EPI_LOSS) {
          const float d = v - (tg[i][j][q] - mc) / sc;
          loss += d * d;
          v = 2.f * d * scale;
        }
        C[at] = v;
      }
  }
  if constexpr (EPI == EPI_LOSS) {
    __shared__ float red[GT / 64];
    const float s = admmi::wave_sum(loss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      float t = red[0];
#pragma unroll
      for (int q = 1; q < GT / 64; ++q) t += red[q];
      part[blockIdx.x] = t;
    }
  }
}

// Part of [0, K) of sharer w of n: whole steps of 32; its chunks are as many
// as the first one's.
__host__ __device__ inline int k_share(int K, int n) { return tiles(tiles(K, n), 32) * 32; }

// The tiles of a workgroup's groups meet in LDS (over the operands' space)
// and are added in group order.
template <int BN, int KW>
union SplitSmem {
  GroupSmem<BN> g[KW];
  float t[KW][BM][BN + 1];
};

template <int BN, int KW>
__device__ __forceinline__ void split_store(SplitSmem<BN, KW>& sm, const Tile<BN>& tile) {
  const int g = threadIdx.x / GT;
#pragma unroll
  for (int i = 0; i < Tile<BN>::MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        sm.t[g][Tile<BN>::row(i, q)][Tile<BN>::col(j)] = tile.acc[i][j][q];
}

template <int BN, int KW>
__device__ __forceinline__ float split_sum(const SplitSmem<BN, KW>& sm, int e) {
  float s = sm.t[0][e / BN][e % BN];
#pragma unroll
  for (int q = 1; q < KW; ++q) s += sm.t[q][e / BN][e % BN];
  return s;
}

// Backward through a layer: D [M][N] = (G W) where the layer's input was
// positive, else 0; G [M][K] the gradient of its outputs, W [K][N] its
// weights.  One 64 x 32 tile per workgroup, K shared by its groups.  What
// bounds it: as above.  Batch 2048: K = 1100 and 256 10.9 us on average (17.9
// with split products in memory and their sum in a second launch; 15.5 with
// a 64-wide tile, 12.3 with one group).
template <int BW, int KW>
__global__ __launch_bounds__(KW * GT) void back_kernel(int M, int N, int K, Operand G,
                                                       Operand W, const float* __restrict__ h,
                                                       float* __restrict__ D) {
  __shared__ SplitSmem<BW, KW> sm;
  const int gm = tiles(M, BM), g = threadIdx.x / GT;
  const int m0 = (int)blockIdx.x % gm * BM, n0 = (int)blockIdx.x / gm * BW;
  const int ks = k_share(K, KW), k0 = min(K, g * ks);
  Tile<BW> tile;
  float asum;
  group_product<false, true, false>(G, M, W, N, m0, n0, k0, min(K, k0 + ks), tiles(ks, KC),
                                    sm.g[g], tile, asum);
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < Tile<BW>::MI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = m0 + Tile<BW>::row(i, q), col = n0 + Tile<BW>::col(j);
          if (row < M && col < N) {
            const int64_t at = (int64_t)row * N + col;
            D[at] = h[at] > 0.f ? tile.acc[i][j][q] : 0.f;
          }
        }
  } else {
    __syncthreads();
    split_store(sm, tile);
    __syncthreads();
#pragma unroll
    for (int x = 0; x < BM * BW / (KW * GT); ++x) {
      const int e = threadIdx.x + x * KW * GT, row = m0 + e / BW, col = n0 + e % BW;
      if (row < M && col < N) {
        const int64_t at = (int64_t)row * N + col;
        D[at] = h[at] > 0.f ? split_sum(sm, e) : 0.f;
      }
    }
  }
}

// Gradients of every layer's weights and biases in one launch: for layer l,
// dW [M][N] = G^T H summed over the batch, G [batch][M] the gradient of its
// outputs and H [batch][N] its inputs, and db [M] = G summed over the batch
// (by the workgroups of the first column of tiles, from the operands before
// rounding).  One 64 x 64 tile per workgroup; the batch is shared by
// `splits` workgroups, whose results go to consecutive parameter-sized rows
// of ws.  The last workgroup adds the loss partials.  What bounds it: the
// traffic of the operands, each read by 4 to 18 tiles, and a chunk's round
// trip.  Batch 2048, hidden 256, n_out 1100: 12.2 us (19.0 with two groups
// per workgroup; twelve launches and some 75 us as separate products, sums and
// column sums).
struct GradLayer {
  Operand G, H;
  int M, N, tn, blk0;   // tiles per row of tiles, first workgroup of a split
  int64_t oW, ob;       // offsets in the parameter vector
};
struct GradArgs {
  GradLayer l[3];
  int batch, blocks, splits;   // blocks: workgroups per split
  float* ws;
  int64_t n_params;
  const float* part;
  int64_t n_part;
  float scale;
  float* loss;
};

__global__ __launch_bounds__(GT) void grad_kernel(GradArgs a) {
  constexpr int BN = 64;
  __shared__ GroupSmem<BN> sm;
  __shared__ float rs[GT / 64][BM];
  const int t = threadIdx.x, w = t >> 6;
  if ((int)blockIdx.x == a.blocks * a.splits) {
    // strided sums, then the wavefronts' in order
    float s = 0.f;
    for (int64_t i = t; i < a.n_part; i += GT) s += a.part[i];
    s = admmi::wave_sum(s);
    if ((t & 63) == 0) rs[0][w] = s;
    __syncthreads();
    if (t == 0) {
      float r = rs[0][0];
#pragma unroll
      for (int q = 1; q < GT / 64; ++q) r += rs[0][q];
      *a.loss = r * a.scale;
    }
    return;
  }
  const int split = (int)blockIdx.x % a.splits, blk = (int)blockIdx.x / a.splits;
  const GradLayer L = a.l[blk >= a.l[2].blk0 ? 2 : (blk >= a.l[1].blk0 ? 1 : 0)];
  const int m0 = (blk - L.blk0) / L.tn * BM, n0 = (blk - L.blk0) % L.tn * BN;
  const int ks = k_share(a.batch, a.splits);
  const int k0 = min(a.batch, split * ks), k1 = min(a.batch, k0 + ks);
  float* out = a.ws + split * a.n_params;
  Tile<BN> tile;
  float asum;
  if (n0 == 0)
    group_product<true, true, true>(L.G, L.M, L.H, L.N, m0, n0, k0, k1, tiles(ks, KC), sm, tile, asum);
  else
    group_product<true, true, false>(L.G, L.M, L.H, L.N, m0, n0, k0, k1, tiles(ks, KC), sm, tile, asum);
#pragma unroll
  for (int i = 0; i < Tile<BN>::MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = m0 + Tile<BN>::row(i, q), col = n0 + Tile<BN>::col(j);
        if (row < L.M && col < L.N) out[L.oW + (int64_t)row * L.N + col] = tile.acc[i][j][q];
      }
  if (n0 == 0) {   // uniform
    rs[w][t & 63] = asum;
    __syncthreads();
    if (t < BM && m0 + t < L.M) out[L.ob + m0 + t] = (rs[0][t] + rs[1][t]) + (rs[2][t] + rs[3][t]);
  }
}

// The splits' gradients in order, and what becomes of them: stored in g, or
// (ADAM) the step they give (Kingma and Ba, bias-corrected) on the flat
// parameter vector.
template <bool ADAM>
__global__ __launch_bounds__(256) void step_kernel(int64_t n, int splits,
                                                   const float* __restrict__ ws, float* g, float* p,
                                                   float* m, float* v, float lr, float b1, float b2,
                                                   float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float gi = ws[i];
  for (int s = 1; s < splits; ++s) gi += ws[s * n + i];
  if constexpr (ADAM) {
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  } else {
    g[i] = gi;
  }
}

// Per-column statistics of a [rows][cols] array in two deterministic
// stages.  colpart: part[k][c] = sum over the rows of chunk k, in order, of
// (a[r][c] - shift[c])^pw (pw = 1 or 2, shift = 0 when NULL), in FP64.
__global__ void colpart_kernel(int64_t rows, int cols, int64_t chunk, const float* __restrict__ a,
                               const double* __restrict__ shift, int pw,
                               double* __restrict__ part) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= cols) return;
  const int64_t r0 = (int64_t)blockIdx.y * chunk;
  const int64_t r1 = r0 + chunk < rows ? r0 + chunk : rows;
  const double sh = shift ? shift[c] : 0.0;
  double s = 0.0;
  for (int64_t r = r0; r < r1; ++r) {
    const double d = (double)a[r * cols + c] - sh;
    s += pw == 1 ? d : d * d;
  }
  part[(int64_t)blockIdx.y * cols + c] = s;
}

// Sums the chunk partials in chunk order.  stage 0: mean (kept in FP64 as
// the shift of the second stage); stage 1: standard deviation, floored.
__global__ void colfinish_kernel(int cols, int nk, int64_t rows, const double* __restrict__ part,
                                 int stage, double* __restrict__ mean_d, float* __restrict__ mu,
                                 float* __restrict__ sd, float sd_min) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= cols) return;
  double s = 0.0;
  for (int k = 0; k < nk; ++k) s += part[(int64_t)k * cols + c];
  if (stage == 0) {
    const double m = s / (double)rows;
    mean_d[c] = m;
    mu[c] = (float)m;
  } else {
    const double v = sqrt(s / (double)rows);
    sd[c] = (float)(v > sd_min ? v : sd_min);
  }
}

__global__ void fill_kernel(int n, float v, float* a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

}  // namespace

// Workspace of admm_mlp_fit_output_scaling_noalloc: a fixed array in device
// memory, one copy per device for the life of the process, shared by every
// call on that device.  Host code uses only its device address, looked up
// once per device with that device current; the symbol itself is a host
// stand-in and is never passed to a kernel or a copy.
constexpr int64_t SCRATCH_DOUBLES = int64_t(1) << 20;   // 8 MiB
static __device__ __align__(256) double scratch[SCRATCH_DOUBLES];

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex scratch_mu;
double* scratch_dev[SCRATCH_MAX_DEVICES] = {};

// Device address of `scratch` on `device` (which must be current).
admm_status scratch_address(int device, double** out) {
  if (device < 0 || device >= SCRATCH_MAX_DEVICES)
    return admmi::set_err(ADMM_E_ARG, "device %d out of range", device);
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_dev[device]) {
    void* p = nullptr;
    ADMM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return admmi::set_err(ADMM_E_HIP, "no device address for the workspace");
    scratch_dev[device] = static_cast<double*>(p);
  }
  *out = scratch_dev[device];
  return ADMM_OK;
}
}  // namespace

struct admm_mlp {
  int device = 0;
  int n_in = 0, hid = 0, n_out = 0, max_batch = 0;
  int64_t n_params = 0;
  int64_t oW1, ob1, oW2, ob2, oW3, ob3;
  float *p = nullptr, *am = nullptr, *av = nullptr;
  float* ws = nullptr;                 // gradients of each split of the batch
  float *h1 = nullptr, *h2 = nullptr, *dy = nullptr, *dh1 = nullptr, *dh2 = nullptr;
  float* part = nullptr;               // loss partials, one per workgroup
  float *mu = nullptr, *sd = nullptr;  // fixed output affine y = mu + sd * yhat
  int64_t step = 0;
  std::vector<void*> allocs;
  ~admm_mlp() {
    if (!allocs.empty()) {
      hipSetDevice(device);
      for (void* q : allocs) hipFree(q);
    }
  }
};

namespace {

admm_status mlp_alloc(admm_mlp* n, float** q, int64_t count) {
  ADMM_HIP(hipMalloc((void**)q, (size_t)std::max<int64_t>(count, 1) * sizeof(float)));
  n->allocs.push_back(*q);
  return ADMM_OK;
}

// Columns of a product's tile.  A tile twice as wide reads half as much, a
// narrow one has twice the workgroups and wavefronts: 64 from four workgroups
// per CU on (hidden 256, 8192 rows: forward 41.5 us, 44.2 with 32; 1024 hidden,
// 2048 rows and 512 or 576 tiles: 58.5, 51.9 with 64, but 256 -> 1100 outputs at
// as many 68.6, with 32 66.2 per step).
int layer_tile(int M, int N) { return (int64_t)tiles(M, BM) * tiles(N, 64) >= 1024 ? 64 : 32; }

// The loss epilogue holds the targets as well, so that its wider tile pays by
// the product's size (a step at 1024 -> 1100 with 16,384 rows 1.22 ms, 1.35 with
// 32; at 256 -> 1100 0.271 and 0.264).
int loss_tile(int M, int N, int K) {
  return (int64_t)tiles(M, BM) * tiles(N, 64) * K >= 1 << 21 ? layer_tile(M, N) : 32;
}

template <int EPI>
void layer(int M, int N, int K, const float* A, const float* B, const float* bias, float* C,
           hipStream_t st, const float* mu = nullptr, const float* sd = nullptr,
           const float* target = nullptr, float scale = 0.f, float* part = nullptr) {
  const int ln = EPI == EPI_LOSS ? loss_tile(M, N, K) : layer_tile(M, N);
  (ln == 64 ? layer_kernel<EPI, 64> : layer_kernel<EPI, 32>)<<<tiles(M, BM) * tiles(N, ln), GT, 0, st>>>(
      M, N, K, operand(A, K), operand(B, K), bias, C, mu, sd, target, scale, part);
}

// Gradients through a layer, as wide a tile as its forward pass.
void back(int M, int N, int K, const float* G, const float* W, const float* h, float* D,
          hipStream_t st) {
  const Operand g = operand(G, K), w = operand(W, N);
  const int gm = tiles(M, BM);
  if (layer_tile(M, N) == 64)
    back_kernel<64, 1><<<gm * tiles(N, 64), GT, 0, st>>>(M, N, K, g, w, h, D);
  else
    back_kernel<32, BSPLIT><<<gm * tiles(N, 32), BSPLIT * GT, 0, st>>>(M, N, K, g, w, h, D);
}

// h1 = relu(x W1^T + b1), h2 = relu(h1 W2^T + b2)
void hidden_layers(admm_mlp* n, const float* x, int batch, hipStream_t st) {
  layer<EPI_RELU>(batch, n->hid, n->n_in, x, n->p + n->oW1, n->p + n->ob1, n->h1, st);
  layer<EPI_RELU>(batch, n->hid, n->hid, n->h1, n->p + n->oW2, n->p + n->ob2, n->h2, st);
}

// y = mu + sd * (h2 W3^T + b3)
void forward(admm_mlp* n, const float* x, int batch, float* y, hipStream_t st) {
  hidden_layers(n, x, batch, st);
  layer<EPI_AFFINE>(batch, n->n_out, n->hid, n->h2, n->p + n->oW3, n->p + n->ob3, y, st, n->mu,
                    n->sd);
}

// Workgroups that share the batch in the gradient launch, at least 32 rows
// each.  Consecutive workgroups go to different XCDs, so with eight each XCD
// reads its own eighth of the activations and gradients (19.0 us against 23.4 with
// five and the splits in order, measured with two groups per workgroup).
// Networks whose tiles fill the chip by themselves take fewer, nine workgroups
// per CU at most: every split writes all gradients once and the step reads
// them (2048-4096-2048, 512 rows: 0.69 ms, 1.32 with eight; 8-1024-1100, 256
// rows, 560 tiles: 91 us with four, 113 with eight, 78 with one, but 2048 rows
// 219 with four, 229 with one).
constexpr int MAX_SPLITS = 8, MAX_GRAD_BLOCKS = 9 * 256;
int grad_splits(const admm_mlp* n, int batch) {
  const int64_t h = tiles(n->hid, BM);
  const int64_t blocks = h * (tiles(n->n_out, BM) + h + tiles(n->n_in, 64));
  int most = MAX_SPLITS;
  while (most > 1 && most * blocks > MAX_GRAD_BLOCKS) most /= 2;
  // (not decreasing with the batch: the workspace is that of max_batch)
  return std::max(1, std::min(most, batch / 32));
}

// gradients of mean((y - t)^2) into g, or, with lr > 0, the Adam step they
// give; loss (device scalar) when non-null
void backward(admm_mlp* n, const float* x, const float* tg, int batch, float* loss, float* g,
              float lr, hipStream_t st) {
  hidden_layers(n, x, batch, st);
  const float scale = 1.f / (float)((int64_t)batch * n->n_out);
  layer<EPI_LOSS>(batch, n->n_out, n->hid, n->h2, n->p + n->oW3, n->p + n->ob3, n->dy, st, n->mu,
                  n->sd, tg, scale, n->part);
  back(batch, n->hid, n->n_out, n->dy, n->p + n->oW3, n->h2, n->dh2, st);
  back(batch, n->hid, n->hid, n->dh2, n->p + n->oW2, n->h1, n->dh1, st);
  GradArgs a{};
  const float* G[3] = {n->dy, n->dh2, n->dh1};
  const float* H[3] = {n->h2, n->h1, x};
  const int M[3] = {n->n_out, n->hid, n->hid}, N[3] = {n->hid, n->hid, n->n_in};
  const int64_t oW[3] = {n->oW3, n->oW2, n->oW1}, ob[3] = {n->ob3, n->ob2, n->ob1};
  for (int l = 0; l < 3; ++l) {
    a.l[l] = GradLayer{operand(G[l], M[l]), operand(H[l], N[l]), M[l], N[l], tiles(N[l], 64),
                       a.blocks, oW[l], ob[l]};
    a.blocks += tiles(M[l], BM) * tiles(N[l], 64);
  }
  a.batch = batch;
  a.splits = grad_splits(n, batch);
  a.ws = n->ws;
  a.n_params = n->n_params;
  a.part = n->part;
  a.n_part = (int64_t)tiles(batch, BM) * tiles(n->n_out, loss_tile(batch, n->n_out, n->hid));
  a.scale = scale;
  a.loss = loss;
  grad_kernel<<<a.blocks * a.splits + (loss ? 1 : 0), GT, 0, st>>>(a);
  const unsigned gp = (unsigned)((n->n_params + 255) / 256);
  if (lr > 0.f) {
    n->step += 1;
    const float c1 = 1.f - (float)std::pow(0.9, (double)n->step);
    const float c2 = 1.f - (float)std::pow(0.999, (double)n->step);
    step_kernel<true><<<gp, 256, 0, st>>>(n->n_params, a.splits, n->ws, nullptr, n->p, n->am, n->av,
                                          lr, 0.9f, 0.999f, 1e-8f, c1, c2);
  } else if (g) {
    step_kernel<false><<<gp, 256, 0, st>>>(n->n_params, a.splits, n->ws, g, nullptr, nullptr, nullptr,
                                           0.f, 0.f, 0.f, 0.f, 1.f, 1.f);
  }
}

}  // namespace

extern "C" {

admm_status admm_mlp_create(int32_t n_in, int32_t hidden, int32_t n_out, int32_t max_batch,
                            int32_t device, admm_mlp** out) {
  admmi::clear_err();
  if (!out) return admmi::set_err(ADMM_E_ARG, "out is NULL");
  *out = nullptr;
  if (n_in < 1 || hidden < 1 || n_out < 1 || max_batch < 1)
    return admmi::set_err(ADMM_E_ARG, "sizes must be >= 1");
  if ((int64_t)max_batch * std::max(std::max(n_in, hidden), n_out) >= (1LL << 31))
    return admmi::set_err(ADMM_E_UNSUPPORTED, "max_batch x layer width must stay below 2^31");
  std::unique_ptr<admm_mlp> n(new admm_mlp());
  n->device = device;
  n->n_in = n_in;
  n->hid = hidden;
  n->n_out = n_out;
  n->max_batch = max_batch;
  n->oW1 = 0;
  n->ob1 = n->oW1 + (int64_t)hidden * n_in;
  n->oW2 = n->ob1 + hidden;
  n->ob2 = n->oW2 + (int64_t)hidden * hidden;
  n->oW3 = n->ob2 + hidden;
  n->ob3 = n->oW3 + (int64_t)n_out * hidden;
  n->n_params = n->ob3 + n_out;
  if (admm_status s = admmi::probe_device(device)) return s;
  ADMM_HIP(hipSetDevice(device));
  admm_status s;
  const int64_t B = max_batch;
  if ((s = mlp_alloc(n.get(), &n->p, n->n_params))) return s;
  if ((s = mlp_alloc(n.get(), &n->am, n->n_params))) return s;
  if ((s = mlp_alloc(n.get(), &n->av, n->n_params))) return s;
  if ((s = mlp_alloc(n.get(), &n->h1, B * hidden))) return s;
  if ((s = mlp_alloc(n.get(), &n->h2, B * hidden))) return s;
  if ((s = mlp_alloc(n.get(), &n->dy, B * n_out))) return s;
  if ((s = mlp_alloc(n.get(), &n->dh1, B * hidden))) return s;
  if ((s = mlp_alloc(n.get(), &n->dh2, B * hidden))) return s;
  if ((s = mlp_alloc(n.get(), &n->part, (int64_t)tiles(max_batch, BM) * tiles(n_out, 32)))) return s;
  if ((s = mlp_alloc(n.get(), &n->mu, n_out))) return s;
  if ((s = mlp_alloc(n.get(), &n->ws, n->n_params * grad_splits(n.get(), max_batch)))) return s;
  if ((s = mlp_alloc(n.get(), &n->sd, n_out))) return s;
  fill_kernel<<<(n_out + 255) / 256, 256>>>(n_out, 0.f, n->mu);
  fill_kernel<<<(n_out + 255) / 256, 256>>>(n_out, 1.f, n->sd);
  ADMM_HIP(hipGetLastError());
  ADMM_HIP(hipDeviceSynchronize());
  ADMM_HIP(hipMemset(n->p, 0, n->n_params * sizeof(float)));
  ADMM_HIP(hipMemset(n->am, 0, n->n_params * sizeof(float)));
  ADMM_HIP(hipMemset(n->av, 0, n->n_params * sizeof(float)));
  *out = n.release();
  return ADMM_OK;
}

int64_t admm_mlp_n_params(const admm_mlp* n) { return n ? n->n_params : -1; }

admm_status admm_mlp_set_params(admm_mlp* n, const float* host) {
  admmi::clear_err();
  if (!n || !host) return admmi::set_err(ADMM_E_ARG, "NULL argument");
  ADMM_HIP(hipSetDevice(n->device));
  ADMM_HIP(hipMemcpy(n->p, host, n->n_params * sizeof(float), hipMemcpyHostToDevice));
  ADMM_HIP(hipMemset(n->am, 0, n->n_params * sizeof(float)));
  ADMM_HIP(hipMemset(n->av, 0, n->n_params * sizeof(float)));
  n->step = 0;
  return ADMM_OK;
}

admm_status admm_mlp_get_params(admm_mlp* n, float* host) {
  admmi::clear_err();
  if (!n || !host) return admmi::set_err(ADMM_E_ARG, "NULL argument");
  ADMM_HIP(hipSetDevice(n->device));
  ADMM_HIP(hipMemcpy(host, n->p, n->n_params * sizeof(float), hipMemcpyDeviceToHost));
  return ADMM_OK;
}

admm_status admm_mlp_forward(admm_mlp* n, const float* x, int32_t batch, float* y, void* stream) {
  admmi::clear_err();
  if (!n || !x || !y) return admmi::set_err(ADMM_E_ARG, "NULL argument");
  if (batch < 1 || batch > n->max_batch) return admmi::set_err(ADMM_E_ARG, "batch out of [1, max_batch]");
  ADMM_HIP(hipSetDevice(n->device));
  forward(n, x, batch, y, (hipStream_t)stream);
  ADMM_HIP(hipGetLastError());
  return ADMM_OK;
}

admm_status admm_mlp_grads(admm_mlp* n, const float* x, const float* target, int32_t batch,
                           float* grads, float* loss, void* stream) {
  admmi::clear_err();
  if (!n || !x || !target) return admmi::set_err(ADMM_E_ARG, "NULL argument");
  if (batch < 1 || batch > n->max_batch) return admmi::set_err(ADMM_E_ARG, "batch out of [1, max_batch]");
  ADMM_HIP(hipSetDevice(n->device));
  hipStream_t st = (hipStream_t)stream;
  backward(n, x, target, batch, loss, grads, 0.f, st);
  ADMM_HIP(hipGetLastError());
  return ADMM_OK;
}

admm_status admm_mlp_train_step(admm_mlp* n, const float* x, const float* target, int32_t batch,
                                float lr, float* loss, void* stream) {
  admmi::clear_err();
  if (!n || !x || !target) return admmi::set_err(ADMM_E_ARG, "NULL argument");
  if (batch < 1 || batch > n->max_batch) return admmi::set_err(ADMM_E_ARG, "batch out of [1, max_batch]");
  if (!(lr > 0.f)) return admmi::set_err(ADMM_E_ARG, "lr must be > 0");
  ADMM_HIP(hipSetDevice(n->device));
  backward(n, x, target, batch, loss, nullptr, lr, (hipStream_t)stream);
  ADMM_HIP(hipGetLastError());
  return ADMM_OK;
}

admm_status admm_mlp_fit_output_scaling(admm_mlp* n, const float* targets, int64_t rows,
                                        float sd_min, void* stream) {
  admmi::clear_err();
  if (!n || !targets || rows < 1) return admmi::set_err(ADMM_E_ARG, "bad arguments");
  if (!(sd_min > 0.f)) return admmi::set_err(ADMM_E_ARG, "sd_min must be > 0");
  ADMM_HIP(hipSetDevice(n->device));
  // chunks of at least 256 rows, at most 1024 chunks
  const int64_t nk = std::min<int64_t>(1024, (rows + 255) / 256);
  const int64_t chunk = (rows + nk - 1) / nk;
  const int nkk = (int)((rows + chunk - 1) / chunk);
  double* tmp = nullptr;
  ADMM_HIP(hipMalloc((void**)&tmp, ((size_t)nkk + 1) * n->n_out * sizeof(double)));
  double* mean_d = tmp + (int64_t)nkk * n->n_out;
  hipStream_t st = (hipStream_t)stream;
  const dim3 gp((n->n_out + 255) / 256, nkk);
  const unsigned gf = (n->n_out + 255) / 256;
  colpart_kernel<<<gp, 256, 0, st>>>(rows, n->n_out, chunk, targets, nullptr, 1, tmp);
  colfinish_kernel<<<gf, 256, 0, st>>>(n->n_out, nkk, rows, tmp, 0, mean_d, n->mu, n->sd, sd_min);
  colpart_kernel<<<gp, 256, 0, st>>>(rows, n->n_out, chunk, targets, mean_d, 2, tmp);
  colfinish_kernel<<<gf, 256, 0, st>>>(n->n_out, nkk, rows, tmp, 1, mean_d, n->mu, n->sd, sd_min);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  hipFree(tmp);
  if (e != hipSuccess) return admmi::set_err(ADMM_E_HIP, "output scaling: %s", hipGetErrorString(e));
  ADMM_HIP(hipGetLastError());
  return ADMM_OK;
}

admm_status admm_mlp_fit_output_scaling_noalloc(admm_mlp* n, const float* targets, int64_t rows,
                                                float sd_min, void* stream) {
  admmi::clear_err();
  if (!n || !targets || rows < 1) return admmi::set_err(ADMM_E_ARG, "bad arguments");
  if (!(sd_min > 0.f)) return admmi::set_err(ADMM_E_ARG, "sd_min must be > 0");
  if (2 * (int64_t)n->n_out > SCRATCH_DOUBLES)
    return admmi::set_err(ADMM_E_UNSUPPORTED,
                          "n_out = %d: the fixed workspace holds at most %lld outputs", n->n_out,
                          (long long)(SCRATCH_DOUBLES / 2));
  ADMM_HIP(hipSetDevice(n->device));
  double* ws = nullptr;
  if (admm_status s = scratch_address(n->device, &ws)) return s;
  // the chunking of admm_mlp_fit_output_scaling, with at most as many
  // chunks as the workspace holds partial rows (one more row keeps the mean)
  const int64_t nk = std::min<int64_t>(std::min<int64_t>(1024, (rows + 255) / 256),
                                       SCRATCH_DOUBLES / n->n_out - 1);
  const int64_t chunk = (rows + nk - 1) / nk;
  const int nkk = (int)((rows + chunk - 1) / chunk);
  double* mean_d = ws + (int64_t)nkk * n->n_out;
  hipStream_t st = (hipStream_t)stream;
  const dim3 gp((n->n_out + 255) / 256, nkk);
  const unsigned gf = (n->n_out + 255) / 256;
  colpart_kernel<<<gp, 256, 0, st>>>(rows, n->n_out, chunk, targets, nullptr, 1, ws);
  colfinish_kernel<<<gf, 256, 0, st>>>(n->n_out, nkk, rows, ws, 0, mean_d, n->mu, n->sd, sd_min);
  colpart_kernel<<<gp, 256, 0, st>>>(rows, n->n_out, chunk, targets, mean_d, 2, ws);
  colfinish_kernel<<<gf, 256, 0, st>>>(n->n_out, nkk, rows, ws, 1, mean_d, n->mu, n->sd, sd_min);
  ADMM_HIP(hipGetLastError());
  return ADMM_OK;
}

admm_status admm_mlp_set_output_scaling(admm_mlp* n, const float* mean, const float* sd) {
  admmi::clear_err();
  if (!n || !mean || !sd) return admmi::set_err(ADMM_E_ARG, "NULL argument");
  for (int i = 0; i < n->n_out; ++i)
    if (!(sd[i] > 0.f)) return admmi::set_err(ADMM_E_ARG, "sd must be > 0");
  ADMM_HIP(hipSetDevice(n->device));
  ADMM_HIP(hipMemcpy(n->mu, mean, n->n_out * sizeof(float), hipMemcpyHostToDevice));
  ADMM_HIP(hipMemcpy(n->sd, sd, n->n_out * sizeof(float), hipMemcpyHostToDevice));
  return ADMM_OK;
}

admm_status admm_mlp_get_output_scaling(admm_mlp* n, float* mean, float* sd) {
  admmi::clear_err();
  if (!n || !mean || !sd) return admmi::set_err(ADMM_E_ARG, "NULL argument");
  ADMM_HIP(hipSetDevice(n->device));
  ADMM_HIP(hipMemcpy(mean, n->mu, n->n_out * sizeof(float), hipMemcpyDeviceToHost));
  ADMM_HIP(hipMemcpy(sd, n->sd, n->n_out * sizeof(float), hipMemcpyDeviceToHost));
  return ADMM_OK;
}

admm_status admm_mlp_destroy(admm_mlp* n) {
  admmi::clear_err();
  delete n;
  return ADMM_OK;
}

}  // extern "C"
