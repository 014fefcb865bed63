// Per-column corrector network on gfx950: multilayer perceptron with GELU
// hidden layers, BF16 operands and FP32 accumulation on the matrix cores
// (v_mfma_f32_16x16x32_bf16), forward, backward and Adam on the GPU.
//
// Layout: weights W[out][in] and activations [batch][width], row-major.  One
// GEMM kernel C[M][N] = sum_k A(m, k) B(n, k) reads either operand with k
// contiguous (A[m][k], B[n][k]) or with k as the outer index (A[k][m],
// B[k][n]) through LDS, so no transposed copies are kept:
//   forward    Z  = H_prev W^T     A = H_prev [B][in],   B = W [out][in]
//   input grad dH = dZ W           A = dZ [B][out],      B = W read as [k=out][n=in]
//   weight grad dW = dZ^T H_prev   A = dZ read as [k=B][m=out], B = H_prev read as [k=B][n=in]
// Pre-activation gradients are formed in the epilogues of the products before
// them, and the gradients of all layers and the update take one launch each.
// For the corrector's shape the forward and backward products are one launch
// too (k_mlp_train4): an Adam step on 4096 rows is 3 launches and 45 us, where
// a kernel per layer and purpose took 35 and 260.
// The weight gradient reduces over the batch in fixed chunks (split K) whose
// partial sums are added in a fixed order, so results are reproducible.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "internal.h"

namespace thor {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;    // C tile per workgroup (4 wavefronts of 32 x 32)
constexpr int kStepK = 64;   // k per staged tile (two MFMA k-steps of 32)
constexpr int kRow = kStepK + 8;   // LDS row of a staged tile (bf16), padded
constexpr int kMaxSplit = 8;       // batch chunks of the weight gradient
constexpr int kBiasSplit = 32;     // batch chunks of the bias gradient
constexpr int kMaxLayers = 16;
// Bytes of split-K partial sums that layers share a gradient launch within
// (the corrector's four take 15 MB).  Larger networks go through it in groups,
// their partial sums in the same place one group after another, so that 16
// layers of 4096 x 4096 need 0.5 GiB for them and not 8.  A group of this size
// has 2048 product tiles per batch chunk, eight per compute unit; with 64 MiB
// an Adam step of three 1024 x 1024 layers on 32 rows, then two groups, took
// 102 us against 95 in one.
constexpr size_t kSplitBytes = (size_t)256 << 20;

enum Epilogue { EPI_STORE = 0, EPI_GELU = 1, EPI_GELU_ONLY = 2, EPI_LOSS = 3, EPI_ACT_GRAD = 4 };

// erf by Abramowitz & Stegun 7.1.26: erf x = 1 - t (a1 + t (a2 + ... a5 t))
// e^(-x^2), t = 1 / (1 + p x) for x >= 0, odd in x; absolute error below
// 1.5e-7, far under the BF16 rounding of the activations it feeds, and
// branch-free (the epilogues evaluate it for every hidden activation).
__device__ __forceinline__ float erf_as(float x) {
  const float a = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(1.f + 0.3275911f * a);
  const float poly =
      t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float e = 1.f - poly * __expf(-a * a);
  return copysignf(e, x);
}
__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.f + erf_as(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  return 0.5f * (1.f + erf_as(z * 0.70710678118654752f)) + z * 0.39894228040143268f * __expf(-0.5f * z * z);
}

// Piece h (0, 1) of a 64 x 64 operand tile, 16 bytes per thread (256
// threads), read from global memory: rows r0.. of an operand with `rows`
// rows, k from k0.  KOUTER: stored [k][row] with leading dimension ld, else
// [row][k].  Rows past the end repeat the last ones (their products are not
// stored), k past k_hi the tile's first k (tile_store writes zeros there), so
// that the loads are unconditional and nothing waits on a branch.
template <bool KOUTER>
__device__ __forceinline__ int tile_k(int h) {
  const int t = threadIdx.x;
  return KOUTER ? 2 * (t >> 3) + h : (t & 3) * 16 + 8 * h;
}
template <bool KOUTER>
__device__ __forceinline__ bf16x8 tile_load(const __bf16 *P, int ld, int rows, int r0, int k0, int k_hi, int h) {
  const int t = threadIdx.x;
  const int kk = k0 + tile_k<KOUTER>(h), k = kk < k_hi ? kk : k0;
  if (!KOUTER) return *reinterpret_cast<const bf16x8 *>(P + (size_t)min(r0 + (t >> 2), rows - 1) * ld + k);
  return *reinterpret_cast<const bf16x8 *>(P + (size_t)k * ld + min(r0 + (t & 7) * 8, rows - 8));   // rows % 8 == 0
}

// Position of (row, k) in the LDS tile, rows of kRow values.  A KOUTER tile is
// transposed on the way in, two k at a time; its 8-value chunks are permuted
// by the row's group of eight, so that a wavefront's 32-bit stores (8 row
// groups, 8 k pairs) meet 64 different banks.
template <bool KOUTER>
__device__ __forceinline__ int tile_at(int row, int k) {
  return row * kRow + (KOUTER ? k ^ (row & 56) : k);
}

// Both pieces into the LDS tile, zeros from k = k_n on (k_n = 64 or a
// multiple of 32 below).
template <bool KOUTER>
__device__ __forceinline__ void tile_store(__bf16 *S, const bf16x8 vin[2], int k_n) {
  const int t = threadIdx.x;
  bf16x8 v[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) v[h] = tile_k<KOUTER>(h) < k_n ? vin[h] : bf16x8{};
  if (!KOUTER) {
#pragma unroll
    for (int h = 0; h < 2; ++h) *reinterpret_cast<bf16x8 *>(S + (t >> 2) * kRow + (t & 3) * 16 + 8 * h) = v[h];
  } else {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const int k = 2 * (t >> 3), rc = (t & 7) * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<bf16x2 *>(S + tile_at<true>(rc + i, k)) = bf16x2{v[0][i], v[1][i]};
  }
}

// What the epilogues read and write beside C.
struct Epi {
  const float *bias = nullptr;   // [N]
  __bf16 *H = nullptr;           // EPI_GELU*: activations; EPI_LOSS, EPI_ACT_GRAD: gradient of the pre-activations
  const float *ref = nullptr;    // EPI_LOSS: targets [M][N]; EPI_ACT_GRAD: pre-activations [M][N]
  float *loss = nullptr;         // EPI_LOSS: partial loss sums, [column tile][row tile]
  float scale = 0.f;             // EPI_LOSS: M N (the gradient is 2 d / (M N))
};

// C tile (m0, n0) of the product over k in [k_lo, k_hi), 4 wavefronts, LDS
// double-buffered in tiles of 64 k.  Wavefront w owns rows 32 (w / 2) .. + 31 and columns
// 32 (w % 2) .. + 31 of the tile as 2 x 2 MFMA tiles of 16 x 16; lane l holds
// A(row l % 16, k0 + 8 (l / 16) .. + 7), B(col l % 16, same k) and
// accumulates D[4 (l / 16) + i][l % 16], i = 0..3.
//   EPI_STORE: C = acc (+ bias).
//   EPI_GELU:  C = acc + bias (pre-activation), H = gelu(C) in bf16.
//   EPI_GELU_ONLY: H only (inference keeps no pre-activation).
//   EPI_LOSS: y = acc + bias, d = y - target, C = 2 d / (M N), H = C in bf16, and the sums of d^2.
//   EPI_ACT_GRAD: C = acc gelu'(ref), H = C in bf16.
// The last two form the gradient where its product is, so that neither y nor
// dH goes through memory for a kernel of its own.
template <bool AK, bool BK, int EPI>
__device__ __forceinline__ void gemm_tile(const __bf16 *__restrict__ A, int lda, const __bf16 *__restrict__ B, int ldb,
                                          float *__restrict__ C, int ldc, const Epi &epi, int M, int N, int k_lo,
                                          int k_hi, int tm, int tn) {
  __shared__ __align__(16) __bf16 As[2][kTile * kRow];
  __shared__ __align__(16) __bf16 Bs[2][kTile * kRow];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int m0 = tm * kTile, n0 = tn * kTile;
  const int wm = 32 * (w >> 1), wn = 32 * (w & 1);
  const int r = lane & 15, kq = (lane >> 4) * 8;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Tile i sits in LDS buffer i % 2; tile i + 1 is in registers since the
  // iteration before and goes to LDS after the products of tile i, while the
  // loads of tile i + 2 are in flight for a whole iteration.  The last two
  // iterations load nothing and the last stores nothing: with the last tile
  // loaded again there, products of few tiles read up to three times their
  // operands (inference through two layers of 256, 16384 rows, 23.0 -> 22.0
  // us; 1120 to 160, 32 rows, 11.2 -> 10.5; an Adam step of 1120-128-128-128-
  // 160 on 16384 rows 116.6 -> 110.7).
  bf16x8 ra[2][2], rb[2][2];
  const int nt = (k_hi - k_lo + kStepK - 1) / kStepK;
  auto load = [&](int i, bf16x8 a[2], bf16x8 b[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      a[h] = tile_load<AK>(A, lda, M, m0, k_lo + i * kStepK, k_hi, h);
      b[h] = tile_load<BK>(B, ldb, N, n0, k_lo + i * kStepK, k_hi, h);
    }
  };
  auto products = [&](auto sc) __attribute__((always_inline)) {
    constexpr int s = decltype(sc)::value;
#pragma unroll
    for (int kk = 0; kk < kStepK; kk += 32) {
      bf16x8 a[2], b[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        a[q] = *reinterpret_cast<const bf16x8 *>(&As[s][tile_at<AK>(wm + 16 * q + r, kk + kq)]);
        b[q] = *reinterpret_cast<const bf16x8 *>(&Bs[s][tile_at<BK>(wn + 16 * q + r, kk + kq)]);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[q][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[q], b[j], acc[q][j], 0, 0, 0);
    }
  };
  auto store = [&](int i, auto sc) __attribute__((always_inline)) {   // tile i, in registers and LDS buffer s
    constexpr int s = decltype(sc)::value;
    const int k_n = k_hi - k_lo - i * kStepK;
    tile_store<AK>(As[s], ra[s], k_n);
    tile_store<BK>(Bs[s], rb[s], k_n);
    __syncthreads();
  };
  constexpr std::integral_constant<int, 0> even;
  constexpr std::integral_constant<int, 1> odd;
  load(0, ra[0], rb[0]);   // k_lo < k_hi
  if (nt == 1) {
    store(0, even);
    products(even);
  } else {
    load(1, ra[1], rb[1]);
    store(0, even);
    int i = 0;
    for (; i + 3 < nt; i += 2) {
      load(i + 2, ra[0], rb[0]);
      products(even);
      store(i + 1, odd);
      load(i + 3, ra[1], rb[1]);
      products(odd);
      store(i + 2, even);
    }
    // two or three tiles are left
    if (i + 2 < nt) {
      load(i + 2, ra[0], rb[0]);
      products(even);
      store(i + 1, odd);
      products(odd);
      store(i + 2, even);
      products(even);
    } else {
      products(even);
      store(i + 1, odd);
      products(odd);
    }
  }
  double sq = 0.0;   // this lane's squared errors, rounded once per tile
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + wn + 16 * j + r;
      if (col >= N) continue;
      const float bb = epi.bias ? epi.bias[col] : 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = m0 + wm + 16 * i + (lane >> 4) * 4 + q;
        if (row >= M) continue;
        const float z = acc[i][j][q] + bb;
        if (EPI == EPI_STORE || EPI == EPI_GELU) C[(size_t)row * ldc + col] = z;
        if (EPI == EPI_GELU || EPI == EPI_GELU_ONLY) epi.H[(size_t)row * N + col] = (__bf16)gelu_f(z);
        if (EPI == EPI_LOSS || EPI == EPI_ACT_GRAD) {
          const float ref = epi.ref[(size_t)row * N + col];
          float g;
          if (EPI == EPI_LOSS) {
            const float d = z - ref;
            sq += (double)d * d;
            g = 2.f * d / epi.scale;
          } else {
            g = z * gelu_grad_f(ref);
          }
          C[(size_t)row * ldc + col] = g;
          epi.H[(size_t)row * N + col] = (__bf16)g;
        }
      }
    }
  if (EPI == EPI_LOSS) {
    double *sm = reinterpret_cast<double *>(As[0]);
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    __syncthreads();   // every wavefront has read its operand tiles
    if (lane == 0) sm[w] = sq;
    __syncthreads();
    if (threadIdx.x == 0) epi.loss[(size_t)tn * ((M + kTile - 1) / kTile) + tm] = (float)(((sm[0] + sm[1]) + sm[2]) + sm[3]);
  }
}

template <bool AK, bool BK, int EPI>
__global__ __launch_bounds__(256) void k_gemm(const __bf16 *__restrict__ A, int lda, const __bf16 *__restrict__ B,
                                              int ldb, float *__restrict__ C, int ldc, Epi epi, int M, int N, int K) {
  gemm_tile<AK, BK, EPI>(A, lda, B, ldb, C, ldc, epi, M, N, 0, K, blockIdx.x, blockIdx.y);
}

// Column sums of X[B][N] over row chunk `chunk` into part[chunk][N]: 64
// columns from n0, 4 row groups combined in a fixed order.
__device__ __forceinline__ void colsum_tile(const float *X, int B, int N, int rows_per, int n0, int chunk, float *part) {
  __shared__ float sm[4][64];
  const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int n = n0 + c;
  const int b0 = chunk * rows_per, b1 = min(B, b0 + rows_per);
  float s = 0.f;
  if (n < N) {
#pragma unroll 8
    for (int b = b0 + g; b < b1; b += 4) s += X[(size_t)b * N + n];
  }
  sm[g][c] = s;
  __syncthreads();
  if (g == 0 && n < N) part[(size_t)chunk * N + n] = ((sm[0][c] + sm[1][c]) + sm[2][c]) + sm[3][c];
}

// Weight and bias gradients of every layer of a group (kSplitBytes; all layers
// of the corrector's networks) in one launch (they only need the
// pre-activation gradients and the activations, which all exist by then, and
// one layer's 16-72 tiles fill few compute units).  dW[N][K] = dZ^T H_prev,
// both operands read with the batch as outer index, in S batch chunks of
// `chunk` rows whose partial products go to split + z N K; db = the column
// sums of dZ in kBiasSplit chunks of `rows_per` rows.  The first S x (tiles)
// workgroups take the products, the rest the sums.  Consecutive workgroups go
// to the eight L2 caches in turn, so the batch chunk is the workgroup's number
// modulo S: with 8 chunks (2048 rows up) each cache reads one of them, where
// all read all when the chunk was the slower index (an Adam step on 4096 /
// 8192 rows 52.8 / 76.5 -> 45.2 / 61.4 us, on 1024 rows 36.2 -> 35.8).
struct GradLayer {
  const __bf16 *dZb, *prev;
  const float *dZ;
  float *split, *bsum;
  int N, K, tn, first, bfirst;   // widths; column tiles; first product and sum workgroup of the layer
};
struct GradNet {
  GradLayer l[kMaxLayers];
  int nl, tiles, S;   // product workgroups per batch chunk
};
__global__ __launch_bounds__(256) void k_grad(GradNet net, int B, int chunk, int rows_per) {
  const int wg = blockIdx.x, products = net.tiles * net.S;
  if (wg < products) {
    const int z = wg % net.S, i = wg / net.S;
    int l = 0;
    while (l + 1 < net.nl && i >= net.l[l + 1].first) ++l;
    const GradLayer &g = net.l[l];
    const int t = i - g.first, k_lo = z * chunk;
    gemm_tile<true, true, EPI_STORE>(g.dZb, g.N, g.prev, g.K, g.split + (size_t)z * g.N * g.K, g.K, Epi{}, g.N, g.K,
                                     k_lo, min(B, k_lo + chunk), t / g.tn, t % g.tn);
  } else {
    const int i = wg - products;
    int l = 0;
    while (l + 1 < net.nl && i >= net.l[l + 1].bfirst) ++l;
    const GradLayer &g = net.l[l];
    const int t = i - g.bfirst;
    colsum_tile(g.dZ, B, g.N, rows_per, t / kBiasSplit * 64, t % kBiasSplit, g.bsum);
  }
}

// Position of W[n][k], N rows, in the transposed copy in fragment order (see
// k_weights_frag_t).
__device__ __forceinline__ size_t frag_t(int n, int k, int N) {
  return (((size_t)(k / 16) * (N / 32) + n / 32) * 64 + k % 16 + 16 * (n % 32 / 8)) * 8 + n % 8;
}

// The end of a backward pass, kUpd consecutive parameters per thread: the
// gradient as the sum of its partial sums in order, then (ADAM) Adam on the
// packed fp32 parameters and the bf16 copies of the weights, row-major and in
// fragment order; else the gradient alone.  One launch where reductions,
// Adam and copies of each layer were eighteen.
constexpr int kUpd = 4;
struct UpdateLayer {
  const float *split, *bias;   // S partial weight gradients; kBiasSplit partial bias gradients
  __bf16 *Wb, *Wf, *Wt;        // Wt: null unless the fused training pass reads it
  size_t woff;                 // weights at woff, biases at woff + N K
  int N, K;
};
struct UpdateNet {
  UpdateLayer l[kMaxLayers];
  int nl, S;
  size_t p0, p1;   // the group's range of the packed parameters
};
struct Adam {
  float lr, b1, b2, eps, c1, c2;
};
template <bool ADAM>
__global__ __launch_bounds__(256) void k_update(UpdateNet net, float *p, float *m, float *v, float *grad, Adam a) {
  const size_t i = net.p0 + (blockIdx.x * (size_t)blockDim.x + threadIdx.x) * kUpd;
  if (i >= net.p1) return;
  int l = 0;
  while (l + 1 < net.nl && i >= net.l[l + 1].woff) ++l;
  const UpdateLayer &L = net.l[l];
  const size_t j = i - L.woff, nw = (size_t)L.N * L.K;
  const bool weight = j < nw;
  const float *src = weight ? L.split + j : L.bias + (j - nw);
  const size_t step = weight ? nw : (size_t)L.N;
  const int parts = weight ? net.S : kBiasSplit;
  float g[kUpd] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int z = 0; z < parts; ++z) {
    const float4 x = *reinterpret_cast<const float4 *>(src + z * step);
    g[0] += x.x; g[1] += x.y; g[2] += x.z; g[3] += x.w;
  }
  if (!ADAM) {
    *reinterpret_cast<float4 *>(grad + i) = make_float4(g[0], g[1], g[2], g[3]);
    return;
  }
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  float pi[kUpd], mi[kUpd], vi[kUpd];
  bf16x4 b;
#pragma unroll
  for (int e = 0; e < kUpd; ++e) {
    mi[e] = a.b1 * m[i + e] + (1.f - a.b1) * g[e];
    vi[e] = a.b2 * v[i + e] + (1.f - a.b2) * g[e] * g[e];
    pi[e] = p[i + e] - a.lr * (mi[e] / a.c1) / (sqrtf(vi[e] / a.c2) + a.eps);
    b[e] = (__bf16)pi[e];
  }
  *reinterpret_cast<float4 *>(m + i) = make_float4(mi[0], mi[1], mi[2], mi[3]);
  *reinterpret_cast<float4 *>(v + i) = make_float4(vi[0], vi[1], vi[2], vi[3]);
  *reinterpret_cast<float4 *>(p + i) = make_float4(pi[0], pi[1], pi[2], pi[3]);
  if (!weight) return;
  *reinterpret_cast<bf16x4 *>(L.Wb + j) = b;
  // fragment order of k_weights_frag: half of the 8 values from W[row][k & ~7]
  const int row = (int)(j / L.K), k = (int)(j % L.K);
  const size_t f = ((size_t)(row / 16) * (L.K / 32) + k / 32) * 64 + row % 16 + 16 * (k % 32 / 8);
  *reinterpret_cast<bf16x4 *>(L.Wf + f * 8 + k % 8) = b;
  if (L.Wt) {
    __bf16 *t = L.Wt + frag_t(row, k, L.N);
#pragma unroll
    for (int e = 0; e < kUpd; ++e) t[8 * e] = b[e];
  }
}

// ---------------------------------------------------------------------------
// Fused inference of a 4-layer network whose hidden widths are all kFH =
// 256 (the corrector's shape): one workgroup of kFW = 8 wavefronts (2 per
// SIMD) per tile of kFM = 48 rows runs every layer (214 workgroups for the
// g5 corrector's 10242 columns, one per CU, against 161 for 64-row tiles).
//   * The tile's inputs (48 rows x in, bf16) are staged once into LDS by
//     direct global-to-LDS loads (global_load_lds_dwordx4), all issued
//     before the first wait, laid out [k / 8][row slot][8] with 64 row slots
//     (one per lane of the loading wavefront), so that a wavefront's 16-byte
//     operand reads hit 64 distinct banks.
//   * The hidden activations then live in the same LDS ([row][k], rows
//     padded) from one layer to the next, so only the inputs, the weights
//     (from L2) and the outputs cross the memory hierarchy.
//   * The weights are read from a copy in MFMA fragment order
//     (k_weights_frag), one contiguous KiB per wavefront load.  Each layer
//     is its own loop over k in substeps of 32; a wavefront streams its
//     weight fragments through a ring of kFD substeps in registers, kFD - 1
//     substeps in flight while one is multiplied, with no barrier inside a
//     layer, and the next layer's first kFD substeps go in flight before the
//     current layer's epilogue.
// Wavefront w owns the 16-column tiles w + kFW j (j < kFT) of a layer
// below its width / 16, over the tile's rows (kFI MFMA tiles of 16 x 16
// each).  Per tile the products and their order (k ascending in steps of
// 32) equal k_gemm's, so the outputs equal the layer-by-layer path bit for
// bit.
// ---------------------------------------------------------------------------
#ifndef MLP_FI
#define MLP_FI 3
#endif
constexpr int kFI = MLP_FI;          // 16-row MFMA tiles per workgroup
constexpr int kFM = 16 * kFI;        // rows per workgroup
constexpr int kFR = 64;              // row slots per staged k block (one per lane of a wavefront)
constexpr int kFH = 256;             // hidden width
#ifndef MLP_FW
#define MLP_FW 8
#endif
constexpr int kFW = MLP_FW;          // wavefronts per workgroup
constexpr int kFT = kFH / 16 / kFW;  // 16-column tiles per wavefront (2)
constexpr int kFK0Max = 1152;        // widest input the LDS tile holds
#ifndef MLP_FD
#define MLP_FD 6
#endif
constexpr int kFD = MLP_FD;          // 32-k substeps in the weight ring
constexpr int kHRow = kFH + 8;       // LDS row of the hidden activations, padded
constexpr int kFLds = kFK0Max / 8 * kFR * 8;   // bf16 values of the LDS tile (147,456 bytes)
static_assert(kFM * kHRow <= kFLds, "hidden activations must fit the input tile's LDS");

struct FusedNet {
  const __bf16 *W[4];   // bf16 in MFMA fragment order (k_weights_frag)
  const float *b[4];
  int in, out;          // widths of the input and output layers
};

// A wavefront's weight stream of one layer: its fragment of tile j at
// substep 0 and the layer's number of 32-k substeps.
struct FusedW {
  const __bf16 *row[kFT];
  int nsub;
};

__device__ __forceinline__ FusedW fused_w(const __bf16 *W, int K, const int tile[kFT]) {
  FusedW fw;
  fw.nsub = K >> 5;
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int j = 0; j < kFT; ++j) fw.row[j] = W + ((size_t)tile[j] * fw.nsub * 64 + lane) * 8;
  return fw;
}

// Substep t's fragments (a substep past the end reloads the last one).
__device__ __forceinline__ void fused_load(const FusedW &fw, int t, bf16x8 fr[kFT]) {
  const int tt = min(t, fw.nsub - 1);
#pragma unroll
  for (int j = 0; j < kFT; ++j) fr[j] = *reinterpret_cast<const bf16x8 *>(fw.row[j] + (size_t)tt * 512);
}

// acc[i][j] += A(rows 16 i + .., k) W(rows 16 tile[j] + .., k) over the
// layer's k, with ring[d] holding substep d on entry (the caller issues
// those loads early: before the input tile's wait, or before the previous
// layer's epilogue).  KC: the layer's k width if known at compile time,
// else 0.  XS: A is the staged input tile ([k / 8][SLOTS rows][8]), else the
// hidden activations ([row][kHRow]).  FI: 16-row tiles of the workgroup.  Tiles with use[j] false are loaded
// (from a valid row) but not multiplied.  The ring is refilled
// unconditionally, so every substep issues the same loads and the wait
// before a substep's products covers only its own fragments, kFD substeps
// old.
template <bool XS, int KC, int FI, int SLOTS>
__device__ __forceinline__ void fused_layer(const FusedW &fw, const bool use[kFT], const __bf16 *lds,
                                            f32x4 acc[FI][kFT], bf16x8 ring[kFD][kFT]) {
  const int lane = threadIdx.x & 63, r = lane & 15, kq = (lane >> 4) * 8;
  const int nsub = KC ? KC >> 5 : fw.nsub, nfull = nsub / kFD;
  auto mul = [&](int t, const bf16x8 fr[kFT]) {
    bf16x8 a[FI];
#pragma unroll
    for (int i = 0; i < FI; ++i)
      a[i] = XS ? *reinterpret_cast<const bf16x8 *>(lds + ((((32 * t + kq) >> 3) * SLOTS) + 16 * i + r) * 8)
                : *reinterpret_cast<const bf16x8 *>(lds + (16 * i + r) * kHRow + 32 * t + kq);
#pragma unroll
    for (int j = 0; j < kFT; ++j)
      if (use[j])
#pragma unroll
        for (int i = 0; i < FI; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], fr[j], acc[i][j], 0, 0, 0);
  };
  for (int b = 0; b < nfull; ++b) {
#pragma unroll
    for (int d = 0; d < kFD; ++d) {
      const int t = b * kFD + d;
      mul(t, ring[d]);
      if (!KC || t + kFD < nsub) fused_load(fw, t + kFD, ring[d]);
    }
  }
#pragma unroll
  for (int d = 0; d < kFD; ++d)
    if (nfull * kFD + d < nsub) mul(nfull * kFD + d, ring[d]);
}

// Tiles of wavefront w in layer l (out of n_tiles): w + kFW j.
__device__ __forceinline__ void fused_tiles(int w, int n_tiles, int tile[kFT], bool use[kFT]) {
#pragma unroll
  for (int j = 0; j < kFT; ++j) {
    use[j] = w + kFW * j < n_tiles;
    tile[j] = use[j] ? w + kFW * j : 0;
  }
}

__global__ __launch_bounds__(64 * kFW) void k_mlp_fused4(FusedNet net, const __bf16 *__restrict__ X, int B,
                                                         float *__restrict__ Y) {
  __shared__ __align__(16) __bf16 lds[kFLds];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 15;
  const int m0 = blockIdx.x * kFM;
  const int K0 = net.in, N3 = net.out;
  // stage the input tile: wavefront w takes k blocks w, w + kFW, ...; lane =
  // row (lanes past the tile or the batch repeat its last row; their outputs
  // are dropped)
  {
    const __bf16 *xrow = X + (size_t)min(m0 + min(lane, kFM - 1), B - 1) * K0;
    for (int kb = w; kb < K0 / 8; kb += kFW)
      __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void *)(xrow + 8 * kb),
                                       (__attribute__((address_space(3))) void *)(lds + kb * (kFR * 8)), 16, 0, 0);
  }
  int tile[kFT];
  bool use[kFT];
  fused_tiles(w, kFH / 16, tile, use);
  FusedW fw = fused_w(net.W[0], K0, tile);
  bf16x8 ring[kFD][kFT];
#pragma unroll
  for (int d = 0; d < kFD; ++d) fused_load(fw, d, ring[d]);
  __builtin_amdgcn_s_waitcnt(0);   // the direct-to-LDS loads (and the first weights) have landed
  __syncthreads();
  f32x4 acc[kFI][kFT];
  for (int l = 0; l < 4; ++l) {
#pragma unroll
    for (int i = 0; i < kFI; ++i)
#pragma unroll
      for (int j = 0; j < kFT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (l == 0)
      fused_layer<true, 0, kFI, kFR>(fw, use, lds, acc, ring);
    else
      fused_layer<false, kFH, kFI, kFR>(fw, use, lds, acc, ring);
    // the next layer's first weights go in flight before this epilogue
    int tile_n[kFT];
    bool use_n[kFT];
    FusedW fw_n = fw;
    if (l < 3) {
      fused_tiles(w, (l == 2 ? N3 : kFH) / 16, tile_n, use_n);
      fw_n = fused_w(net.W[l + 1], kFH, tile_n);
#pragma unroll
      for (int d = 0; d < kFD; ++d) fused_load(fw_n, d, ring[d]);
    }
    const float *bias = net.b[l];
    if (l < 3) __syncthreads();   // every wavefront is done reading this layer's input
#pragma unroll
    for (int j = 0; j < kFT; ++j) {
      if (!use[j]) continue;
      const int col = 16 * tile[j] + r;
      const float bb = bias[col];
#pragma unroll
      for (int i = 0; i < kFI; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 16 * i + (lane >> 4) * 4 + q;
          const float z = acc[i][j][q] + bb;
          if (l < 3)
            lds[row * kHRow + col] = (__bf16)gelu_f(z);
          else if (m0 + row < B)
            Y[(size_t)(m0 + row) * N3 + col] = z;
        }
    }
    if (l < 3) {
      __syncthreads();   // the activations are the next layer's input
      fw = fw_n;
#pragma unroll
      for (int j = 0; j < kFT; ++j) {
        tile[j] = tile_n[j];
        use[j] = use_n[j];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Forward and backward pass of the same networks in one launch: a workgroup
// takes 16 FI rows through the four layers and back to the gradient of the
// first layer's pre-activation, seven products whose operand passes from one
// to the next in LDS (two buffers in turn, so one barrier a product) while
// the next product's first weights are in flight.  A wavefront owns the same
// column tiles in every hidden layer, so the pre-activations that the
// backward pass needs stay in its registers.  To memory go the activations
// and the gradients of the pre-activations, for the weight gradients.  The
// backward products read W with the output index as k, from a transposed
// copy in fragment order.
// As seven products of 64 x 64 tiles, each a launch of 256 workgroups or
// fewer that waits on its operands for most of 8-17 us, they took 75 us at
// 4096 rows; this takes 23, and an Adam step 100 -> 53 (256 rows 76 -> 33,
// 8192 rows 133 -> 77).  Here the bound is the weights' way from L2, 1.26 MB
// per workgroup at the corrector's widths, 8 us at 64 bytes per clock, and
// the seven latencies.
// Products and their order equal k_gemm's, so the results do bit for bit.
// ---------------------------------------------------------------------------
struct TrainNet {
  const __bf16 *W[4], *Wt[4];   // fragment order; Wt: transposed (unused for the first layer)
  const float *b[4];
  __bf16 *H[3], *dZb[4];
  float *dZ[4];
  int in, out;
};

// Largest batch in 16-row workgroups: up to one workgroup per compute unit
// they leave fewer units idle (an Adam step on 2048 / 4096 rows 41.6 / 52.8
// us against 45.9 / 55.4 with 32), past that 32 rows per workgroup fetch the
// weights half as often (6144 / 8192 rows 65.0 / 76.5 us against 77.5 / 88.8).
constexpr int kTrain16 = 16 * 256;

// R rows of N bf16 values from LDS rows of kHRow to dst[R][N], N % 8 == 0.
template <int R>
__device__ __forceinline__ void store_rows(const __bf16 *src, __bf16 *dst, int N) {
  const int per = N / 8;
  for (int i = threadIdx.x; i < R * per; i += 64 * kFW) {
    const int row = i / per, c = 8 * (i - row * per);
    *reinterpret_cast<bf16x8 *>(dst + (size_t)row * N + c) = *reinterpret_cast<const bf16x8 *>(src + row * kHRow + c);
  }
}

template <int FI>
__global__ __launch_bounds__(64 * kFW) void k_mlp_train4(TrainNet net, const __bf16 *__restrict__ X,
                                                         const float *__restrict__ T, float scale,
                                                         float *__restrict__ loss) {
  constexpr int R = 16 * FI, KB = 64 / R;   // rows; 8-value k blocks per wavefront load
  __shared__ __align__(16) __bf16 xs[kFK0Max * R];
  __shared__ __align__(16) __bf16 hid[2][R * kHRow];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = lane & 15, r4 = (lane >> 4) * 4;
  const size_t m0 = (size_t)blockIdx.x * R;
  const int K0 = net.in, N3 = net.out;
  {
    // input tile [k / 8][row][8]: lane = (k block, row)
    const __bf16 *src = X + (m0 + lane % R) * K0 + 8 * (lane / R);
    for (int i = w; i < K0 / (8 * KB); i += kFW)
      __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void *)(src + 8 * KB * i),
                                       (__attribute__((address_space(3))) void *)(xs + i * 512), 16, 0, 0);
  }
  int tile[kFT], tile3[kFT];
  bool use[kFT], use3[kFT];
  fused_tiles(w, kFH / 16, tile, use);
  fused_tiles(w, N3 / 16, tile3, use3);
  bf16x8 ring[kFD][kFT];
  FusedW fw;
  auto weights = [&](const __bf16 *W, int K, const int t[kFT]) {
    fw = fused_w(W, K, t);
#pragma unroll
    for (int d = 0; d < kFD; ++d) fused_load(fw, d, ring[d]);
  };
  weights(net.W[0], K0, tile);
  __builtin_amdgcn_s_waitcnt(0);   // the direct-to-LDS loads have landed
  __syncthreads();
  f32x4 acc[FI][kFT], z[3][FI][kFT];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int j = 0; j < kFT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    clear();
    if (l == 0)
      fused_layer<true, 0, FI, R>(fw, use, xs, acc, ring);
    else
      fused_layer<false, kFH, FI, R>(fw, use, hid[(l - 1) & 1], acc, ring);
    weights(net.W[l + 1], kFH, l < 2 ? tile : tile3);
#pragma unroll
    for (int j = 0; j < kFT; ++j) {
      const int col = 16 * tile[j] + r;
      const float bb = net.b[l][col];
#pragma unroll
      for (int i = 0; i < FI; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          z[l][i][j][q] = acc[i][j][q] + bb;
          hid[l & 1][(16 * i + r4 + q) * kHRow + col] = (__bf16)gelu_f(z[l][i][j][q]);
        }
    }
    __syncthreads();
    store_rows<R>(hid[l & 1], net.H[l] + m0 * kFH, kFH);
  }
  clear();
  fused_layer<false, kFH, FI, R>(fw, use3, hid[0], acc, ring);
  weights(net.Wt[3], N3, tile);
  double sq = 0.0;   // squared errors, rounded once per workgroup
#pragma unroll
  for (int j = 0; j < kFT; ++j) {
    if (!use3[j]) continue;
    const int col = 16 * tile3[j] + r;
    const float bb = net.b[3][col];
#pragma unroll
    for (int i = 0; i < FI; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 16 * i + r4 + q;
        const size_t o = (m0 + row) * N3 + col;
        const float y = acc[i][j][q] + bb;
        const float d = y - T[o];
        sq += (double)d * d;
        const float g = 2.f * d / scale;
        net.dZ[3][o] = g;
        hid[1][row * kHRow + col] = (__bf16)g;
      }
  }
  for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
  double *sums = reinterpret_cast<double *>(xs);   // the input tile is free
  if (lane == 0) sums[w] = sq;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < kFW; ++i) s += sums[i];
    loss[blockIdx.x] = (float)s;
  }
  store_rows<R>(hid[1], net.dZb[3] + m0 * N3, N3);
#pragma unroll
  for (int l = 2; l >= 0; --l) {
    // gradient of layer l's pre-activation from that of layer l + 1
    const __bf16 *in = hid[(l + 1) & 1];
    __bf16 *out = hid[l & 1];
    clear();
    if (l == 2)
      fused_layer<false, 0, FI, R>(fw, use, hid[1], acc, ring);
    else
      fused_layer<false, kFH, FI, R>(fw, use, in, acc, ring);
    if (l > 0) weights(net.Wt[l], kFH, tile);
#pragma unroll
    for (int j = 0; j < kFT; ++j) {
      const int col = 16 * tile[j] + r;
#pragma unroll
      for (int i = 0; i < FI; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 16 * i + r4 + q;
          const float g = acc[i][j][q] * gelu_grad_f(z[l][i][j][q]);
          net.dZ[l][(m0 + row) * kFH + col] = g;
          out[row * kHRow + col] = (__bf16)g;
        }
    }
    __syncthreads();
    store_rows<R>(out, net.dZb[l] + m0 * kFH, kFH);
  }
}

// bf16 copy of one layer's fp32 weights.
__global__ void k_weights_bf16(const float *W, __bf16 *Wb, size_t n) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  Wb[i] = (__bf16)W[i];
}

// W[N][K] (FP32) into BF16 MFMA fragment order for the fused kernel:
// fragment (tile j, 32-k substep t, lane l) holds the 8 values
// W[16 j + l % 16][32 t + 8 (l / 16) .. + 7] at ((j K/32 + t) 64 + l) 8,
// so a wavefront's operand load for one tile and substep is 1 KiB
// contiguous.  N % 16 == 0, K % 32 == 0.
__global__ void k_weights_frag(const float *W, __bf16 *Wf, int N, int K) {
  const size_t f = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const int nsub = K / 32;
  if (f >= (size_t)N * K / 8) return;
  const int lane = (int)(f % 64), t = (int)((f / 64) % nsub), j = (int)(f / 64 / nsub);
  const float *src = W + (size_t)(16 * j + lane % 16) * K + 32 * t + 8 * (lane / 16);
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (__bf16)src[e];
  *reinterpret_cast<bf16x8 *>(Wf + f * 8) = v;
}

// The same of the transpose of W[N][K]: rows of K, the N as 32-k substeps.
__global__ void k_weights_frag_t(const float *W, __bf16 *Wt, int N, int K) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= (size_t)N * K) return;
  const int n = (int)(i / K), k = (int)(i % K);
  Wt[frag_t(n, k, N)] = (__bf16)W[i];
}

inline size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }
inline unsigned nb(size_t n, unsigned t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace
}  // namespace thor

using namespace thor;

struct thor_mlp {
  int nl = 0;                    // layers
  std::vector<int> w;            // widths, nl + 1
  int max_batch = 0;
  size_t n_params = 0;
  std::vector<size_t> woff, boff;   // offsets of W_l, b_l in the packed arrays
  float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
  std::vector<__bf16 *> Wb;      // bf16 copies of W_l [out][in]
  std::vector<__bf16 *> Wf;      // the same in MFMA fragment order (fused inference and training)
  std::vector<__bf16 *> Wt;      // W_l^T in fragment order (fused training; null where it is not read)
  std::vector<float *> Z;        // pre-activations of the hidden layers, [B][w_{l+1}]
  std::vector<__bf16 *> H;       // hidden activations, [B][w_{l+1}]
  std::vector<float *> dZ;       // gradients of the pre-activations
  std::vector<__bf16 *> dZb;
  std::vector<int> group;        // first layer of each gradient launch, and the number of layers
  std::vector<float *> split;    // partial sums of the weight gradient, [kMaxSplit][w_{l+1}][w_l], shared by the groups
  std::vector<float *> bsum;     // and of the bias gradient, [kBiasSplit][w_{l+1}]
  float *partial = nullptr;      // loss partial sums, one per output tile or workgroup of the fused pass
  int adam_t = 0;
  bool fused = true;             // k_mlp_fused4 and k_mlp_train4 where the shape allows
  hipStream_t stream = nullptr;
};

namespace {

bool mlp_ok(hipError_t e, const char *what) {
  if (e == hipSuccess) return true;
  set_error(std::string(what) + ": " + hipGetErrorString(e));
  return false;
}

// The fused kernels serve 4-layer networks with hidden widths kFH, an input
// width of at most kFK0Max and an output width of at most kFH.
bool fused_shape(const thor_mlp *M) {
  return M->nl == 4 && M->w[0] <= kFK0Max && M->w[1] == kFH && M->w[2] == kFH && M->w[3] == kFH &&
         M->w[4] <= kFH;
}

// Sizes every device array; with base == nullptr only counts bytes.
size_t mlp_layout(thor_mlp *M, char *base) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> char * {
    char *ptr = base ? base + off : nullptr;
    off += a256(bytes);
    return ptr;
  };
  const int B = M->max_batch, nl = M->nl;
  const size_t tiles = ((size_t)B + kTile - 1) / kTile;
  M->p = (float *)take(M->n_params * 4);
  M->g = (float *)take(M->n_params * 4);
  M->m = (float *)take(M->n_params * 4);
  M->v = (float *)take(M->n_params * 4);
  M->Wb.assign(nl, nullptr);
  M->Wf.assign(nl, nullptr);
  M->Wt.assign(nl, nullptr);
  M->Z.assign(nl, nullptr);
  M->H.assign(nl, nullptr);
  M->dZ.assign(nl, nullptr);
  M->dZb.assign(nl, nullptr);
  M->split.assign(nl, nullptr);
  M->bsum.assign(nl, nullptr);
  M->group.clear();
  std::vector<size_t> at(nl);   // of a layer's partial sums in the shared area
  size_t used = 0, most = 0;
  for (int l = 0; l < nl; ++l) {
    const size_t bytes = a256((size_t)kMaxSplit * M->w[l] * M->w[l + 1] * 4);
    if (l == 0 || used + bytes > kSplitBytes) {
      M->group.push_back(l);
      used = 0;
    }
    at[l] = used;
    used += bytes;
    most = std::max(most, used);
  }
  M->group.push_back(nl);
  for (int l = 0; l < nl; ++l) {
    const size_t wsz = (size_t)M->w[l] * M->w[l + 1];
    M->Wb[l] = (__bf16 *)take(wsz * 2);
    M->Wf[l] = (__bf16 *)take(wsz * 2);
    if (l > 0 && fused_shape(M)) M->Wt[l] = (__bf16 *)take(wsz * 2);
    if (l + 1 < nl) {
      M->Z[l] = (float *)take((size_t)B * M->w[l + 1] * 4);
      M->H[l] = (__bf16 *)take((size_t)B * M->w[l + 1] * 2);
    }
    M->dZ[l] = (float *)take((size_t)B * M->w[l + 1] * 4);
    M->dZb[l] = (__bf16 *)take((size_t)B * M->w[l + 1] * 2);
    M->bsum[l] = (float *)take((size_t)kBiasSplit * M->w[l + 1] * 4);
  }
  char *const split = take(most);
  if (base)
    for (int l = 0; l < nl; ++l) M->split[l] = (float *)(split + at[l]);
  M->partial = (float *)take(std::max(tiles * ((M->w[nl] + kTile - 1) / kTile), ((size_t)B + 15) / 16) * 4);
  return off;
}

bool mlp_shape(thor_mlp *M, int n_layers, const int *widths, int max_batch) {
  if (n_layers < 1 || n_layers > kMaxLayers || !widths || max_batch < 1) {
    set_error("thor_mlp: need 1..16 layers, widths and max_batch >= 1");
    return false;
  }
  M->nl = n_layers;
  M->w.assign(widths, widths + n_layers + 1);
  for (int x : M->w)
    if (x < 1 || x % 32) {
      set_error("thor_mlp: every width must be a positive multiple of 32");
      return false;
    }
  M->max_batch = max_batch;
  M->n_params = 0;
  M->woff.clear();
  M->boff.clear();
  for (int l = 0; l < n_layers; ++l) {
    M->woff.push_back(M->n_params);
    M->n_params += (size_t)M->w[l] * M->w[l + 1];
    M->boff.push_back(M->n_params);
    M->n_params += M->w[l + 1];
  }
  return true;
}

void refresh_bf16(thor_mlp *M) {
  for (int l = 0; l < M->nl; ++l) {
    const size_t n = (size_t)M->w[l] * M->w[l + 1];
    hipLaunchKernelGGL(k_weights_bf16, dim3(nb(n)), dim3(256), 0, M->stream, M->p + M->woff[l], M->Wb[l], n);
    hipLaunchKernelGGL(k_weights_frag, dim3(nb(n / 8)), dim3(256), 0, M->stream, M->p + M->woff[l], M->Wf[l],
                       M->w[l + 1], M->w[l]);
    if (M->Wt[l])
      hipLaunchKernelGGL(k_weights_frag_t, dim3(nb(n)), dim3(256), 0, M->stream, M->p + M->woff[l], M->Wt[l],
                         M->w[l + 1], M->w[l]);
  }
}

// C[M][N] = sum_k A(m, k) B(n, k); see gemm_tile for the operand forms.
template <bool AK, bool BK, int EPI>
void gemm(const __bf16 *A, int lda, const __bf16 *B, int ldb, float *C, int ldc, const Epi &epi, int Mr, int N, int K,
          hipStream_t s) {
  dim3 grid((Mr + kTile - 1) / kTile, (N + kTile - 1) / kTile);
  hipLaunchKernelGGL((k_gemm<AK, BK, EPI>), grid, dim3(256), 0, s, A, lda, B, ldb, C, ldc, epi, Mr, N, K);
}

// Number of batch chunks of a weight gradient: chunks of at least 256 rows.
int grad_splits(int B) { return std::max(1, std::min(kMaxSplit, B / 256)); }

// Inference: the output layer's pre-activation to y (hidden pre-activations
// are not kept).
void infer(thor_mlp *M, const __bf16 *X, int B, float *y) {
  if (fused_shape(M) && M->fused) {
    FusedNet net;
    for (int l = 0; l < 4; ++l) {
      net.W[l] = M->Wf[l];
      net.b[l] = M->p + M->boff[l];
    }
    net.in = M->w[0];
    net.out = M->w[4];
    hipLaunchKernelGGL(k_mlp_fused4, dim3((B + kFM - 1) / kFM), dim3(64 * kFW), 0, M->stream, net, X, B, y);
    return;
  }
  const __bf16 *in = X;
  for (int l = 0; l < M->nl; ++l) {
    const int K = M->w[l], N = M->w[l + 1];
    Epi e;
    e.bias = M->p + M->boff[l];
    if (l + 1 < M->nl) {
      e.H = M->H[l];
      gemm<false, false, EPI_GELU_ONLY>(in, K, M->Wb[l], K, nullptr, N, e, B, N, K, M->stream);
      in = M->H[l];
    } else {
      gemm<false, false, EPI_STORE>(in, K, M->Wb[l], K, y, N, e, B, N, K, M->stream);
    }
  }
}

// Forward and backward pass of the mean-squared loss up to the gradients of
// the pre-activations and the partial sums of the loss (M->partial), layer by
// layer; returns the number of those sums.
int passes_by_layer(thor_mlp *M, const __bf16 *X, const float *T, int B) {
  const int nl = M->nl;
  hipStream_t s = M->stream;
  for (int l = 0; l < nl; ++l) {
    const int K = M->w[l], N = M->w[l + 1];
    const __bf16 *in = l ? M->H[l - 1] : X;
    Epi e;
    e.bias = M->p + M->boff[l];
    if (l + 1 < nl) {
      e.H = M->H[l];
      gemm<false, false, EPI_GELU>(in, K, M->Wb[l], K, M->Z[l], N, e, B, N, K, s);
    } else {
      e.H = M->dZb[l];
      e.ref = T;
      e.loss = M->partial;
      e.scale = (float)B * (float)N;
      gemm<false, false, EPI_LOSS>(in, K, M->Wb[l], K, M->dZ[l], N, e, B, N, K, s);
    }
  }
  for (int l = nl - 1; l > 0; --l) {
    const int K = M->w[l], N = M->w[l + 1];
    // dH[B][K] = dZ W, W read as [k = out][n = in], through the activation
    Epi e;
    e.H = M->dZb[l - 1];
    e.ref = M->Z[l - 1];
    gemm<false, true, EPI_ACT_GRAD>(M->dZb[l], N, M->Wb[l], K, M->dZ[l - 1], K, e, B, K, N, s);
  }
  return (B + kTile - 1) / kTile * ((M->w[nl] + kTile - 1) / kTile);
}

// The same in one launch; B % 32 == 0.
int passes_fused(thor_mlp *M, const __bf16 *X, const float *T, int B) {
  TrainNet net{};
  for (int l = 0; l < 4; ++l) {
    net.W[l] = M->Wf[l];
    net.Wt[l] = M->Wt[l];
    net.b[l] = M->p + M->boff[l];
    net.dZ[l] = M->dZ[l];
    net.dZb[l] = M->dZb[l];
    if (l < 3) net.H[l] = M->H[l];
  }
  net.in = M->w[0];
  net.out = M->w[4];
  const float scale = (float)B * (float)net.out;
  const int wg = B <= kTrain16 ? B / 16 : B / 32;
  if (B <= kTrain16)
    hipLaunchKernelGGL(k_mlp_train4<1>, dim3(wg), dim3(64 * kFW), 0, M->stream, net, X, T, scale, M->partial);
  else
    hipLaunchKernelGGL(k_mlp_train4<2>, dim3(wg), dim3(64 * kFW), 0, M->stream, net, X, T, scale, M->partial);
  return wg;
}

// Gradients of every parameter from the passes' results, group by group: into
// M->g, or (ADAM) into an Adam step.
template <bool ADAM>
void gradients(thor_mlp *M, const __bf16 *X, int B, const Adam &a) {
  const int splits = grad_splits(B);
  const int chunk = ((B + splits - 1) / splits + kStepK - 1) / kStepK * kStepK, S = (B + chunk - 1) / chunk;
  for (size_t k = 0; k + 1 < M->group.size(); ++k) {
    const int l0 = M->group[k], l1 = M->group[k + 1];
    GradNet g{};
    UpdateNet u{};
    g.nl = u.nl = l1 - l0;
    g.S = u.S = S;
    u.p0 = M->woff[l0];
    u.p1 = l1 < M->nl ? M->woff[l1] : M->n_params;
    int sums = 0;
    for (int l = l0; l < l1; ++l) {
      const int K = M->w[l], N = M->w[l + 1], tn = (K + kTile - 1) / kTile;
      g.l[l - l0] = GradLayer{M->dZb[l], l ? M->H[l - 1] : X, M->dZ[l], M->split[l], M->bsum[l], N, K, tn, g.tiles, sums};
      u.l[l - l0] = UpdateLayer{M->split[l], M->bsum[l], M->Wb[l], M->Wf[l], M->Wt[l], M->woff[l], N, K};
      g.tiles += (N + kTile - 1) / kTile * tn;
      sums += (N + 63) / 64 * kBiasSplit;
    }
    hipLaunchKernelGGL(k_grad, dim3(g.tiles * S + sums), dim3(256), 0, M->stream, g, B, chunk,
                       (B + kBiasSplit - 1) / kBiasSplit);
    hipLaunchKernelGGL(k_update<ADAM>, dim3(nb((u.p1 - u.p0) / kUpd)), dim3(256), 0, M->stream, u, M->p, M->m, M->v,
                       M->g, a);
  }
}

// Forward and backward pass of the mean-squared loss; the number of its
// partial sums.
int passes(thor_mlp *M, const __bf16 *X, const float *T, int B) {
  return fused_shape(M) && M->fused ? passes_fused(M, X, T, B) : passes_by_layer(M, X, T, B);
}

// SplitMix64 stream and Box-Muller normals for the initial weights.
struct Rng {
  uint64_t s;
  uint64_t next() {
    uint64_t z = (s += 0x9E3779B97F4A7C15ULL);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
    return z ^ (z >> 31);
  }
  double uniform() { return ((next() >> 11) + 0.5) * 0x1.0p-53; }
  double normal() { return std::sqrt(-2.0 * std::log(uniform())) * std::cos(2.0 * M_PI * uniform()); }
};

}  // namespace

namespace thor {
void mlp_shape_of(const thor_mlp *m, int *in, int *out, int *max_batch) {
  *in = m->w.front();
  *out = m->w.back();
  *max_batch = m->max_batch;
}
}  // namespace thor

extern "C" {

int thor_mlp_bytes(int n_layers, const int *widths, int max_batch, size_t *bytes) {
  clear_error();
  if (!bytes) { set_error("thor_mlp_bytes: NULL argument"); return THOR_EINVAL; }
  thor_mlp M;
  if (!mlp_shape(&M, n_layers, widths, max_batch)) return THOR_EINVAL;
  *bytes = mlp_layout(&M, nullptr);
  return THOR_OK;
}

int thor_mlp_init(int n_layers, const int *widths, int max_batch, uint64_t seed, void *dev_buf,
                  size_t dev_bytes, void *hip_stream, thor_mlp **out) {
  clear_error();
  if (!out || !dev_buf) { set_error("thor_mlp_init: NULL argument"); return THOR_EINVAL; }
  *out = nullptr;
  thor_mlp *M = new (std::nothrow) thor_mlp;
  if (!M) { set_error("thor_mlp_init: out of host memory"); return THOR_ENOMEM; }
  if (!mlp_shape(M, n_layers, widths, max_batch)) { delete M; return THOR_EINVAL; }
  if (dev_bytes < mlp_layout(M, nullptr)) {
    delete M;
    set_error("thor_mlp_init: dev_bytes smaller than thor_mlp_bytes");
    return THOR_ENOMEM;
  }
  if (((uintptr_t)dev_buf & 255) != 0) { delete M; set_error("thor_mlp_init: dev_buf must be 256-byte aligned"); return THOR_EINVAL; }
  mlp_layout(M, (char *)dev_buf);
  M->stream = (hipStream_t)hip_stream;
  // He-style normal weights (std sqrt(2 / in)), zero biases; Adam moments 0
  std::vector<float> host(M->n_params, 0.f);
  Rng rng{seed};
  for (int l = 0; l < M->nl; ++l) {
    const double sd = std::sqrt(2.0 / M->w[l]);
    for (size_t i = 0; i < (size_t)M->w[l] * M->w[l + 1]; ++i) host[M->woff[l] + i] = (float)(sd * rng.normal());
  }
  std::vector<float> zeros(M->n_params, 0.f);
  bool ok = mlp_ok(hipMemcpyAsync(M->p, host.data(), M->n_params * 4, hipMemcpyHostToDevice, M->stream), "copy params") &&
            mlp_ok(hipMemcpyAsync(M->m, zeros.data(), M->n_params * 4, hipMemcpyHostToDevice, M->stream), "copy m") &&
            mlp_ok(hipMemcpyAsync(M->v, zeros.data(), M->n_params * 4, hipMemcpyHostToDevice, M->stream), "copy v");
  if (ok) refresh_bf16(M);
  ok = ok && mlp_ok(hipStreamSynchronize(M->stream), "mlp init synchronize");
  if (!ok) { delete M; return THOR_EHIP; }
  *out = M;
  return THOR_OK;
}

size_t thor_mlp_param_count(const thor_mlp *m) { return m ? m->n_params : 0; }

int thor_mlp_set_params(thor_mlp *m, const float *host) {
  clear_error();
  if (!m || !host) { set_error("thor_mlp_set_params: NULL argument"); return THOR_EINVAL; }
  if (!mlp_ok(hipMemcpyAsync(m->p, host, m->n_params * 4, hipMemcpyHostToDevice, m->stream), "copy params")) return THOR_EHIP;
  refresh_bf16(m);
  m->adam_t = 0;
  std::vector<float> zeros(m->n_params, 0.f);
  bool ok = mlp_ok(hipMemcpyAsync(m->m, zeros.data(), m->n_params * 4, hipMemcpyHostToDevice, m->stream), "zero m") &&
            mlp_ok(hipMemcpyAsync(m->v, zeros.data(), m->n_params * 4, hipMemcpyHostToDevice, m->stream), "zero v") &&
            mlp_ok(hipStreamSynchronize(m->stream), "set params synchronize");
  return ok ? THOR_OK : THOR_EHIP;
}

int thor_mlp_get_params(thor_mlp *m, float *host) {
  clear_error();
  if (!m || !host) { set_error("thor_mlp_get_params: NULL argument"); return THOR_EINVAL; }
  bool ok = mlp_ok(hipMemcpyAsync(host, m->p, m->n_params * 4, hipMemcpyDeviceToHost, m->stream), "copy params") &&
            mlp_ok(hipStreamSynchronize(m->stream), "get params synchronize");
  return ok ? THOR_OK : THOR_EHIP;
}

int thor_mlp_forward(thor_mlp *m, const void *x_bf16, int B, float *y) {
  clear_error();
  if (!m || !x_bf16 || !y) { set_error("thor_mlp_forward: NULL argument"); return THOR_EINVAL; }
  if (B < 1 || B > m->max_batch) { set_error("thor_mlp_forward: batch outside 1..max_batch"); return THOR_EINVAL; }
  if (((uintptr_t)x_bf16 & 15) != 0) { set_error("thor_mlp_forward: inputs must be 16-byte aligned"); return THOR_EINVAL; }
  infer(m, (const __bf16 *)x_bf16, B, y);
  return mlp_ok(hipGetLastError(), "mlp forward") ? THOR_OK : THOR_EHIP;
}

int thor_mlp_loss_grad(thor_mlp *m, const void *x_bf16, const float *t, int B, double *loss, float *grad_host) {
  clear_error();
  if (!m || !x_bf16 || !t) { set_error("thor_mlp_loss_grad: NULL argument"); return THOR_EINVAL; }
  if (B < 1 || B > m->max_batch || B % 32) { set_error("thor_mlp_loss_grad: batch must be a multiple of 32 within max_batch"); return THOR_EINVAL; }
  if (((uintptr_t)x_bf16 & 15) != 0) { set_error("thor_mlp_loss_grad: inputs must be 16-byte aligned"); return THOR_EINVAL; }
  const size_t np = passes(m, (const __bf16 *)x_bf16, t, B);
  gradients<false>(m, (const __bf16 *)x_bf16, B, Adam{});
  std::vector<float> part(np);
  if (!mlp_ok(hipMemcpyAsync(part.data(), m->partial, np * 4, hipMemcpyDeviceToHost, m->stream), "copy loss"))
    return THOR_EHIP;
  if (grad_host && !mlp_ok(hipMemcpyAsync(grad_host, m->g, m->n_params * 4, hipMemcpyDeviceToHost, m->stream), "copy grad"))
    return THOR_EHIP;
  if (!mlp_ok(hipStreamSynchronize(m->stream), "loss synchronize")) return THOR_EHIP;
  double s = 0.0;
  for (float v : part) s += v;
  if (loss) *loss = s / ((double)B * m->w[m->nl]);
  return THOR_OK;
}

int thor_mlp_train_step(thor_mlp *m, const void *x_bf16, const float *t, int B, float lr) {
  clear_error();
  if (!m || !x_bf16 || !t) { set_error("thor_mlp_train_step: NULL argument"); return THOR_EINVAL; }
  if (B < 1 || B > m->max_batch || B % 32 || !(lr > 0)) { set_error("thor_mlp_train_step: batch must be a multiple of 32 within max_batch, lr > 0"); return THOR_EINVAL; }
  if (((uintptr_t)x_bf16 & 15) != 0) { set_error("thor_mlp_train_step: inputs must be 16-byte aligned"); return THOR_EINVAL; }
  passes(m, (const __bf16 *)x_bf16, t, B);
  m->adam_t += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, (float)m->adam_t), c2 = 1.f - std::pow(b2, (float)m->adam_t);
  gradients<true>(m, (const __bf16 *)x_bf16, B, Adam{lr, b1, b2, 1e-8f, c1, c2});
  return mlp_ok(hipGetLastError(), "train step") ? THOR_OK : THOR_EHIP;
}

int thor_mlp_set_fused(thor_mlp *m, int on) {
  clear_error();
  if (!m) { set_error("thor_mlp_set_fused: NULL network"); return THOR_EINVAL; }
  m->fused = on != 0;
  return THOR_OK;
}

void thor_mlp_free(thor_mlp *m) { delete m; }

}  // extern "C"
