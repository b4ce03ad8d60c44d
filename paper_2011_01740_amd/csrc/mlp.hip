// Surrogate network kernels (BF16 matrix cores, FP32 accumulation) and the
// C ABI declared in include/sur.h.
//
// Every product of the network has the form
//     C[r][c] = sum_k X[r][k] * Y[c][k]
// with X and Y BF16 operands:
//   forward      Z = A W^T       X = A  [batch][in],   Y = W   [out][in]
//   data grad    dA = dZ W       X = dZ [batch][out],  Y = W^T [in][out]
//   weight grad  dW = dZ^T A     X = dZ^T [out][batch], Y = A^T [in][batch]
// Every operand that a kernel reads from global memory is stored in fragment
// order (below), so that a wave's load of an MFMA operand is 1 KB contiguous.
// A training step is 3 launches.  The work local to a batch row (the feature
// layer, the forward products, the loss gradient, the data gradients) runs in
// one kernel per 16-row tile with the activations in LDS (k_train_fb), which
// also writes each activation and gradient transposed for the weight
// gradients.  Those are split over the batch (k_gemm, the three products in
// one launch, one wave per 32 x 32 output tile, a whole group of K steps
// loaded at a time); bias gradients are column sums per
// 16-row tile; one kernel then reduces every partial sum in a fixed order, so
// every result is deterministic, and takes each parameter's Adam step on the
// FP32 master copy at once, refreshing its BF16 copies.  The first layer is a fixed random
// Fourier-feature map of the two inputs (sin of x W1^T + b1, on the vector
// unit) and is not trained, so no gradient is propagated to it.  Inference
// runs the whole network in one kernel (k_net).
//
// MFMA 16x16x32 BF16 operand layout (lane l, 64 lanes): A fragment = row
// (l mod 16), k = 8 (l / 16) + 0..7; B fragment = column (l mod 16), same k;
// accumulator element q = row 4 (l / 16) + q, column (l mod 16).
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include <rocprim/device/device_radix_sort.hpp>

#include "../../include/sur.h"
#include "ens_internal.h"
#include "records.h"

namespace {

typedef __bf16 bf16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
// four floats of a caller's array, aligned as its floats are
typedef f32x4 __attribute__((aligned(4))) f32x4_of_floats;

using ens::kOut;
using ens::sorted_records;
constexpr int kIn = SUR_IN, kH = SUR_HIDDEN;
// packed parameter offsets: W1, b1, W2, b2, W3, b3, W4, b4
constexpr int64_t oW1 = 0, ob1 = oW1 + kH * kIn, oW2 = ob1 + kH, ob2 = oW2 + kH * kH,
                  oW3 = ob2 + kH, ob3 = oW3 + kH * kH, oW4 = ob3 + kH, ob4 = oW4 + kOut * kH,
                  kNP = ob4 + kOut;
static_assert(kNP == SUR_N_PARAMS, "parameter count");

// Loss weight of output column c: the first output (the largest of the
// recorded maxima, the value the screen labels by) counts kW0 times, the
// others once, normalised to mean 1.
constexpr float kW0 = 32.0f;
__device__ __forceinline__ float out_weight(int c) {
  return (c == 0 ? kW0 : 1.0f) * ((float)kOut / (kW0 + (float)(kOut - 1)));
}

// The network's two nonlinear functions, in the form every kernel uses:
//
// Fourier feature sin(v): the hardware sine (v_sin_f32, which takes its
// argument in turns) of the fractional part of v / (2 pi).  Rounding v / (2 pi)
// to FP32 moves the angle by at most |v| 2^-24 (under 1e-5 for the |v| < 200
// the features reach), the size of the rounding of v itself, and far below
// the BF16 unit (2^-8) the feature is rounded to.
__device__ __forceinline__ float feature_sin(float v) {
  return __builtin_amdgcn_sinf(__builtin_amdgcn_fractf(v * 0.15915494309189534f));
}

// GELU(z) = z Phi(z), Phi the standard normal CDF.  The tail
// T(z) = Phi(-|z|) = erfc(|z| / sqrt 2) / 2 comes from the rational-times-
// Gaussian approximation of Abramowitz and Stegun (eq. 7.1.26, after
// Hastings; |error in erfc| <= 1.5e-7):
//   erfc(u) ~ t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-u^2),
//   t = 1 / (1 + p u),
// evaluated with u' = u sqrt(log2 e) so that exp(-u^2) = 2^(-u'^2) (p scaled
// to match, the a_i halved).  Then GELU(z) = max(z, 0) - |z| T(z), which
// holds for either sign and forms the small negative tail without the
// cancellation of 1 + erf.  Branch-free: one reciprocal, one exp2.
constexpr float kTailU = 0.84932180028801907f;   // sqrt(log2 e / 2)
constexpr float kTailP = 0.27273748f;            // 0.3275911 / sqrt(log2 e)
constexpr float kTailA1 = 0.127414796f, kTailA2 = -0.142248368f, kTailA3 = 0.7107068705f,
                kTailA4 = -0.7265760135f, kTailA5 = 0.5307027145f;
__device__ __forceinline__ float normal_tail(float z, float *gauss = nullptr) {
  const float u = fabsf(z) * kTailU;
  const float t = __builtin_amdgcn_rcpf(fmaf(kTailP, u, 1.0f));
  float p = fmaf(t, kTailA5, kTailA4);
  p = fmaf(t, p, kTailA3);
  p = fmaf(t, p, kTailA2);
  p = fmaf(t, p, kTailA1);
  const float e = __builtin_amdgcn_exp2f(-(u * u));   // exp(-z^2 / 2)
  if (gauss) *gauss = e;
  return (t * p) * e;
}
// max(z, 0) as a median, which takes z as it is: fmaxf first quiets it with
// an instruction of its own.
__device__ __forceinline__ float gelu_f(float z) {
  return fmaf(-fabsf(z), normal_tail(z), __builtin_amdgcn_fmed3f(z, 0.0f, INFINITY));
}
// d GELU / dz = Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_grad_f(float z) {
  float e;
  const float tail = normal_tail(z, &e);
  const float cdf = z < 0.0f ? tail : 1.0f - tail;
  return fmaf(z, e * 0.39894228040143268f, cdf);
}

// ------------------------------------------------------------ fragment order
// An operand matrix [rows][K] as the MFMA fragments that its products read:
// fragment (fb, c) covers rows 16 fb .. 16 fb + 15 and k = 32 c .. 32 c + 31,
// and holds for lane l the 8 values of row 16 fb + l mod 16 that the lane
// supplies, 16 bytes per lane, 1 KB in all.  Standard k order: lane group g =
// l / 16, slot s <-> k = 32 c + 8 g + s.  Permuted order (the inputs of layers
// 3 and 4 in k_net): k = 32 c + 16 (s / 4) + 4 g + s mod 4.
// In both, element (row, k) within its fragment:
__device__ __forceinline__ int frag_std(int row, int k) {
  return ((((k >> 3) & 3) << 4) | (row & 15)) * 8 + (k & 7);
}
__device__ __forceinline__ int frag_perm(int row, int k) {
  return ((((k >> 2) & 3) << 4) | (row & 15)) * 8 + (((k >> 4) & 1) << 2 | (k & 3));
}
constexpr int kFrag = 512;   // elements of a fragment

// The BF16 copies of the weights, all in fragment order, fragments of a row
// block after each other ([fb][c]): W2, W3, W4 [out][in] and W3, W4 transposed
// [in][out] for training, W3 and W4 in the permuted order for inference (which
// shares W2).  Whoever changes a master weight writes its copies.
struct WeightCopies {
  bf16 *W2, *W3, *W4, *W3T, *W4T, *W3p, *W4p;
};
// Layer (2, 3 or 4) weights [o][in .. in + 3] (in a multiple of 4) = v in all
// their copies.
template <int LAYER>
__device__ __forceinline__ void put_weights(const WeightCopies &c, int o, int in, bf16x4 v) {
  constexpr int NC = kH / 32, NT = (LAYER == 4 ? kOut : kH) / 32;
  const int at = ((o >> 4) * NC + (in >> 5)) * kFrag;
  bf16 *W = LAYER == 2 ? c.W2 : (LAYER == 3 ? c.W3 : c.W4);
  *(bf16x4 *)(W + at + frag_std(o, in)) = v;
  if (LAYER == 2) return;
  bf16 *Wp = LAYER == 3 ? c.W3p : c.W4p, *WT = LAYER == 3 ? c.W3T : c.W4T;
  *(bf16x4 *)(Wp + at + frag_perm(o, in)) = v;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    WT[((in >> 4) * NT + (o >> 5)) * kFrag + frag_std(in + q, o)] = v[q];
}

// ---------------------------------------------------------------- GEMM tile
// Weight-gradient products: C = sum_k X[r][k] Y[c][k] over one share of the
// batch (k), written as a partial sum.
struct GemmArgs {
  const bf16 *X, *Y;     // batch-major fragments: [k / 32][R / 16], [k / 32][16]
  int R;                 // C[R][256], reduction over the batch
  float *out_f32;        // [split][R][256] partial sums
};

constexpr int kTile = 32;  // output tile edge per wave
constexpr int kLSplit = 3, kSplit = 1 << kLSplit;  // largest batch split

// The constants of one Adam step (Kingma and Ba, 2015), for k_reduce_grads:
// h = lr, beta1, beta2, eps, 1 / (1 - beta1^t), 1 / (1 - beta2^t) with
// t = t_base + step + 1.  With hyper != NULL the learning rate, betas, epsilon
// and t_base are read from device memory (hyper[0..4]), so a captured epoch
// replays with new values.  h == NULL: no step follows.
struct AdamHyper {
  const double *hyper;
  double lr, b1, b2, eps, t_base;
  int step;
  float *h;
};
__device__ __forceinline__ void adam_constants(const AdamHyper &a) {
  double lr = a.lr, b1 = a.b1, b2 = a.b2, eps = a.eps, t0 = a.t_base;
  if (a.hyper) {
    lr = a.hyper[0];
    b1 = a.hyper[1];
    b2 = a.hyper[2];
    eps = a.hyper[3];
    t0 = a.hyper[4];
  }
  const double t = t0 + (double)a.step + 1.0;
  a.h[0] = (float)lr;
  a.h[1] = (float)b1;
  a.h[2] = (float)b2;
  a.h[3] = (float)eps;
  a.h[4] = (float)(1.0 / (1.0 - pow(b1, t)));
  a.h[5] = (float)(1.0 / (1.0 - pow(b2, t)));
}

// Three products in one launch (a training step's weight gradients), each
// split over the batch rows in `split` equal parts of `kchunk` rows.
struct GemmBatch {
  GemmArgs g[3];
  int ntile[3];  // tiles of each product: (R/32) (256/32)
  int lsplit;    // log2 split
  int kchunk;
  AdamHyper ad;
};

// One wave per 32 x 32 output tile and part of the batch (2 x 2 accumulators).
// Consecutive blocks take the parts: blocks go round the 8 XCDs, and with 8
// parts every XCD multiplies the rows that its own k_train_fb blocks wrote, out of
// its own L2.  The K range is taken KG MFMA steps (32 each) at a time: all
// operand loads of a group are issued before its products, so one memory
// latency covers KG steps.  One block more than the products need forms the
// step's Adam constants (two FP64 powers) beside the products.
// At 4096 rows: 6.6 us, before 12.0 us with row-major operands and the parts
// spread over all XCDs; 75 MB through L2.
template <int KG>
__global__ __launch_bounds__(64) void k_gemm(GemmBatch bt) {
  int tile = (int)blockIdx.x >> bt.lsplit;
  if (tile >= bt.ntile[0] + bt.ntile[1] + bt.ntile[2]) {
    if (threadIdx.x == 0 && bt.ad.h) adam_constants(bt.ad);
    return;
  }
  const int bz = (int)blockIdx.x & ((1 << bt.lsplit) - 1);
  const int p = tile < bt.ntile[0] ? 0 : (tile < bt.ntile[0] + bt.ntile[1] ? 1 : 2);
  tile -= p == 0 ? 0 : (p == 1 ? bt.ntile[0] : bt.ntile[0] + bt.ntile[1]);
  const GemmArgs g = p == 0 ? bt.g[0] : (p == 1 ? bt.g[1] : bt.g[2]);
  // every product has kH columns
  const int c0 = (tile % (kH / kTile)) * kTile, r0 = (tile / (kH / kTile)) * kTile;
  const int nx = g.R / 16, ny = kH / 16;   // fragments per 32 rows of the batch
  const int kb = bz * (bt.kchunk / 32), ke = kb + bt.kchunk / 32;
  const int l = threadIdx.x & 63;
  const int lc = l & 15, lrow = (l >> 4) * 4;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bf16 *xp = g.X + (r0 / 16) * kFrag + l * 8;
  const bf16 *yp = g.Y + (c0 / 16) * kFrag + l * 8;
  for (int k = kb; k < ke; k += KG) {
    bf16x8 a[KG][2], b[KG][2];
#pragma unroll
    for (int u = 0; u < KG; ++u) {
#pragma unroll
      for (int i = 0; i < 2; ++i) a[u][i] = *(const bf16x8 *)(xp + ((k + u) * nx + i) * kFrag);
#pragma unroll
      for (int j = 0; j < 2; ++j) b[u][j] = *(const bf16x8 *)(yp + ((k + u) * ny + j) * kFrag);
    }
    // keep the whole group of loads ahead of the products
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < KG; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][i], b[u][j], acc[i][j], 0, 0, 0);
  }
  float *o = g.out_f32 + bz * g.R * kH;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = c0 + 16 * j + lc;
      const int rb = r0 + 16 * i + lrow;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[(rb + q) * kH + c] = acc[i][j][q];
    }
}

// ------------------------------------------------ fused training tile
// One training step's work that is local to a row of the batch, for a tile
// of 16 rows per block (a batch of 4096 rows fills every CU): the feature
// layer, the forward products of layers 2 to 4, the loss gradient of the
// output layer, and the data gradients back through layers 3 and 2.  The
// block has 16 waves, 4 on each SIMD (a wave alone on its SIMD issues only
// every fifth cycle), and wave w computes output features 16 w .. 16 w + 15
// of a 256-wide layer, so it already holds, in the accumulator layout, the
// GELU derivatives of exactly the positions whose data gradient it forms on
// the way back.  The activations and gradients that feed the next product
// stay in LDS (two BF16 row-major tiles, rows padded to 264 so that the 16
// rows of an operand fragment fall on different banks), and each product's
// weight fragments are loaded into registers a layer ahead.  What leaves the
// block is what the weight-gradient products and the reduction need: the
// activations and gradients in fragment order over the batch (BF16; a tile
// is half of the 32 rows of a fragment), the column sums of each
// gradient over the tile (bias gradients), and the tile's weighted squared
// error.  Activations and gradients are rounded to BF16 where they become
// operands; every product accumulates in FP32, its MFMA steps in increasing
// k.
// At 4096 rows (one block per CU): 10.2 us, before 20.5 us with 4 waves a block
// and row-major weights (16 rows of 64 bytes to a load).  Of its 20k cycles
// about half go to the 448 KB of weights that every CU reads from L2 (some 40
// bytes a cycle), the rest to the chain of 7 phases between barriers.  More
// prefetching (W3 at the start, W3T a layer earlier) was slower: the waves wait
// to issue loads then, instead of for their data.
constexpr int kTileLd = kH + 8;
constexpr int kTR = 16;                  // rows per tile
constexpr int kFbWaves = kH / 16;        // one 16-feature block of a layer per wave

struct TrainArgs {
  const float *x;          // inputs [*][2]: batch row r is dataset row rows[r] (or r)
  const int64_t *rows;     // dataset rows of the batch, or NULL
  const float *tgt;        // targets [*][64], indexed like x
  const float *P;          // FP32 parameters (W1, b1 .. b4 read here)
  WeightCopies W;
  int m;                   // batch rows
  int lsplit;              // log2 of the parts of the batch that k_gemm splits it in
  bf16 *a1, *a2, *a3;      // [m / 32][16] fragments
  bf16 *dz4;               // [m / 32][4] fragments
  bf16 *dz3, *dz2;         // [m / 32][16] fragments
  float *cp4, *cp3, *cp2;  // [m/16][64], [m/16][256], [m/16][256]
  float *lpart;            // [m/16]
};

// The B operands of a tile product: the fragments of weight row block fb for
// every MFMA step of K.  Loaded a whole layer ahead: the weights do not
// depend on the activations, so a layer's loads are issued before the
// previous layer's epilogue and barrier, which hides their latency.
template <int K>
__device__ __forceinline__ void tile_weights(const bf16 *__restrict__ W, int fb, int l,
                                             bf16x8 (&b)[K / 32]) {
  const bf16 *wp = W + fb * (K / 32) * kFrag + l * 8;
#pragma unroll
  for (int s = 0; s < K / 32; ++s) b[s] = *(const bf16x8 *)(wp + s * kFrag);
}

// The tile's 16 rows times the weight rows of b over k = 0 .. K, the A
// operands from the LDS tile, the MFMA steps in increasing k.
template <int K>
__device__ __forceinline__ f32x4 tile_product(const bf16 (*in)[kTileLd],
                                              const bf16x8 (&b)[K / 32], int l) {
  const int lr = l & 15, lk = (l >> 4) * 8;
  f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 a[K / 32];
#pragma unroll
  for (int s = 0; s < K / 32; ++s) a[s] = *(const bf16x8 *)&in[lr][32 * s + lk];
#pragma unroll
  for (int s = 0; s < K / 32; ++s)
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s], b[s], acc, 0, 0, 0);
  return acc;
}

// Rows 4 rq .. 4 rq + 3 of feature f of the tile (nf features wide) to its
// place in the batch's fragments.
__device__ __forceinline__ void put_rows(bf16 *F, int nf, int tile, int f, int rq, bf16x4 v) {
  const int row = (tile & 1) * 16 + 4 * rq;
  *(bf16x4 *)(F + ((tile >> 1) * (nf / 16) + (f >> 4)) * kFrag + frag_std(f, row)) = v;
}

// Column sums over the tile's rows of v (the accumulator layout: lane l
// holds rows 4 (l / 16) + q of column l mod 16): the lane's rows, then the 4
// lane groups, in a fixed order; lanes 0 .. 15 hold the sums.
__device__ __forceinline__ float tile_colsum(const float (&v)[4]) {
  float s0 = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) s0 += v[q];
  s0 += __shfl_xor(s0, 16);
  s0 += __shfl_xor(s0, 32);
  return s0;
}

__global__ __launch_bounds__(64 * kFbWaves) void k_train_fb(TrainArgs g) {
  __shared__ bf16 act[2][kTR][kTileLd];
  __shared__ float lw[kOut / 16];
  // consecutive blocks (which go round the XCDs) take tiles of different
  // parts of the batch, as k_gemm's blocks do
  const int m = g.m, b = (int)blockIdx.x;
  const int tile = (b & ((1 << g.lsplit) - 1)) * (m / kTR >> g.lsplit) + (b >> g.lsplit);
  const int r0 = tile * kTR;
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  const int lc = l & 15, lg = l >> 4;
  const int c = 16 * w + lc;    // the lane's output feature
  // layer 1: wave w takes rows 4 (w / 4) .. + 3, lane l feature 64 (w mod 4) + l.
  // The rows and inputs are the same in all lanes (scalar loads).
  const int f = t & (kH - 1), rq = __builtin_amdgcn_readfirstlane(t / kH);
  int64_t src[4], trow[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    src[q] = r0 + 4 * rq + q;
    trow[q] = r0 + 4 * lg + q;
  }
  if (g.rows) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      src[q] = g.rows[src[q]];
      trow[q] = g.rows[trow[q]];
    }
  }
  float xin[4][2];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    xin[q][0] = g.x[2 * src[q]];
    xin[q][1] = g.x[2 * src[q] + 1];
  }
  const float w0 = g.P[oW1 + 2 * f], w1 = g.P[oW1 + 2 * f + 1], bb = g.P[ob1 + f];
  // biases of the lane's output positions
  const float b23[2] = {g.P[ob2 + c], g.P[ob3 + c]}, b4c = g.P[ob4 + (c & (kOut - 1))];
  bf16x8 bw[kH / 32];           // the next 256-wide product's weights
  tile_weights<kH>(g.W.W2, w, l, bw);
  float tq[4] = {0.f, 0.f, 0.f, 0.f};
  if (w < kOut / 16) {
#pragma unroll
    for (int q = 0; q < 4; ++q) tq[q] = g.tgt[trow[q] * kOut + c];
  }
  {
    bf16x4 col;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bf16 v = (bf16)feature_sin(fmaf(xin[q][1], w1, fmaf(xin[q][0], w0, bb)));
      act[0][4 * rq + q][f] = v;
      col[q] = v;
    }
    put_rows(g.a1, kH, tile, f, rq, col);
  }
  __syncthreads();
  // layers 2 and 3: z = a W^T + b, a' = GELU(z); keep GELU'(z) for the way back
  float gp[2][4];  // [layer 2, 3][q]
  f32x4 acc;
#pragma unroll
  for (int L = 0; L < 2; ++L) {
    acc = tile_product<kH>(act[L], bw, l);
    if (L == 0)
      tile_weights<kH>(g.W.W3, w, l, bw);
    else if (w < kOut / 16)
      tile_weights<kH>(g.W.W4, w, l, bw);
    bf16x4 col;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float z = acc[q] + b23[L];
      gp[L][q] = gelu_grad_f(z);
      const bf16 a = (bf16)gelu_f(z);
      act[1 - L][4 * lg + q][c] = a;
      col[q] = a;
    }
    put_rows(L == 0 ? g.a2 : g.a3, kH, tile, c, lg, col);
    __syncthreads();
  }
  // layer 4 and the loss gradient 2 w_c (out - t) / (m * 64): waves 0 .. 3
  // take the 64 output columns
  bf16x8 bwt[kOut / 32];  // W4^T for the first product back
  tile_weights<kOut>(g.W.W4T, w, l, bwt);
  if (w < kOut / 16) {
    acc = tile_product<kH>(act[0], bw, l);
    const float wc = out_weight(c);
    const float scale = 2.0f * wc / (float)((int64_t)m * kOut);
    float gv[4];
    float sq = 0.f;
    bf16x4 col;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float d = (acc[q] + b4c) - tq[q];
      sq = fmaf(wc * d, d, sq);
      gv[q] = scale * d;
      const bf16 gb = (bf16)gv[q];
      act[1][4 * lg + q][c] = gb;
      col[q] = gb;
    }
    put_rows(g.dz4, kOut, tile, c, lg, col);
    const float cs = tile_colsum(gv);
    if (l < 16) g.cp4[tile * kOut + c] = cs;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if (l == 0) lw[w] = sq;
  }
  __syncthreads();
  if (t == 0) g.lpart[tile] = ((lw[0] + lw[1]) + lw[2]) + lw[3];
  // back through layer 3 (dA3 = dZ4 W4, K = 64), then layer 2 (dA2 = dZ3 W3)
#pragma unroll
  for (int L = 1; L >= 0; --L) {
    if (L == 1) {
      acc = tile_product<kOut>(act[1], bwt, l);
      tile_weights<kH>(g.W.W3T, w, l, bw);
    } else {
      acc = tile_product<kH>(act[0], bw, l);
    }
    float dz[4];
    bf16x4 col;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      dz[q] = acc[q] * gp[L][q];
      const bf16 gb = (bf16)dz[q];
      if (L == 1) act[0][4 * lg + q][c] = gb;
      col[q] = gb;
    }
    put_rows(L == 1 ? g.dz3 : g.dz2, kH, tile, c, lg, col);
    const float cs = tile_colsum(dz);
    if (l < 16) (L == 1 ? g.cp3 : g.cp2)[tile * kH + c] = cs;
    if (L == 1) __syncthreads();
  }
}

// ---------------------------------------------------------------- small kernels
// Gradients of all trained parameters (W2 onwards) from the partial sums of
// one batch of m rows (T = m / 16 row tiles, S weight-gradient splits), each
// summed in a fixed order, and the batch loss; acc (optional) accumulates the
// loss.  ADAM: each summed gradient also takes its Adam step on the FP32
// master parameters at once, and the BF16 copies follow the updated values.
struct GradParts {
  const float *w2, *w3;           // [S][256][256]
  const float *b2, *b3;           // [T][256]
  const float *w4;                // [S][64][256]
  const float *b4;                // [T][64]
  const float *lpart;             // [T]
};
struct AdamArgs {
  float *P, *Mm, *V;
  const float *h;                 // the step's constants (adam_constants)
  WeightCopies W;
};

// One parameter p with moments m and v and gradient gr.
__device__ __forceinline__ void adam_one(const float (&h)[6], float gr, float &p, float &m,
                                         float &v) {
  const float lr = h[0], b1 = h[1], b2 = h[2], eps = h[3], c1 = h[4], c2 = h[5];
  m = fmaf(b1, m, (1.0f - b1) * gr);
  v = fmaf(b2, v, (1.0f - b2) * gr * gr);
  p = p - lr * (m * c1) / (sqrtf(v * c2) + eps);
}

// Weights [o][in .. in + 3] of a layer: a block takes 16 rows and 64 columns,
// 2 whole fragments of the copies.
constexpr int kRedTiles = kH / 16 * (kH / 64), kRedTiles4 = kOut / 16 * (kH / 64);
constexpr int kRedWBlocks = 2 * kRedTiles + kRedTiles4;
constexpr int kRedCols = 16;   // tile-summed columns (b2, b3, b4) of a block
constexpr int kRedBlocks = kRedWBlocks + (2 * kH + kOut) / kRedCols + 1;

template <int LAYER, bool ADAM>
__device__ __forceinline__ void reduce_weights(const float *__restrict__ part, int S, int64_t base,
                                               int tile, float *G, const AdamArgs &ad) {
  const int64_t stride = (LAYER == 4 ? kOut : kH) * kH;
  const int o = (tile / (kH / 64)) * 16 + ((int)threadIdx.x >> 4);
  const int in = (tile % (kH / 64)) * 64 + 4 * ((int)threadIdx.x & 15);
  const int64_t k = (int64_t)o * kH + in, i = base + k;
  f32x4 p, m, v, d[kSplit];
#pragma unroll
  for (int u = 0; u < kSplit; ++u) d[u] = *(const f32x4 *)(part + (u < S ? u : 0) * stride + k);
  float h[6];
  if (ADAM) {
    p = *(const f32x4 *)(ad.P + i);
    m = *(const f32x4 *)(ad.Mm + i);
    v = *(const f32x4 *)(ad.V + i);
#pragma unroll
    for (int u = 0; u < 6; ++u) h[u] = ad.h[u];
  }
  f32x4 g{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < kSplit; ++u)
    if (u < S) g += d[u];
  *(f32x4 *)(G + i) = g;
  if (!ADAM) return;
  bf16x4 wb;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float pq = p[q], mq = m[q], vq = v[q];
    adam_one(h, g[q], pq, mq, vq);
    p[q] = pq;
    m[q] = mq;
    v[q] = vq;
    wb[q] = (bf16)pq;
  }
  *(f32x4 *)(ad.P + i) = p;
  *(f32x4 *)(ad.Mm + i) = m;
  *(f32x4 *)(ad.V + i) = v;
  put_weights<LAYER>(ad.W, o, in, wb);
}

// Blocks [0, kRedWBlocks): weights.  The next blocks: kRedCols tile-summed
// columns each, 16 threads a column.  The order of a column's sum: 64 partial
// sums l, of tiles l, l + 64, ..., then a tree that adds l + 32, 16, .. 1;
// thread t holds those with l = t / 16 mod 16 of column t mod 16.  The last
// block: the loss, in the same order.  Bound by the latency of one round of
// loads (8 MB in all, each thread's in flight at once).  At 4096 rows: 4.4 us,
// before 8.7 us with the Adam constants formed in every block and a column's
// tiles read by the lanes of one wave, 64 lines to a load.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_reduce_grads(GradParts p, int64_t T, int S,
                                                      float count, float *G, float *loss,
                                                      float *acc, int first, AdamArgs ad) {
  const int b = (int)blockIdx.x;
  if (b < kRedTiles) {
    reduce_weights<2, ADAM>(p.w2, S, oW2, b, G, ad);
    return;
  }
  if (b < 2 * kRedTiles) {
    reduce_weights<3, ADAM>(p.w3, S, oW3, b - kRedTiles, G, ad);
    return;
  }
  if (b < kRedWBlocks) {
    reduce_weights<4, ADAM>(p.w4, S, oW4, b - 2 * kRedTiles, G, ad);
    return;
  }
  if (b == kRedBlocks - 1) {
    if (threadIdx.x >= 64) return;
    float v = 0.f;
    for (int64_t t = threadIdx.x; t < T; t += 64) v += p.lpart[t];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (threadIdx.x == 0) {
      const float lv = v / count;
      *loss = lv;
      if (acc) *acc = first ? lv : *acc + lv;
    }
    return;
  }
  __shared__ float red[4][64];
  const int e0 = (b - kRedWBlocks) * kRedCols, e = e0 + ((int)threadIdx.x & 15);
  const int l0 = (int)threadIdx.x >> 4;
  const float *src;
  int64_t ld, i;
  if (e0 < kH) {
    src = p.b2 + e; ld = kH; i = ob2 + e;
  } else if (e0 < 2 * kH) {
    src = p.b3 + (e - kH); ld = kH; i = ob3 + (e - kH);
  } else {
    src = p.b4 + (e - 2 * kH); ld = kOut; i = ob4 + (e - 2 * kH);
  }
  float h[6], pe = 0.f, me = 0.f, ve = 0.f;
  if (ADAM && threadIdx.x < kRedCols) {
    pe = ad.P[i];
    me = ad.Mm[i];
    ve = ad.V[i];
#pragma unroll
    for (int u = 0; u < 6; ++u) h[u] = ad.h[u];
  }
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t t = 0; t < T; t += 256) {
    float d[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int64_t r = t + l0 + 16 * k;
      d[k] = src[(r < T ? r : T - 1) * ld];
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (t + l0 + 16 * k < T) v[k & 3] += d[k];
  }
  const float s = (v[0] + v[2]) + (v[1] + v[3]);   // l + 32, l + 16
  red[threadIdx.x >> 6][threadIdx.x & 63] = s;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int l = threadIdx.x;
  float gr = (red[0][l] + red[2][l]) + (red[1][l] + red[3][l]);   // l + 8, l + 4
  gr += __shfl_xor(gr, 32);                                        // l + 2
  gr += __shfl_xor(gr, 16);                                        // l + 1
  if (l >= kRedCols) return;
  G[i] = gr;
  if (ADAM) {
    adam_one(h, gr, pe, me, ve);
    ad.P[i] = pe;
    ad.Mm[i] = me;
    ad.V[i] = ve;
  }
}

// The BF16 copies of W2, W3, W4 from the master weights: 4 weights a thread.
__global__ void k_refresh(const float *__restrict__ P, WeightCopies W) {
  const int i = ((int)blockIdx.x * (int)blockDim.x + (int)threadIdx.x) * 4;
  if (i >= kH * kH) return;
  const int o = i / kH, in = i % kH;
  bf16x4 a, b, c;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    a[q] = (bf16)P[oW2 + i + q];
    b[q] = (bf16)P[oW3 + i + q];
  }
  put_weights<2>(W, o, in, a);
  put_weights<3>(W, o, in, b);
  if (i >= kOut * kH) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) c[q] = (bf16)P[oW4 + i + q];
  put_weights<4>(W, o, in, c);
}

// ---------------------------------------------------------------- dataset
// The recorded maxima of a point in decreasing order are the network's
// targets (the first output then is the point's largest maximum; the order
// does not depend on the phase of a periodic or chaotic response within the
// window).  One point per lane: the 64 loads of a wave are 512 bytes
// contiguous each, and the bitonic network (672 exchanges) runs in registers.
//
// 262144 points (134 MB of records in, 67 MB of targets out; 28 and 42 us at
// the 4.8 TB/s of a copy): k_moments 68 us, k_dataset 57 us, bound by the
// instructions of the network and the logarithms at 2 waves per SIMD.  Before,
// a kernel with one wave per point sorted (249 us, 64 lines to a load) and
// wrote the records out again, twice, and one block per output took all
// logarithms for the mean (436 us) and for the deviation (458 us), and a
// thread per target once more (145 us).
//
// A wave takes 64 points (a tile) and all 64 outputs, in groups of 16, or,
// where the points are too few for the SIMDs (few below), one group of them,
// so that 4 waves sort the same points and share the logarithms.
constexpr int kGrp = 16;              // outputs passed at a time
constexpr int kDsWaves = 4;           // waves of a block
constexpr int kGroups = kOut / kGrp;
constexpr int kRowLd = kOut + 4;      // 16 lanes' rows on different banks

static_assert(kDsWaves == kGroups, "few points: one group per wave of a block");
// Few points: the grid of one group per wave still is at most one wave per
// SIMD (16384 points: k_dataset 11 us, 20 us with all groups in a wave).
inline bool few_points(int64_t n) { return n <= 64 * 256; }

// ln x for finite normal x > 0, from a table and a short series (the method of
// Tang, 1990).  x = 2^e m with m in [1/2, 1); the top 7 bits
// of m's fraction choose a table entry with inv ~ 1 / m of few bits, and
//     ln x = k ln 2 + L + log1p(f),   f = m inv - 1,  |f| <= 2^-7,
// k = e with L = -ln inv for the upper part of the interval, and k = e - 1
// with L = -ln (inv / 2) below sqrt(1/2), so that k = L = 0 on both sides of
// x = 1.  ln 2 and L are split: the high parts are multiples of 2^-42, so
// k ln2_hi + L_hi is exact; the sum with f keeps its rounding error, and the
// Taylor series of log1p(f) - f is small beside it.  Error at most 0.63 ulp
// (0.64 for the library's log, of 4 times as many instructions), measured
// against 64-bit mantissas over 1e-130 .. 1e130 and near 1.
struct LnEntry {
  double hi;
  float lo, inv;
};
constexpr int kLnTab = 128, kLnLow = 53;   // entries; those below sqrt(1/2)
constexpr double kLn2Hi = 0x1.62e42fefa38p-1, kLn2Lo = 0x1.ef35793c7673p-45;

void ln_table(LnEntry *t) {
  for (int i = 0; i < kLnTab; ++i) {
    const double centre = 0.5 + (i + 0.5) / (2 * kLnTab);
    double inv = std::round(1024.0 / centre) / 1024.0;
    if (i == 0) inv = 2.0;             // next to x = 1 on either side
    if (i == kLnTab - 1) inv = 1.0;
    const long double L = -std::log((long double)(i < kLnLow ? inv / 2 : inv));
    t[i].hi = (double)(std::round(L * 0x1p42L) / 0x1p42L);
    t[i].lo = (float)(L - (long double)t[i].hi);
    t[i].inv = (float)inv;
  }
}

__device__ __forceinline__ double ln_normal(const LnEntry *tab, double x) {
  const int i = (__double2hiint(x) >> 13) & (kLnTab - 1);
  const LnEntry t = tab[i];
  const double k = (double)(__builtin_amdgcn_frexp_exp(x) - (i < kLnLow ? 1 : 0));
  const double f = fma(__builtin_amdgcn_frexp_mant(x), (double)t.inv, -1.0);
  double q = -1.0 / 8;
  q = fma(q, f, 1.0 / 7);
  q = fma(q, f, -1.0 / 6);
  q = fma(q, f, 1.0 / 5);
  q = fma(q, f, -1.0 / 4);
  q = fma(q, f, 1.0 / 3);
  q = fma(q, f, -1.0 / 2);
  const double h = fma(k, kLn2Hi, t.hi), lo = fma(k, kLn2Lo, (double)t.lo);
  const double s = h + f, r = (h - s) + f;
  return s + (r + fma(f * f, q, lo));
}
// Sorted records all finite, normal and positive in every lane (a NaN among
// them does not outlive the sort unless all are)?
__device__ __forceinline__ bool all_normal(const double (&v)[kOut]) {
  return __all(v[kOut - 1] >= 0x1p-1022 && v[0] < (double)INFINITY);
}

// Orders the wave's LDS writes before its lanes' reads of each other's values.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The output normalisation: y = (ln record - mean) / stdv.
struct Norm {
  double mean[kOut], stdv[kOut], rstd[kOut];   // rstd = 1 / stdv
  float fmean[kOut], fstd[kOut];
};

// (passed by value: no copy from the caller's memory to wait for)
__global__ void k_set_norm(Norm nm, Norm *out) {
  const int j = threadIdx.x;
  out->mean[j] = nm.mean[j];
  out->stdv[j] = nm.stdv[j];
  out->rstd[j] = nm.rstd[j];
  out->fmean[j] = nm.fmean[j];
  out->fstd[j] = nm.fstd[j];
}

// Network inputs and targets of n points: (p_A, ln f) mapped to [-1, 1]
// (k_net<.., true> normalises its inputs the same way), and y[i][j] =
// (ln rec[j][i] - mean_j) / std_j of the sorted records.  The rows of y are
// gathered in LDS (each lane has one) and stored 1 KB contiguous: storing 16
// bytes of every lane's row at a time took 72 us for 262144 points with the
// sort and the logarithms left out.
struct DatasetArgs {
  const double *prm, *rec;
  const Norm *norm;
  int64_t n;
  double lo0, sc0, lo1, sc1;
  float *x, *y;
  const LnEntry *lntab;
  bool plain;   // no step of the division by way of rstd leaves the normal range
  bool few;
};
__global__ __launch_bounds__(64 * kDsWaves, 2) void k_dataset(DatasetArgs a) {
  __shared__ LnEntry lntab[kLnTab];
  __shared__ float rows[kDsWaves][64][kRowLd];
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (a.few ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * kDsWaves + w) * 64;
  const int64_t i = i0 + l;
  const bool mine = i < a.n;
  if (threadIdx.x < kLnTab) lntab[threadIdx.x] = a.lntab[threadIdx.x];
  __syncthreads();
  if (i0 >= a.n) return;   // the whole wave
  double v[kOut];
  sorted_records(a.rec, a.n, i, v);
  if (mine && (!a.few || w == 0)) {
    a.x[2 * i] = (float)(fma(a.prm[i] - a.lo0, a.sc0, -1.0));
    a.x[2 * i + 1] = (float)(fma(log(a.prm[a.n + i]) - a.lo1, a.sc1, -1.0));
  }
  const Norm &nm = *a.norm;
  const bool normal = a.plain && all_normal(v);
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    if (a.few && g != w) continue;
    if (normal) {
#pragma unroll
      for (int j = kGrp * g; j < kGrp * (g + 1); j += 4) {
        f32x4 o;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          // the quotient by way of the reciprocal and one correction of the
          // residual (Markstein, 1990)
          const double d = ln_normal(lntab, v[j + u]) - nm.mean[j + u], q = d * nm.rstd[j + u];
          o[u] = (float)fma(fma(-q, nm.stdv[j + u], d), nm.rstd[j + u], q);
        }
        *(f32x4 *)&rows[w][l][j] = o;
      }
    } else {
#pragma unroll
      for (int j = kGrp * g; j < kGrp * (g + 1); j += 4) {
#pragma unroll 1
        for (int u = 0; u < 4; ++u) {
          const double x = u < 2 ? (u == 0 ? v[j] : v[j + 1]) : (u == 2 ? v[j + 2] : v[j + 3]);
          rows[w][l][j + u] = (float)((log(x) - nm.mean[j + u]) / nm.stdv[j + u]);
        }
      }
    }
  }
  wave_lds_sync();
  // whole rows: 4 a store, or the wave's quarter of 16
  const int c = a.few ? kGrp * w + 4 * (l & 3) : 4 * (l & 15);
  const int step = a.few ? 16 : 4;
  for (int r = a.few ? l >> 2 : l >> 4; r < 64 && i0 + r < a.n; r += step)
    *(f32x4_of_floats *)(a.y + (i0 + r) * kOut + c) = *(const f32x4 *)&rows[w][r][c];
}

// Count, mean and sum of squares about the mean of two sets together (Chan,
// Golub and LeVeque, 1983).
struct Moments {
  double n, mean, m2;
};
__device__ __forceinline__ Moments merged(const Moments &a, const Moments &b) {
  if (b.n == 0.0) return a;
  Moments c;
  c.n = a.n + b.n;
  const double d = b.mean - a.mean;
  c.mean = fma(d, b.n / c.n, a.mean);
  c.m2 = (a.m2 + b.m2) + d * d * (a.n * b.n / c.n);
  return c;
}

// Moments of ln (sorted records) of each output over n points: each wave's
// tile in two passes (the mean from the differences to the tile's first
// point) by 4 lanes per output, the block's tiles merged, to
// part[output][block].
__global__ __launch_bounds__(64 * kDsWaves, 2) void k_moments(const double *__restrict__ rec,
                                                              int64_t n, bool few,
                                                              const LnEntry *__restrict__ tab,
                                                              Moments *__restrict__ part) {
  // rows 65 apart: 16 outputs' values fall on different banks
  __shared__ double lds[kDsWaves][kGrp][65];
  __shared__ Moments tile[kDsWaves][kOut];
  __shared__ LnEntry lntab[kLnTab];
  if (threadIdx.x < kLnTab) lntab[threadIdx.x] = tab[threadIdx.x];
  __syncthreads();
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (few ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * kDsWaves + w) * 64;
  if (i0 < n) {
    const int jj = l & (kGrp - 1), q = l / kGrp;
    double *row = lds[w][jj];
    const int cnt = n - i0 < 64 ? (int)(n - i0) : 64;
    const int ke = cnt - 16 * q;   // the lane's values: k = 0 .. 15 with k < ke
    double v[kOut];
    sorted_records(rec, n, i0 + l, v);
    const bool normal = all_normal(v);
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      if (few && g != w) continue;
#pragma unroll
      for (int r = 0; r < kGrp; ++r)
        lds[w][r][l] = normal ? ln_normal(lntab, v[kGrp * g + r]) : v[kGrp * g + r];
      if (!normal)
#pragma unroll 1
        for (int r = 0; r < kGrp; ++r) lds[w][r][l] = log(lds[w][r][l]);
      wave_lds_sync();
      // the lane's 16 values, as differences to the tile's first point
      const double p = row[0];
      double d[16], sum = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        d[k] = k < ke ? row[16 * q + k] - p : 0.0;
        sum += d[k];
      }
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
      const double dm = sum / (double)cnt;
      double m2 = 0.0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double e = k < ke ? d[k] - dm : 0.0;
        m2 = fma(e, e, m2);
      }
      m2 += __shfl_xor(m2, 16);
      m2 += __shfl_xor(m2, 32);
      if (q == 0) tile[few ? 0 : w][kGrp * g + jj] = Moments{(double)cnt, p + dm, m2};
      wave_lds_sync();
      __builtin_amdgcn_sched_barrier(0);   // one group's values in registers at a time
    }
  } else if (!few) {
    tile[w][l] = Moments{0.0, 0.0, 0.0};
  }
  __syncthreads();
  if (threadIdx.x >= kOut) return;
  Moments m = tile[0][threadIdx.x];
  if (!few)
#pragma unroll
    for (int k = 1; k < kDsWaves; ++k) m = merged(m, tile[k][threadIdx.x]);
  part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = m;
}

// Mean and standard deviation of each output (one block each) from the
// moments of nb blocks, merged in a fixed order.
__global__ __launch_bounds__(256) void k_mean_std(const Moments *__restrict__ part, int64_t nb,
                                                  double *fit) {
  __shared__ Moments red[256];
  const int j = blockIdx.x, t = threadIdx.x;
  Moments m{0.0, 0.0, 0.0};
  for (int64_t i = t; i < nb; i += 256) m = merged(m, part[j * nb + i]);
  red[t] = m;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (t < k) red[t] = merged(red[t], red[t + k]);
    __syncthreads();
  }
  if (t == 0) {
    fit[j] = red[0].mean;
    fit[kOut + j] = sqrt(red[0].m2 / red[0].n);
  }
}

// ---------------------------------------------------------------- fused inference
// The whole network in one kernel, for a tile of 16 NJ points per block.
// The products are taken transposed, Z^T = W A^T (MFMA rows = output features,
// columns = points), so the accumulator of feature block fb and point block j
// holds, in lane 16 g + i, features 16 fb + 4 g + q of point 16 j + i.  Packed
// pairwise ((fb, fb + 1) = (2c, 2c + 1)) these are already the B fragments of
// the next layer's k chunk c, in the permuted k order
//     k slot 8 g + s  <->  feature 32 c + 16 (s / 4) + 4 g + s mod 4,
// so the weights of layers 3 and 4 are read with their columns permuted the
// same way; the feature layer's fragments are formed directly in the standard
// order.  A wave takes NF of a layer's 16 feature blocks, whose weights it
// loads into registers (in fragment order, while it forms the activations of
// the layer before), and all points of the tile; between layers the
// activations wait in LDS.  The arithmetic of every element is the training
// path's (same features, GELU and roundings to BF16) except for the order of
// the FP32 sums: the bias starts the accumulation here, and the k order inside
// an MFMA differs for layers 3 and 4.
//
// Many points: NJ = 4, NF = 2 (two blocks of 8 waves per CU).  4096 x 4096
// points take 7.3 ms (680 TFLOP/s): the vector unit, which forms 768 features
// a point, is issuing 77% of the time, beside matrix cores that are busy 30%.
// Before, each wave took 32 points through the whole network and read all
// weights for them (7.6 ms).  NJ = 2, 3, 6, 8, one feature block per wave, and
// blocks that stay for more tiles were slower (8.1 to 9.3 ms).
// Few points: NJ = 1, then 2, with NF = 1, so that a layer is spread over the
// 16 waves of a block and the points over all CUs: 1000 points 19.8 -> 6.4 us,
// 8192 points 20.3 -> 7.5 us (NJ = 1: 9.3 us; 12288 points with NJ = 4: 13 us).
// What bounds a call then is the 288 KB of weights that each CU reads from L2.

struct FusedArgs {
  int64_t n;                       // points
  const double *prm;               // screen: sweep parameters [2][n] (p_A, f)
  double lo0, sc0, lo1, sc1;       //   and their normalisation
  const float *x;                  // forward: normalised inputs [n][2]
  float *out;                      // forward: network outputs [n][64]
  const float *P;                  // master parameters (W1, b1, b2, b3, b4)
  const bf16 *W2f, *W3f, *W4f;     // BF16 weights in fragment order (3 and 4 k-permuted)
  // screen epilogue (screen_point)
  const float *mean, *stdv;
  float margin, spread, flag_margin, label_margin;
  const int8_t *nlab;
  int GL;
  int8_t *label;
  uint8_t *resolve;
  float *pmax;
  int64_t first;                   // the launch's first point
};

// Label and re-solve mask of point r from its predicted maximum and minimum
// and its normalised inputs.
__device__ __forceinline__ void screen_point(const FusedArgs &a, int64_t r, float xmx, float xmn,
                                             float u0f, float v0f) {
  const float ln2 = 0.69314718055994531f;
  const float d = fabsf(xmx - ln2);
  const bool unsure = d < a.margin;
  bool flag = (xmx - xmn > a.spread) && d < a.flag_margin;
  const int8_t lab = xmx >= ln2 ? 1 : 0;
  if (a.nlab) {
    const int GL = a.GL;
    const float u = (u0f + 1.0f) * 0.5f * (float)(GL - 1);
    const float v = (v0f + 1.0f) * 0.5f * (float)(GL - 1);
    int u0 = (int)floorf(u), v0 = (int)floorf(v);
    u0 = u0 < 0 ? 0 : (u0 > GL - 2 ? GL - 2 : u0);
    v0 = v0 < 0 ? 0 : (v0 > GL - 2 ? GL - 2 : v0);
    const int64_t b = (int64_t)u0 * GL + v0;
    const int k = (a.nlab[b] != lab) + (a.nlab[b + 1] != lab) + (a.nlab[b + GL] != lab) +
                  (a.nlab[b + GL + 1] != lab);
    flag = flag || k == 4 || (k > 0 && d < a.label_margin);
  }
  if (a.label) a.label[r] = lab;
  if (a.resolve) a.resolve[r] = (unsure || flag) ? 1 : 0;
  if (a.pmax) a.pmax[r] = xmx;
}

template <int NJ, int NF, bool SCREEN>
__global__ __launch_bounds__(64 * 16 / NF, 4) void k_net(FusedArgs a) {
  constexpr int NW = 16 / NF;            // waves
  constexpr int NP = 16 * NJ;            // points of the block
  typedef __attribute__((__vector_size__(4 * NF * sizeof(__bf16)))) __bf16 part;
  __shared__ bf16x8 act[2][8][NJ][64];   // [chunk][point block][lane], by turns
  __shared__ float xs[NP][2];            // normalised inputs
  __shared__ float red[2][kOut / 16][NP];   // maxima and minima over 16 outputs
  const int t = threadIdx.x, l = t & 63, g = l >> 4, i = l & 15;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t r0 = a.first + (int64_t)blockIdx.x * NP;
  const float *__restrict__ P = a.P;
  const int half = NF == 1 ? w & 1 : 0, chunk = NF * w >> 1;
  if (t < NP) {
    const int64_t r = r0 + t < a.n ? r0 + t : a.n - 1;
    if (SCREEN) {
      xs[t][0] = (float)(fma(a.prm[r] - a.lo0, a.sc0, -1.0));
      xs[t][1] = (float)(fma(log(a.prm[a.n + r]) - a.lo1, a.sc1, -1.0));
    } else {
      xs[t][0] = a.x[2 * r];
      xs[t][1] = a.x[2 * r + 1];
    }
  }
  // the wave's features of layer 1: 32 chunk + 8 g + 4 half + q
  float w0[4 * NF], w1[4 * NF], bb[4 * NF];
#pragma unroll
  for (int q = 0; q < 4 * NF; ++q) {
    const int f = 32 * chunk + 8 * g + 4 * half + q;
    w0[q] = P[oW1 + 2 * f];
    w1[q] = P[oW1 + 2 * f + 1];
    bb[q] = P[ob1 + f];
  }
  bf16x8 wt[8][NF];
  const int64_t at = (int64_t)NF * w * 8 * kFrag + l * 8;
#pragma unroll
  for (int c = 0; c < 8; ++c)
#pragma unroll
    for (int h = 0; h < NF; ++h) wt[c][h] = *(const bf16x8 *)(a.W2f + at + (h * 8 + c) * kFrag);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const float x0 = xs[16 * j + i][0], x1 = xs[16 * j + i][1];
    part v;
#pragma unroll
    for (int q = 0; q < 4 * NF; ++q)
      v[q] = (bf16)feature_sin(fmaf(x1, w1[q], fmaf(x0, w0[q], bb[q])));
    *((part *)&act[0][chunk][j][l] + half) = v;
  }
  __syncthreads();
  const int ob = w & 3;
#pragma unroll
  for (int L = 0; L < 2; ++L) {
    f32x4 acc[NF][NJ];
#pragma unroll
    for (int h = 0; h < NF; ++h) {
      const f32x4 b = *(const f32x4 *)(P + (L == 0 ? ob2 : ob3) + 16 * (NF * w + h) + 4 * g);
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[h][j] = b;
    }
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bf16x8 in = act[L][c][j][l];
#pragma unroll
        for (int h = 0; h < NF; ++h)
          acc[h][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[c][h], in, acc[h][j], 0, 0, 0);
      }
    // the next layer's weights
    if (L == 0) {
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int h = 0; h < NF; ++h)
          wt[c][h] = *(const bf16x8 *)(a.W3f + at + (h * 8 + c) * kFrag);
    } else if (w < 4 * NJ) {
#pragma unroll
      for (int c = 0; c < 8; ++c)
        wt[c][0] = *(const bf16x8 *)(a.W4f + (ob * 8 + c) * kFrag + l * 8);
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      part v;
#pragma unroll
      for (int h = 0; h < NF; ++h)
#pragma unroll
        for (int q = 0; q < 4; ++q) v[4 * h + q] = (bf16)gelu_f(acc[h][j][q]);
      *((part *)&act[1 - L][chunk][j][l] + half) = v;
    }
    __syncthreads();
  }
  // the output layer: output block ob of point blocks w / 4, w / 4 + NW / 4, ...
  const f32x4 b4 = *(const f32x4 *)(P + ob4 + 16 * ob + 4 * g);
#pragma unroll
  for (int j0 = 0; j0 < NJ; j0 += NW / 4) {
    const int j = j0 + (w >> 2);
    if (j >= NJ) break;
    f32x4 o = b4;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[c][0], act[0][c][j][l], o, 0, 0, 0);
    if (!SCREEN) {
      const int64_t r = r0 + 16 * j + i;
      if (r < a.n) *(f32x4_of_floats *)(a.out + r * kOut + 16 * ob + 4 * g) = o;
    } else {
      // de-standardised maximum and minimum over the wave's 16 outputs: 4 in
      // the lane, then across the four lane groups
      const f32x4 sd = *(const f32x4 *)(a.stdv + 16 * ob + 4 * g);
      const f32x4 mu = *(const f32x4 *)(a.mean + 16 * ob + 4 * g);
      float mx = -INFINITY, mn = INFINITY;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float v = fmaf(o[q], sd[q], mu[q]);
        mx = fmaxf(mx, v);
        mn = fminf(mn, v);
      }
#pragma unroll
      for (int off = 16; off < 64; off <<= 1) {
        mx = fmaxf(mx, __shfl_xor(mx, off));
        mn = fminf(mn, __shfl_xor(mn, off));
      }
      if (g == 0) {
        red[0][ob][16 * j + i] = mx;
        red[1][ob][16 * j + i] = mn;
      }
    }
  }
  if (!SCREEN) return;
  __syncthreads();
  if (t >= NP || r0 + t >= a.n) return;
  float mx = red[0][0][t], mn = red[1][0][t];
#pragma unroll
  for (int k = 1; k < kOut / 16; ++k) {
    mx = fmaxf(mx, red[0][k][t]);
    mn = fminf(mn, red[1][k][t]);
  }
  screen_point(a, r0 + t, mx, mn, xs[t][0], xs[t][1]);
}

// Exact label of each training node: [max_j rec[j][i] >= 2], -1 if a record
// is NaN.
__global__ void k_node_label(const double *__restrict__ rec, int64_t n, int8_t *lab) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double mx = -INFINITY;
  bool bad = false;
  for (int j = 0; j < kOut; ++j) {
    const double v = rec[j * n + i];
    bad = bad || isnan(v);
    mx = v > mx ? v : mx;
  }
  lab[i] = bad ? -1 : (mx >= 2.0 ? 1 : 0);
}

// Deterministic compaction of the re-solve mask: block counts, one-block
// exclusive scan, ordered write.  A thread takes 16 flags.  16.8 million
// flags: k_count 5, k_scan 5, k_write_idx 12 us (46, 41 and 80 us with one
// flag a thread, scans of 10 barriers and the block counts' scan in one
// thread).
constexpr int kScanThreads = 256, kScanPer = 16, kScanBlock = kScanThreads * kScanPer;

// Bit k: flag i0 + k is set (none past n).
__device__ __forceinline__ unsigned flag_bits(const uint8_t *__restrict__ f, int64_t i0, int64_t n) {
  unsigned bits = 0;
  if (i0 + kScanPer <= n && ((uintptr_t)f & 15) == 0) {
    const uint4 v = *(const uint4 *)(f + i0);
    const unsigned q[4] = {v.x, v.y, v.z, v.w};
    // flags are bytes 0 or 1: bit 0 of byte b goes to bit 28 + b
#pragma unroll
    for (int k = 0; k < 4; ++k) bits |= (q[k] * 0x10204080u) >> 28 << (4 * k);
  } else {
    for (int k = 0; k < kScanPer; ++k)
      if (i0 + k < n && f[i0 + k]) bits |= 1u << k;
  }
  return bits;
}

// Sum of v over the threads before this one of the block (T threads), and
// over all of them (*total).
template <int T>
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t *total) {
  __shared__ int64_t wsum[T / 64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t x = v;   // inclusive sum over the wave
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t y = __shfl_up(x, d);
    if (l >= d) x += y;
  }
  if (l == 63) wsum[w] = x;
  __syncthreads();
  int64_t before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < T / 64; ++k) {
    if (k < w) before += wsum[k];
    all += wsum[k];
  }
  *total = all;
  return before + x - v;
}

__global__ __launch_bounds__(kScanThreads) void k_count(const uint8_t *__restrict__ f, int64_t n,
                                                        int64_t *counts) {
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * kScanPer;
  int64_t total;
  block_scan<kScanThreads>(__popc(flag_bits(f, i0, n)), &total);
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_scan(int64_t *counts, int64_t nb, int64_t *total) {
  const int64_t per = (nb + 1023) / 1024;
  const int64_t b = threadIdx.x * per, e = b + per < nb ? b + per : nb;
  int64_t s = 0, all;
  for (int64_t i = b; i < e; ++i) s += counts[i];
  int64_t run = block_scan<1024>(s, &all);
  for (int64_t i = b; i < e; ++i) {
    const int64_t v = counts[i];
    counts[i] = run;
    run += v;
  }
  if (threadIdx.x == 0) *total = all;
}

__global__ __launch_bounds__(kScanThreads) void k_write_idx(const uint8_t *__restrict__ f, int64_t n,
                                                            const int64_t *offs, int64_t *idx) {
  const int64_t i0 = (int64_t)blockIdx.x * kScanBlock + threadIdx.x * kScanPer;
  unsigned bits = flag_bits(f, i0, n);
  int64_t total;
  int64_t at = offs[blockIdx.x] + block_scan<kScanThreads>(__popc(bits), &total);
  for (; bits; bits &= bits - 1) idx[at++] = i0 + (__ffs(bits) - 1);
}

// label[idx[i]] = [max_j rec[j][i] >= 2]; -1 if any record is NaN.
__global__ void k_exact_labels(const double *__restrict__ rec, int64_t k,
                               const int64_t *__restrict__ idx, int8_t *label) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= k) return;
  double mx = -INFINITY;
  bool bad = false;
  for (int j = 0; j < kOut; ++j) {
    const double v = rec[j * k + i];
    bad = bad || isnan(v);
    mx = v > mx ? v : mx;
  }
  label[idx ? idx[i] : i] = bad ? -1 : (mx >= 2.0 ? 1 : 0);
}

}  // namespace

// ======================================================================== API

struct sur_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  int64_t max_batch = 0;
  std::string err;
  double lr = 1e-3, b1 = 0.9, b2 = 0.999, eps = 1e-8;
  int64_t t = 0;
  double in_lo[2] = {0, 0}, in_hi[2] = {1, 1};
  double out_mean[kOut], out_std[kOut];
  bool have_norm = false, norm_plain = false;   // norm_plain: DatasetArgs::plain
  char *arena = nullptr;   // the arrays of fixed size, down to adam_h
  // parameters and optimiser state
  float *P = nullptr, *G = nullptr, *Mm = nullptr, *V = nullptr;
  WeightCopies W = {};
  Norm *norm = nullptr;       // the output normalisation, in device memory
  // one batch: inputs and targets, the activations and gradients in
  // fragment order over the batch for the weight-gradient products
  float *x = nullptr, *tgt = nullptr;
  bf16 *a1 = nullptr, *a2 = nullptr, *a3 = nullptr;
  bf16 *dz4 = nullptr, *dz3 = nullptr, *dz2 = nullptr;
  // partial sums of the gradients: split-K weight products, per-16-row-tile
  // column sums (biases), loss
  float *part2 = nullptr, *part3 = nullptr, *part4 = nullptr;
  float *cp2 = nullptr, *cp3 = nullptr,
        *cp4 = nullptr;
  float *lpart = nullptr;     // loss partials
  float *loss = nullptr;      // device scalar
  float *loss_acc = nullptr;  // device scalar: sum of batch losses of an epoch
  int64_t *scan = nullptr;    // compaction scratch
  int64_t scan_cap = 0;
  int8_t *nlab = nullptr;     // exact labels of the training grid [G][G]
  LnEntry *lntab = nullptr;
  // Pinned host memory that kernels write small results to (the host reads
  // them after its wait, without a copy): means and standard deviations of
  // sur_fit_norm; a screen's number of points to re-solve (an 8-byte copy back
  // took 9 of a small screen's 62 us)
  double *pin = nullptr, *pin_d = nullptr;   // [2 kOut]: host's and device's address
  Moments *mom = nullptr;     // [kOut][blocks] (sur_fit_norm), grown as needed
  int64_t mom_nb = 0;
  int nlab_G = 0;
  // captured training epoch (sur_train_epoch), replayed while the dataset,
  // row list and batch are the same
  hipStream_t cap_stream = nullptr;
  hipGraph_t ep_graph = nullptr;
  hipGraphExec_t ep_exec = nullptr;
  const float *ep_x = nullptr, *ep_y = nullptr;
  const int64_t *ep_perm = nullptr;
  int64_t ep_n = 0, ep_batch = 0;
  double *hyper = nullptr;   // device: lr, beta1, beta2, eps, t_base
  double hyper_host[5] = {0, 0, 0, 0, 0};
  float *adam_h = nullptr;   // device: the running step's constants (adam_constants)
  // inference: staging of host inputs and outputs (sur_forward from host
  // memory: kInferRows rows, allocated on first use)
  float *ix = nullptr, *iout = nullptr;
};

namespace {

// Batch split of a weight-gradient product: chunks of 256 rows where the
// batch allows (at most kSplit of them), else chunks of a multiple of 64 rows
// (m is a multiple of 64).  Returns log2 of the split.
int wgrad_lsplit(int64_t m) {
  for (int ls = kLSplit; ls > 0; --ls)
    if (m % (64 << ls) == 0 && (m >> ls) >= 256) return ls;
  return 0;
}

thread_local std::string g_serr;

int sfail(sur_ctx *s, int code, const std::string &m) {
  g_serr = m;
  if (s) s->err = m;
  return code;
}

#define SUR_HIP(ctx, call)                                                              \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess)                                                               \
      return sfail((ctx), e_ == hipErrorOutOfMemory ? ENS_E_NOMEM : ENS_E_HIP,          \
                   std::string(#call) + ": " + hipGetErrorString(e_));                  \
  } while (0)

struct DevGuard {
  int prev = -1;
  explicit DevGuard(int d) {
    if (hipGetDevice(&prev) == hipSuccess) (void)hipSetDevice(d);
  }
  ~DevGuard() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

template <class T>
hipError_t alloc(T **p, int64_t count) {
  return hipMalloc((void **)p, (size_t)(count > 0 ? count : 1) * sizeof(T));
}

unsigned nblk(int64_t count, int b) { return (unsigned)((count + b - 1) / b); }

// The three products of bt.g (each R a multiple of 32) over m rows of the
// batch in one launch, m / split a multiple of 64 (m <= 65536).
hipError_t gemm3(hipStream_t st, GemmBatch bt, int64_t m, int lsplit) {
  bt.lsplit = lsplit;
  bt.kchunk = (int)(m >> lsplit);
  int total = 0;
  for (int p = 0; p < 3; ++p) {
    bt.ntile[p] = (bt.g[p].R / kTile) * (kH / kTile);
    total += bt.ntile[p] << lsplit;
  }
  total += 1;   // the Adam constants
  if (bt.kchunk % 256 == 0)
    hipLaunchKernelGGL((k_gemm<8>), dim3((unsigned)total), dim3(64), 0, st, bt);
  else
    hipLaunchKernelGGL((k_gemm<2>), dim3((unsigned)total), dim3(64), 0, st, bt);
  return hipGetLastError();
}

constexpr int64_t kInferRows = 65536;

hipError_t ensure_infer(sur_ctx *s) {
  if (s->ix) return hipSuccess;
  hipError_t e = hipMalloc((void **)&s->ix, kInferRows * kIn * sizeof(float));
  if (e == hipSuccess) e = hipMalloc((void **)&s->iout, kInferRows * kOut * sizeof(float));
  if (e != hipSuccess) {
    (void)hipFree(s->ix);
    (void)hipFree(s->iout);
    s->ix = s->iout = nullptr;
  }
  return e;
}

// Compaction scratch (block counts and their scan) for screens of up to n
// points, grown when a larger screen comes.
hipError_t reserve_scan(sur_ctx *s, int64_t n) {
  const int64_t need = (n + kScanBlock - 1) / kScanBlock;
  if (need <= s->scan_cap) return hipSuccess;
  (void)hipFree(s->scan);
  s->scan = nullptr;
  s->scan_cap = 0;
  const hipError_t e = hipMalloc((void **)&s->scan, (size_t)need * sizeof(int64_t));
  if (e == hipSuccess) s->scan_cap = need;
  return e;
}

// The fused inference of n points (n > 0), kNetPoints a launch: a launch's
// threads are counted in 32 bits (a larger grid is cut without an error), and
// k_net<4, 2> takes 8 a point.
constexpr int64_t kNetPoints = 1 << 28;
static_assert(kNetPoints * 8 <= UINT32_MAX && kNetPoints % 64 == 0, "threads of a launch");
hipError_t fused_launch(hipStream_t st, const FusedArgs &a, int64_t count, bool screen) {
  // few points: one tile per CU (256 of them) while that can be had (a screen
  // takes 64 points a block at any size: the smaller tiles have been measured
  // for the forward only)
  const dim3 g1(nblk(count, 16)), g2(nblk(count, 32)), g4(nblk(count, 64));
  if (screen)
    hipLaunchKernelGGL((k_net<4, 2, true>), g4, dim3(512), 0, st, a);
  else if (count <= 16 * 256)
    hipLaunchKernelGGL((k_net<1, 1, false>), g1, dim3(1024), 0, st, a);
  else if (count <= 32 * 256)
    hipLaunchKernelGGL((k_net<2, 1, false>), g2, dim3(1024), 0, st, a);
  else
    hipLaunchKernelGGL((k_net<4, 2, false>), g4, dim3(512), 0, st, a);
  return hipGetLastError();
}
hipError_t fused(sur_ctx *s, FusedArgs a, bool screen) {
  a.P = s->P;
  a.W2f = s->W.W2;
  a.W3f = s->W.W3p;
  a.W4f = s->W.W4p;
  hipError_t e = hipSuccess;
  for (a.first = 0; a.first < a.n && e == hipSuccess; a.first += kNetPoints)
    e = fused_launch(s->stream, a, a.n - a.first < kNetPoints ? a.n - a.first : kNetPoints, screen);
  return e;
}

// The source of a step's Adam constants: hyper-parameters from device memory
// (hyper != NULL, a captured step `step`) or the handle's.
AdamHyper adam_hyper(sur_ctx *s, const double *hyper, int step) {
  return AdamHyper{hyper, s->lr, s->b1, s->b2, s->eps, (double)s->t, step, s->adam_h};
}

// One batch's loss and gradients of all parameters into s->G and s->loss:
// the fused tile kernel (forward, loss gradient, data gradients), then the
// weight gradients (split over the batch) and the fixed-order reduction,
// which with ad != NULL also takes the Adam step.  Inputs: row r of x and
// tgt, or row rows[r] with rows; loss_acc (optional) accumulates the loss
// (first: starts it).
hipError_t train_batch(sur_ctx *s, int64_t m, const float *x, const float *tgt,
                       const int64_t *rows, float *loss_acc = nullptr, bool first = true,
                       const AdamHyper *ad = nullptr) {
  hipStream_t st = s->stream;
  hipError_t e;
  const int lsplit = wgrad_lsplit(m), split = 1 << lsplit;
  const int64_t T = m / kTR;
  TrainArgs a;
  a.x = x;
  a.rows = rows;
  a.tgt = tgt;
  a.P = s->P;
  a.W = s->W;
  a.m = (int)m;
  a.lsplit = lsplit;
  a.a1 = s->a1;
  a.a2 = s->a2;
  a.a3 = s->a3;
  a.dz4 = s->dz4;
  a.dz3 = s->dz3;
  a.dz2 = s->dz2;
  a.cp4 = s->cp4;
  a.cp3 = s->cp3;
  a.cp2 = s->cp2;
  a.lpart = s->lpart;
  hipLaunchKernelGGL(k_train_fb, dim3((unsigned)T), dim3(64 * kFbWaves), 0, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  GemmBatch bt;
  bt.g[0] = GemmArgs{s->dz4, s->a3, kOut, s->part4};
  bt.g[1] = GemmArgs{s->dz3, s->a2, kH, s->part3};
  bt.g[2] = GemmArgs{s->dz2, s->a1, kH, s->part2};
  bt.ad = ad ? *ad : AdamHyper{};
  if ((e = gemm3(st, bt, m, lsplit)) != hipSuccess) return e;
  GradParts p{s->part2, s->part3, s->cp2, s->cp3, s->part4, s->cp4, s->lpart};
  const AdamArgs aa{s->P, s->Mm, s->V, s->adam_h, s->W};
  const dim3 rg(kRedBlocks);
  if (ad)
    hipLaunchKernelGGL(k_reduce_grads<true>, rg, dim3(256), 0, st, p, T, split,
                       (float)(m * kOut), s->G, s->loss, loss_acc, first ? 1 : 0, aa);
  else
    hipLaunchKernelGGL(k_reduce_grads<false>, rg, dim3(256), 0, st, p, T, split,
                       (float)(m * kOut), s->G, s->loss, loss_acc, first ? 1 : 0, aa);
  return hipGetLastError();
}

void free_epoch_graph(sur_ctx *s) {
  if (s->ep_exec) (void)hipGraphExecDestroy(s->ep_exec);
  if (s->ep_graph) (void)hipGraphDestroy(s->ep_graph);
  s->ep_exec = nullptr;
  s->ep_graph = nullptr;
}

hipError_t refresh(sur_ctx *s) {
  hipLaunchKernelGGL(k_refresh, dim3(nblk(kH * kH / 4, 256)), dim3(256), 0, s->stream, s->P, s->W);
  return hipGetLastError();
}

int check_batch(sur_ctx *s, int64_t m) {
  if (m <= 0 || m % 64 || m > s->max_batch)
    return sfail(s, ENS_E_INVAL, "batch must be a positive multiple of 64 <= max_batch");
  return ENS_OK;
}

int load_batch(sur_ctx *s, const float *x, const float *tgt, int64_t m, int where) {
  const hipMemcpyKind k = where == ENS_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
  SUR_HIP(s, hipMemcpyAsync(s->x, x, (size_t)m * kIn * sizeof(float), k, s->stream));
  if (tgt)
    SUR_HIP(s, hipMemcpyAsync(s->tgt, tgt, (size_t)m * kOut * sizeof(float), k, s->stream));
  return ENS_OK;
}

// Captures the launches of one epoch over perm[0 .. n) (once per dataset,
// row-list buffer and batch); replays read the hyper-parameters and the row
// list's contents from device memory.
int ensure_epoch_graph(sur_ctx *s, const float *x, const float *y, int64_t n, const int64_t *perm,
                       int64_t batch) {
  const int64_t nb = n / batch;
  if (s->ep_exec && s->ep_x == x && s->ep_y == y && s->ep_perm == perm && s->ep_n == n &&
      s->ep_batch == batch)
    return ENS_OK;
  free_epoch_graph(s);
  hipStream_t user = s->stream;
  s->stream = s->cap_stream;
  hipError_t e = hipStreamBeginCapture(s->cap_stream, hipStreamCaptureModeThreadLocal);
  for (int64_t b = 0; e == hipSuccess && b < nb; ++b) {
    const int64_t *rows = perm + b * batch;
    // the step's Adam update from the hyper-parameters in s->hyper
    const AdamHyper ad = adam_hyper(s, s->hyper, (int)b);
    e = train_batch(s, batch, x, y, rows, s->loss_acc, b == 0, &ad);
  }
  hipGraph_t gr = nullptr;
  const hipError_t e2 = hipStreamEndCapture(s->cap_stream, &gr);
  s->stream = user;
  if (e != hipSuccess || e2 != hipSuccess) {
    if (gr) (void)hipGraphDestroy(gr);
    return sfail(s, ENS_E_HIP, std::string("training epoch capture: ") +
                                   hipGetErrorString(e != hipSuccess ? e : e2));
  }
  s->ep_graph = gr;
  SUR_HIP(s, hipGraphInstantiate(&s->ep_exec, gr, nullptr, nullptr, 0));
  s->ep_x = x;
  s->ep_y = y;
  s->ep_perm = perm;
  s->ep_n = n;
  s->ep_batch = batch;
  return ENS_OK;
}

// Epoch e's row order: the training rows sorted by a hash of (seed, e, i)
// (SplitMix64's output function of a Weyl sequence), i.e. a seeded uniformly
// random permutation; equal keys keep index order.  The orders of several
// epochs are made at once: all their (epoch, row) pairs are sorted by the
// hash, then, stably, by the epoch.
__global__ void k_epoch_keys(int64_t n, int64_t count, uint64_t seed, int64_t epoch,
                             unsigned long long *key, uint32_t *val) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  uint64_t z = seed + 0x9E3779B97F4A7C15ull * (uint64_t)(epoch * n + p + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  key[p] = (unsigned long long)(z ^ (z >> 31));
  val[p] = (uint32_t)p;
}
// A sorted pair p = epoch n + i as the key and the value of the second sort.
__global__ void k_epoch_rows(const int64_t *__restrict__ rows, uint32_t n, int64_t count,
                             const uint32_t *__restrict__ val, uint32_t *epoch, int64_t *row) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  const uint32_t e = val[p] / n;
  epoch[p] = e;
  row[p] = rows[val[p] - e * n];
}

// The row orders of up to `group` epochs at a time, [epochs][n], in one
// allocation.  At most 2^20 pairs a group: a sort of 65536 pairs is 10 launches
// of some 6 us, bound by their latency, and so is one of 10 times as many.  10
// epochs of 65536 rows in batches of 4096: 4.31 -> 4.05 ms.
constexpr int64_t kOrderPairs = 1 << 20;
// Rows of an epoch: a launch over them, in blocks of 256 threads, has fewer
// than 2^32 threads, and a pair's number fits val.
constexpr int64_t kEpochRows = ((int64_t)1 << 32) - 256;
struct EpochOrders {
  int64_t n, group;
  size_t tmp = 0;
  unsigned long long *key_in, *key_out;
  uint32_t *val_in, *val_out;
  int64_t *rows, *order;   // the second sort's values, in and out
  void *sort_tmp;

  size_t size(int64_t n_, int64_t epochs, hipStream_t st, hipError_t *e) {
    n = n_;
    group = n < kOrderPairs ? kOrderPairs / n : 1;
    group = group < epochs ? group : epochs;
    const size_t m = (size_t)(n * group);
    size_t t1 = 0, t2 = 0;
    *e = rocprim::radix_sort_pairs(nullptr, t1, (const unsigned long long *)nullptr,
                                   (unsigned long long *)nullptr, (const uint32_t *)nullptr,
                                   (uint32_t *)nullptr, m, 0u, 64u, st);
    if (*e == hipSuccess)
      *e = rocprim::radix_sort_pairs(nullptr, t2, (const uint32_t *)nullptr, (uint32_t *)nullptr,
                                     (const int64_t *)nullptr, (int64_t *)nullptr, m, 0u, 32u, st);
    tmp = t1 > t2 ? t1 : t2;
    return 3 * part(m * 8) + 2 * part(m * 4) + tmp;
  }
  static size_t part(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
  void place(char *b) {
    const size_t m = (size_t)(n * group);
    key_in = (unsigned long long *)b;
    key_out = (unsigned long long *)(b + part(m * 8));
    order = (int64_t *)(b + 2 * part(m * 8));
    val_in = (uint32_t *)(b + 3 * part(m * 8));
    val_out = (uint32_t *)(b + 3 * part(m * 8) + part(m * 4));
    rows = (int64_t *)key_in;   // the keys are done with by then
    sort_tmp = b + 3 * part(m * 8) + 2 * part(m * 4);
  }
  // Orders of epochs first .. first + count - 1 (count <= group).
  hipError_t make(const int64_t *rows_in, uint64_t seed, int64_t first, int64_t count,
                  hipStream_t st) {
    const int64_t m = n * count;
    hipLaunchKernelGGL(k_epoch_keys, dim3(nblk(m, 256)), dim3(256), 0, st, n, m, seed, first,
                       key_in, val_in);
    hipError_t e = hipGetLastError();
    size_t t = tmp;
    if (e == hipSuccess)
      e = rocprim::radix_sort_pairs(sort_tmp, t, key_in, key_out, val_in, val_out, (size_t)m, 0u,
                                    64u, st);
    if (e != hipSuccess) return e;
    // one epoch: its rows are in order
    int64_t *to = count > 1 ? rows : order;
    hipLaunchKernelGGL(k_epoch_rows, dim3(nblk(m, 256)), dim3(256), 0, st, rows_in, (uint32_t)n, m,
                       val_out, val_in, to);
    e = hipGetLastError();
    if (e != hipSuccess || count == 1) return e;
    unsigned bits = 0;
    while (((int64_t)1 << bits) < count) ++bits;
    t = tmp;
    return rocprim::radix_sort_pairs(sort_tmp, t, val_in, val_out, rows, order, (size_t)m, 0u,
                                     bits, st);
  }
};

}  // namespace

extern "C" {

const char *sur_last_error(sur_t s) { return s ? s->err.c_str() : g_serr.c_str(); }

int sur_create(int32_t device, void *hip_stream, int64_t max_batch, sur_t *out) {
  if (!out) return sfail(nullptr, ENS_E_INVAL, "sur_create: out is NULL");
  *out = nullptr;
  if (max_batch <= 0 || max_batch % 64 || max_batch > 65536)
    return sfail(nullptr, ENS_E_INVAL, "sur_create: max_batch must be a multiple of 64 in [64, 65536]");
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0)
    return sfail(nullptr, ENS_E_HIP, "sur_create: no HIP device");
  if (device < 0 || device >= ndev) return sfail(nullptr, ENS_E_INVAL, "sur_create: bad device");
  sur_ctx *s = new (std::nothrow) sur_ctx();
  if (!s) return sfail(nullptr, ENS_E_NOMEM, "sur_create: out of host memory");
  s->device = device;
  s->stream = (hipStream_t)hip_stream;
  s->max_batch = max_batch;
  for (int j = 0; j < kOut; ++j) {
    s->out_mean[j] = 0.0;
    s->out_std[j] = 1.0;
  }
  DevGuard dg(device);
  const int64_t B = max_batch;
  hipError_t e = hipSuccess;
  // every device array in one allocation (a handle for batches of 4096 takes 75
  // us to create, 180 us with one allocation each), placed by the second
  // of two passes, the first of which adds up the sizes
  size_t at = 0;
  for (int pass = 0; pass < 2 && e == hipSuccess; ++pass) {
    at = 0;
    const auto A = [&](auto &ptr, int64_t count) {
      if (pass) ptr = (std::remove_reference_t<decltype(ptr)>)(s->arena + at);
      at += ((size_t)count * sizeof(*ptr) + 255) & ~(size_t)255;
    };
    A(s->P, kNP); A(s->G, kNP); A(s->Mm, kNP); A(s->V, kNP);
    A(s->W.W2, kH * kH); A(s->W.W3, kH * kH); A(s->W.W3T, kH * kH); A(s->W.W3p, kH * kH);
    A(s->W.W4, kOut * kH); A(s->W.W4T, kOut * kH); A(s->W.W4p, kOut * kH);
    A(s->norm, 1); A(s->lntab, kLnTab);
    A(s->x, B * kIn); A(s->tgt, B * kOut);
    A(s->a1, B * kH); A(s->a2, B * kH); A(s->a3, B * kH);
    A(s->dz4, B * kOut); A(s->dz3, B * kH); A(s->dz2, B * kH);
    A(s->part2, (int64_t)kSplit * kH * kH); A(s->part3, (int64_t)kSplit * kH * kH);
    A(s->part4, (int64_t)kSplit * kOut * kH);
    A(s->cp2, B / kTR * kH); A(s->cp3, B / kTR * kH); A(s->cp4, B / kTR * kOut);
    A(s->lpart, B / kTR); A(s->loss, 1); A(s->loss_acc, 1);
    A(s->hyper, 5); A(s->adam_h, 6);
    if (!pass) e = alloc(&s->arena, (int64_t)at);
  }
  if (e == hipSuccess)
    e = hipHostMalloc((void **)&s->pin, 2 * kOut * sizeof(double), hipHostMallocMapped);
  if (e == hipSuccess) e = hipHostGetDevicePointer((void **)&s->pin_d, s->pin, 0);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&s->cap_stream, hipStreamNonBlocking);
  // P, G, Mm, V (the feature layer's gradients stay 0: no kernel writes them)
  if (e == hipSuccess)
    e = hipMemsetAsync(s->P, 0, (char *)s->W.W2 - (char *)s->P, s->stream);
  if (e == hipSuccess) e = refresh(s);
  LnEntry lntab[kLnTab];
  ln_table(lntab);
  if (e == hipSuccess)
    e = hipMemcpyAsync(s->lntab, lntab, sizeof(lntab), hipMemcpyHostToDevice, s->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
  if (e != hipSuccess) {
    int code = sfail(nullptr, e == hipErrorOutOfMemory ? ENS_E_NOMEM : ENS_E_HIP,
                     std::string("sur_create: ") + hipGetErrorString(e));
    sur_destroy(s);
    return code;
  }
  *out = s;
  return ENS_OK;
}

int sur_destroy(sur_t s) {
  if (!s) return ENS_OK;
  DevGuard dg(s->device);
  (void)hipStreamSynchronize(s->stream);
  void *ptrs[] = {s->arena, s->scan, s->nlab, s->mom, s->ix, s->iout};
  for (void *p : ptrs) (void)hipFree(p);
  free_epoch_graph(s);
  if (s->pin) (void)hipHostFree(s->pin);
  if (s->cap_stream) (void)hipStreamDestroy(s->cap_stream);
  delete s;
  return ENS_OK;
}

int sur_set_params(sur_t s, const double *flat) {
  if (!s || !flat) return sfail(s, ENS_E_INVAL, "sur_set_params: NULL argument");
  std::vector<float> f(kNP);
  for (int64_t i = 0; i < kNP; ++i) {
    if (!std::isfinite(flat[i])) return sfail(s, ENS_E_INVAL, "sur_set_params: non-finite value");
    f[i] = (float)flat[i];
  }
  DevGuard dg(s->device);
  SUR_HIP(s, hipMemcpyAsync(s->P, f.data(), kNP * sizeof(float), hipMemcpyHostToDevice, s->stream));
  SUR_HIP(s, hipMemsetAsync(s->Mm, 0, kNP * sizeof(float), s->stream));
  SUR_HIP(s, hipMemsetAsync(s->V, 0, kNP * sizeof(float), s->stream));
  SUR_HIP(s, refresh(s));
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  s->t = 0;
  return ENS_OK;
}

int sur_get_params(sur_t s, double *flat) {
  if (!s || !flat) return sfail(s, ENS_E_INVAL, "sur_get_params: NULL argument");
  std::vector<float> f(kNP);
  DevGuard dg(s->device);
  SUR_HIP(s, hipMemcpyAsync(f.data(), s->P, kNP * sizeof(float), hipMemcpyDeviceToHost, s->stream));
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  for (int64_t i = 0; i < kNP; ++i) flat[i] = f[i];
  return ENS_OK;
}

int sur_set_norm(sur_t s, const double *in_lo, const double *in_hi, const double *out_mean,
                 const double *out_std) {
  if (!s || !in_lo || !in_hi || !out_mean || !out_std)
    return sfail(s, ENS_E_INVAL, "sur_set_norm: NULL argument");
  for (int i = 0; i < 2; ++i)
    if (!(in_hi[i] > in_lo[i]) || !std::isfinite(in_lo[i]) || !std::isfinite(in_hi[i]))
      return sfail(s, ENS_E_INVAL, "sur_set_norm: need finite in_lo < in_hi");
  for (int j = 0; j < kOut; ++j)
    if (!(out_std[j] > 0.0) || !std::isfinite(out_mean[j]) || !std::isfinite(out_std[j]))
      return sfail(s, ENS_E_INVAL, "sur_set_norm: need finite mean and std > 0");
  Norm nm;
  s->norm_plain = true;
  for (int i = 0; i < 2; ++i) {
    s->in_lo[i] = in_lo[i];
    s->in_hi[i] = in_hi[i];
  }
  for (int j = 0; j < kOut; ++j) {
    s->out_mean[j] = out_mean[j];
    s->out_std[j] = out_std[j];
    nm.mean[j] = out_mean[j];
    nm.stdv[j] = out_std[j];
    nm.rstd[j] = 1.0 / out_std[j];
    nm.fmean[j] = (float)out_mean[j];
    nm.fstd[j] = (float)out_std[j];
    s->norm_plain = s->norm_plain && out_std[j] >= 1e-100 && out_std[j] <= 1e100 &&
                    std::fabs(out_mean[j]) <= 1e100;
  }
  DevGuard dg(s->device);
  hipLaunchKernelGGL(k_set_norm, dim3(1), dim3(kOut), 0, s->stream, nm, s->norm);
  SUR_HIP(s, hipGetLastError());
  s->have_norm = true;
  return ENS_OK;
}

int sur_build_dataset(sur_t s, const double *params, const double *records, int64_t n, float *x,
                      float *y) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_build_dataset: NULL handle");
  if (!s->have_norm) return sfail(s, ENS_E_ORDER, "sur_build_dataset: call sur_set_norm first");
  if (n < 0 || (n > 0 && (!params || !records || !x || !y)))
    return sfail(s, ENS_E_INVAL, "sur_build_dataset: bad arguments");
  if (n == 0) return ENS_OK;
  DevGuard dg(s->device);
  const double sc0 = 2.0 / (s->in_hi[0] - s->in_lo[0]), sc1 = 2.0 / (s->in_hi[1] - s->in_lo[1]);
  const DatasetArgs a{params, records, s->norm, n, s->in_lo[0], sc0, s->in_lo[1], sc1,
                      x, y, s->lntab, s->norm_plain, few_points(n)};
  hipLaunchKernelGGL(k_dataset, dim3(nblk(n, a.few ? 64 : 64 * kDsWaves)), dim3(64 * kDsWaves), 0, s->stream, a);
  SUR_HIP(s, hipGetLastError());
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  return ENS_OK;
}

int sur_set_adam(sur_t s, double lr, double beta1, double beta2, double eps) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_set_adam: NULL handle");
  if (!(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0))
    return sfail(s, ENS_E_INVAL, "sur_set_adam: bad hyper-parameters");
  s->lr = lr;
  s->b1 = beta1;
  s->b2 = beta2;
  s->eps = eps;
  return ENS_OK;
}

int sur_gradients(sur_t s, const float *x, const float *target, int64_t m, float *grads,
                  float *loss, int32_t where) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_gradients: NULL handle");
  if (int rc = check_batch(s, m)) return rc;
  if (!x || !target) return sfail(s, ENS_E_INVAL, "sur_gradients: NULL input");
  DevGuard dg(s->device);
  if (int rc = load_batch(s, x, target, m, where)) return rc;
  SUR_HIP(s, train_batch(s, m, s->x, s->tgt, nullptr));
  const hipMemcpyKind k = where == ENS_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  if (grads) SUR_HIP(s, hipMemcpyAsync(grads, s->G, kNP * sizeof(float), k, s->stream));
  if (loss) SUR_HIP(s, hipMemcpyAsync(loss, s->loss, sizeof(float), k, s->stream));
  if (where == ENS_HOST) SUR_HIP(s, hipStreamSynchronize(s->stream));
  return ENS_OK;
}

int sur_train_step(sur_t s, const float *x, const float *target, int64_t m, float *loss,
                   int32_t where) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_train_step: NULL handle");
  if (int rc = check_batch(s, m)) return rc;
  if (!x || !target) return sfail(s, ENS_E_INVAL, "sur_train_step: NULL input");
  DevGuard dg(s->device);
  if (int rc = load_batch(s, x, target, m, where)) return rc;
  const AdamHyper ad = adam_hyper(s, nullptr, 0);
  SUR_HIP(s, train_batch(s, m, s->x, s->tgt, nullptr, nullptr, true, &ad));
  s->t += 1;
  if (loss) {
    const hipMemcpyKind k = where == ENS_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
    SUR_HIP(s, hipMemcpyAsync(loss, s->loss, sizeof(float), k, s->stream));
    if (where == ENS_HOST) SUR_HIP(s, hipStreamSynchronize(s->stream));
  }
  return ENS_OK;
}

int sur_forward(sur_t s, const float *x, int64_t m, float *out, int32_t where) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_forward: NULL handle");
  if (m < 0 || (m > 0 && (!x || !out))) return sfail(s, ENS_E_INVAL, "sur_forward: bad arguments");
  DevGuard dg(s->device);
  if (m == 0) return ENS_OK;
  FusedArgs a;
  std::memset(&a, 0, sizeof(a));
  if (where == ENS_DEVICE) {
    a.n = m;
    a.x = x;
    a.out = out;
    SUR_HIP(s, fused(s, a, false));
    return ENS_OK;
  }
  // host buffers: staged through the handle's buffers kInferRows rows at a time
  SUR_HIP(s, ensure_infer(s));
  for (int64_t first = 0; first < m; first += kInferRows) {
    const int64_t rows = m - first < kInferRows ? m - first : kInferRows;
    SUR_HIP(s, hipMemcpyAsync(s->ix, x + first * kIn, rows * kIn * sizeof(float),
                              hipMemcpyHostToDevice, s->stream));
    a.n = rows;
    a.x = s->ix;
    a.out = s->iout;
    SUR_HIP(s, fused(s, a, false));
    SUR_HIP(s, hipMemcpyAsync(out + first * kOut, s->iout, rows * kOut * sizeof(float),
                              hipMemcpyDeviceToHost, s->stream));
  }
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  return ENS_OK;
}

int sur_reserve(sur_t s, int64_t n_screen) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_reserve: NULL handle");
  if (n_screen < 0) return sfail(s, ENS_E_INVAL, "sur_reserve: n_screen must be >= 0");
  DevGuard dg(s->device);
  SUR_HIP(s, reserve_scan(s, n_screen));
  return ENS_OK;
}

int sur_screen(sur_t s, const double *params, int64_t n, const sur_screen_opts *o, int8_t *label,
               uint8_t *resolve, float *pred_max, int64_t *resolve_idx, int64_t *n_resolve) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_screen: NULL handle");
  if (!o || !n_resolve || n < 0 || (n > 0 && !params))
    return sfail(s, ENS_E_INVAL, "sur_screen: bad arguments");
  if (resolve_idx && !resolve)
    return sfail(s, ENS_E_INVAL, "sur_screen: resolve_idx needs the resolve mask");
  if (!s->have_norm) return sfail(s, ENS_E_ORDER, "sur_screen: call sur_set_norm first");
  if (!(o->margin >= 0) || !(o->spread >= 0) || !(o->flag_margin >= 0) ||
      std::isnan(o->label_margin))
    return sfail(s, ENS_E_INVAL, "sur_screen: margins must be >= 0");
  *n_resolve = 0;
  if (n == 0) return ENS_OK;
  DevGuard dg(s->device);
  const double sc0 = 2.0 / (s->in_hi[0] - s->in_lo[0]), sc1 = 2.0 / (s->in_hi[1] - s->in_lo[1]);
  const bool use_labels = s->nlab && o->label_margin >= 0.0;
  FusedArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n = n;
  a.prm = params;
  a.lo0 = s->in_lo[0];
  a.sc0 = sc0;
  a.lo1 = s->in_lo[1];
  a.sc1 = sc1;
  a.mean = s->norm->fmean;
  a.stdv = s->norm->fstd;
  a.margin = (float)o->margin;
  a.spread = (float)o->spread;
  a.flag_margin = (float)o->flag_margin;
  a.label_margin = (float)o->label_margin;
  a.nlab = use_labels ? s->nlab : nullptr;
  a.GL = s->nlab_G;
  a.label = label;
  a.resolve = resolve;
  a.pmax = pred_max;
  SUR_HIP(s, fused(s, a, true));
  if (resolve) {
    const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    SUR_HIP(s, reserve_scan(s, n));
    hipLaunchKernelGGL(k_count, dim3((unsigned)nb), dim3(kScanThreads), 0, s->stream, resolve, n,
                       s->scan);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s->stream, s->scan, nb,
                       (int64_t *)s->pin_d);
    if (resolve_idx)
      hipLaunchKernelGGL(k_write_idx, dim3((unsigned)nb), dim3(kScanThreads), 0, s->stream,
                         resolve, n, s->scan, resolve_idx);
    SUR_HIP(s, hipGetLastError());
  }
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  if (resolve) std::memcpy(n_resolve, s->pin, sizeof(int64_t));
  return ENS_OK;
}

int sur_fit_norm(sur_t s, const double *in_lo, const double *in_hi, const double *records,
                 int64_t n, double *out_mean, double *out_std) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_fit_norm: NULL handle");
  if (!in_lo || !in_hi || !records || n <= 0)
    return sfail(s, ENS_E_INVAL, "sur_fit_norm: bad arguments");
  DevGuard dg(s->device);
  const bool few = few_points(n);
  const int64_t nb = nblk(n, few ? 64 : 64 * kDsWaves);
  if (nb > s->mom_nb) {
    (void)hipFree(s->mom);
    s->mom = nullptr;
    s->mom_nb = 0;
    SUR_HIP(s, alloc(&s->mom, nb * kOut));
    s->mom_nb = nb;
  }
  hipLaunchKernelGGL(k_moments, dim3((unsigned)nb), dim3(64 * kDsWaves), 0, s->stream, records, n,
                     few, s->lntab, s->mom);
  hipLaunchKernelGGL(k_mean_std, dim3(kOut), dim3(256), 0, s->stream, s->mom, nb, s->pin_d);
  SUR_HIP(s, hipGetLastError());
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  double m[kOut], sd[kOut];
  const auto results = [&] {
    std::memcpy(m, s->pin, sizeof(m));
    std::memcpy(sd, s->pin + kOut, sizeof(sd));
  };
  results();
  // spreads within 4 ulp of the logarithms (one point has none)
  uint64_t ranks = 0;
  for (int j = 0; j < kOut; ++j)
    ranks |= (uint64_t)(sd[j] <= 0x1p-50 * std::fabs(m[j])) << j;
  if (ranks && n > 1) {
    SUR_HIP(s, ens::launch_rounding_spread(records, n, ranks, s->pin_d, s->stream));
    SUR_HIP(s, hipStreamSynchronize(s->stream));
    results();
  }
  for (int j = 0; j < kOut; ++j)
    if (!(sd[j] > 0.0) || !std::isfinite(m[j]))
      return sfail(s, ENS_E_INVAL, "sur_fit_norm: records give a non-positive or non-finite spread");
  if (int rc = sur_set_norm(s, in_lo, in_hi, m, sd)) return rc;
  if (out_mean) std::memcpy(out_mean, m, sizeof(m));
  if (out_std) std::memcpy(out_std, sd, sizeof(sd));
  return ENS_OK;
}

int sur_train_epoch(sur_t s, const float *x, const float *y, int64_t n, const int64_t *perm,
                    int64_t batch, float *mean_loss) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_train_epoch: NULL handle");
  if (int rc = check_batch(s, batch)) return rc;
  if (!x || !y || !perm || n < batch) return sfail(s, ENS_E_INVAL, "sur_train_epoch: bad arguments");
  DevGuard dg(s->device);
  const int64_t nb = n / batch;
  if (int rc = ensure_epoch_graph(s, x, y, n, perm, batch)) return rc;
  s->hyper_host[0] = s->lr;
  s->hyper_host[1] = s->b1;
  s->hyper_host[2] = s->b2;
  s->hyper_host[3] = s->eps;
  s->hyper_host[4] = (double)s->t;
  SUR_HIP(s, hipMemcpyAsync(s->hyper, s->hyper_host, sizeof(s->hyper_host),
                            hipMemcpyHostToDevice, s->stream));
  SUR_HIP(s, hipGraphLaunch(s->ep_exec, s->stream));
  s->t += nb;
  if (mean_loss) {
    float acc = 0.f;
    SUR_HIP(s, hipMemcpyAsync(&acc, s->loss_acc, sizeof(float), hipMemcpyDeviceToHost, s->stream));
    SUR_HIP(s, hipStreamSynchronize(s->stream));
    *mean_loss = acc / (float)nb;
  }
  return ENS_OK;
}

int sur_train_epochs(sur_t s, const float *x, const float *y, const int64_t *rows, int64_t n,
                     int64_t batch, int64_t epochs, const double *lr, uint64_t seed,
                     float *losses) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_train_epochs: NULL handle");
  if (int rc = check_batch(s, batch)) return rc;
  if (!x || !y || !rows || n < batch || epochs < 0 || (epochs > 0 && !lr))
    return sfail(s, ENS_E_INVAL, "sur_train_epochs: bad arguments");
  if (n > kEpochRows)
    return sfail(s, ENS_E_INVAL, "sur_train_epochs: more than 2^32 - 256 rows");
  for (int64_t e = 0; e < epochs; ++e)
    if (!(lr[e] > 0)) return sfail(s, ENS_E_INVAL, "sur_train_epochs: learning rates must be > 0");
  if (epochs == 0) return ENS_OK;
  DevGuard dg(s->device);
  const int64_t nb = n / batch;
  // device buffers of this call: the epochs' orders, the running epoch's, the
  // per-epoch hyper-parameters, the per-epoch losses
  EpochOrders eo;
  hipError_t oe;
  const size_t ob = (eo.size(n, epochs, s->stream, &oe) + 255) & ~(size_t)255;
  SUR_HIP(s, oe);
  // (orders made one at a time are read in place)
  const size_t kb = eo.group > 1 ? ((size_t)n * 8 + 255) & ~(size_t)255 : 0;
  const size_t hb = ((size_t)epochs * 5 * sizeof(double) + 255) & ~(size_t)255;
  const size_t lb = ((size_t)epochs * sizeof(float) + 255) & ~(size_t)255;
  char *buf = nullptr;
  SUR_HIP(s, hipMalloc((void **)&buf, ob + kb + hb + lb));
  eo.place(buf);
  auto *order = eo.group > 1 ? (int64_t *)(buf + ob) : eo.order;
  auto *hyp = (double *)(buf + ob + kb);
  auto *loss_d = (float *)(buf + ob + kb + hb);
  std::vector<double> h((size_t)epochs * 5);
  for (int64_t e = 0; e < epochs; ++e) {
    h[5 * e + 0] = lr[e];
    h[5 * e + 1] = s->b1;
    h[5 * e + 2] = s->b2;
    h[5 * e + 3] = s->eps;
    h[5 * e + 4] = (double)(s->t + e * nb);
  }
  hipError_t err = hipMemcpyAsync(hyp, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice,
                                  s->stream);
  int rc = ENS_OK;
  if (err == hipSuccess) rc = ensure_epoch_graph(s, x, y, n, order, batch);
  for (int64_t e = 0; err == hipSuccess && rc == ENS_OK && e < epochs; ++e) {
    if (e % eo.group == 0)
      err = eo.make(rows, seed, e, epochs - e < eo.group ? epochs - e : eo.group, s->stream);
    if (err == hipSuccess && eo.group > 1)
      err = hipMemcpyAsync(order, eo.order + e % eo.group * n, (size_t)n * sizeof(int64_t),
                           hipMemcpyDeviceToDevice, s->stream);
    if (err == hipSuccess)
      err = hipMemcpyAsync(s->hyper, hyp + 5 * e, 5 * sizeof(double), hipMemcpyDeviceToDevice,
                           s->stream);
    if (err == hipSuccess) err = hipGraphLaunch(s->ep_exec, s->stream);
    if (err == hipSuccess)
      err = hipMemcpyAsync(loss_d + e, s->loss_acc, sizeof(float), hipMemcpyDeviceToDevice,
                           s->stream);
  }
  std::vector<float> lh((size_t)epochs);
  if (err == hipSuccess && rc == ENS_OK)
    err = hipMemcpyAsync(lh.data(), loss_d, epochs * sizeof(float), hipMemcpyDeviceToHost, s->stream);
  if (err == hipSuccess) err = hipStreamSynchronize(s->stream);
  // the epoch graph reads `order`, which is freed here: drop it
  free_epoch_graph(s);
  s->ep_perm = nullptr;
  (void)hipFree(buf);
  if (rc != ENS_OK) return rc;
  if (err != hipSuccess)
    return sfail(s, err == hipErrorOutOfMemory ? ENS_E_NOMEM : ENS_E_HIP,
                 std::string("sur_train_epochs: ") + hipGetErrorString(err));
  s->t += epochs * nb;
  if (losses)
    for (int64_t e = 0; e < epochs; ++e) losses[e] = lh[e] / (float)nb;
  return ENS_OK;
}

int sur_exact_labels(sur_t s, const double *records, int64_t k, const int64_t *idx,
                     int8_t *label) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_exact_labels: NULL handle");
  if (k < 0 || (k > 0 && (!records || !label)))
    return sfail(s, ENS_E_INVAL, "sur_exact_labels: bad arguments");
  if (k == 0) return ENS_OK;
  DevGuard dg(s->device);
  hipLaunchKernelGGL(k_exact_labels, dim3(nblk(k, 256)), dim3(256), 0, s->stream, records, k,
                     idx, label);
  SUR_HIP(s, hipGetLastError());
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  return ENS_OK;
}

int sur_fit_label_map(sur_t s, const double *records, int32_t G, int8_t *map_out) {
  if (!s) return sfail(nullptr, ENS_E_INVAL, "sur_fit_label_map: NULL handle");
  if (!records || G < 2 || G > 65536) return sfail(s, ENS_E_INVAL, "sur_fit_label_map: bad arguments");
  const int64_t n = (int64_t)G * G;
  DevGuard dg(s->device);
  if (s->nlab_G != G) {
    (void)hipFree(s->nlab);
    s->nlab = nullptr;
    s->nlab_G = 0;
    SUR_HIP(s, hipMalloc((void **)&s->nlab, n));
    s->nlab_G = G;
  }
  hipLaunchKernelGGL(k_node_label, dim3(nblk(n, 256)), dim3(256), 0, s->stream, records, n, s->nlab);
  SUR_HIP(s, hipGetLastError());
  if (map_out) SUR_HIP(s, hipMemcpyAsync(map_out, s->nlab, n, hipMemcpyDeviceToDevice, s->stream));
  SUR_HIP(s, hipStreamSynchronize(s->stream));
  return ENS_OK;
}


}  // extern "C"
