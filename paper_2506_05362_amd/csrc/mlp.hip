// Surrogate network on gfx950: BF16 matrix-core GEMMs with FP32 accumulation,
// fused bias / GELU / GELU' epilogues, MSE loss and FP32 Adam.  C ABI in
// include/pd_mlp.h.
//
// Every layer product is one kernel k_gemm: a 256-thread workgroup computes a
// 64 x 64 or 32 x 32 tile of C = A B with gfx950's v_mfma_f32_16x16x32_bf16
// (each wavefront owns a quarter of the tile); A and B are read from FP32 arrays
// in their own layout (so the transposed operands of the backward pass need no
// copies), rounded to BF16 and staged in LDS 64 or 128 columns of K at a time.
// The weight and bias gradients of all layers are one kernel, k_wgrad.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "pd_mlp.h"

namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

typedef float v8f __attribute__((ext_vector_type(8)));

// C += A B on the matrix cores, 16 x 16 x 32 in BF16 with FP32 accumulation.
// Lane l holds 8 consecutive k of row l % 16 of A (group l / 16) and the same
// 8 k of column l % 16 of B, so A and B pair each k alike; the result C[4
// (l / 16) + e][l % 16] lands in element e.
__device__ __forceinline__ v4f mfma_16x16x32(const v8s& a, const v8s& b, const v4f& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// FP32 -> BF16, round to nearest even (the conversion instruction)
__device__ __forceinline__ v8s to_bf16x8(const v8f& x) {
  return __builtin_bit_cast(v8s, __builtin_convertvector(x, v8bf));
}

__device__ __forceinline__ v4s to_bf16x4(const v4f& x) {
  return __builtin_bit_cast(v4s, __builtin_convertvector(x, v4bf));
}

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

struct Gemm {
  const float* A;
  int64_t sam, sak;  // A(m, k) = A[m * sam + k * sak]
  const float* B;
  int64_t sbk, sbn;  // B(k, n) = B[k * sbk + n * sbn]
  int64_t M, N, K;
  float* C;
  int64_t ldc;         // C(m, n) = C[m * ldc + n]
  const float* bias;   // [N]
  float* Zout;         // pre-activation store (ldc), may be null
  const float* Zin;    // pre-activation for GELU' (ldc)
};

enum { EPI_BIAS = 1, EPI_BIAS_GELU = 2, EPI_GELU_GRAD = 3 };

// How an operand's 8 consecutive k are read: one by one with the rows side by
// side in memory (any stride), one by one along k, or as two float4 along k
// (K a multiple of 8, rows 16-byte aligned).
enum { ROWS = 0, ALONG_K = 1, ALONG_K4 = 2 };

// The k0..k0+KC-1 columns of T rows of an operand (row i at p + i * srow), 8 k
// per thread and group.  Where k is the contiguous direction the KC / 8 threads
// of a row sit side by side; where the rows are, the threads of one group of
// 8 k do, so that each of its 8 loads is one coalesced run.  Every load is
// issued without a branch (rows and k past the end read the last one, and are
// zeroed on the way to LDS): behind a branch each would wait for the one before.
template <int T, int KC, int MODE>
struct Stage {
  static constexpr int kGroups = T * KC / 8 / 256;
  v8f x[kGroups];
  const float* q[kGroups];
  __device__ __forceinline__ static void place(int g, int& row, int& kk) {
    const int id = threadIdx.x + g * 256;
    row = MODE == ROWS ? id % T : id / (KC / 8);
    kk = (MODE == ROWS ? id / T : id % (KC / 8)) * 8;
  }
  __device__ __forceinline__ void init(const float* p, int64_t srow, int64_t r0, int64_t R) {
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      int row, kk;
      place(g, row, kk);
      q[g] = p + (r0 + row < R ? r0 + row : R - 1) * srow;
    }
  }
  __device__ __forceinline__ void load(int64_t sk, int k0, int K) {
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      int row, kk;
      place(g, row, kk);
      if (MODE == ALONG_K4) {
        const int k = k0 + kk < K ? k0 + kk : K - 8;
        const v4f a = *reinterpret_cast<const v4f*>(q[g] + k), b = *reinterpret_cast<const v4f*>(q[g] + k + 4);
        x[g] = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int k = k0 + kk + e < K ? k0 + kk + e : K - 1;
          x[g][e] = q[g][MODE == ROWS ? k * sk : (int64_t)k];
        }
      }
    }
  }
  __device__ __forceinline__ void store(short (*s)[KC + 8], int k0, int K) const {
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      int row, kk;
      place(g, row, kk);
      v8s v = to_bf16x8(x[g]);
      if (k0 + KC > K) {  // the last chunk's missing k add exact zeros
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (k0 + kk + e >= K) v[e] = 0;
      }
      *reinterpret_cast<v8s*>(&s[row][kk]) = v;
    }
  }
};

// One KC-deep chunk from LDS: wavefront w owns the quarter (w / 2, w % 2) of the
// T x T tile as NB x NB matrix-core blocks.  Every element adds its k in
// steps of 32, ascending, into one accumulator, whatever T and KC are.
template <int T, int KC, int NB>
__device__ __forceinline__ void gemm_chunk(const short (*As)[KC + 8], const short (*Bs)[KC + 8], int wm, int wn,
                                           int lane, v4f (&acc)[NB][NB]) {
#pragma unroll
  for (int k = 0; k < KC; k += 32) {
    v8s a[NB], b[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) a[i] = *reinterpret_cast<const v8s*>(&As[wm + i * 16 + (lane & 15)][k + 8 * (lane >> 4)]);
#pragma unroll
    for (int j = 0; j < NB; ++j) b[j] = *reinterpret_cast<const v8s*>(&Bs[wn + j * 16 + (lane & 15)][k + 8 * (lane >> 4)]);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[i][j] = mfma_16x16x32(a[i], b[j], acc[i][j]);
  }
}

// KC k at a time; the next chunk's loads travel while this one is multiplied.
// Bound by the latency of its one or few rounds of loads at small batches (512 x
// 256 x 256: 5.4 us, 25 us with 32 k a round and one workgroup on every eighth
// CU), by its FP32 operands and the exact-erf GELU at large ones (16384 x 256 x
// 256: 19.5 us for 50 MB, 33 us before).
template <int EPI, int T, int KC, int MA, int MB>
__global__ __launch_bounds__(256) void k_gemm(Gemm g) {
  __shared__ __align__(16) short As[T][KC + 8];  // As[m][k]
  __shared__ __align__(16) short Bs[T][KC + 8];  // Bs[n][k] (B transposed)
  constexpr int NB = T / 32;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t m0 = (int64_t)blockIdx.y * T, n0 = (int64_t)blockIdx.x * T;
  const int wm = (wv >> 1) * (T / 2), wn = (wv & 1) * (T / 2);
  v4f acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  const int K = (int)g.K;
  Stage<T, KC, MA> sa;
  Stage<T, KC, MB> sb;
  sa.init(g.A, g.sam, m0, g.M);
  sb.init(g.B, g.sbn, n0, g.N);
  sa.load(g.sak, 0, K);
  sb.load(g.sbk, 0, K);
  for (int k0 = 0; k0 < K; k0 += KC) {
    sa.store(As, k0, K);
    sb.store(Bs, k0, K);
    __syncthreads();
    if (k0 + KC < K) {
      sa.load(g.sak, k0 + KC, K);
      sb.load(g.sbk, k0 + KC, K);
    }
    gemm_chunk<T, KC, NB>(As, Bs, wm, wn, lane, acc);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t m = m0 + wm + i * 16 + 4 * (lane >> 4) + e;
        const int64_t n = n0 + wn + j * 16 + (lane & 15);
        if (m >= g.M || n >= g.N) continue;
        const float v = acc[i][j][e];
        const int64_t o = m * g.ldc + n;
        if (EPI == EPI_BIAS) {
          g.C[o] = v + g.bias[n];
        } else if (EPI == EPI_BIAS_GELU) {
          const float z = v + g.bias[n];
          if (g.Zout) g.Zout[o] = z;
          g.C[o] = gelu(z);
        } else {
          g.C[o] = v * gelu_grad(g.Zin[o]);
        }
      }
}

// ---------------------------------------------------------------------------
// Weight and bias gradients of every layer in one launch: dW_l = A_{l-1}^T dZ_l
// and db_l = column sums of dZ_l.  Each element is one sum over the batch, in
// row order: a matrix-core accumulator taking 32 rows at a time for dW, plain
// FP32 additions of the unrounded dZ for db.  What bounds it is the latency of
// walking the batch, so the outputs are cut small (32 x 32 tiles of dW, 64
// columns of db, in workgroups of their own since an addition chain is slower
// than the matrix cores) and each workgroup keeps kWD chunks of kWK rows in
// flight in registers.  All four layers of 6-256-256-256-7: 8.8 us at 512 rows,
// 162 us at 16384 (four dW and four column-sum launches one after the other: 650
// us and 22.9 ms).  At 16384 rows its 157 workgroups read 0.6 GB, every column block
// once for each tile that needs it, at 3.7 TB/s; the 512 dependent matrix instructions
// of a tile are a few us of that.  Splitting the batch over workgroups as well took 46 us at
// 16384 rows, but sums in another order: the difference of 4e-7 in the gradient
// passes through Adam's first steps, which for gradients near eps is 1e-3 of a
// weight.
// ---------------------------------------------------------------------------

constexpr int kWT = 32, kWK = 128, kWD = 4;
constexpr int kBT = 64, kBD = 4;   // columns of a bias workgroup, its chunks in flight
constexpr int kGroupLayers = 8;    // layers per launch

struct WGrad {
  const float* A;   // layer input, din of lda columns
  const float* dZ;  // dl of ldz columns
  int32_t din, lda, dl, ldz;
  int32_t tiles_n, tiles_w;  // tiles of dW across, and in all; bias workgroups follow
  float *dW, *db;
};
struct WGradGroup {
  WGrad l[kGroupLayers];
  int32_t block0[kGroupLayers + 1];  // workgroups before layer l
  int32_t layers;
  int64_t batch;
};

// One chunk of T columns of a row-major [batch][ld] array in registers: blocks of
// 4 rows x 4 columns, T / 4 threads side by side (ld a multiple of 4, 16-byte
// aligned).  Loads are issued without a branch, as above; columns past ld feed
// only outputs that are not stored, rows past the batch are zeroed on the way to
// LDS.
template <int T>
struct Rows {
  static constexpr int kBlocks = T * kWK / 16 / 256;
  v4f x[kBlocks][4];
  __device__ __forceinline__ static int col() { return threadIdx.x % (T / 4) * 4; }
  __device__ __forceinline__ static int row(int g) { return (threadIdx.x / (T / 4) + g * (256 / (T / 4))) * 4; }
  __device__ __forceinline__ void load(const float* p, int ld, int c0, int64_t b0, int64_t batch) {
    const int c = c0 + col() < ld ? c0 + col() : ld - 4;
#pragma unroll
    for (int g = 0; g < kBlocks; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t r = b0 + row(g) + e;
        x[g][e] = *reinterpret_cast<const v4f*>(p + (r < batch ? r : batch - 1) * ld + c);
      }
  }
  __device__ __forceinline__ void mask(int64_t b0, int64_t batch) {
#pragma unroll
    for (int g = 0; g < kBlocks; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (b0 + row(g) + e >= batch) x[g][e] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  // column k of block g: its four rows
  __device__ __forceinline__ v4f column(int g, int k) const { return v4f{x[g][0][k], x[g][1][k], x[g][2][k], x[g][3][k]}; }
};

__device__ __forceinline__ void wgrad_bias(const WGrad& L, int n0, int64_t batch, char* lds) {
  float(*s)[kBT][kWK + 4] = reinterpret_cast<float(*)[kBT][kWK + 4]>(lds);  // s[buffer][n][k]
  using R = Rows<kBT>;
  R x[kBD];
#pragma unroll
  for (int d = 0; d < kBD; ++d) x[d].load(L.dZ, L.ldz, n0, d * kWK, batch);
  float sum = 0.0f;
  // rounds of kBD chunks, the last one masked (a branch in the others would have
  // every load waited for): rows past the batch hold zeros, which change no sum
  auto round = [&](int64_t c0, auto masked) {
#pragma unroll
    for (int d = 0; d < kBD; ++d) {
      const int64_t b0 = c0 + d * kWK;
      const int buf = d & 1;
      if (masked && b0 >= batch) return;  // (the same for the workgroup)
      if (masked) x[d].mask(b0, batch);
#pragma unroll
      for (int g = 0; g < R::kBlocks; ++g)
#pragma unroll
        for (int k = 0; k < 4; ++k) *reinterpret_cast<v4f*>(&s[buf][R::col() + k][R::row(g)]) = x[d].column(g, k);
      __syncthreads();  // the other buffer was read before this barrier's arrival
      if (!masked) x[d].load(L.dZ, L.ldz, n0, b0 + kBD * kWK, batch);
      if (threadIdx.x < kBT) {
#pragma unroll
        for (int r = 0; r < kWK; r += 4) {
          const v4f v = *reinterpret_cast<const v4f*>(&s[buf][threadIdx.x][r]);
#pragma unroll
          for (int e = 0; e < 4; ++e) sum += v[e];
        }
      }
    }
  };
  int64_t c0 = 0;
  for (; c0 + kBD * kWK <= batch; c0 += kBD * kWK) round(c0, std::false_type{});
  if (c0 < batch) round(c0, std::true_type{});
  if (threadIdx.x < kBT && n0 + (int)threadIdx.x < L.dl) L.db[n0 + threadIdx.x] = sum;
}

__device__ __forceinline__ void wgrad_tile(const WGrad& L, int m0, int n0, int64_t batch, char* lds) {
  short(*As)[kWT][kWK + 8] = reinterpret_cast<short(*)[kWT][kWK + 8]>(lds);  // As[buffer][m][k]
  short(*Bs)[kWT][kWK + 8] = As + 2;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wm = (wv >> 1) * (kWT / 2), wn = (wv & 1) * (kWT / 2);
  v4f acc[1][1] = {{v4f{0.f, 0.f, 0.f, 0.f}}};
  using R = Rows<kWT>;
  R a[kWD], b[kWD];
#pragma unroll
  for (int d = 0; d < kWD; ++d) {
    a[d].load(L.A, L.lda, m0, d * kWK, batch);
    b[d].load(L.dZ, L.ldz, n0, d * kWK, batch);
  }
  auto round = [&](int64_t c0, auto masked) {
#pragma unroll
    for (int d = 0; d < kWD; ++d) {
      const int64_t b0 = c0 + d * kWK;
      const int buf = d & 1;
      if (masked && b0 >= batch) return;
      if (masked) {
        a[d].mask(b0, batch);
        b[d].mask(b0, batch);
      }
#pragma unroll
      for (int g = 0; g < R::kBlocks; ++g)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          *reinterpret_cast<v4s*>(&As[buf][R::col() + k][R::row(g)]) = to_bf16x4(a[d].column(g, k));
          *reinterpret_cast<v4s*>(&Bs[buf][R::col() + k][R::row(g)]) = to_bf16x4(b[d].column(g, k));
        }
      __syncthreads();  // the other buffer was read before this barrier's arrival
      if (!masked) {
        a[d].load(L.A, L.lda, m0, b0 + kWD * kWK, batch);
        b[d].load(L.dZ, L.ldz, n0, b0 + kWD * kWK, batch);
      }
      gemm_chunk<kWT, kWK, 1>(As[buf], Bs[buf], wm, wn, lane, acc);
    }
  };
  int64_t c0 = 0;
  for (; c0 + kWD * kWK <= batch; c0 += kWD * kWK) round(c0, std::false_type{});
  if (c0 < batch) round(c0, std::true_type{});
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int m = m0 + wm + 4 * (lane >> 4) + e, n = n0 + wn + (lane & 15);
    if (m < L.din && n < L.dl) L.dW[m * L.dl + n] = acc[0][0][e];
  }
}

__global__ __launch_bounds__(256) void k_wgrad(WGradGroup G) {
  constexpr int kTileBytes = 2 * 2 * kWT * (kWK + 8) * (int)sizeof(short), kBiasBytes = 2 * kBT * (kWK + 4) * (int)sizeof(float);
  __shared__ __align__(16) char smem[kTileBytes > kBiasBytes ? kTileBytes : kBiasBytes];
  int li = 0;
  while (li + 1 < G.layers && (int)blockIdx.x >= G.block0[li + 1]) ++li;
  const WGrad L = G.l[li];
  const int t = (int)blockIdx.x - G.block0[li];
  if (t >= L.tiles_w) wgrad_bias(L, (t - L.tiles_w) * kBT, G.batch, smem);
  else wgrad_tile(L, t / L.tiles_n * kWT, t % L.tiles_n * kWT, G.batch, smem);
}

// residual, loss partial sums and dY = 2 (Y_hat - Y) / (B * d) in rows of ldd
// (the columns past d zero); with xp, also the input copied to rows of ldx: what
// k_wgrad reads four columns at a time
__global__ __launch_bounds__(256) void k_loss(const float* yh, const float* y, float* dy, int64_t rows, int d, int ldd,
                                               float scale, double* partial, const float* x, int dx, float* xp,
                                               int ldx) {
  __shared__ double red[256];
  const int tid = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * 256 + tid, step = (int64_t)gridDim.x * 256;
  double s = 0.0;
  for (int64_t i = i0; i < rows * ldd; i += step) {
    const int64_t m = i / ldd;
    const int n = (int)(i % ldd);
    const float r = n < d ? yh[m * d + n] - y[m * d + n] : 0.0f;
    dy[i] = scale * r;
    s += (double)r * (double)r;
  }
  if (xp)
    for (int64_t i = i0; i < rows * ldx; i += step) {
      const int64_t m = i / ldx;
      const int n = (int)(i % ldx);
      xp[i] = n < dx ? x[m * dx + n] : 0.0f;
    }
  red[tid] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (tid < o) red[tid] += red[tid + o];
    __syncthreads();
  }
  if (tid == 0) partial[blockIdx.x] = red[0];
}

// Adam with decoupled weight decay: p -= lr (m_hat / (sqrt(v_hat) + eps) + wd p)
__global__ void k_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, float wd, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i];
  p[i] = pi - lr * ((mi / c1) / (sqrtf(vi / c2) + eps) + wd * pi);
}

// ---------------------------------------------------------------------------
// Fused inference for din <= 16 -> 256 -> 256 -> 256 -> dout <= 16, one launch.
// A workgroup of eight wavefronts keeps W2 and W3 in registers (wavefront w the
// 32 columns from 32 w, as matrix-core operands: 128 VGPRs) and walks tiles of
// 16 R rows.  Layer 1 runs on the vector units (its 6-wide products are too small
// for the matrix cores), a wavefront computing its 32 hidden units; activations
// pass between the layers through LDS in BF16, one barrier each; layer 4 is one
// wavefront's work per 16 rows.  Weights take the matrix cores' A side, so that a
// lane ends up with four neighbouring units of one row: one 8-byte LDS store.
// Operands are rounded to BF16 exactly where the layer-by-layer path rounds them
// (x, W1, activations, W2..W4) and every sum runs in its order; accumulation is
// FP32.
//
// Bound by the vector units: 768 exact-erf GELUs a row, some 44 instructions each.
// 1e7 rows: 8.0 ms (as two kernels with the weights in LDS, the second hidden
// layer's activations stored between them and 2-byte stores: 12.9 ms); 100 rows,
// which those two kernels put on one CU: 30 us a call instead of 71.
// ---------------------------------------------------------------------------

constexpr int kH = 256;          // hidden width of the fused path
constexpr int kHRow = kH + 8;    // LDS row of activations (bf16), 16-byte aligned, banks staggered
constexpr int kIW = 8;           // wavefronts per workgroup, 32 hidden units each

__device__ __forceinline__ float round_bf16(float x) { return (float)(__bf16)x; }

struct Infer {
  const float* x;
  int64_t M;
  int din, dout;
  const float *W1, *b1, *W2, *b2, *W3, *b3, *W4, *b4;  // fp32, W [fan_in][fan_out]
  float* y;  // [M][dout]
};

// operand of the 16 units from n0 for all k: lane l holds unit n0 + l % 16, k = 32
// kk + 8 (l / 16) + j
__device__ __forceinline__ void load_units(const float* W, int n0, v8s (&f)[kH / 32]) {
  const int lane = threadIdx.x & 63;
  const float* p = W + (int64_t)8 * (lane >> 4) * kH + n0 + (lane & 15);
#pragma unroll
  for (int kk = 0; kk < kH / 32; ++kk) {
    v8f v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p[(kk * 32 + j) * kH];
    f[kk] = to_bf16x8(v);
  }
}

// one hidden layer of the wavefront's 32 units: GELU(W^T act + b) into out
template <int R>
__device__ __forceinline__ void hidden(const v8s (&w)[2][kH / 32], const float* bias, int n0,
                                       const short (*in)[kHRow], short (*out)[kHRow]) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  v4f acc[R][2];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r][0] = acc[r][1] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < kH / 32; ++kk)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const v8s act = *reinterpret_cast<const v8s*>(&in[16 * r + lr][kk * 32 + 8 * lg]);
#pragma unroll
      for (int c = 0; c < 2; ++c) acc[r][c] = mfma_16x16x32(w[c][kk], act, acc[r][c]);
    }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int n = n0 + 16 * c + 4 * lg;  // the lane's four units
    const v4f b = *reinterpret_cast<const v4f*>(bias + n);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      v4f g;
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] = gelu(acc[r][c][e] + b[e]);
      *reinterpret_cast<v4s*>(&out[16 * r + lr][n]) = to_bf16x4(g);
    }
  }
}

template <int DINP, int R>
__global__ __launch_bounds__(64 * kIW) void k_infer(Infer a) {
  __shared__ __align__(16) short act[3][16 * R][kHRow];
  __shared__ __align__(16) short sW4[16][kHRow];   // transposed, units >= dout zero
  __shared__ __align__(16) float sW1[DINP][kH];
  __shared__ __align__(16) float sb[3][kH];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), n0 = 32 * wv;
  v8s w2[2][kH / 32], w3[2][kH / 32];
#pragma unroll
  for (int c = 0; c < 2; ++c) load_units(a.W2, n0 + 16 * c, w2[c]);
  for (int i = tid; i < DINP * kH; i += 64 * kIW) (&sW1[0][0])[i] = i < a.din * kH ? round_bf16(a.W1[i]) : 0.0f;
  for (int i = tid; i < kH; i += 64 * kIW) {
    sb[0][i] = a.b1[i];
    sb[1][i] = a.b2[i];
    sb[2][i] = a.b3[i];
  }
  for (int i = tid; i < 16 * kH; i += 64 * kIW) {
    const int k = i / 16, n = i % 16;
    sW4[n][k] = __builtin_bit_cast(short, (__bf16)(n < a.dout ? a.W4[(int64_t)k * a.dout + n] : 0.0f));
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) load_units(a.W3, n0 + 16 * c, w3[c]);
  const int64_t ntiles = (a.M + 16 * R - 1) / (16 * R);
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    // layer 1: the lane's row lr of each 16, hidden units n0 + 8 lg + 0..7
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = t * 16 * R + 16 * r + lr;
      float xv[DINP];
#pragma unroll
      for (int i = 0; i < DINP; ++i) {
        const float v = a.x[(row < a.M ? row : a.M - 1) * a.din + (i < a.din ? i : 0)];
        xv[i] = i < a.din ? round_bf16(v) : 0.0f;
      }
      float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < DINP; ++i) {
        const v8f w = *reinterpret_cast<const v8f*>(&sW1[i][n0 + 8 * lg]);
#pragma unroll
        for (int j = 0; j < 8; ++j) z[j] = fmaf(xv[i], w[j], z[j]);
      }
      const v8f b = *reinterpret_cast<const v8f*>(&sb[0][n0 + 8 * lg]);
      v8f g;
#pragma unroll
      for (int j = 0; j < 8; ++j) g[j] = gelu(z[j] + b[j]);
      *reinterpret_cast<v8s*>(&act[0][16 * r + lr][n0 + 8 * lg]) = to_bf16x8(g);
    }
    __syncthreads();
    hidden<R>(w2, sb[1], n0, act[0], act[1]);
    __syncthreads();
    hidden<R>(w3, sb[2], n0, act[1], act[2]);
    __syncthreads();
    // layer 4 (the next tile's first write to act[2] is two barriers away)
    if (wv < R) {
      v4f o = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < kH / 32; ++kk)
        o = mfma_16x16x32(*reinterpret_cast<const v8s*>(&sW4[lr][kk * 32 + 8 * lg]),
                          *reinterpret_cast<const v8s*>(&act[2][16 * wv + lr][kk * 32 + 8 * lg]), o);
      const int64_t row = t * 16 * R + 16 * wv + lr;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = 4 * lg + e;
        if (row < a.M && n < a.dout) a.y[row * a.dout + n] = o[e] + a.b4[n];
      }
    }
  }
}

}  // namespace

struct pdm_net {
  std::vector<int32_t> dims;
  int64_t max_batch = 0, n_params = 0;
  hipStream_t stream = nullptr;
  int own_stream = 0;
  std::string err;
  float *params = nullptr, *grad = nullptr, *m = nullptr, *v = nullptr;
  std::vector<float*> Z, Aout, dZ;  // per layer, [max_batch][row4(dims[l+1])]
  float* yhat = nullptr;            // [max_batch][d_out]
  float* xrows = nullptr;           // the training input with rows padded to 4 columns
  double* partial = nullptr;
  int nloss_blocks = 0;
  std::vector<int64_t> woff, boff;  // offsets of W_l, b_l in the parameter vector
  float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f, weight_decay = 0.0f;
  // fused inference path (din <= 16 -> 256 -> 256 -> 256 -> dout <= 16)
  int fused_ok = 0, use_fused = 0, cus = 0;
  int64_t t = 0;
  std::vector<void*> owned;
  pd_alloc_fn alloc = nullptr;  // caller's device allocator (hipMalloc when none)
  pd_free_fn free_fn = nullptr;
  void* alloc_user = nullptr;
};

namespace {

pd_status fail(pdm_net* n, pd_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (n) n->err = buf;
  return st;
}

#define HIPCHK(net, call)                                                                    \
  do {                                                                                       \
    hipError_t e_ = (call);                                                                  \
    if (e_ != hipSuccess)                                                                    \
      return fail((net), PD_ERR_HIP, "%s failed: %s", #call, hipGetErrorName(e_));           \
  } while (0)

template <typename T>
pd_status alloc(pdm_net* n, T** p, int64_t count) {
  void* q = nullptr;
  const size_t bytes = (sizeof(T) * (size_t)(count > 0 ? count : 1) + 255) & ~size_t(255);
  if (n->alloc) q = n->alloc(bytes, n->alloc_user);
  else if (hipMalloc(&q, bytes) != hipSuccess) q = nullptr;
  if (!q) return fail(n, PD_ERR_OOM, "device allocation of %lld elements failed", (long long)count);
  n->owned.push_back(q);
  *p = static_cast<T*>(q);
  return PD_OK;
}

#define TRY(e)                        \
  do {                                \
    pd_status s_ = (e);               \
    if (s_ != PD_OK) return s_;       \
  } while (0)

// 64 x 64 tiles where they give every CU a workgroup, else 32 x 32 with chunks
// of 128 k (a quarter of the work per workgroup, half the trips to memory): at
// 512 x 256 x 256 the small tiles take 5.4 us
template <int EPI, int MA, int MB>
void gemm_modes(const Gemm& g, hipStream_t s) {
  auto grid = [&](int t) { return dim3((unsigned)((g.N + t - 1) / t), (unsigned)((g.M + t - 1) / t)); };
  const dim3 g64 = grid(64);
  if ((int64_t)g64.x * g64.y >= 256) hipLaunchKernelGGL((k_gemm<EPI, 64, 64, MA, MB>), g64, dim3(256), 0, s, g);
  else hipLaunchKernelGGL((k_gemm<EPI, 32, 128, MA, MB>), grid(32), dim3(256), 0, s, g);
}

template <int EPI>
hipError_t gemm(const Gemm& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  const auto vec = [&](const float* p, int64_t srow) {
    return g.K % 8 == 0 && srow % 4 == 0 && (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
  };
  // A is an activation or dZ, contiguous along k; so is W^T in the backward
  // product, while the forward product's W is contiguous along its columns
  if (EPI == EPI_GELU_GRAD) {
    if (vec(g.A, g.sam) && vec(g.B, g.sbn)) gemm_modes<EPI, ALONG_K4, ALONG_K4>(g, s);
    else gemm_modes<EPI, ALONG_K, ALONG_K>(g, s);
  } else {
    if (vec(g.A, g.sam)) gemm_modes<EPI, ALONG_K4, ROWS>(g, s);
    else gemm_modes<EPI, ALONG_K, ROWS>(g, s);
  }
  return hipGetLastError();
}

int n_layers(const pdm_net* n) { return (int)n->dims.size() - 1; }

// row length of the network's own activation buffers: what k_wgrad can read four
// columns at a time (the padding is never read into a result)
int row4(int64_t w) { return (int)((w + 3) & ~int64_t(3)); }

// forward of `batch` rows (<= max_batch) from x into y (device pointers)
pd_status forward_chunk(pdm_net* n, const float* x, int64_t batch, float* y, bool keep_z) {
  const int L = n_layers(n);
  const float* A = x;
  for (int l = 0; l < L; ++l) {
    const int64_t din = n->dims[l], dout = n->dims[l + 1];
    Gemm g{};
    g.A = A;
    g.sam = l == 0 ? din : row4(din);
    g.sak = 1;
    g.B = n->params + n->woff[l];
    g.sbk = dout;
    g.sbn = 1;
    g.M = batch;
    g.N = dout;
    g.K = din;
    g.bias = n->params + n->boff[l];
    g.ldc = l < L - 1 ? row4(dout) : dout;
    if (l < L - 1) {
      g.C = n->Aout[l];
      g.Zout = keep_z ? n->Z[l] : nullptr;
      HIPCHK(n, gemm<EPI_BIAS_GELU>(g, n->stream));
      A = n->Aout[l];
    } else {
      g.C = y;
      HIPCHK(n, gemm<EPI_BIAS>(g, n->stream));
    }
  }
  return PD_OK;
}

// loss and gradient into n->grad for one batch
pd_status loss_and_grad(pdm_net* n, const float* x, const float* y, int64_t batch, float* loss) {
  const int L = n_layers(n);
  const int64_t dout = n->dims[L];
  TRY(forward_chunk(n, x, batch, n->yhat, true));
  const int64_t cnt = batch * dout;
  const bool copy_x = n->dims[0] % 4 != 0 || (reinterpret_cast<uintptr_t>(x) & 15u) != 0;
  hipLaunchKernelGGL(k_loss, dim3(n->nloss_blocks), dim3(256), 0, n->stream, n->yhat, y, n->dZ[L - 1], batch, (int)dout,
                     row4(dout), 2.0f / (float)cnt, n->partial, x, n->dims[0], copy_x ? n->xrows : nullptr,
                     row4(n->dims[0]));
  HIPCHK(n, hipGetLastError());
  for (int l = L - 1; l > 0; --l) {
    const int64_t din = n->dims[l], dl = n->dims[l + 1];
    // dZ_{l-1} = (dZ_l W_l^T) * GELU'(Z_{l-1})
    Gemm gx{};
    gx.A = n->dZ[l];
    gx.sam = row4(dl);
    gx.sak = 1;
    gx.B = n->params + n->woff[l];
    gx.sbk = 1;
    gx.sbn = dl;
    gx.M = batch;
    gx.N = din;
    gx.K = dl;
    gx.C = n->dZ[l - 1];
    gx.ldc = row4(din);
    gx.Zin = n->Z[l - 1];
    HIPCHK(n, gemm<EPI_GELU_GRAD>(gx, n->stream));
  }
  WGradGroup G{};
  G.batch = batch;
  for (int l0 = 0; l0 < L; l0 += kGroupLayers) {
    G.layers = std::min(kGroupLayers, L - l0);
    G.block0[0] = 0;
    for (int k = 0; k < G.layers; ++k) {
      const int l = l0 + k;
      WGrad& w = G.l[k];
      w.A = l > 0 ? n->Aout[l - 1] : copy_x ? n->xrows : x;
      w.dZ = n->dZ[l];
      w.din = n->dims[l];
      w.lda = row4(w.din);
      w.dl = n->dims[l + 1];
      w.ldz = row4(w.dl);
      w.dW = n->grad + n->woff[l];
      w.db = n->grad + n->boff[l];
      w.tiles_n = (w.dl + kWT - 1) / kWT;
      w.tiles_w = ((w.din + kWT - 1) / kWT) * w.tiles_n;
      G.block0[k + 1] = G.block0[k] + w.tiles_w + (w.dl + kBT - 1) / kBT;
    }
    hipLaunchKernelGGL(k_wgrad, dim3((unsigned)G.block0[G.layers]), dim3(256), 0, n->stream, G);
    HIPCHK(n, hipGetLastError());
  }
  if (loss) {
    std::vector<double> part((size_t)n->nloss_blocks);
    HIPCHK(n, hipMemcpyAsync(part.data(), n->partial, sizeof(double) * part.size(), hipMemcpyDeviceToHost,
                             n->stream));
    HIPCHK(n, hipStreamSynchronize(n->stream));
    double s = 0.0;
    for (double p : part) s += p;
    *loss = (float)(s / (double)cnt);
  }
  return PD_OK;
}

}  // namespace

extern "C" {

pd_status pdm_create(pdm_net** out, const int32_t* dims, int32_t n_dims, int64_t max_batch, pd_alloc_fn alloc_fn,
                     pd_free_fn free_fn, void* alloc_user, void* stream) {
  if (!out) return PD_ERR_INVALID;
  *out = nullptr;
  if ((alloc_fn == nullptr) != (free_fn == nullptr)) return PD_ERR_INVALID;
  pdm_net* n = new (std::nothrow) pdm_net();
  if (!n) return PD_ERR_OOM;
  *out = n;
  n->alloc = alloc_fn;
  n->free_fn = free_fn;
  n->alloc_user = alloc_user;
  if (!dims || n_dims < 2) return fail(n, PD_ERR_INVALID, "need at least two layer widths");
  for (int k = 0; k < n_dims; ++k)
    if (dims[k] < 1 || dims[k] > 1024) return fail(n, PD_ERR_INVALID, "layer width %d out of [1, 1024]", dims[k]);
  if (max_batch < 1 || max_batch > (1 << 24)) return fail(n, PD_ERR_INVALID, "max_batch out of range");
  n->dims.assign(dims, dims + n_dims);
  n->max_batch = max_batch;
  n->stream = static_cast<hipStream_t>(stream);
  if (!n->stream) {
    if (hipStreamCreate(&n->stream) != hipSuccess) return fail(n, PD_ERR_HIP, "hipStreamCreate failed");
    n->own_stream = 1;
  }
  const int L = n_dims - 1;
  int64_t o = 0;
  for (int l = 0; l < L; ++l) {
    n->woff.push_back(o);
    o += (int64_t)dims[l] * dims[l + 1];
    n->boff.push_back(o);
    o += dims[l + 1];
  }
  n->n_params = o;
  TRY(alloc(n, &n->params, o));
  TRY(alloc(n, &n->grad, o));
  TRY(alloc(n, &n->m, o));
  TRY(alloc(n, &n->v, o));
  n->Z.resize(L);
  n->Aout.resize(L);
  n->dZ.resize(L);
  for (int l = 0; l < L; ++l) {
    TRY(alloc(n, &n->Z[l], max_batch * row4(dims[l + 1])));
    TRY(alloc(n, &n->Aout[l], max_batch * row4(dims[l + 1])));
    TRY(alloc(n, &n->dZ[l], max_batch * row4(dims[l + 1])));
  }
  TRY(alloc(n, &n->yhat, max_batch * dims[L]));
  TRY(alloc(n, &n->xrows, max_batch * row4(dims[0])));
  if (n_dims == 5 && dims[1] == kH && dims[2] == kH && dims[3] == kH && dims[0] <= 16 && dims[4] <= 16) {
    // (the LDS of gfx950; the kernel's 77 KB are more than other devices give a workgroup)
    int dev = 0, lds = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess &&
        hipDeviceGetAttribute(&n->cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && lds >= 160 * 1024)
      n->fused_ok = n->use_fused = 1;
    (void)hipGetLastError();
  }
  n->nloss_blocks = 256;
  TRY(alloc(n, &n->partial, n->nloss_blocks));
  HIPCHK(n, hipMemsetAsync(n->params, 0, sizeof(float) * o, n->stream));
  HIPCHK(n, hipMemsetAsync(n->m, 0, sizeof(float) * o, n->stream));
  HIPCHK(n, hipMemsetAsync(n->v, 0, sizeof(float) * o, n->stream));
  HIPCHK(n, hipStreamSynchronize(n->stream));
  return PD_OK;
}

int64_t pdm_param_count(const pdm_net* n) { return n ? n->n_params : 0; }

pd_status pdm_set_params(pdm_net* n, const float* p, int64_t cnt) {
  if (!n || !p) return PD_ERR_INVALID;
  if (cnt != n->n_params) return fail(n, PD_ERR_INVALID, "expected %lld parameters", (long long)n->n_params);
  HIPCHK(n, hipMemcpyAsync(n->params, p, sizeof(float) * cnt, hipMemcpyHostToDevice, n->stream));
  HIPCHK(n, hipMemsetAsync(n->m, 0, sizeof(float) * cnt, n->stream));
  HIPCHK(n, hipMemsetAsync(n->v, 0, sizeof(float) * cnt, n->stream));
  HIPCHK(n, hipStreamSynchronize(n->stream));
  n->t = 0;
  return PD_OK;
}

pd_status pdm_get_params(pdm_net* n, float* p, int64_t cnt) {
  if (!n || !p) return PD_ERR_INVALID;
  if (cnt < n->n_params) return fail(n, PD_ERR_INVALID, "expected room for %lld parameters", (long long)n->n_params);
  HIPCHK(n, hipMemcpyAsync(p, n->params, sizeof(float) * n->n_params, hipMemcpyDeviceToHost, n->stream));
  HIPCHK(n, hipStreamSynchronize(n->stream));
  return PD_OK;
}

pd_status pdm_set_adam(pdm_net* n, float b1, float b2, float eps, float weight_decay) {
  if (!n) return PD_ERR_INVALID;
  if (!(b1 >= 0 && b1 < 1 && b2 >= 0 && b2 < 1 && eps > 0 && weight_decay >= 0))
    return fail(n, PD_ERR_INVALID, "bad Adam parameters");
  n->weight_decay = weight_decay;
  n->beta1 = b1;
  n->beta2 = b2;
  n->eps = eps;
  return PD_OK;
}

pd_status pdm_set_inference(pdm_net* n, int32_t fused) {
  if (!n) return PD_ERR_INVALID;
  if (fused && !n->fused_ok)
    return fail(n, PD_ERR_UNSUPPORTED, "the fused inference path needs dims din<=16,256,256,256,dout<=16 "
                                       "and enough LDS per workgroup");
  n->use_fused = fused ? 1 : 0;
  return PD_OK;
}

pd_status pdm_forward(pdm_net* n, const float* x, int64_t batch, float* y) {
  if (!n || (!x && batch > 0) || (!y && batch > 0) || batch < 0) return PD_ERR_INVALID;
  const int64_t din = n->dims.front(), dout = n->dims.back();
  // Workgroups of the fused kernel write outputs while others have yet to read their
  // inputs.  Where the two arrays overlap the layer-by-layer kernels give the same
  // values: they read a chunk's inputs before its outputs are written.  (Equal rows in
  // place are one workgroup's own.)
  const bool overlap = x < y + batch * dout && y < x + batch * din && !(x == y && din == dout);
  if (n->use_fused && batch > 0 && !overlap) {
    Infer a{};
    a.x = x;
    a.M = batch;
    a.din = (int)din;
    a.dout = (int)dout;
    a.W1 = n->params + n->woff[0];
    a.b1 = n->params + n->boff[0];
    a.W2 = n->params + n->woff[1];
    a.b2 = n->params + n->boff[1];
    a.W3 = n->params + n->woff[2];
    a.b3 = n->params + n->boff[2];
    a.W4 = n->params + n->woff[3];
    a.b4 = n->params + n->boff[3];
    a.y = y;
    // 32 rows a tile once they give every CU a workgroup, one workgroup a CU
    const int64_t cus = std::max(n->cus, 1);
    const bool wide = batch > 32 * cus;
    const int64_t tiles = wide ? (batch + 31) / 32 : (batch + 15) / 16;
    const dim3 grid((unsigned)std::min<int64_t>(tiles, wide ? cus : 2 * cus)), block(64 * kIW);
    if (din <= 8) {
      if (wide) hipLaunchKernelGGL((k_infer<8, 2>), grid, block, 0, n->stream, a);
      else hipLaunchKernelGGL((k_infer<8, 1>), grid, block, 0, n->stream, a);
    } else {
      if (wide) hipLaunchKernelGGL((k_infer<16, 2>), grid, block, 0, n->stream, a);
      else hipLaunchKernelGGL((k_infer<16, 1>), grid, block, 0, n->stream, a);
    }
    HIPCHK(n, hipGetLastError());
  } else {
    for (int64_t b0 = 0; b0 < batch; b0 += n->max_batch) {
      const int64_t cb = batch - b0 < n->max_batch ? batch - b0 : n->max_batch;
      TRY(forward_chunk(n, x + b0 * din, cb, y + b0 * dout, false));
    }
  }
  HIPCHK(n, hipStreamSynchronize(n->stream));
  return PD_OK;
}

pd_status pdm_gradients(pdm_net* n, const float* x, const float* y, int64_t batch, float* loss, float* grad) {
  if (!n || !x || !y || !grad) return PD_ERR_INVALID;
  if (batch < 1 || batch > n->max_batch) return fail(n, PD_ERR_INVALID, "batch must be in [1, max_batch]");
  TRY(loss_and_grad(n, x, y, batch, loss));
  HIPCHK(n, hipMemcpyAsync(grad, n->grad, sizeof(float) * n->n_params, hipMemcpyDeviceToHost, n->stream));
  HIPCHK(n, hipStreamSynchronize(n->stream));
  return PD_OK;
}

pd_status pdm_train_step(pdm_net* n, const float* x, const float* y, int64_t batch, float lr, float* loss) {
  if (!n || !x || !y) return PD_ERR_INVALID;
  if (batch < 1 || batch > n->max_batch) return fail(n, PD_ERR_INVALID, "batch must be in [1, max_batch]");
  if (!(lr > 0)) return fail(n, PD_ERR_INVALID, "learning rate must be > 0");
  TRY(loss_and_grad(n, x, y, batch, loss));
  n->t += 1;
  const float c1 = 1.0f - powf(n->beta1, (float)n->t), c2 = 1.0f - powf(n->beta2, (float)n->t);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((n->n_params + 255) / 256)), dim3(256), 0, n->stream, n->params,
                     n->grad, n->m, n->v, n->n_params, lr, n->beta1, n->beta2, n->eps, n->weight_decay, c1, c2);
  HIPCHK(n, hipGetLastError());
  if (!loss) HIPCHK(n, hipStreamSynchronize(n->stream));
  return PD_OK;
}

void pdm_destroy(pdm_net* n) {
  if (!n) return;
  (void)hipStreamSynchronize(n->stream);
  for (void* p : n->owned) {
    if (n->free_fn) n->free_fn(p, n->alloc_user);
    else (void)hipFree(p);
  }
  if (n->own_stream) (void)hipStreamDestroy(n->stream);
  delete n;
}

const char* pdm_last_error(const pdm_net* n) { return n ? n->err.c_str() : "null network"; }

}  // extern "C"
