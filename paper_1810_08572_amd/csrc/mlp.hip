// Learned warm start (not part of the paper's method; conjugate gradients
// always finishes the solve, so the network can only change the iteration
// count).  A dense network n_in -> width (x n_hidden, SiLU) -> 1 (linear)
// maps per-cell features to the next pressure increment.
//
//   training   FP32 matrix cores (deterministic split-K over the rows),
//              SiLU, mean-squared-error gradient, Adam;
//   inference  the width x width hidden layers on BF16 MFMA
//              (v_mfma_f32_32x32x8bf16_1k, FP32 accumulation), the first and
//              last (thin) layers in FP32 on the vector ALUs;
//   features   of every active cell, from the solver's mesh adjacency.
//
// Parameters are FP32, packed layer by layer: W ([out][in], row-major), b.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>

struct ppe_mlp {
  int n_in = 0, width = 0, n_hidden = 0;
  hipStream_t stream = nullptr;
  int64_t n_params = 0;
  std::vector<int> dims;                 // n_in, width, ..., width, 1
  std::vector<int64_t> woff, boff;       // offsets of W_l, b_l in the packed vector
  ppe::DevBuf params, grad, m, v, bf16;  // bf16: hidden weight matrices in BF16
  ppe::DevBuf act, pre, gbuf, part, lossbuf;
  double* loss_h = nullptr;  // pinned: the last batch's loss
  int64_t adam_t = 0;
  size_t lds_max = 0;  // LDS one workgroup may use (0: not queried yet)
  int cus = 0;         // compute units of the device
  std::string err;
};

namespace ppe {
namespace {

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu_f(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s + z * s * (1.0f - s);
}

// ---- training and FP32 inference
// A batch is a handful of thin products (8,192 rows, width 128: 1.7 GFLOP
// with the gradients, 26 MB of activations), so what bounds it is the number
// of dispatches and how many compute units each one fills.  Every product
// runs on the FP32 matrix cores (FP32 products and sums, the vector ALUs'
// accuracy), a layer's as two v_mfma_f32_16x16x4f32 tiles side by side per wave,
// the weight gradients as one v_mfma_f32_32x32x2f32 tile per wave, and takes
// what follows it along: bias and SiLU with the forward layers, silu' with
// the backward ones, the whole output layer with the loss.  The weight and
// bias gradients of all layers are one dispatch over (tile, chunk of rows),
// their chunks added in order by a second: eight dispatches for three hidden
// layers.  Loss and gradient of 8,192 rows take 90 us; the vector-ALU tiles
// this replaces (64 x 64 outputs per workgroup, eight workgroups for a weight
// gradient, a separate pass for every bias, activation and column sum) took
// 3.87 ms.
typedef float float16_t __attribute__((ext_vector_type(16)));

constexpr int kTile = 32;  // rows of a workgroup's tile; rows and columns of a gradient wave's
constexpr int kTileN = 4 * kTile;  // columns of a workgroup's tile (4 waves)
constexpr int kTileK = 64;         // depth staged in LDS at a time

// Operands of v_mfma_f32_32x32x2f32: lane l holds A[l % 32][l / 32] and
// B[l / 32][l % 32]; accumulator r of lane l is
// C[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
__device__ __forceinline__ int acc_row(int r, int lane) {
  return 8 * (r / 4) + 4 * (lane / 32) + r % 4;
}

// A ROWS x COLS tile of a row-major matrix on its way through T threads into
// LDS: fetch requests it all (zeros past `rows` and `cols`), put stores it.
// Four columns per load where the matrix allows it (vec: its leading
// dimension and address are multiples of four floats; one by one, a layer of
// width 128 took 14.4 us, with them 11.5).
template <int ROWS, int COLS, int T>
struct Staged {
  static constexpr int U = ROWS * COLS / (4 * T), kRow = COLS / 4, kStep = T / kRow;
  static_assert(U * 4 * T == ROWS * COLS && kStep * kRow == T, "whole rounds only");
  float4 v[U];
  __device__ __forceinline__ void fetch(const float* __restrict__ src, int ld, int rows, int cols,
                                        bool vec) {
    const int r0 = (int)threadIdx.x / kRow, c = 4 * ((int)threadIdx.x % kRow);
    if (vec) {  // no branch inside, so the loads issue together
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * kStep;
        const bool ok = r < rows && c < cols;  // cols is a multiple of four too
        v[u] = *reinterpret_cast<const float4*>(src + (ok ? r * ld + c : 0));
        if (!ok) v[u] = float4{0.0f, 0.0f, 0.0f, 0.0f};
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u * kStep;
        float w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool ok = r < rows && c + q < cols;
          w[q] = src[ok ? r * ld + c + q : 0];
          if (!ok) w[q] = 0.0f;
        }
        v[u] = float4{w[0], w[1], w[2], w[3]};
      }
    }
  }
  __device__ __forceinline__ void put(float* dst, int pitch) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float* d = dst + ((int)threadIdx.x / kRow + u * kStep) * pitch + 4 * ((int)threadIdx.x % kRow);
      d[0] = v[u].x;
      d[1] = v[u].y;
      d[2] = v[u].z;
      d[3] = v[u].w;
    }
  }
};
__device__ __forceinline__ bool vec4(const float* p, int ld) {
  return ld % 4 == 0 && reinterpret_cast<uintptr_t>(p) % 16 == 0;
}

// One layer over rows of a batch.  Forward (BACK = false): z = X W^T + b with
// W [N][K]; z (if wanted) and silu(z) are stored.  Backward (BACK = true):
// Z = (X W) silu'(Z) in place, W [K][N].  A workgroup takes ROWS rows and 4,096 /
// ROWS columns.  32 x 128: 256 workgroups for 8,192 rows and a width up to 128,
// one per compute unit, so its eight waves (16 rows and 32 columns each) are all
// there is to cover the loads' and the epilogue's latency (four waves of 32 x 32:
// 11.5 us for a width of 128, eight 9.6).  Narrower layers take taller tiles
// (tile_rows), whose waves all have columns.
// Operands of v_mfma_f32_16x16x4f32: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator r of lane l is C[4 (l / 16) + r][l % 16].
typedef float float4_v __attribute__((ext_vector_type(4)));
constexpr int kLayerT = 512;
template <bool BACK, int ROWS>
__global__ void __launch_bounds__(kLayerT) k_layer(int n, int N, int K,
                                                   const float* __restrict__ X,
                                                   const float* __restrict__ W,
                                                   const float* __restrict__ bias,
                                                   float* __restrict__ Z, float* __restrict__ H) {
  constexpr int COLS = kTile * kTileN / ROWS, kAcross = COLS / 32;  // waves across
  // rows of X and (forward) of W are stored one word apart from a multiple of
  // the bank count: a tile's lanes read its rows at one depth
  __shared__ float Xs[ROWS][kTileK + 1];
  __shared__ float Ws[COLS * (kTileK + 1)];
  const int t = threadIdx.x, lane = t % 64, wv = t / 64, c = lane % 16, kq = lane / 16;
  const int64_t i0 = (int64_t)blockIdx.x * ROWS;
  const int iw = 16 * (wv / kAcross);                       // the wave's rows
  const int j0 = blockIdx.y * COLS, jw = 32 * (wv % kAcross);  // and columns
  const bool live = j0 + jw < N;
  const int rows = (int)min((int64_t)ROWS, n - i0);
  const bool vx = vec4(X, K), vw = vec4(W, BACK ? N : K);
  Staged<ROWS, kTileK, kLayerT> xs;
  Staged<BACK ? kTileK : COLS, BACK ? COLS : kTileK, kLayerT> ws;
  auto fetch = [&](int k0) {  // entries past the matrix are zeros
    const int kn = min(kTileK, K - k0);
    xs.fetch(X + i0 * K + k0, K, rows, kn, vx);
    if (BACK)
      ws.fetch(W + (int64_t)k0 * N + j0, N, kn, N - j0, vw);
    else
      ws.fetch(W + (int64_t)j0 * K + k0, K, N - j0, kn, vw);
  };
  float4_v acc[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += kTileK) {
    const int kn = min(kTileK, K - k0);
    __syncthreads();  // the last chunk's readers are done
    xs.put(&Xs[0][0], kTileK + 1);
    ws.put(Ws, BACK ? COLS : kTileK + 1);
    __syncthreads();
    if (k0 + kTileK < K) fetch(k0 + kTileK);
    if (live) {
      for (int kk = 0; kk < kn; kk += 16) {
#pragma unroll
        for (int u = 0; u < 16; u += 4) {
          const int k = kk + u + kq;
          const float a = Xs[iw + c][k];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int j = jw + 16 * h + c;
            const float b = BACK ? Ws[k * COLS + j] : Ws[j * (kTileK + 1) + k];
            acc[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[h], 0, 0, 0);
          }
        }
      }
    }
  }
  if (!live) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = j0 + jw + 16 * h + c;
    if (j >= N) continue;
    const float bj = BACK ? 0.0f : bias[j];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t i = i0 + iw + 4 * kq + r;
      if (i >= n) continue;
      const int64_t e = i * N + j;
      if (BACK) {
        Z[e] = acc[h][r] * dsilu_f(Z[e]);
      } else {
        const float z = acc[h][r] + bj;
        if (Z) Z[e] = z;
        H[e] = silu_f(z);
      }
    }
  }
}

// The output layer y = H w + b, 16 lanes per row.  Training (t given): also
// g = 2/n (y - t), the gradient g w silu'(Z) of the last hidden layer's
// pre-activations in place of Z, and the block's share of the squared error.
constexpr int kOutLanes = 16, kOutRows = kBlock / kOutLanes;
__global__ void __launch_bounds__(kBlock) k_output(int n, int width, const float* __restrict__ H,
                                                   const float* __restrict__ w,
                                                   float* __restrict__ y,
                                                   const float* __restrict__ t,
                                                   float* __restrict__ g, float* __restrict__ Z,
                                                   double* __restrict__ partials) {
  const int lane = threadIdx.x % kOutLanes, sub = threadIdx.x / kOutLanes;
  const float b = w[width];
  double loss = 0.0;
  const int64_t rows = ((int64_t)n + kOutRows - 1) / kOutRows;
  for (int64_t q = blockIdx.x; q < rows; q += gridDim.x) {
    const int64_t i = q * kOutRows + sub;
    float s = 0.0f;
    if (i < n)
      for (int j = lane; j < width; j += kOutLanes) s = s + H[i * width + j] * w[j];
#pragma unroll
    for (int o = kOutLanes / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kOutLanes);
    if (i >= n) continue;
    const float yi = s + b;
    if (!t) {
      if (lane == 0) y[i] = yi;
      continue;
    }
    const float e = yi - t[i];
    const float gi = (2.0f / (float)n) * e;
    if (lane == 0) {
      g[i] = gi;
      loss += (double)e * (double)e;
    }
    for (int j = lane; j < width; j += kOutLanes) {
      const int64_t at = i * width + j;
      Z[at] = gi * w[j] * dsilu_f(Z[at]);
    }
  }
  if (t) {
    double v[1] = {loss};
    write_partials<kBlock, 1>(v, partials);
  }
}

// Weight and bias gradients of every layer: layer l's dW [M][N] = G^T Hin and
// db [M] = column sums of G over a chunk of rows (blockIdx.y), as that
// chunk's copy of the packed gradient.  blockIdx.x counts the layers' tiles of
// 32 x 128 outputs.
constexpr int kMaxLayers = 16;  // layers of one k_grads dispatch
struct GradLayer {
  const float* G;   // [n][M]
  const float* Hin; // [n][N]
  int64_t woff, boff;
  int M, N, tile0;  // first tile of the layer
};
struct GradArgs {
  GradLayer l[kMaxLayers];
  int layers;
};
__global__ void __launch_bounds__(256) k_grads(GradArgs a, int n, int chunk, int64_t n_params,
                                               float* __restrict__ parts) {
  __shared__ float Gs[kTileK][kTile];
  __shared__ float Hs[kTileK][kTileN];
  __shared__ float bs[8][kTile];
  int li = 0;
  while (li + 1 < a.layers && (int)blockIdx.x >= a.l[li + 1].tile0) ++li;
  const GradLayer L = a.l[li];
  const int tn = (L.N + kTileN - 1) / kTileN, tile = blockIdx.x - L.tile0;
  const int o0 = (tile / tn) * kTile, j0 = (tile % tn) * kTileN;
  const int t = threadIdx.x, lane = t % 64, wv = t / 64, c = lane % 32, half = lane / 32;
  const int jw = wv * kTile;
  const bool live = j0 + jw < L.N;
  const int64_t r0 = (int64_t)blockIdx.y * chunk, r1 = r0 + chunk < n ? r0 + chunk : n;
  const bool vg = vec4(L.G, L.M), vh = vec4(L.Hin, L.N);
  float16_t acc = {0};
  float db = 0.0f;
  Staged<kTileK, kTile, 256> gs;
  Staged<kTileK, kTileN, 256> hs;
  auto fetch = [&](int64_t k0) {
    const int rows = (int)min((int64_t)kTileK, r1 - k0);
    gs.fetch(L.G + k0 * L.M + o0, L.M, rows, L.M - o0, vg);
    hs.fetch(L.Hin + k0 * L.N + j0, L.N, rows, L.N - j0, vh);
  };
  fetch(r0);
  for (int64_t k0 = r0; k0 < r1; k0 += kTileK) {
    __syncthreads();  // the last chunk's readers are done
    gs.put(&Gs[0][0], kTile);
    hs.put(&Hs[0][0], kTileN);
    __syncthreads();
    if (k0 + kTileK < r1) fetch(k0 + kTileK);
    if (j0 == 0)  // eight runs of rows per column, added below
      for (int kk = t / kTile; kk < kTileK; kk += 8) db = db + Gs[kk][t % kTile];
    if (live) {
#pragma unroll 8
      for (int kk = 0; kk < kTileK; kk += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(Gs[kk + half][c], Hs[kk + half][jw + c], acc, 0,
                                                   0, 0);
    }
  }
  float* out = parts + (size_t)blockIdx.y * n_params;
  if (j0 == 0) {
    bs[t / kTile][t % kTile] = db;
    __syncthreads();
    if (t < kTile && o0 + t < L.M) {
      float s = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) s = s + bs[k][t];
      out[L.boff + o0 + t] = s;
    }
  }
  const int j = j0 + jw + c;
  if (!live || j >= L.N) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int o = o0 + acc_row(r, lane);
    if (o < L.M) out[L.woff + (int64_t)o * L.N + j] = acc[r];
  }
}

// grad[e] = sum over the chunks of parts, in chunk order; the last block adds
// the loss partials.
__global__ void __launch_bounds__(kBlock) k_sum_grads(int64_t len, int nz,
                                                      const float* __restrict__ parts,
                                                      float* __restrict__ grad,
                                                      const double* __restrict__ partials, int g,
                                                      int n, double* __restrict__ loss) {
  if (blockIdx.x == gridDim.x - 1) {
    const double s = sum_partials<kBlock>(partials, g);
    if (threadIdx.x == 0) *loss = s / n;
    return;
  }
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= len) return;
  float s = 0.0f;
#pragma unroll 8
  for (int z = 0; z < nz; ++z) s = s + parts[(size_t)z * len + e];
  grad[e] = s;
}

__global__ void k_adam(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, float lr, float c1, float c2) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n) return;
  const float b1 = 0.9f, b2 = 0.999f;
  const float mm = b1 * m[e] + (1.0f - b1) * g[e];
  const float vv = b2 * v[e] + (1.0f - b2) * g[e] * g[e];
  m[e] = mm;
  v[e] = vv;
  p[e] = p[e] - lr * (mm / c1) / (sqrtf(vv / c2) + 1e-8f);
}

__global__ void k_to_bf16(int64_t n, const float* __restrict__ a, uint16_t* __restrict__ b) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= n) return;
  // round to nearest even
  uint32_t u = __float_as_uint(a[e]);
  u += 0x7FFFu + ((u >> 16) & 1u);
  b[e] = (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------- BF16 inference
typedef short short4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

constexpr int kW = 128;      // hidden width of the MFMA path
constexpr int kIn = 10;      // input features of the MFMA path
constexpr int kWaves = 4;    // waves per workgroup, 32 cells each

// One wave per tile of 32 cells; hidden activations live in LDS as
// [cell][feature] bf16.  For a hidden layer, out^T (features x cells) =
// W (width x width) . h^T: 4 output tiles of 32 features, 16 k-steps of 8.
// Operand layout of v_mfma_f32_32x32x8bf16_1k: lane l holds A[l%32][4(l/32)+v]
// and B[4(l/32)+v][l%32] (v = 0..3); accumulator r of lane l is
// C[8(r/4) + 4(l/32) + r%4][l%32].
__global__ void __launch_bounds__(64 * kWaves) k_mlp_infer_bf16(
    int n, int n_hidden, const float* __restrict__ x, const float* __restrict__ params,
    const uint16_t* __restrict__ wbf, float* __restrict__ y) {
  __shared__ uint16_t hA[kWaves][32 * kW];
  __shared__ uint16_t hB[kWaves][32 * kW];
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  const int cell = lane % 32, half = lane / 32;
  const float* W1 = params;
  const float* b1 = W1 + kW * kIn;
  const int64_t hid = (int64_t)kW * kW + kW;
  const float* last = b1 + kW + (n_hidden - 1) * hid;  // W_out [1 x kW], then b_out
  const int ntile = (n + 31) / 32;
  // every wave of the workgroup runs the same trip count (the barriers below
  // are workgroup-wide); tiles past the end compute on zeros and store nothing
  for (int base = blockIdx.x * kWaves; base < ntile; base += gridDim.x * kWaves) {
    const int tile = base + wv;
    const int c = tile * 32 + cell;
    // layer 1 (n_in -> width) in FP32: this lane does features half*64 .. +63
    float xin[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) xin[k] = c < n ? x[(size_t)c * kIn + k] : 0.0f;
    for (int f = half * 64; f < half * 64 + 64; ++f) {
      float s = b1[f];
#pragma unroll
      for (int k = 0; k < kIn; ++k) s = s + W1[f * kIn + k] * xin[k];
      hA[wv][cell * kW + f] = f2bf(silu_f(s));
    }
    __syncthreads();
    uint16_t* hin = hA[wv];
    uint16_t* hout = hB[wv];
    for (int l = 0; l < n_hidden - 1; ++l) {
      const uint16_t* W = wbf + (size_t)l * kW * kW;
      const float* bias = b1 + kW + l * hid + kW * kW;
      for (int mt = 0; mt < kW / 32; ++mt) {
        float16_t acc = {0};
        for (int kt = 0; kt < kW / 8; ++kt) {
          const int kk = kt * 8 + 4 * half;
          short4_t a, b;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            a[v] = (short)W[(size_t)(mt * 32 + cell) * kW + kk + v];
            b[v] = (short)hin[cell * kW + kk + v];
          }
          acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int f = mt * 32 + 8 * (r / 4) + 4 * half + (r % 4);
          hout[cell * kW + f] = f2bf(silu_f(acc[r] + bias[f]));
        }
      }
      __syncthreads();
      uint16_t* tmp = hin;
      hin = hout;
      hout = tmp;
    }
    // output layer (width -> 1) in FP32 from the bf16 activations
    float s = 0.0f;
    for (int f = half * 64; f < half * 64 + 64; ++f)
      s = s + last[f] * __uint_as_float((uint32_t)hin[cell * kW + f] << 16);
    s = s + __shfl_down(s, 32, 64);
    if (half == 0 && c < n) y[c] = s + last[kW];
    __syncthreads();
  }
}

// The inference pass used at every timestep.  With out^T = W h^T (features x
// cells), a lane's accumulators r = 4q .. 4q+3 of tile mt hold features
// 32 mt + 8 q + 4 (lane / 32) + 0..3 of one cell: exactly the four values that
// lane supplies as the next layer's B operand in k-step 4 mt + q.  So a wave
// keeps its 32 cells' activations in registers from the first layer to the
// last; LDS holds only what all waves share, the BF16 weights as quads of 8
// bytes (weight (f, k) in quad (k/4) 128 + f: one conflict-free read per lane
// and operand), the first layer's split weights, the biases and the output
// weights.
//
// Bound by the vector ALUs: a cell's 384 SiLUs (five operations and two
// transcendentals each) cost more cycles than its matrix products.  What the
// layout buys is the room for waves to run one's products beside another's
// SiLUs: with the activations in LDS as well (8 KB per wave) and the split
// weights in registers, eight waves fitted a compute unit and took turns;
// twelve run now, 600 k cells in 123 us (148 before), the same results
// bit for bit.
//
// Roundings are those of the pass above: the first layer is formed to FP32
// accuracy on the matrix cores from three-way BF16 splits of x and W1
// (x = x0 + x1 + x2, 8 bits each; the six products x_i w_j with i + j <= 2,
// exact in the FP32 accumulator; the dropped ones are below 2^-24 of the
// sum), every hidden activation and the width x width weights are BF16,
// the output layer is an FP32 dot product with the last BF16 activations.
// SiLU uses the hardware exp2 and reciprocal (about 1 ulp of FP32 each,
// far below the BF16 rounding that follows).
// Waves of a workgroup, one workgroup per compute unit.  A wave's tiles are its
// rounds, and a round of twelve waves takes 4/3 of one of eight (two mid layers
// and one: 14.0 and 10.3 us, three: 19.3 and 14.6), so twelve run where that
// makes up for itself in fewer rounds: 80 k cells and four hidden layers 40 us
// with twelve and 49 with eight, 100 k 58 and 49, 600 k 154 and 163.
constexpr int kWavesM = 12, kWavesFew = 8;
inline int infer_waves(int tiles, int cus) {
  const auto rounds = [&](int waves) { return (tiles + cus * waves - 1) / (cus * waves); };
  return 4 * rounds(kWavesM) < 3 * rounds(kWavesFew) ? kWavesM : kWavesFew;
}

__device__ __forceinline__ float silu_hw(float z) {
  const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * z);
  return z * __builtin_amdgcn_rcpf(1.0f + e);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Two FP32 values rounded to BF16 (nearest, ties to even) in one gfx950
// conversion (v_cvt_pk_bf16_f32), the first in the low half.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(float2_t{a, b}, bf16x2_t));
}

// LDS: n_mid weight matrices, then the first layer's split operands
// [part][mt][kt][lane], then the biases of every layer and the output weights.
constexpr int kQuads = kW * kW / 4;       // quads of one width x width matrix
constexpr int kSplitQuads = 3 * 4 * 2 * 64;
inline size_t infer_lds(int n_mid) {
  return 8 * ((size_t)n_mid * kQuads + kSplitQuads) + 4 * ((size_t)(n_mid + 2) * kW + 4);
}

__global__ void __launch_bounds__(64 * kWavesM) k_mlp_infer_mfma(
    int n, int n_mid, const float* __restrict__ x, const float* __restrict__ params,
    const uint16_t* __restrict__ wbf, float* __restrict__ y) {
  extern __shared__ uint64_t lds_q[];
  uint64_t* wq = lds_q;                                  // n_mid matrices
  uint64_t* split = wq + (size_t)n_mid * kQuads;         // first-layer A operands
  float* vecs = reinterpret_cast<float*>(split + kSplitQuads);  // n_mid + 1 biases, W_out, b_out
  const int lane = threadIdx.x % 64, wv = threadIdx.x / 64;
  const int cell = lane % 32, half = lane / 32;
  // W_l[f][4kq .. 4kq+3] is 8 contiguous bytes
  for (int q = threadIdx.x; q < n_mid * kQuads; q += blockDim.x) {
    const int l = q / kQuads, rem = q % kQuads, kq = rem / kW, f = rem % kW;
    wq[q] = *reinterpret_cast<const uint64_t*>(wbf + (size_t)l * kW * kW + (size_t)f * kW + 4 * kq);
  }
  const float* W1 = params;
  const float* b1 = W1 + kW * kIn;
  const int64_t hid = (int64_t)kW * kW + kW;
  const float* last = b1 + kW + (int64_t)n_mid * hid;  // W_out [kW], then b_out
  // A[f][k] = W1[mt 32 + cell][8 kt + 4 half + v], zero for k >= n_in, in
  // three BF16 parts
  for (int e = threadIdx.x; e < 4 * 2 * 64; e += blockDim.x) {
    const int mt = e / 128, kt = (e / 64) % 2, ln = e % 64;
    uint64_t part[3] = {0, 0, 0};
    for (int v = 0; v < 4; ++v) {
      const int k = kt * 8 + 4 * (ln / 32) + v;
      float w = k < kIn ? W1[(mt * 32 + ln % 32) * kIn + k] : 0.0f;
      for (int p = 0; p < 3; ++p) {
        const uint16_t h = f2bf(w);
        part[p] |= (uint64_t)h << (16 * v);
        w = w - bf2f(h);
      }
    }
    for (int p = 0; p < 3; ++p) split[(p * 8 + mt * 2 + kt) * 64 + ln] = part[p];
  }
  for (int e = threadIdx.x; e < (n_mid + 2) * kW + 1; e += blockDim.x) {
    const int l = e / kW;
    vecs[e] = l == 0 ? b1[e]
              : l <= n_mid ? b1[kW + (int64_t)(l - 1) * hid + kW * kW + e % kW]
                           : last[e - (n_mid + 1) * kW];
  }
  __syncthreads();
  const int ntile = (n + 31) / 32;
  // this lane's inputs of a tile: x[c][8 kt + 4 half + v] (zero past n_in)
  float xin[2][4];
  auto fetch = [&](int tile) {
    const int c = tile * 32 + cell;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = kt * 8 + 4 * half + v;
        xin[kt][v] = c < n && k < kIn ? x[(size_t)c * kIn + k] : 0.0f;
      }
  };
  const int waves = blockDim.x / 64, all = gridDim.x * waves;
  int tile = blockIdx.x * waves + wv;
  if (tile < ntile) fetch(tile);
  for (; tile < ntile; tile += all) {
    const int c = tile * 32 + cell;
    // layer 1: B[k][cell] in three BF16 parts
    short4_t b1p[3][2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float xv = xin[kt][v];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const uint16_t h = f2bf(xv);
          b1p[p][kt][v] = (short)h;
          xv = xv - bf2f(h);
        }
      }
    if (tile + all < ntile) fetch(tile + all);
    float16_t acc[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      acc[mt] = float16_t{0};
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {  // smallest products first
        short4_t a[3];
#pragma unroll
        for (int p = 0; p < 3; ++p)
          a[p] = __builtin_bit_cast(short4_t, split[(p * 8 + mt * 2 + kt) * 64 + lane]);
        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[0], b1p[2][kt], acc[mt], 0, 0, 0);
        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[1], b1p[1][kt], acc[mt], 0, 0, 0);
        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[2], b1p[0][kt], acc[mt], 0, 0, 0);
        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[0], b1p[1][kt], acc[mt], 0, 0, 0);
        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[1], b1p[0][kt], acc[mt], 0, 0, 0);
        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a[0], b1p[0][kt], acc[mt], 0, 0, 0);
      }
    }
    const float* bias = vecs;
    for (int l = 0; l < n_mid; ++l, bias += kW) {
      // SiLU of the accumulators (bias added), rounded to BF16: quad 4 mt + q
      uint64_t h[16];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 bq = *reinterpret_cast<const float4*>(bias + mt * 32 + 8 * q + 4 * half);
          const uint32_t lo = bf16_pair(silu_hw(acc[mt][4 * q] + bq.x), silu_hw(acc[mt][4 * q + 1] + bq.y));
          const uint32_t hi = bf16_pair(silu_hw(acc[mt][4 * q + 2] + bq.z), silu_hw(acc[mt][4 * q + 3] + bq.w));
          h[4 * mt + q] = (uint64_t)lo | ((uint64_t)hi << 32);
        }
      // hidden layer l: out^T = W_l h^T, all four output tiles in registers
      const uint64_t* W = wq + (size_t)l * kQuads;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) acc[mt] = float16_t{0};
#pragma unroll
      for (int kt = 0; kt < kW / 8; ++kt) {
        const short4_t b = __builtin_bit_cast(short4_t, h[kt]);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const short4_t a = __builtin_bit_cast(short4_t, W[(2 * kt + half) * kW + mt * 32 + cell]);
          acc[mt] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, acc[mt], 0, 0, 0);
        }
      }
    }
    // the last hidden layer feeds the output layer
    const float* wout = bias + kW;
    float s = 0.0f;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f0 = mt * 32 + 8 * q + 4 * half;
        const float4 bq = *reinterpret_cast<const float4*>(bias + f0);
        const float4 wo = *reinterpret_cast<const float4*>(wout + f0);
        const uint32_t lo = bf16_pair(silu_hw(acc[mt][4 * q] + bq.x), silu_hw(acc[mt][4 * q + 1] + bq.y));
        const uint32_t hi = bf16_pair(silu_hw(acc[mt][4 * q + 2] + bq.z), silu_hw(acc[mt][4 * q + 3] + bq.w));
        s = s + wo.x * __uint_as_float(lo << 16);
        s = s + wo.y * __uint_as_float(lo & 0xFFFF0000u);
        s = s + wo.z * __uint_as_float(hi << 16);
        s = s + wo.w * __uint_as_float(hi & 0xFFFF0000u);
      }
    s = s + __shfl_down(s, 32, 64);
    if (half == 0 && c < n) y[c] = s + wout[kW];
  }
}

// ---------------------------------------------------------------- warm-start features
// Pressure fields are referenced to each pocket's current pin (p = 0 there):
// a previous field is re-referenced by subtracting its value at the pin of
// the cell's pocket (comp[c]), which removes the constant jump a pocket's
// pressure takes when its lowest cell, and so its pin, changes.
__global__ void k_ws_stats(int na, const int* __restrict__ perm, const int* __restrict__ comp,
                           const double* __restrict__ dp, const double* __restrict__ rhs,
                           const double* __restrict__ vol, double* __restrict__ partials) {
  double s[3] = {0.0, 0.0, 0.0};
  for (int r = blockIdx.x * kBlock + threadIdx.x; r < na; r += gridDim.x * kBlock) {
    const int c = perm[r];
    const double d = dp[c] - dp[comp[c]];
    s[0] += d * d;
    s[1] += rhs[c] * rhs[c];
    s[2] += vol[c];
  }
  write_partials<kBlock, 3>(s, partials);
}

// The statistics from their partials; the first also goes to *host, pinned
// memory that the host reads once the stream has been waited for.
__global__ void k_ws_stats_final(const double* __restrict__ partials, int g, int na,
                                 double* __restrict__ out, double* __restrict__ host) {
  const double* const parts[3] = {partials, partials + g, partials + 2 * g};
  double s[3];
  sum_partials_n<kBlock, 3>(parts, g, s);
  if (threadIdx.x == 0) {
    out[0] = sqrt(s[0] / na);  // RMS of the previous increment
    out[1] = sqrt(s[1] / na);  // RMS of the right-hand side
    out[2] = s[2] / na;        // mean cell volume
    *host = out[0];
  }
}

// Features of active cell r (cell c), before standardisation:
//   0 previous increment (re-referenced) / its RMS, 1 rhs / its RMS, 2 liquid fraction,
//   3 volume / mean volume, 4..9 the six largest open-face coefficients of
//   the cell divided by their sum (descending, 0 where fewer).
// Bound by memory: about 190 bytes per cell, most of them gathered.  With DEG
// > 0 (no cell has more neighbours) a thread requests all neighbours, then all
// their flags and coefficients, where the plain loop waited for three loads in
// turn per neighbour; the features leave through LDS, so that a wave's stores
// are contiguous instead of 40 bytes apart.  600 k cells: 37 -> 23 us.
template <int DEG>
__global__ void __launch_bounds__(kBlock) k_ws_features(
    int na, const int* __restrict__ perm, const int* __restrict__ comp,
    const int* __restrict__ adj_ptr, const int* __restrict__ adj_nbr,
    const int* __restrict__ adj_face, const int* __restrict__ active,
    const double* __restrict__ dp, const double* __restrict__ rhs, const double* __restrict__ fl,
    const double* __restrict__ vol, const double* __restrict__ coeff,
    const double* __restrict__ st, const float* __restrict__ mu, const float* __restrict__ sigma,
    float* __restrict__ out) {
  __shared__ float rows[kBlock * 10];
  const int r0 = blockIdx.x * kBlock, r = r0 + threadIdx.x;
  if (r < na) {
    const int c = perm[r];
    const int k0 = adj_ptr[c], k1 = adj_ptr[c + 1];
    double top[6] = {0, 0, 0, 0, 0, 0};
    double sum = 0.0;
    auto take = [&](double v) {
      sum += v;
#pragma unroll
      for (int q = 0; q < 6; ++q)  // insert into the descending top-6
        if (v > top[q]) { const double t = top[q]; top[q] = v; v = t; }
    };
    if constexpr (DEG > 0) {
      int nb[DEG], fc[DEG], on[DEG];
      double v[DEG];
#pragma unroll
      for (int u = 0; u < DEG; ++u) {
        nb[u] = k0 + u < k1 ? adj_nbr[k0 + u] : -1;
        fc[u] = k0 + u < k1 ? adj_face[k0 + u] : -1;
      }
#pragma unroll
      for (int u = 0; u < DEG; ++u) {
        on[u] = nb[u] >= 0 ? active[nb[u]] : 0;
        v[u] = fc[u] >= 0 ? coeff[fc[u]] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < DEG; ++u)
        if (on[u]) take(v[u]);
    } else {
      for (int k = k0; k < k1; ++k)
        if (active[adj_nbr[k]]) take(coeff[adj_face[k]]);
    }
    float f[10];
    f[0] = st[0] > 0.0 ? (float)((dp[c] - dp[comp[c]]) / st[0]) : 0.0f;
    f[1] = st[1] > 0.0 ? (float)(rhs[c] / st[1]) : 0.0f;
    f[2] = (float)fl[c];
    f[3] = st[2] > 0.0 ? (float)(vol[c] / st[2]) : 0.0f;
#pragma unroll
    for (int q = 0; q < 6; ++q) f[4 + q] = sum > 0.0 ? (float)(top[q] / sum) : 0.0f;
#pragma unroll
    for (int k = 0; k < 10; ++k) rows[threadIdx.x * 10 + k] = (f[k] - mu[k]) / sigma[k];
  }
  __syncthreads();
  const int cnt = min(kBlock, na - r0) * 10;
  for (int e = threadIdx.x; e < cnt; e += kBlock) out[(size_t)r0 * 10 + e] = rows[e];
}

// x0 = p_prev (re-referenced) + scale * y on active non-pin cells, 0 elsewhere
__global__ void k_ws_apply(int nc, const int* __restrict__ cid, const int* __restrict__ comp,
                           const double* __restrict__ p_prev, const float* __restrict__ yv,
                           double scale, double* __restrict__ x0) {
  const int c = blockIdx.x * kBlock + threadIdx.x;
  if (c >= nc) return;
  const int r = cid[c];
  x0[c] = (r < 0 || comp[c] == c) ? 0.0 : (p_prev[c] - p_prev[comp[c]]) + scale * (double)yv[r];
}

// training target of active cell r: (p_new - p_prev re-referenced) / scale
__global__ void k_ws_targets(int na, const int* __restrict__ perm, const int* __restrict__ comp,
                             const double* __restrict__ p_new, const double* __restrict__ p_prev,
                             double scale, float* __restrict__ t) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= na) return;
  const int c = perm[r];
  t[r] = scale > 0.0 ? (float)((p_new[c] - (p_prev[c] - p_prev[comp[c]])) / scale) : 0.0f;
}

// ---------------------------------------------------------------- host side
// Workspace of ppe_warm_start_features_noalloc: the statistics' block
// partials (at most kRedBlocks per statistic) and the three statistics, in a
// static device array instead of solver memory.  Each device holds its own
// copy for the life of the process; host code reaches it only through the
// address hipGetSymbolAddress gives on that device (the array's name is a
// host-side stand-in there).
constexpr int kWsScratch = 3 * kRedBlocks + 3;
static __device__ __align__(256) double scratch[kWsScratch];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch[kMaxDevices] = {};

// The device address of `scratch` on `device`, looked up once per device
// with that device current.
double* ws_scratch(int device) {
  require(device >= 0 && device < kMaxDevices, PPE_ERR_ARG, "device index out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[device]) {
    int prev = -1;
    PPE_HIP(hipGetDevice(&prev));
    if (prev != device) PPE_HIP(hipSetDevice(device));
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (prev != device) (void)hipSetDevice(prev);
    PPE_HIP(e);
    require(ptr != nullptr, PPE_ERR_HIP, "hipGetSymbolAddress gave no address for the workspace");
    g_scratch[device] = static_cast<double*>(ptr);
  }
  return g_scratch[device];
}

// The warm-start features of the assembled solver's active cells with the
// statistics' partials in `part` (3 red_grid(n_active) + 3 doubles, written
// before they are read: nothing needs clearing).  *dp_scale comes back through
// the solver's pinned box.
ppe_status ws_features(ppe_solver* s, const double* dp_prev, const double* rhs,
                       const double* face_coeff, const double* fl, const double* cell_volume,
                       const float* mu, const float* sigma, float* features, double* dp_scale,
                       double* part) {
  const int na = s->n_active;
  if (na == 0) {
    *dp_scale = 0.0;
    return PPE_OK;
  }
  const int g = red_grid(na);
  hipLaunchKernelGGL(k_ws_stats, dim3(g), dim3(kBlock), 0, s->stream, na, s->perm.as<int>(),
                     s->comp_full.as<int>(), dp_prev, rhs, cell_volume, part);
  PPE_LAUNCH_CHECK();
  ensure_box(s, kBoxScale + 2);  // made by the assembly: nothing is allocated here
  hipLaunchKernelGGL(k_ws_stats_final, dim3(1), dim3(kBlock), 0, s->stream, part, g, na,
                     part + 3 * g, reinterpret_cast<double*>(s->box_d + kBoxScale));
  PPE_LAUNCH_CHECK();
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid_for(na)), dim3(kBlock), 0, s->stream, na,
                       s->perm.as<int>(), s->comp_full.as<int>(), s->adj_ptr.as<int>(),
                       s->adj_nbr.as<int>(), s->adj_face.as<int>(), s->active.as<int>(), dp_prev,
                       rhs, fl, cell_volume, face_coeff, part + 3 * g, mu, sigma, features);
  };
  if (s->max_deg <= 6)
    run(k_ws_features<6>);
  else
    run(k_ws_features<0>);
  PPE_LAUNCH_CHECK();
  PPE_HIP(hipStreamSynchronize(s->stream));
  std::memcpy(dp_scale, s->box_h + kBoxScale, sizeof(double));
  return PPE_OK;
}

// Rows of a layer's tile: as tall as its columns allow where the rows still give
// every compute unit one (256 of them).  One million rows forward, 32 rows and as
// below: width 1 235 and 87 us, three layers of 16 610 and 205, of 64 1,132 and
// 593; 8,192 rows do not change (their tiles would leave compute units idle).
int tile_rows(int n, int N) {
  if (N <= 32 && n >= 128 * 256) return 128;
  if (N <= 64 && n >= 64 * 256) return 64;
  return kTile;
}

// Rows of one launch: a grid holds at most 2^32 threads along a dimension, and
// 32 rows take 512.
constexpr int kLayerRows = 1 << 27;

template <bool BACK>
void layer(ppe_mlp* m, int n, int N, int K, const float* X, const float* W, const float* bias,
           float* Z, float* H) {
  const int rows = tile_rows(n, N), cols = kTile * kTileN / rows;
  auto run = [&](auto kernel) {
    for (int64_t i = 0; i < n; i += kLayerRows) {
      const int part = (int)std::min<int64_t>(n - i, kLayerRows);
      const dim3 grid((unsigned)((part + (int64_t)rows - 1) / rows), (N + cols - 1) / cols);
      hipLaunchKernelGGL(kernel, grid, dim3(kLayerT), 0, m->stream, part, N, K, X + i * K, W, bias,
                         Z ? Z + i * N : nullptr, H ? H + i * N : nullptr);
      PPE_LAUNCH_CHECK();
    }
  };
  if (rows == 128)
    run(k_layer<BACK, 128>);
  else if (rows == 64)
    run(k_layer<BACK, 64>);
  else
    run(k_layer<BACK, kTile>);
}

// The hidden layers of n rows: activations into m->act and, for the backward
// pass, pre-activations into m->pre.  Returns the last hidden activations.
const float* hidden_layers(ppe_mlp* m, int n, const float* x, bool keep_pre) {
  const int64_t len = (int64_t)n * m->width;
  float* act = m->act.get<float>((size_t)len * m->n_hidden);
  float* pre = keep_pre ? m->pre.get<float>((size_t)len * m->n_hidden) : nullptr;
  const float* P = m->params.as<float>();
  const float* h = x;
  for (int l = 0; l < m->n_hidden; ++l) {
    layer<false>(m, n, m->width, m->dims[l], h, P + m->woff[l], P + m->boff[l],
                 pre ? pre + l * len : nullptr, act + l * len);
    h = act + l * len;
  }
  return h;
}

int output_grid(int n) {
  const int64_t g = ((int64_t)n + kOutRows - 1) / kOutRows;
  return (int)std::min<int64_t>(g, kRedBlocks);
}

// FP32 forward of n rows into y.
void forward_fp32(ppe_mlp* m, int n, const float* x, float* y) {
  const float* h = hidden_layers(m, n, x, false);
  hipLaunchKernelGGL(k_output, dim3(output_grid(n)), dim3(kBlock), 0, m->stream, n, m->width, h,
                     m->params.as<float>() + m->woff[m->n_hidden], y, (const float*)nullptr,
                     (float*)nullptr, (float*)nullptr, (double*)nullptr);
  PPE_LAUNCH_CHECK();
}

// Chunks of rows of the weight gradients: at least 128 rows each, at most 64
// chunks, and at most 128 MB of partial gradients (they are written and read
// once each; a network that large fills the device with its tiles alone).
constexpr int kGradRows = 128, kGradChunks = 64;
int grad_chunk(const ppe_mlp* m, int n) {
  const int64_t most = std::clamp<int64_t>((int64_t(1) << 25) / m->n_params, 1, kGradChunks);
  return std::max(kGradRows, (int)((n + most - 1) / most));
}

// Queues the packed gradient of the mean-squared error into grad and the
// loss into *m->loss_h (pinned: read it once the stream has been waited for).
void loss_grad(ppe_mlp* m, int n, const float* x, const float* t, float* grad) {
  const int L = m->n_hidden;  // the output layer
  const int64_t len = (int64_t)n * m->width;
  if (!m->loss_h) PPE_HIP(hipHostMalloc(reinterpret_cast<void**>(&m->loss_h), sizeof(double)));
  const float* P = m->params.as<float>();
  const float* h = hidden_layers(m, n, x, true);
  float* act = m->act.as<float>();
  float* pre = m->pre.as<float>();
  float* g = m->gbuf.get<float>(n);
  const int go = output_grid(n);
  double* lp = m->lossbuf.get<double>(go);
  hipLaunchKernelGGL(k_output, dim3(go), dim3(kBlock), 0, m->stream, n, m->width, h,
                     P + m->woff[L], (float*)nullptr, t, g, pre + (L - 1) * len, lp);
  PPE_LAUNCH_CHECK();
  // pre[l] turns into the gradient of layer l's pre-activations, last to first
  for (int l = L - 1; l > 0; --l) {
    layer<true>(m, n, m->width, m->width, pre + l * len, P + m->woff[l], nullptr,
                pre + (l - 1) * len, nullptr);
  }
  const int chunk = grad_chunk(m, n);
  const int nz = (int)(((int64_t)n + chunk - 1) / chunk);
  float* parts = m->part.get<float>((size_t)nz * m->n_params);
  for (int l0 = 0; l0 <= L; l0 += kMaxLayers) {
    GradArgs a{};
    int tiles = 0;
    a.layers = std::min(kMaxLayers, L + 1 - l0);
    for (int k = 0; k < a.layers; ++k) {
      const int l = l0 + k;
      a.l[k] = GradLayer{l == L ? g : pre + l * len, l == 0 ? x : act + (l - 1) * len, m->woff[l],
                         m->boff[l], m->dims[l + 1], m->dims[l], tiles};
      tiles += ((m->dims[l + 1] + kTile - 1) / kTile) * ((m->dims[l] + kTileN - 1) / kTileN);
    }
    hipLaunchKernelGGL(k_grads, dim3(tiles, nz), dim3(256), 0, m->stream, a, n, chunk,
                       m->n_params, parts);
    PPE_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(k_sum_grads, dim3(grid_for(m->n_params) + 1), dim3(kBlock), 0, m->stream,
                     m->n_params, nz, parts, grad, lp, go, n, m->loss_h);
  PPE_LAUNCH_CHECK();
}

void refresh_bf16(ppe_mlp* m) {
  if (m->n_in != kIn || m->width != kW || m->n_hidden < 1) return;
  const int nh = m->n_hidden - 1;  // width x width matrices
  if (nh <= 0) return;
  uint16_t* w = m->bf16.get<uint16_t>((size_t)nh * kW * kW);
  for (int l = 0; l < nh; ++l) {
    hipLaunchKernelGGL(k_to_bf16, dim3(grid_for((int64_t)kW * kW)), dim3(kBlock), 0, m->stream,
                       (int64_t)kW * kW, m->params.as<float>() + m->woff[l + 1],
                       w + (size_t)l * kW * kW);
    PPE_LAUNCH_CHECK();
  }
}

template <class F>
ppe_status mlp_guard(ppe_mlp* m, F&& f) {
  try {
    if (m) m->err.clear();
    return f();
  } catch (const Error& e) {
    if (m) m->err = e.what();
    return e.status;
  } catch (const std::exception& e) {
    if (m) m->err = e.what();
    return PPE_ERR_INTERNAL;
  }
}

}  // namespace
}  // namespace ppe

using namespace ppe;

extern "C" {

ppe_status ppe_mlp_create(int32_t n_in, int32_t width, int32_t n_hidden, void* stream,
                          ppe_mlp** out) {
  if (!out) return PPE_ERR_ARG;
  *out = nullptr;
  if (n_in < 1 || width < 1 || n_hidden < 1 || width > 4096 || n_in > 4096) return PPE_ERR_ARG;
  auto* m = new ppe_mlp();
  m->n_in = n_in;
  m->width = width;
  m->n_hidden = n_hidden;
  m->stream = static_cast<hipStream_t>(stream);
  m->dims.push_back(n_in);
  for (int k = 0; k < n_hidden; ++k) m->dims.push_back(width);
  m->dims.push_back(1);
  int64_t off = 0;
  for (size_t l = 0; l + 1 < m->dims.size(); ++l) {
    m->woff.push_back(off);
    off += (int64_t)m->dims[l + 1] * m->dims[l];
    m->boff.push_back(off);
    off += m->dims[l + 1];
  }
  m->n_params = off;
  ppe_status st = mlp_guard(m, [&]() -> ppe_status {
    float* p = m->params.get<float>(off);
    float* mm = m->m.get<float>(off);
    float* vv = m->v.get<float>(off);
    PPE_HIP(hipMemsetAsync(p, 0, sizeof(float) * off, m->stream));
    PPE_HIP(hipMemsetAsync(mm, 0, sizeof(float) * off, m->stream));
    PPE_HIP(hipMemsetAsync(vv, 0, sizeof(float) * off, m->stream));
    PPE_HIP(hipStreamSynchronize(m->stream));
    return PPE_OK;
  });
  if (st != PPE_OK) {
    delete m;
    return st;
  }
  *out = m;
  return PPE_OK;
}

void ppe_mlp_destroy(ppe_mlp* m) {
  if (!m) return;
  (void)hipStreamSynchronize(m->stream);
  if (m->loss_h) (void)hipHostFree(m->loss_h);
  delete m;
}

int64_t ppe_mlp_num_params(const ppe_mlp* m) { return m ? m->n_params : -1; }

const char* ppe_mlp_last_error(const ppe_mlp* m) { return m ? m->err.c_str() : ""; }

ppe_status ppe_mlp_set_params(ppe_mlp* m, const float* params) {
  if (!m || !params) return PPE_ERR_ARG;
  return mlp_guard(m, [&]() -> ppe_status {
    PPE_HIP(hipMemcpyAsync(m->params.as<float>(), params, sizeof(float) * m->n_params,
                           hipMemcpyDeviceToDevice, m->stream));
    PPE_HIP(hipMemsetAsync(m->m.as<float>(), 0, sizeof(float) * m->n_params, m->stream));
    PPE_HIP(hipMemsetAsync(m->v.as<float>(), 0, sizeof(float) * m->n_params, m->stream));
    m->adam_t = 0;
    refresh_bf16(m);
    PPE_HIP(hipStreamSynchronize(m->stream));
    return PPE_OK;
  });
}

ppe_status ppe_mlp_get_params(const ppe_mlp* m, float* params) {
  if (!m || !params) return PPE_ERR_ARG;
  ppe_mlp* mm = const_cast<ppe_mlp*>(m);
  return mlp_guard(mm, [&]() -> ppe_status {
    PPE_HIP(hipMemcpyAsync(params, m->params.as<float>(), sizeof(float) * m->n_params,
                           hipMemcpyDeviceToDevice, m->stream));
    PPE_HIP(hipStreamSynchronize(m->stream));
    return PPE_OK;
  });
}

ppe_status ppe_mlp_forward(ppe_mlp* m, int32_t n, const float* x, float* y, int bf16) {
  if (!m || n < 0 || (n > 0 && (!x || !y))) return PPE_ERR_ARG;
  if (n == 0) return PPE_OK;
  return mlp_guard(m, [&]() -> ppe_status {
    if (bf16) {
      require(m->n_in == kIn && m->width == kW && m->n_hidden >= 2, PPE_ERR_ARG,
              "the BF16 MFMA path needs 10 inputs, width 128 and >= 2 hidden layers");
      const int tiles = (n + 31) / 32;
      const int n_mid = m->n_hidden - 1;
      const size_t lds = infer_lds(n_mid);
      if (m->lds_max == 0) {
        int dev = 0, v = 0;
        PPE_HIP(hipGetDevice(&dev));
        PPE_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
        int cus = 0;
        PPE_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        m->lds_max = (size_t)v;
        m->cus = cus;
      }
      if (lds <= m->lds_max) {
        // one workgroup per compute unit holds the staged weights; waves
        // stride over the 32-cell tiles
        const int waves = infer_waves(tiles, m->cus);
        int g = (tiles + waves - 1) / waves;
        if (g > m->cus) g = m->cus;
        hipLaunchKernelGGL(k_mlp_infer_mfma, dim3(g), dim3(64 * waves), lds, m->stream, n,
                           n_mid, x, m->params.as<float>(), m->bf16.as<uint16_t>(), y);
      } else {  // deeper networks than the staged weights fit
        int g = (tiles + kWaves - 1) / kWaves;
        if (g > 2048) g = 2048;
        hipLaunchKernelGGL(k_mlp_infer_bf16, dim3(g), dim3(64 * kWaves), 0, m->stream, n,
                           m->n_hidden, x, m->params.as<float>(), m->bf16.as<uint16_t>(), y);
      }
      PPE_LAUNCH_CHECK();
    } else {
      forward_fp32(m, n, x, y);
    }
    PPE_HIP(hipStreamSynchronize(m->stream));
    return PPE_OK;
  });
}

ppe_status ppe_mlp_loss_grad(ppe_mlp* m, int32_t n, const float* x, const float* t, float* grad,
                             double* loss) {
  if (!m || n < 1 || !x || !t || !grad) return PPE_ERR_ARG;
  return mlp_guard(m, [&]() -> ppe_status {
    loss_grad(m, n, x, t, grad);
    PPE_HIP(hipStreamSynchronize(m->stream));
    if (loss) *loss = *m->loss_h;
    return PPE_OK;
  });
}

ppe_status ppe_mlp_train_step(ppe_mlp* m, int32_t n, const float* x, const float* t, float lr,
                              double* loss) {
  if (!m || n < 1 || !x || !t || !(lr > 0)) return PPE_ERR_ARG;
  return mlp_guard(m, [&]() -> ppe_status {
    loss_grad(m, n, x, t, m->grad.get<float>(m->n_params));
    m->adam_t += 1;
    const float c1 = 1.0f - std::pow(0.9f, (float)m->adam_t);
    const float c2 = 1.0f - std::pow(0.999f, (float)m->adam_t);
    hipLaunchKernelGGL(k_adam, dim3(grid_for(m->n_params)), dim3(kBlock), 0, m->stream, m->n_params,
                       m->params.as<float>(), m->grad.as<float>(), m->m.as<float>(),
                       m->v.as<float>(), lr, c1, c2);
    PPE_LAUNCH_CHECK();
    refresh_bf16(m);
    PPE_HIP(hipStreamSynchronize(m->stream));
    if (loss) *loss = *m->loss_h;
    return PPE_OK;
  });
}

ppe_status ppe_warm_start_features(ppe_solver* s, const double* dp_prev, const double* rhs,
                                   const double* face_coeff, const double* fl,
                                   const double* cell_volume, const float* mu, const float* sigma,
                                   float* features, double* dp_scale) {
  if (!s || !dp_prev || !rhs || !face_coeff || !fl || !cell_volume || !mu || !sigma || !features ||
      !dp_scale)
    return PPE_ERR_ARG;
  if (!s->assembled || s->shifted) return PPE_ERR_STATE;  // needs a pinned pressure system
  AllocScope scope(&s->allocator);
  try {
    const int na = s->n_active;
    double* part =
        na > 0 ? s->tmp_d[0].get<double>((size_t)3 * red_grid(na) + 3) : nullptr;
    return ppe::ws_features(s, dp_prev, rhs, face_coeff, fl, cell_volume, mu, sigma, features,
                            dp_scale, part);
  } catch (const Error& e) {
    s->err = e.what();
    return e.status;
  }
}

ppe_status ppe_warm_start_features_noalloc(ppe_solver* s, const double* dp_prev,
                                           const double* rhs, const double* face_coeff,
                                           const double* fl, const double* cell_volume,
                                           const float* mu, const float* sigma, float* features,
                                           double* dp_scale) {
  if (!s || !dp_prev || !rhs || !face_coeff || !fl || !cell_volume || !mu || !sigma || !features ||
      !dp_scale)
    return PPE_ERR_ARG;
  if (!s->assembled || s->shifted) return PPE_ERR_STATE;  // needs a pinned pressure system
  try {
    const int na = s->n_active;
    const size_t need = na > 0 ? (size_t)3 * red_grid(na) + 3 : 0;
    require(need <= (size_t)ppe::kWsScratch, PPE_ERR_ARG,
            "ppe_warm_start_features_noalloc: " + std::to_string(need) +
                " workspace doubles needed, the static workspace holds " +
                std::to_string(ppe::kWsScratch));
    double* part = na > 0 ? ppe::ws_scratch(s->device) : nullptr;
    return ppe::ws_features(s, dp_prev, rhs, face_coeff, fl, cell_volume, mu, sigma, features,
                            dp_scale, part);
  } catch (const Error& e) {
    s->err = e.what();
    return e.status;
  }
}

ppe_status ppe_warm_start_apply(ppe_solver* s, const double* p_prev, const float* y,
                                double dp_scale, double* x0) {
  if (!s || !p_prev || !x0 || (s->n_active > 0 && !y)) return PPE_ERR_ARG;
  if (!s->assembled || s->shifted) return PPE_ERR_STATE;  // needs a pinned pressure system
  try {
    hipLaunchKernelGGL(k_ws_apply, dim3(grid_for(s->n_cells)), dim3(kBlock), 0, s->stream,
                       s->n_cells, s->cid.as<int>(), s->comp_full.as<int>(), p_prev, y, dp_scale,
                       x0);
    PPE_LAUNCH_CHECK();
    PPE_HIP(hipStreamSynchronize(s->stream));
    return PPE_OK;
  } catch (const Error& e) {
    s->err = e.what();
    return e.status;
  }
}

ppe_status ppe_warm_start_targets(ppe_solver* s, const double* p_new, const double* p_prev,
                                  double dp_scale, float* targets) {
  if (!s || !p_new || !p_prev || (s->n_active > 0 && !targets)) return PPE_ERR_ARG;
  if (!s->assembled || s->shifted) return PPE_ERR_STATE;  // needs a pinned pressure system
  try {
    if (s->n_active) {
      hipLaunchKernelGGL(k_ws_targets, dim3(grid_for(s->n_active)), dim3(kBlock), 0, s->stream,
                         s->n_active, s->perm.as<int>(), s->comp_full.as<int>(), p_new, p_prev,
                         dp_scale, targets);
      PPE_LAUNCH_CHECK();
    }
    PPE_HIP(hipStreamSynchronize(s->stream));
    return PPE_OK;
  } catch (const Error& e) {
    s->err = e.what();
    return e.status;
  }
}

}  // extern "C"
