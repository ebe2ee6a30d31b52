// Learned control variate for the stochastic diagonal estimator (no counterpart in
// the paper): cheap local features, exact diagonals for training, and a small MLP
// 8 -> 64 -> 64 -> 1 (tanh) trained with hand-written forward / backward / Adam kernels.
//
// Features of node i (structural quantities scaled by the operator parameter s, so one
// network serves graphs of different spectral radius):
//   x0 = log1p(s d_i)              degree
//   x1 = log1p(s^2 d_i)            = s^2 diag(A^2)_i
//   x2 = log1p(s^3 2 t_i)          = s^3 diag(A^3)_i, t_i triangles through i
//   x3 = log1p(s^2 S2_i)           S2_i = sum_{j in N(i)} d_j  (2-walk count (A^2 1)_i)
//   x4 = log1p(s mean_j d_j)       neighbour-degree moments
//   x5 = log1p(s sqrt(mean_j d_j^2))
//   x6 = log1p(s max_j d_j)
//   x7 = 2 t_i / (d_i (d_i - 1))   local clustering (0 if d_i < 2)
// Parameter vector layout: W1 (64x8 row-major), b1 (64), W2 (64x64), b2 (64), W3 (1x64), b3.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <type_traits>
#include <vector>

#include "wl_internal.h"

namespace {

constexpr int NIN = 8, NH = 64;
constexpr int OW1 = 0, OB1 = OW1 + NH * NIN, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH, OB3 = OW3 + NH;
constexpr int NPARAM = OB3 + 1;  // 4801

// triangles: for every stored edge (i, j) count |N(i) cap N(j)| by binary-searching the
// shorter list in the longer one; integer atomics keep the sum exact.
__global__ void k_triangles(int64_t n, int64_t nnz, const int32_t* __restrict__ rowptr,
                            const int32_t* __restrict__ colidx, const int32_t* __restrict__ rowof,
                            unsigned long long* __restrict__ tri2) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * blockDim.x) {
    const int32_t i = rowof[e], j = colidx[e];
    int32_t a0 = rowptr[i], a1 = rowptr[i + 1], b0 = rowptr[j], b1 = rowptr[j + 1];
    if (a1 - a0 > b1 - b0) {
      int32_t t0 = a0, t1 = a1;
      a0 = b0;
      a1 = b1;
      b0 = t0;
      b1 = t1;
    }
    unsigned long long c = 0;
    for (int32_t p = a0; p < a1; ++p) {
      const int32_t v = colidx[p];
      int32_t lo = b0, hi = b1 - 1;
      while (lo <= hi) {
        const int32_t mid = (lo + hi) >> 1;
        const int32_t w = colidx[mid];
        if (w == v) {
          ++c;
          break;
        }
        if (w < v) lo = mid + 1; else hi = mid - 1;
      }
    }
    if (c) atomicAdd(&tri2[i], c);  // each triangle at i is seen from both of its edges at i
  }
}

__global__ void k_rowof(int64_t n, const int32_t* __restrict__ rowptr, int32_t* __restrict__ rowof) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    for (int32_t k = rowptr[i]; k < rowptr[i + 1]; ++k) rowof[k] = (int32_t)i;
}

__device__ __forceinline__ double wave_add(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sums over the neighbours of row i: s1 = sum d_j, s2 = sum d_j^2, mx = max d_j, by a group
// of G lanes (every lane gets the result) or by a workgroup (G = 256, result in all threads).
// The sums are integers below 2^53, so their order does not matter.  Rows of up to
// ROWSUM_LONG neighbours take 16 lanes (of up to 64 one lane, in sparse graphs), the others (first
// in the decreasing-degree list) a workgroup each: with one thread for every row a hub's chain of
// dependent loads set the time (R-MAT of 2^19 nodes, degree 30: features 6235 us and surrogate
// 5858 us; now 146 and 98 us).
constexpr int ROWSUM_LONG = 512;
struct RowSums {
  double s1, s2, mx;
};

template <int G>
__device__ __forceinline__ RowSums row_sums(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                            int32_t a, int32_t b, int sub) {
  RowSums r{0.0, 0.0, 0.0};
  for (int64_t k = a + sub; k < b; k += G) {
    const int32_t j = colidx[k];
    const double dj = rowptr[j + 1] - rowptr[j];
    r.s1 += dj;
    r.s2 += dj * dj;
    r.mx = fmax(r.mx, dj);
  }
#pragma unroll
  for (int off = (G < 64 ? G : 64) / 2; off > 0; off >>= 1) {
    r.s1 += __shfl_xor(r.s1, off, 64);
    r.s2 += __shfl_xor(r.s2, off, 64);
    r.mx = fmax(r.mx, __shfl_xor(r.mx, off, 64));
  }
  if constexpr (G == 256) {
    __shared__ double red[4][3];
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
      red[wave][0] = r.s1;
      red[wave][1] = r.s2;
      red[wave][2] = r.mx;
    }
    __syncthreads();
    r.s1 = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
    r.s2 = (red[0][1] + red[1][1]) + (red[2][1] + red[3][1]);
    r.mx = fmax(fmax(red[0][2], red[1][2]), fmax(red[2][2], red[3][2]));
  }
  return r;
}

// f(row, this thread's place in its group, lanes of the group, neighbour sums) for every row: the
// first n_long workgroups take one row of more than long_deg neighbours each, the others 256 / W
// rows at a time, W lanes each (a launch is limited to 2^32 threads, which 16 lanes per row would
// reach at 2^28 rows).
constexpr int64_t ROWSUM_WGS = 1 << 20;
template <int W, typename F>
__device__ __forceinline__ void for_rows(int64_t n, const int32_t* __restrict__ rowptr,
                                         const int32_t* __restrict__ colidx, const int32_t* __restrict__ long_rows,
                                         int n_long, int long_deg, F f) {
  if ((int)blockIdx.x < n_long) {
    const int64_t row = long_rows[blockIdx.x];
    f(row, (int)threadIdx.x, std::integral_constant<int, 256>(),
      row_sums<256>(rowptr, colidx, rowptr[row], rowptr[row + 1], threadIdx.x));
    return;
  }
  const int sub = threadIdx.x % W;
  const int64_t step = ((int64_t)gridDim.x - n_long) * (256 / W);
  for (int64_t row = ((int64_t)blockIdx.x - n_long) * (256 / W) + threadIdx.x / W; row < n; row += step) {
    const int32_t a = rowptr[row], b = rowptr[row + 1];  // (the lanes of a group stay together)
    if (b - a <= long_deg) f(row, sub, std::integral_constant<int, W>(), row_sums<W>(rowptr, colidx, a, b, sub));
  }
}

template <int W>
__global__ __launch_bounds__(256) void k_features(int64_t n, const int32_t* __restrict__ rowptr,
                                                  const int32_t* __restrict__ colidx,
                                                  const unsigned long long* __restrict__ tri2, double s,
                                                  float* __restrict__ feat, const int32_t* __restrict__ long_rows,
                                                  int n_long, int long_deg) {
  for_rows<W>(n, rowptr, colidx, long_rows, n_long, long_deg, [&](int64_t i, int sub, auto lanes, const RowSums& rs) {
    const double d = rowptr[i + 1] - rowptr[i];
    const double t = tri2 ? 0.5 * (double)tri2[i] : 0.0;
#pragma unroll
    for (int f = sub; f < NIN; f += decltype(lanes)::value) {
      double x;
      switch (f) {
        case 0: x = s * d; break;
        case 1: x = s * s * d; break;
        case 2: x = s * s * s * 2.0 * t; break;
        case 3: x = s * s * rs.s1; break;
        case 4: x = s * (d > 0 ? rs.s1 / d : 0.0); break;
        case 5: x = s * (d > 0 ? sqrt(rs.s2 / d) : 0.0); break;
        case 6: x = s * rs.mx; break;
        default: x = d >= 2 ? 2.0 * t / (d * (d - 1.0)) : 0.0; break;
      }
      feat[i * NIN + f] = (float)(f < 7 ? log1p(x) : x);
    }
  });
}

// out[j] = Y[nodes[j0 + j], j] for the unit-vector block e_{nodes[j0 .. j0+b)}
template <typename T>
__global__ void k_unit_block(int64_t n, int b, const int32_t* __restrict__ nodes, int64_t j0, int64_t count,
                             T* __restrict__ E) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * b; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / b;
    const int c = (int)(e - r * b);
    const int64_t jj = j0 + c;
    E[e] = (jj < count && nodes[jj] == r) ? T(1) : T(0);
  }
}

template <typename T>
__global__ void k_extract_diag(int b, const int32_t* __restrict__ nodes, int64_t j0, int64_t count,
                               const T* __restrict__ Y, T* __restrict__ out) {
  const int c = threadIdx.x;
  const int64_t jj = j0 + c;
  if (c < b && jj < count) out[jj] = Y[(int64_t)nodes[jj] * b + c];
}

// ------------------------------------------------------------------ MLP
// The network is three small contractions and runs on the FP32 matrix cores
// (v_mfma_f32_16x16x4f32: A 16x4, B 4x16; lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and holds D[4 (l / 16) + v][l % 16], v = 0..3).  A wave takes tiles of
// 16 samples with units as rows and samples as columns: with g = l / 16, c = l % 16 lane l
// holds units 16 t + 4 g + v (t, v = 0..3) of sample c, in every layer.  That is already the
// B operand of the next layer's step (t, v), which sums over the units {16 t + 4 g + v : g};
// the matching A operands W2[16 T + c][16 t + 4 g + v] (and W2^T for the backward pass) sit
// lane-ordered in LDS as 16-byte vectors, so a layer costs no data movement.  Bound: FP32
// matrix-core rate (27 kflop per sample forward and backward, 157 TFLOP/s) beside 128 tanhf
// per sample on the vector units.
// Measured on 204 800 samples, loss and gradient: one sample per thread with LDS sums
// 6620 us; this form 200 us.
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int MLP_TILE = 16;  // samples per tile
// No instruction moves across: without these marks the compiler interleaves all the tanhf and
// operand loads of a tile, and k_mlp_forward takes 136 + 56 registers instead of 74 + 24.
// k_mlp_grad is the same either way: 256 registers with 133 spilled to scratch.
#define MLP_STEP() __builtin_amdgcn_sched_barrier(0)

// Lane-ordered operands: sW2[(4 T + t) 64 + l] = W2[16 T + c][16 t + 4 g ..+3],
// sW2t[(4 T + t) 64 + l] = W2[16 t + 4 g ..+3][16 T + c] (optional); sb = b1, b2, W3, b3.
__device__ __forceinline__ void mlp_stage(const float* __restrict__ P, float4* sW2, float4* sW2t, float* sb) {
  for (int e = threadIdx.x; e < 16 * 64; e += 256) {
    const int l = e & 63, tt = e >> 6, T = tt >> 2, t = tt & 3, g = l >> 4, c = l & 15;
    const float* r = P + OW2 + (16 * T + c) * NH + 16 * t + 4 * g;
    sW2[e] = make_float4(r[0], r[1], r[2], r[3]);
    if (sW2t) {
      const float* q = P + OW2 + (16 * t + 4 * g) * NH + 16 * T + c;
      sW2t[e] = make_float4(q[0], q[NH], q[2 * NH], q[3 * NH]);
    }
  }
  for (int e = threadIdx.x; e < NH; e += 256) {
    sb[e] = P[OB1 + e];
    sb[NH + e] = P[OB2 + e];
    sb[2 * NH + e] = P[OW3 + e];
  }
  if (threadIdx.x == 0) sb[3 * NH] = P[OB3];
}

// W1 operands of lane l: W1[16 T + c][2 g], W1[16 T + c][2 g + 1] (step s sums over the
// features {2 g + s}).
__device__ __forceinline__ void mlp_w1(const float* __restrict__ P, int lane, float (&w1)[4][2]) {
#pragma unroll
  for (int T = 0; T < 4; ++T)
#pragma unroll
    for (int s = 0; s < 2; ++s) w1[T][s] = P[OW1 + (16 * T + (lane & 15)) * NIN + 2 * (lane >> 4) + s];
}

__device__ __forceinline__ v4f mlp_row4(const float* p) {
  const float4 b = *reinterpret_cast<const float4*>(p);
  return v4f{b.x, b.y, b.z, b.w};
}

// D_T = init_T + sum over units of (lane-ordered matrix) x act, for the four row tiles T.
__device__ __forceinline__ void mlp_contract(const float4* sM, int lane, const v4f (&act)[4], v4f (&d)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    float4 a[4];
#pragma unroll
    for (int T = 0; T < 4; ++T) a[T] = sM[(4 * T + t) * 64 + lane];
#pragma unroll
    for (int T = 0; T < 4; ++T) d[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[T].x, act[t][0], d[T], 0, 0, 0);
#pragma unroll
    for (int T = 0; T < 4; ++T) d[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[T].y, act[t][1], d[T], 0, 0, 0);
#pragma unroll
    for (int T = 0; T < 4; ++T) d[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[T].z, act[t][2], d[T], 0, 0, 0);
#pragma unroll
    for (int T = 0; T < 4; ++T) d[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[T].w, act[t][3], d[T], 0, 0, 0);
    MLP_STEP();
  }
}

// Forward pass of one tile: hidden layers h1, h2 and the output of sample l % 16 (in every
// lane).  x0, x1: features 2 g, 2 g + 1 of that sample.
__device__ __forceinline__ float mlp_tile(const float (&w1)[4][2], const float4* sW2, const float* sb, int lane,
                                          float x0, float x1, v4f (&h1)[4], v4f (&h2)[4]) {
  const int g = lane >> 4;
#pragma unroll
  for (int T = 0; T < 4; ++T) {
    v4f z = mlp_row4(sb + 16 * T + 4 * g);
    z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[T][0], x0, z, 0, 0, 0);
    z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[T][1], x1, z, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) h1[T][v] = tanhf(z[v]);
    h2[T] = mlp_row4(sb + NH + 16 * T + 4 * g);
    MLP_STEP();
  }
  mlp_contract(sW2, lane, h1, h2);
  float y = 0.f;
#pragma unroll
  for (int T = 0; T < 4; ++T) {
    const v4f w3 = mlp_row4(sb + 2 * NH + 16 * T + 4 * g);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      h2[T][v] = tanhf(h2[T][v]);
      y += w3[v] * h2[T][v];
    }
    MLP_STEP();
  }
  y += __shfl_xor(y, 16, 64);
  y += __shfl_xor(y, 32, 64);
  return y + sb[3 * NH];
}

__global__ __launch_bounds__(256) void k_mlp_forward(int64_t n, const float* __restrict__ P,
                                                     const float* __restrict__ X, float* __restrict__ out) {
  __shared__ float4 sW2[16 * 64];
  __shared__ __align__(16) float sb[3 * NH + 4];
  mlp_stage(P, sW2, nullptr, sb);
  __syncthreads();
  const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
  float w1[4][2];
  mlp_w1(P, lane, w1);
  const int64_t ntiles = (n + MLP_TILE - 1) / MLP_TILE;
  for (int64_t tile = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); tile < ntiles; tile += (int64_t)gridDim.x * 4) {
    const int64_t i = tile * MLP_TILE + c;
    const bool ok = i < n;
    const float x0 = ok ? X[i * NIN + 2 * g] : 0.f, x1 = ok ? X[i * NIN + 2 * g + 1] : 0.f;
    v4f h1[4], h2[4];
    const float y = mlp_tile(w1, sW2, sb, lane, x0, x1, h1, h2);
    if (ok && g == 0) out[i] = y;
  }
}

// Forward and backward.  dh1 = W2^T dz2 has the layout of the forward layers.  The weight
// gradients sum over samples (dW2[m][k] = sum_s dz2[m][s] h1[k][s]), so both factors are
// turned through the wave's own LDS slice: lane l reads samples 4 g .. 4 g + 3 of unit
// 16 T + c (16 bytes) and step v sums over the samples {4 g + v}.  dW1 takes the features as
// B operand, with a column of ones behind them that gives db1.  A wave sums at most
// MLP_MAXT tiles (128 samples) in FP32; the four waves and the rounds are then added in FP64
// and every workgroup writes one partial (fixed order, the sum of squared residuals last).
constexpr int MLP_MAXT = 8;
constexpr int MLP_TS = 20;       // floats per unit row of a turned tile (16 samples, padded)
constexpr int MLP_WGS = 512;     // two workgroups on each of the 256 CUs
__global__ __launch_bounds__(256, 2) void k_mlp_grad(int64_t n, const float* __restrict__ P,
                                                     const float* __restrict__ X, const float* __restrict__ tgt,
                                                     double inv_n, int tiles_per_wave,
                                                     double* __restrict__ partials) {
  constexpr size_t W_BYTES = 2 * 16 * 64 * sizeof(float4);                 // W2 and its transpose
  constexpr size_t T_BYTES = (size_t)4 * 2 * NH * MLP_TS * sizeof(float);  // two turned tiles per wave
  static_assert(W_BYTES + T_BYTES >= (NPARAM + 1) * sizeof(double), "the reduction reuses the space");
  __shared__ __align__(16) unsigned char smem[W_BYTES + T_BYTES];
  __shared__ __align__(16) float sb[3 * NH + 4];
  float4* sW2 = reinterpret_cast<float4*>(smem);
  float4* sW2t = sW2 + 16 * 64;
  double* red = reinterpret_cast<double*>(smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, c = lane & 15;
  float* tA = reinterpret_cast<float*>(smem + W_BYTES) + (size_t)wave * 2 * NH * MLP_TS;
  float* tB = tA + NH * MLP_TS;
  float w1[4][2];
  mlp_w1(P, lane, w1);
  const int64_t ntiles = (n + MLP_TILE - 1) / MLP_TILE;
  const int64_t per = (int64_t)4 * tiles_per_wave;
  double* out = partials + (int64_t)blockIdx.x * (NPARAM + 1);
  const float dys = (float)(2.0 * inv_n);
  for (int64_t base = (int64_t)blockIdx.x * per; base < ntiles; base += (int64_t)gridDim.x * per) {
    mlp_stage(P, sW2, sW2t, sb);
    __syncthreads();
    v4f gW2[4][4], gW1[4], gb2[4], gW3[4];
#pragma unroll
    for (int T = 0; T < 4; ++T) {
      gW1[T] = gb2[T] = gW3[T] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int J = 0; J < 4; ++J) gW2[T][J] = v4f{0.f, 0.f, 0.f, 0.f};
    }
    double gb3 = 0.0, loss = 0.0;
    for (int q = 0; q < tiles_per_wave; ++q) {
      const int64_t tile = base + (int64_t)q * 4 + wave;
      if (tile >= ntiles) break;  // whole wave
      const int64_t i = tile * MLP_TILE + c;
      const bool ok = i < n;
      const float x0 = ok ? X[i * NIN + 2 * g] : 0.f, x1 = ok ? X[i * NIN + 2 * g + 1] : 0.f;
      float xs[4];  // B operand of dW1: feature c (column 8: ones) of sample 4 g + v
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t s = tile * MLP_TILE + 4 * g + v;
        xs[v] = (s < n && c < NIN) ? X[s * NIN + c] : (c == NIN ? 1.f : 0.f);
      }
      v4f h1[4], h2[4];
      const float y = mlp_tile(w1, sW2, sb, lane, x0, x1, h1, h2);
      const float r = ok ? y - tgt[i] : 0.f;
      const float dy = dys * r;
      if (g == 0) {
        loss += (double)r * (double)r;
        gb3 += (double)dy;
      }
      // output layer and dz2 = dy W3 (1 - h2^2), in place
#pragma unroll
      for (int T = 0; T < 4; ++T) {
        const v4f w3 = mlp_row4(sb + 2 * NH + 16 * T + 4 * g);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float h = h2[T][v];
          gW3[T][v] += dy * h;
          const float dz = dy * w3[v] * (1.f - h * h);
          gb2[T][v] += dz;
          h2[T][v] = dz;
          tA[(16 * T + 4 * g + v) * MLP_TS + c] = dz;
          tB[(16 * T + 4 * g + v) * MLP_TS + c] = h1[T][v];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      {
        v4f b[4];
#pragma unroll
        for (int J = 0; J < 4; ++J) b[J] = mlp_row4(tB + (16 * J + c) * MLP_TS + 4 * g);
#pragma unroll
        for (int T = 0; T < 4; ++T) {
          const v4f a = mlp_row4(tA + (16 * T + c) * MLP_TS + 4 * g);
#pragma unroll
          for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int J = 0; J < 4; ++J)
              gW2[T][J] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v], b[J][v], gW2[T][J], 0, 0, 0);
          MLP_STEP();
        }
      }
      v4f d[4];
#pragma unroll
      for (int T = 0; T < 4; ++T) d[T] = v4f{0.f, 0.f, 0.f, 0.f};
      mlp_contract(sW2t, lane, h2, d);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int T = 0; T < 4; ++T)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          tA[(16 * T + 4 * g + v) * MLP_TS + c] = d[T][v] * (1.f - h1[T][v] * h1[T][v]);  // dz1
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int T = 0; T < 4; ++T) {
        const v4f a = mlp_row4(tA + (16 * T + c) * MLP_TS + 4 * g);
#pragma unroll
        for (int v = 0; v < 4; ++v) gW1[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v], xs[v], gW1[T], 0, 0, 0);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    gb3 = wave_add(gb3);
    loss = wave_add(loss);
    __syncthreads();
#pragma unroll 1
    for (int w = 0; w < 4; ++w) {
      if (wave == w) {
        auto put = [&](int at, double v) { red[at] = (w == 0 ? 0.0 : red[at]) + v; };
#pragma unroll
        for (int T = 0; T < 4; ++T)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int unit = 16 * T + 4 * g + v;
#pragma unroll
            for (int J = 0; J < 4; ++J) put(OW2 + unit * NH + 16 * J + c, (double)gW2[T][J][v]);
            if (c < NIN) put(OW1 + unit * NIN + c, (double)gW1[T][v]);
            if (c == NIN) put(OB1 + unit, (double)gW1[T][v]);
            double s2 = (double)gb2[T][v], s3 = (double)gW3[T][v];
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
              s2 += __shfl_xor(s2, off, 64);
              s3 += __shfl_xor(s3, off, 64);
            }
            if (c == 0) {
              put(OB2 + unit, s2);
              put(OW3 + unit, s3);
            }
            MLP_STEP();
          }
        if (lane == 0) {
          put(OB3, gb3);
          put(NPARAM, loss);
        }
      }
      __syncthreads();
    }
    const bool first = base == (int64_t)blockIdx.x * per;
    for (int p = threadIdx.x; p <= NPARAM; p += 256) out[p] = (first ? 0.0 : out[p]) + red[p];
    __syncthreads();
  }
}

// g[p] = sum of the partials of p, in a fixed order: 16 parameters per workgroup, 16 phases
// of partials each (one thread per parameter walking all of them took 170 us for 512).
__global__ __launch_bounds__(256) void k_mlp_grad_finalize(int nparts, const double* __restrict__ partials,
                                                           double* __restrict__ g) {
  __shared__ double s[256];
  const int el = threadIdx.x & 15, ph = threadIdx.x >> 4;
  const int p = blockIdx.x * 16 + el;
  double v = 0.0;
  if (p <= NPARAM)
    for (int q = ph; q < nparts; q += 16) v += partials[(int64_t)q * (NPARAM + 1) + p];
  s[threadIdx.x] = v;
  __syncthreads();
  for (int h = 8; h > 0; h >>= 1) {
    if (ph < h) s[threadIdx.x] += s[threadIdx.x + 16 * h];
    __syncthreads();
  }
  if (ph == 0 && p <= NPARAM) g[p] = s[el];
}

__global__ void k_adam(float* __restrict__ P, const double* __restrict__ g, double* __restrict__ m,
                       double* __restrict__ v, double lr, double b1, double b2, double eps, double c1, double c2) {
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < NPARAM; p += gridDim.x * blockDim.x) {
    const double gp = g[p];
    const double mp = b1 * m[p] + (1.0 - b1) * gp;
    const double vp = b2 * v[p] + (1.0 - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    P[p] = (float)((double)P[p] - lr * (mp / c1) / (sqrt(vp / c2) + eps));
  }
}

}  // namespace

struct wl_mlp {
  wl_ctx* ctx = nullptr;
  DevBuf params, m, v, grad, partials;
  int64_t step = 0;
};

namespace {
wl_status mlp_grad(wl_mlp* net, const float* feat, const float* tgt, int64_t n, double* loss) {
  wl_ctx* ctx = net->ctx;
  // one tile per wave while that fills the chip's MLP_WGS workgroups, then up to MLP_MAXT
  const int64_t ntiles = (n + MLP_TILE - 1) / MLP_TILE;
  const int tpw = (int)std::min<int64_t>(MLP_MAXT, (ntiles + 4 * MLP_WGS - 1) / (4 * MLP_WGS));
  const int grid = (int)std::min<int64_t>(MLP_WGS, (ntiles + 4 * tpw - 1) / (4 * tpw));
  WL_TRY(net->partials.ensure((size_t)grid * (NPARAM + 1) * sizeof(double)));
  WL_TRY(net->grad.ensure((size_t)(NPARAM + 1) * sizeof(double)));
  hipLaunchKernelGGL(k_mlp_grad, dim3(grid), dim3(256), 0, ctx->stream, n, net->params.as<float>(), feat, tgt,
                     1.0 / (double)n, tpw, net->partials.as<double>());
  WL_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_mlp_grad_finalize, dim3((NPARAM + 16) / 16), dim3(256), 0, ctx->stream, grid,
                     net->partials.as<double>(), net->grad.as<double>());
  WL_HIP(hipGetLastError());
  if (loss) {
    double l = 0.0;
    WL_HIP(hipMemcpyAsync(&l, net->grad.as<double>() + NPARAM, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
    WL_HIP(hipStreamSynchronize(ctx->stream));
    *loss = l / (double)n;
  }
  return WL_OK;
}
// Degree-3 series diagonal and the scale of the remainder at row r (the exact low-order
// part of diag phi and the size of what is left, which the network learns):
//   base  = 1 + c2m d + c3 tri2           (diag q_2 = (1 - mu) d, diag q_3 = (A^3)_rr)
//   scale = c4 max(1, d^2 + S2),  S2 = sum_{j in N(r)} d_j   (bounds the 4-walk count)
__device__ inline void surrogate_terms(double d, double s2, double tri2, double c2m, double c3, double c4,
                                       double* base, double* scale) {
  *base = 1.0 + c2m * d + c3 * tri2;
  *scale = c4 * fmax(1.0, d * d + s2);
}

template <typename T, int W>
__global__ __launch_bounds__(256) void k_surrogate_diag(int64_t n, const int32_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ colidx,
                                                        const unsigned long long* __restrict__ tri2, double c2m,
                                                        double c3, double c4, T* __restrict__ base,
                                                        T* __restrict__ scale,
                                                        const int32_t* __restrict__ long_rows, int n_long,
                                                        int long_deg) {
  for_rows<W>(n, rowptr, colidx, long_rows, n_long, long_deg, [&](int64_t r, int sub, auto, const RowSums& rs) {
    if (sub != 0) return;
    double bs, sc;
    surrogate_terms(rowptr[r + 1] - rowptr[r], rs.s1, (double)tri2[r], c2m, c3, c4, &bs, &sc);
    if (base) base[r] = (T)bs;
    if (scale) scale[r] = (T)sc;
  });
}

// out[j] = (d[j] - base(nodes[j])) / scale(nodes[j]) in place (d: diag phi at the nodes)
// (one wave per node: the nodes are a caller's sample, hubs among them)
template <typename T>
__global__ __launch_bounds__(256) void k_surrogate_target(int64_t count, const int32_t* __restrict__ nodes,
                                                          const int32_t* __restrict__ rowptr,
                                                          const int32_t* __restrict__ colidx,
                                                          const unsigned long long* __restrict__ tri2, double c2m,
                                                          double c3, double c4, T* __restrict__ d) {
  const int lane = threadIdx.x & 63;
  for (int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); j < count; j += (int64_t)gridDim.x * 4) {
    const int64_t r = nodes[j];
    const int32_t a = rowptr[r], b = rowptr[r + 1];
    const RowSums rs = row_sums<64>(rowptr, colidx, a, b, lane);
    if (lane != 0) continue;
    double bs, sc;
    surrogate_terms(b - a, rs.s1, (double)tri2[r], c2m, c3, c4, &bs, &sc);
    d[j] = (T)(((double)d[j] - bs) / sc);
  }
}

__global__ void k_affine(int64_t n, const float* __restrict__ base, const float* __restrict__ scale,
                         float* __restrict__ y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (base ? base[i] : 0.f) + (scale ? scale[i] : 1.f) * y[i];
}

// Launch of the neighbour-sum kernels: lanes a short row, rows of a workgroup each, workgroups.
// One lane a row where rows are short (below a mean degree of one_lane_deg) and many enough to
// fill the chip; us with 1 / 16 lanes: features, lattice of 1M nodes 57 / 153, 500k nodes of degree 12
// 83 / 90, of 16 107 / 94; surrogate, degree 6 23 / 31, 8 31 / 33, 12 52 / 40; features of 3000 nodes
// of degree 8 22 / 18.
constexpr double FEATURES_ONE_LANE = 14.0, SURROGATE_ONE_LANE = 8.0;
constexpr int64_t ROWSUM_SMALL = 1 << 15;
struct RowSumShape {
  int lanes, long_deg, n_long;
  dim3 grid;
};
RowSumShape rowsum_shape(const wl_graph* g, double one_lane_deg) {
  RowSumShape s;
  s.lanes = g->n >= ROWSUM_SMALL && g->mean_deg < one_lane_deg ? 1 : 16;
  s.long_deg = s.lanes == 1 ? g->long_min_thr : ROWSUM_LONG;
  const auto& dd = g->h_long_deg;  // decreasing
  s.n_long = (int)(std::lower_bound(dd.begin(), dd.end(), s.long_deg, [](int32_t d, int t) { return d > t; }) -
                   dd.begin());
  const int rows = 256 / s.lanes;
  s.grid = dim3((unsigned)(s.n_long + std::min((g->n + rows - 1) / rows, ROWSUM_WGS)));
  return s;
}

// c_2 (1 - mu), c_3, c_4 of the operator's weights
void surrogate_coeffs(const wl_op* op, double* c2m, double* c3, double* c4) {
  const double p = op->d.param;
  const bool ex = op->d.func == WL_F_EXP;
  if (op->d.func == WL_F_LINEAR) {  // c_k = 0 for k >= 2
    *c2m = *c3 = *c4 = 0.0;
    return;
  }
  *c2m = (ex ? p * p / 2.0 : p * p) * (1.0 - op->d.mu);
  *c3 = ex ? p * p * p / 6.0 : p * p * p;
  *c4 = ex ? p * p * p * p / 24.0 : p * p * p * p;
}

}  // namespace

wl_status graph_tri2(wl_graph* g, const unsigned long long** out) {
  hipStream_t st = g->ctx->stream;
  if (!g->tri2_valid) {
    WL_TRY(g->tri2.ensure((size_t)std::max<int64_t>(g->n, 1) * 8));
    if (g->n > 0) WL_HIP(hipMemsetAsync(g->tri2.p, 0, (size_t)g->n * 8, st));
    if (g->nnz > 0) {
      DevBuf rowof;
      WL_TRY(rowof.ensure((size_t)g->nnz * 4));
      const int gb = (int)std::min<int64_t>(8192, (g->n + 255) / 256);
      hipLaunchKernelGGL(k_rowof, dim3(gb), dim3(256), 0, st, g->n, g->rowptr, rowof.as<int32_t>());
      WL_HIP(hipGetLastError());
      const int ge = (int)std::min<int64_t>(65536, (g->nnz + 255) / 256);
      hipLaunchKernelGGL(k_triangles, dim3(ge), dim3(256), 0, st, g->n, g->nnz, g->rowptr, g->colidx,
                         rowof.as<int32_t>(), g->tri2.as<unsigned long long>());
      WL_HIP(hipGetLastError());
      // rowof is released (after a device synchronisation) when it leaves scope
    }
    g->tri2_valid = true;
  }
  *out = g->tri2.as<unsigned long long>();
  return WL_OK;
}

extern "C" {

wl_status wl_features(wl_graph* g, double scale, void* d_feat) {
  WL_CHECK(g, WL_EINVAL, "wl_features: graph is null");
  WL_CHECK(std::isfinite(scale) && scale > 0, WL_EINVAL, "wl_features: scale must be > 0");
  WL_CHECK(g->n == 0 || d_feat, WL_EINVAL, "wl_features: output is null");
  if (g->n == 0) return WL_OK;
  (void)hipSetDevice(g->ctx->device);
  hipStream_t st = g->ctx->stream;
  const unsigned long long* tri = nullptr;
  WL_TRY(graph_tri2(g, &tri));
  const RowSumShape sh = rowsum_shape(g, FEATURES_ONE_LANE);
  hipLaunchKernelGGL((sh.lanes == 1 ? k_features<1> : k_features<16>), sh.grid, dim3(256), 0, st, g->n, g->rowptr,
                     g->colidx, tri, scale, (float*)d_feat, g->long_rows.as<int32_t>(), sh.n_long, sh.long_deg);
  WL_HIP(hipGetLastError());
  WL_HIP(hipStreamSynchronize(st));
  return WL_OK;
}

wl_status wl_diag_exact(wl_op* op, const int32_t* d_nodes, int64_t count, int32_t width, void* d_out) {
  WL_CHECK(op, WL_EINVAL, "wl_diag_exact: op is null");
  WL_CHECK(count >= 0 && (count == 0 || (d_nodes && d_out)), WL_EINVAL, "wl_diag_exact: bad node list");
  WL_CHECK(width >= 1 && width <= 64, WL_EINVAL, "wl_diag_exact: width must lie in [1, 64]");
  if (count == 0) return WL_OK;
  wl_graph* g = op->g;
  (void)hipSetDevice(g->ctx->device);
  const int64_t n = g->n;
  const size_t es = op->d.prec == WL_FP32 ? 4 : 8;
  DevBuf E, Y;
  WL_TRY(E.ensure((size_t)n * width * es));
  WL_TRY(Y.ensure((size_t)n * width * es));
  hipStream_t st = g->ctx->stream;
  const int gb = (int)std::min<int64_t>(8192, (n * width + 255) / 256);
  for (int64_t j0 = 0; j0 < count; j0 += width) {
    if (op->d.prec == WL_FP32) {
      hipLaunchKernelGGL((k_unit_block<float>), dim3(gb), dim3(256), 0, st, n, width, d_nodes, j0, count,
                         E.as<float>());
      WL_HIP(hipGetLastError());
      WL_TRY(wl_apply_phi(op, E.p, Y.p, width));
      hipLaunchKernelGGL((k_extract_diag<float>), dim3(1), dim3(64), 0, st, width, d_nodes, j0, count,
                         Y.as<float>(), (float*)d_out);
    } else {
      hipLaunchKernelGGL((k_unit_block<double>), dim3(gb), dim3(256), 0, st, n, width, d_nodes, j0, count,
                         E.as<double>());
      WL_HIP(hipGetLastError());
      WL_TRY(wl_apply_phi(op, E.p, Y.p, width));
      hipLaunchKernelGGL((k_extract_diag<double>), dim3(1), dim3(64), 0, st, width, d_nodes, j0, count,
                         Y.as<double>(), (double*)d_out);
    }
    WL_HIP(hipGetLastError());
  }
  WL_HIP(hipStreamSynchronize(st));
  return WL_OK;
}

wl_status wl_surrogate_diag(wl_op* op, void* d_base, void* d_scale) {
  WL_CHECK(op, WL_EINVAL, "wl_surrogate_diag: op is null");
  wl_graph* g = op->g;
  WL_CHECK(g->n == 0 || d_base || d_scale, WL_EINVAL, "wl_surrogate_diag: no output");
  if (g->n == 0) return WL_OK;
  (void)hipSetDevice(g->ctx->device);
  const unsigned long long* tri = nullptr;
  WL_TRY(graph_tri2(g, &tri));
  double c2m, c3, c4;
  surrogate_coeffs(op, &c2m, &c3, &c4);
  const RowSumShape sh = rowsum_shape(g, SURROGATE_ONE_LANE);
  if (op->d.prec == WL_FP32)
    hipLaunchKernelGGL((sh.lanes == 1 ? k_surrogate_diag<float, 1> : k_surrogate_diag<float, 16>), sh.grid, dim3(256),
                       0, g->ctx->stream, g->n, g->rowptr, g->colidx, tri, c2m, c3, c4, (float*)d_base,
                       (float*)d_scale, g->long_rows.as<int32_t>(), sh.n_long, sh.long_deg);
  else
    hipLaunchKernelGGL((sh.lanes == 1 ? k_surrogate_diag<double, 1> : k_surrogate_diag<double, 16>), sh.grid,
                       dim3(256), 0, g->ctx->stream, g->n, g->rowptr, g->colidx, tri, c2m, c3, c4, (double*)d_base,
                       (double*)d_scale, g->long_rows.as<int32_t>(), sh.n_long, sh.long_deg);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status wl_surrogate_target(wl_op* op, const int32_t* d_nodes, int64_t count, int32_t width, void* d_out) {
  WL_TRY(wl_diag_exact(op, d_nodes, count, width, d_out));
  if (count == 0) return WL_OK;
  wl_graph* g = op->g;
  const unsigned long long* tri = nullptr;
  WL_TRY(graph_tri2(g, &tri));
  double c2m, c3, c4;
  surrogate_coeffs(op, &c2m, &c3, &c4);
  const int gb = (int)std::min<int64_t>(8192, (count + 255) / 256);
  if (op->d.prec == WL_FP32)
    hipLaunchKernelGGL(k_surrogate_target<float>, dim3(gb), dim3(256), 0, g->ctx->stream, count, d_nodes,
                       g->rowptr, g->colidx, tri, c2m, c3, c4, (float*)d_out);
  else
    hipLaunchKernelGGL(k_surrogate_target<double>, dim3(gb), dim3(256), 0, g->ctx->stream, count, d_nodes,
                       g->rowptr, g->colidx, tri, c2m, c3, c4, (double*)d_out);
  WL_HIP(hipGetLastError());
  WL_HIP(hipStreamSynchronize(g->ctx->stream));
  return WL_OK;
}

wl_status wl_mlp_predict(wl_mlp* net, const void* d_feat, int64_t n, const void* d_base, const void* d_scale,
                         void* d_out) {
  WL_TRY(wl_mlp_forward(net, d_feat, n, d_out));
  if (n == 0) return WL_OK;
  const int grid = (int)std::min<int64_t>(4096, (n + 255) / 256);
  hipLaunchKernelGGL(k_affine, dim3(grid), dim3(256), 0, net->ctx->stream, n, (const float*)d_base,
                     (const float*)d_scale, (float*)d_out);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status wl_mlp_create(wl_ctx* ctx, const float* h_params, wl_mlp** out) {
  WL_CHECK(ctx && out, WL_EINVAL, "wl_mlp_create: null argument");
  (void)hipSetDevice(ctx->device);
  auto* net = new wl_mlp;
  net->ctx = ctx;
  std::vector<float> init(NPARAM, 0.f);
  if (h_params) init.assign(h_params, h_params + NPARAM);
  std::vector<double> zeros(NPARAM, 0.0);
  wl_status s = net->params.ensure(NPARAM * sizeof(float));
  if (s == WL_OK) s = net->m.ensure(NPARAM * sizeof(double));
  if (s == WL_OK) s = net->v.ensure(NPARAM * sizeof(double));
  if (s != WL_OK) {
    delete net;
    return s;
  }
  if (hipMemcpy(net->params.p, init.data(), NPARAM * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(net->m.p, zeros.data(), NPARAM * sizeof(double), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(net->v.p, zeros.data(), NPARAM * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
    delete net;
    wl_set_error("wl_mlp_create: upload failed");
    return WL_EDEVICE;
  }
  ++ctx->refs;
  *out = net;
  return WL_OK;
}

wl_status wl_mlp_destroy(wl_mlp* net) {
  if (!net) return WL_OK;
  wl_ctx* ctx = net->ctx;
  (void)hipSetDevice(ctx->device);
  (void)hipStreamSynchronize(ctx->stream);
  delete net;
  ctx_release(ctx);
  return WL_OK;
}

int32_t wl_mlp_num_params(void) { return NPARAM; }

wl_status wl_mlp_get_params(const wl_mlp* net, float* h_params) {
  WL_CHECK(net && h_params, WL_EINVAL, "wl_mlp_get_params: null argument");
  (void)hipSetDevice(net->ctx->device);
  WL_HIP(hipStreamSynchronize(net->ctx->stream));
  WL_HIP(hipMemcpy(h_params, net->params.p, NPARAM * sizeof(float), hipMemcpyDeviceToHost));
  return WL_OK;
}

wl_status wl_mlp_forward(wl_mlp* net, const void* d_feat, int64_t n, void* d_out) {
  WL_CHECK(net, WL_EINVAL, "wl_mlp_forward: net is null");
  WL_CHECK(n >= 0 && (n == 0 || (d_feat && d_out)), WL_EINVAL, "wl_mlp_forward: bad arguments");
  if (n == 0) return WL_OK;
  (void)hipSetDevice(net->ctx->device);
  const int grid = (int)std::min<int64_t>(1024, (n + 4 * MLP_TILE - 1) / (4 * MLP_TILE));
  hipLaunchKernelGGL(k_mlp_forward, dim3(grid), dim3(256), 0, net->ctx->stream, n, net->params.as<float>(),
                     (const float*)d_feat, (float*)d_out);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status wl_mlp_loss_grad(wl_mlp* net, const void* d_feat, const void* d_target, int64_t n, double* loss,
                           double* h_grad) {
  WL_CHECK(net && d_feat && d_target && n >= 1, WL_EINVAL, "wl_mlp_loss_grad: bad arguments");
  (void)hipSetDevice(net->ctx->device);
  WL_TRY(mlp_grad(net, (const float*)d_feat, (const float*)d_target, n, loss));
  if (h_grad) {
    WL_HIP(hipMemcpy(h_grad, net->grad.p, NPARAM * sizeof(double), hipMemcpyDeviceToHost));
  }
  return WL_OK;
}

wl_status wl_mlp_train_step(wl_mlp* net, const void* d_feat, const void* d_target, int64_t n, double lr,
                            double* loss) {
  WL_CHECK(net && d_feat && d_target && n >= 1, WL_EINVAL, "wl_mlp_train_step: bad arguments");
  WL_CHECK(std::isfinite(lr) && lr > 0, WL_EINVAL, "wl_mlp_train_step: lr must be > 0");
  (void)hipSetDevice(net->ctx->device);
  WL_TRY(mlp_grad(net, (const float*)d_feat, (const float*)d_target, n, loss));
  net->step += 1;
  const double b1 = 0.9, b2 = 0.999;
  const double c1 = 1.0 - std::pow(b1, (double)net->step), c2 = 1.0 - std::pow(b2, (double)net->step);
  hipLaunchKernelGGL(k_adam, dim3((NPARAM + 255) / 256), dim3(256), 0, net->ctx->stream, net->params.as<float>(),
                     net->grad.as<double>(), net->m.as<double>(), net->v.as<double>(), lr, b1, b2, 1e-8, c1, c2);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status wl_mlp_save(const wl_mlp* net, const char* path) {
  WL_CHECK(net && path, WL_EINVAL, "wl_mlp_save: null argument");
  std::vector<float> p(NPARAM);
  WL_TRY(wl_mlp_get_params(net, p.data()));
  FILE* f = std::fopen(path, "wb");
  WL_CHECK(f, WL_EINVAL, "wl_mlp_save: cannot open %s", path);
  const char magic[8] = {'W', 'L', 'M', 'L', 'P', '0', '0', '1'};
  const int32_t np = NPARAM;
  bool ok = std::fwrite(magic, 1, 8, f) == 8 && std::fwrite(&np, 4, 1, f) == 1 &&
            std::fwrite(p.data(), 4, NPARAM, f) == (size_t)NPARAM;
  std::fclose(f);
  WL_CHECK(ok, WL_EINVAL, "wl_mlp_save: write failed");
  return WL_OK;
}

wl_status wl_mlp_load(wl_ctx* ctx, const char* path, wl_mlp** out) {
  WL_CHECK(ctx && path && out, WL_EINVAL, "wl_mlp_load: null argument");
  FILE* f = std::fopen(path, "rb");
  WL_CHECK(f, WL_EINVAL, "wl_mlp_load: cannot open %s", path);
  char magic[8];
  int32_t np = 0;
  std::vector<float> p(NPARAM);
  bool ok = std::fread(magic, 1, 8, f) == 8 && std::fread(&np, 4, 1, f) == 1 && np == NPARAM &&
            std::fread(p.data(), 4, NPARAM, f) == (size_t)NPARAM;
  std::fclose(f);
  WL_CHECK(ok && std::string(magic, 8) == "WLMLP001", WL_EINVAL, "wl_mlp_load: %s is not a saved network", path);
  return wl_mlp_create(ctx, p.data(), out);
}

}  // extern "C"
