// Tall-skinny block kernels for the Krylov drivers and estimators (gfx950).
//
//  * gram:    X^T Y for n x B blocks (B <= 64), double accumulation, on the FP64 matrix
//             cores in 16-row chunks from five columns on (FP32 blocks of 16, 32 or 64
//             columns staged through LDS); two to four columns stage 32-row tiles in LDS
//             with every thread owning an entry; single columns are 16-byte dot products.
//             Per-workgroup partials are reduced by a second kernel in a fixed
//             order, so results are bitwise reproducible.
//  * update:  Out = w (.) Yin + beta * sum_k X_k C_k, from five columns on as a
//             tall-skinny product on the matrix cores of the block's precision with the
//             FP64 Gram of the result fused (block CholQR needs W^T W right after W is
//             formed); two to four columns hold rows in registers with C_k (B x B) broadcast
//             from LDS; single columns are 16-byte vector updates.
//  * chol:    Cholesky with deflation of a B x B Gram and the inverse of its
//             factor, one workgroup per matrix (batched over graphs or operator groups).
//  * probes:  Philox4x32-10 (Salmon et al., SC'11) Rademacher / Gaussian blocks.
//  * small helpers: fills, scaled row sums, degree vector, CSR validation.
#include <utility>

#include "wl_internal.h"

namespace {

constexpr int GRAM_TR = 32;  // rows per LDS tile in the Gram kernel

// Blocks of up to four columns: a thread per entry (i, j) and row phase.
template <int B>
__global__ __launch_bounds__(256) void k_gram_partial(int64_t n, const float* __restrict__ Xf,
                                                      const double* __restrict__ Xd, int ldx, int64_t sX,
                                                      const float* __restrict__ Yf, const double* __restrict__ Yd,
                                                      int ldy, int bx, int by, double* __restrict__ partials) {
  constexpr int E = B * B;
  static_assert(E < 256, "one entry per thread");
  constexpr int P = 256 / E;  // row phases
  __shared__ double sx[GRAM_TR * B];
  __shared__ double sy[GRAM_TR * B];
  __shared__ double sred[256];
  const int tid = threadIdx.x;
  const int64_t xoff = (int64_t)blockIdx.y * sX;
  const int i = (tid % E) / B, j = (tid % E) % B, p = tid / E;
  double acc = 0.0;
  const int64_t ntiles = (n + GRAM_TR - 1) / GRAM_TR;
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t row0 = t * GRAM_TR;
    for (int idx = tid; idx < GRAM_TR * B; idx += 256) {
      const int r = idx / B, c = idx % B;
      const int64_t row = row0 + r;
      double xv = 0.0, yv = 0.0;
      if (row < n) {
        if (c < bx) xv = Xf ? (double)Xf[xoff + row * ldx + c] : Xd[xoff + row * ldx + c];
        if (c < by) yv = Yf ? (double)Yf[row * ldy + c] : Yd[row * ldy + c];
      }
      sx[idx] = xv;
      sy[idx] = yv;
    }
    __syncthreads();
    if (p < P)
      for (int r = p; r < GRAM_TR; r += P) acc += sx[r * B + i] * sy[r * B + j];
    __syncthreads();
  }
  sred[tid] = p < P ? acc : 0.0;
  __syncthreads();
  if (tid < E) {
    double s = 0.0;
    for (int q = 0; q < P; ++q) s += sred[tid + q * E];
    partials[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * E + tid] = s;
  }
}

// out[(k*bx + i)*by + j] = sum_q partials[k][q][i*B + j].  Fixed-order reduction:
// a block owns EB = min(E, 16) entries; thread (entry, phase p) sums q = p, p + P, ...
// (P = 256 / EB), then the P phase sums are combined by a tree in LDS.
__global__ __launch_bounds__(256) void k_gram_finalize(const double* __restrict__ partials, int nparts, int B,
                                                       int bx, int by, double* __restrict__ out,
                                                       const double* __restrict__ skip) {
  if (skip && *skip != 0.0) return;  // the caller does not need this Gram
  __shared__ double s[256];
  const int E = B * B;
  const int EB = E < 16 ? E : 16;
  const int P = 256 / EB;
  const int k = blockIdx.y;
  const int t = threadIdx.x;
  const int el = t % EB, p = t / EB;
  const int e = blockIdx.x * EB + el;
  double v = 0.0;
  if (e < E) {
    // eight independent sums so that eight loads are in flight per thread
    const double* src = partials + (int64_t)k * nparts * E + e;
    double u[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int q = p;
    for (; q + 7 * P < nparts; q += 8 * P) {
#pragma unroll
      for (int i = 0; i < 8; ++i) u[i] += src[(int64_t)(q + i * P) * E];
    }
    for (; q < nparts; q += P) u[0] += src[(int64_t)q * E];
    v = ((u[0] + u[1]) + (u[2] + u[3])) + ((u[4] + u[5]) + (u[6] + u[7]));
  }
  s[t] = v;
  __syncthreads();
  for (int h = P / 2; h > 0; h >>= 1) {
    if (p < h) s[t] += s[t + h * EB];
    __syncthreads();
  }
  if (p == 0 && e < E) {
    const int i = e / B, j = e % B;
    if (i < bx && j < by) out[((int64_t)k * bx + i) * by + j] = s[t];
  }
}

typedef double v4d __attribute__((ext_vector_type(4)));

// X^T Y for FP32 blocks with B = 16 NT columns on the matrix cores, accumulated in
// FP64 (v_mfma_f64_16x16x4f64: D += A B with A 16x4, B 4x16).  For four consecutive
// rows r..r+3 lane l supplies A[i][kk] = X[r + kk][i] and B[kk][j] = Y[r + kk][j] with
// kk = l / 16 and i = j = l % 16.  D[i][j] sits in lane l, element v with
// i = 4 v + l / 16, j = l % 16 (layout measured on gfx950 with a probe whose inputs
// make every output entry identify its (i, j)).
// NB X blocks (block k at X + k sX) share one pass over Y; the ny groups of NB blocks
// are separate workgroups over the same rows of Y.  Workgroups are dispatched to the 8
// XCDs round-robin, so the 1-D grid of gx ny workgroups (gx row sets, a multiple of 8)
// gives the ny workgroups of one row set ids 8 apart: they run on one XCD at about the
// same time and Y's rows come from HBM once into its L2.  Every wave walks 16-row
// chunks.  When every operand row is exactly B = 16 NT floats (aligned), a chunk is loaded with 16-byte coalesced loads into
// registers one chunk ahead (the loads of chunk i + 1 are in flight while chunk i,
// staged in the wave's own LDS slice, feeds the matrix cores); otherwise one element
// per lane comes straight from memory.  The four waves' accumulators are summed in
// LDS in a fixed order and each workgroup writes one partial (deterministic).
template <int NT, int NB>
__global__ __launch_bounds__(256) void k_gram_mfma(int64_t n, const float* __restrict__ X, int ldx, int64_t sX,
                                                   int nblk, const float* __restrict__ Y, int ldy, int bx, int by,
                                                   double* __restrict__ partials, const double* __restrict__ skip,
                                                   int gx, int ny) {
  if (skip && *skip != 0.0) return;  // the caller does not need this Gram
  const int wg_id = blockIdx.x;
  const int grp = (wg_id >> 3) % ny;                     // group of NB X blocks
  const int rset = ((wg_id >> 3) / ny) * 8 + (wg_id & 7);  // row set, < gx
  constexpr int B = 16 * NT;
  constexpr int TILE = 16 * B;  // floats per 16-row tile of one operand
  constexpr size_t TILE_BYTES = (size_t)4 * (NB + 1) * TILE * sizeof(float);
  constexpr size_t RED_BYTES = (size_t)NB * B * B * sizeof(double);
  __shared__ __align__(16) unsigned char smem[TILE_BYTES > RED_BYTES ? TILE_BYTES : RED_BYTES];
  float(*sm)[NB + 1][TILE] = reinterpret_cast<float(*)[NB + 1][TILE]>(smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kb0 = grp * NB;
  const int nb = (nblk - kb0) < NB ? (nblk - kb0) : NB;
  v4d acc[NB][NT][NT];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int I = 0; I < NT; ++I)
#pragma unroll
      for (int J = 0; J < NT; ++J) acc[q][I][J] = v4d{0.0, 0.0, 0.0, 0.0};
  const int rsub = lane >> 4, c = lane & 15;
  const bool packed = ldx == B && ldy == B && bx == B && by == B && (sX % 4) == 0 &&
                      ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Y)) & 15u) == 0;
  const int64_t nchunks = (n + 15) / 16;
  const int64_t cstride = (int64_t)gx * 4;
  if (packed) {
    // 16 rows x B floats = 4 B float4 per operand, NT per lane
    float4 ry[NT], rx[NB][NT];
    auto fetch = [&](int64_t ch) {
      const int64_t r0 = ch * 16;
#pragma unroll
      for (int s = 0; s < NT; ++s) {
        const int f = s * 64 + lane;  // float4 index inside the tile
        const int64_t row = r0 + (f * 4) / B;
        const bool rok = row < n;
        const int64_t off = r0 * B + (int64_t)f * 4;
        ry[s] = rok ? *reinterpret_cast<const float4*>(Y + off) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int q = 0; q < NB; ++q)
          rx[q][s] = (rok && q < nb) ? *reinterpret_cast<const float4*>(X + (int64_t)(kb0 + q) * sX + off)
                                     : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    };
    int64_t ch = (int64_t)rset * 4 + wave;
    if (ch < nchunks) fetch(ch);
    for (; ch < nchunks; ch += cstride) {
#pragma unroll
      for (int s = 0; s < NT; ++s) {
        const int f = s * 64 + lane;
        *reinterpret_cast<float4*>(&sm[wave][NB][f * 4]) = ry[s];
#pragma unroll
        for (int q = 0; q < NB; ++q) *reinterpret_cast<float4*>(&sm[wave][q][f * 4]) = rx[q][s];
      }
      __builtin_amdgcn_wave_barrier();
      if (ch + cstride < nchunks) fetch(ch + cstride);  // next chunk in flight during the products
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int rl = 4 * m + rsub;
        double yb[NT];
#pragma unroll
        for (int J = 0; J < NT; ++J) yb[J] = (double)sm[wave][NB][rl * B + 16 * J + c];
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int I = 0; I < NT; ++I) {
            const double xa = (double)sm[wave][q][rl * B + 16 * I + c];
#pragma unroll
            for (int J = 0; J < NT; ++J)
              acc[q][I][J] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, yb[J], acc[q][I][J], 0, 0, 0);
          }
      }
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    for (int64_t ch = (int64_t)rset * 4 + wave; ch < nchunks; ch += cstride) {
      const int64_t r0 = ch * 16;
      // every operand element of the chunk is requested before the first product, at
      // addresses clamped into the blocks (a branch around each load would wait for it);
      // out-of-range entries are zeroed afterwards
      float ys[4][NT], xs[4][NB][NT];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int64_t row = min(r0 + 4 * m + rsub, n - 1);
#pragma unroll
        for (int J = 0; J < NT; ++J) ys[m][J] = Y[row * ldy + min(16 * J + c, by - 1)];
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int I = 0; I < NT; ++I)
            xs[m][q][I] = X[(int64_t)(kb0 + min(q, nb - 1)) * sX + row * ldx + min(16 * I + c, bx - 1)];
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const bool rok = r0 + 4 * m + rsub < n;
        double yb[NT];
#pragma unroll
        for (int J = 0; J < NT; ++J) yb[J] = (rok && 16 * J + c < by) ? (double)ys[m][J] : 0.0;
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int I = 0; I < NT; ++I) {
            const double xa = (rok && q < nb && 16 * I + c < bx) ? (double)xs[m][q][I] : 0.0;
#pragma unroll
            for (int J = 0; J < NT; ++J)
              acc[q][I][J] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, yb[J], acc[q][I][J], 0, 0, 0);
          }
      }
    }
  }
  // waves 0..3 add their accumulators into LDS in turn (the tiles are no longer needed)
  __syncthreads();
  double* red = reinterpret_cast<double*>(smem);
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int I = 0; I < NT; ++I)
#pragma unroll
          for (int J = 0; J < NT; ++J)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int idx = q * B * B + (16 * I + 4 * v + rsub) * B + 16 * J + c;
              red[idx] = (w == 0 ? 0.0 : red[idx]) + acc[q][I][J][v];
            }
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < nb * B * B; e += 256) {
    const int q = e / (B * B);
    partials[((int64_t)(kb0 + q) * gx + rset) * (B * B) + (e - q * B * B)] = red[e];
  }
}

// X_k^T Y for any widths up to 16 NT and both precisions on the FP64 matrix cores: the operand
// elements of a 16-row chunk come straight from memory (16 lanes read 16 consecutive
// columns), all requested before the first product, at addresses clamped into the
// blocks; NB blocks X_k share the pass over Y.  Bound: the blocks' bytes.  Partials are
// EB x EB (EB a power of two, at least both widths).  Against LDS tiles with one thread per
// entry, [V_{j-1} V_j W]^T W of 200k rows in FP64, 8 columns: 14.4 us -> 13.5 us.
template <typename T, int NT, int NB>
__global__ __launch_bounds__(256) void k_gram_mx(int64_t n, const T* __restrict__ X, int ldx, int64_t sX, int nblk,
                                                 const T* __restrict__ Y, int ldy, int bx, int by, int EB,
                                                 double* __restrict__ partials) {
  constexpr int B = 16 * NT;
  __shared__ double red[NB * B * B];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kb0 = blockIdx.y * NB;
  const int nb = (nblk - kb0) < NB ? (nblk - kb0) : NB;
  const int g = lane >> 4, c = lane & 15;
  v4d acc[NB][NT][NT];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int I = 0; I < NT; ++I)
#pragma unroll
      for (int J = 0; J < NT; ++J) acc[q][I][J] = v4d{0.0, 0.0, 0.0, 0.0};
  const int64_t nchunks = (n + 15) / 16;
  for (int64_t ch = (int64_t)blockIdx.x * 4 + wave; ch < nchunks; ch += (int64_t)gridDim.x * 4) {
    const int64_t r0 = ch * 16;
    T ys[4][NT], xs[4][NB][NT];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int64_t row = min(r0 + 4 * m + g, n - 1);
#pragma unroll
      for (int J = 0; J < NT; ++J) ys[m][J] = Y[row * ldy + min(16 * J + c, by - 1)];
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int I = 0; I < NT; ++I)
          xs[m][q][I] = X[(int64_t)(kb0 + min(q, nb - 1)) * sX + row * ldx + min(16 * I + c, bx - 1)];
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const bool rok = r0 + 4 * m + g < n;
      double yb[NT];
#pragma unroll
      for (int J = 0; J < NT; ++J) yb[J] = (rok && 16 * J + c < by) ? (double)ys[m][J] : 0.0;
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int I = 0; I < NT; ++I) {
          const double xa = (rok && q < nb && 16 * I + c < bx) ? (double)xs[m][q][I] : 0.0;
#pragma unroll
          for (int J = 0; J < NT; ++J)
            acc[q][I][J] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, yb[J], acc[q][I][J], 0, 0, 0);
        }
    }
  }
  for (int w = 0; w < 4; ++w) {  // the four waves in a fixed order
    if (wave == w) {
#pragma unroll
      for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int I = 0; I < NT; ++I)
#pragma unroll
          for (int J = 0; J < NT; ++J)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int idx = q * B * B + (16 * I + 4 * v + g) * B + 16 * J + c;
              red[idx] = (w == 0 ? 0.0 : red[idx]) + acc[q][I][J][v];
            }
    }
    __syncthreads();
  }
  const int E = EB * EB;
  for (int e = threadIdx.x; e < nb * E; e += 256) {
    const int q = e / E, i = (e - q * E) / EB, j = e % EB;
    partials[((int64_t)(kb0 + q) * gridDim.x + blockIdx.x) * E + (e - q * E)] =
        i < B && j < B ? red[q * B * B + i * B + j] : 0.0;
  }
}

// Coefficient (r, c) of block k: C's, or with a projection step (pj.nbv > 0) what
// k_lanczos_proj would have written for it, taken from the inner products themselves.
__device__ __forceinline__ double coef_at(const double* __restrict__ C, const ProjArgs& pj, int b, int k, int r,
                                          int c) {
  if (pj.nbv == 0) return C[((int64_t)k * b + r) * b + c];
  const double* Pk = pj.P + (int64_t)k * b * b;
  if (k == pj.nbv) return r == c ? 1.0 : 0.0;
  return k + 1 < pj.nbv ? -Pk[r * b + c] : -(0.5 * (Pk[r * b + c] + Pk[c * b + r]));
}

// The other results of the projection step (A_j and the block's scale), by workgroup 0.
__device__ __forceinline__ void proj_outputs(const ProjArgs& pj, int b) {
  if (pj.nbv == 0 || blockIdx.x != 0) return;
  const int t = threadIdx.x;
  const double* Aj = pj.P + (int64_t)(pj.nbv - 1) * b * b;
  const double* Gp = Aj + (int64_t)b * b;
  for (int e = t; e < b * b; e += 256) {
    const int i = e / b, j = e % b;
    pj.Aout[e] = 0.5 * (Aj[i * b + j] + Aj[j * b + i]);
  }
  if (t < 64) {
    double m = t < b ? fmax(0.0, Gp[t * b + t]) : 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if (t == 0) *pj.ref = m;
  }
}

// Out = (wv ? wv[r] : alpha) Yin + beta sum_k X_k C_k for FP32 blocks whose rows are
// exactly B floats (B = 4 LPR): LPR lanes hold one row as float4 fragments (coalesced
// 16-byte accesses across the wave); the row is shared inside its lane group with
// shuffles.  The C_k are staged in LDS (converted to float) once per workgroup when
// they fit (kc blocks at a time otherwise), and the X_k fragments of up to four
// blocks are loaded together so their latencies overlap.
template <int B>
__global__ __launch_bounds__(256) void k_update_f4(int64_t n, const float* X, int64_t sX, int nblk, int kc,
                                                   const double* __restrict__ C, const float* Yin, double alpha,
                                                   const float* __restrict__ wv, double beta, float* Out,
                                                   const double* __restrict__ skip, ProjArgs pj) {
  if (skip && *skip != 0.0) return;  // identity update the caller elides
  constexpr int LPR = B / 4;
  constexpr int RPT = 256 / LPR;  // rows per tile
  extern __shared__ float sC[];   // kc blocks of B x B
  const int sub = threadIdx.x % LPR;
  const int rloc = threadIdx.x / LPR;
  const float tb = (float)beta;
  const bool once = kc >= nblk;
  if (once) {
    for (int e = threadIdx.x; e < nblk * B * B; e += 256)
      sC[e] = (float)coef_at(C, pj, B, e / (B * B), e / B % B, e % B);
    proj_outputs(pj, B);
    __syncthreads();
  }
  const int64_t ntiles = (n + RPT - 1) / RPT;
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t row = t * RPT + rloc;
    const bool ok = row < n;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nblk; c0 += kc) {
      const int c1 = c0 + kc < nblk ? c0 + kc : nblk;
      if (!once) {
        __syncthreads();
        for (int e = threadIdx.x; e < (c1 - c0) * B * B; e += 256) sC[e] = (float)C[(int64_t)c0 * B * B + e];
        __syncthreads();
      }
      for (int k0 = c0; k0 < c1; k0 += 4) {
        float4 xv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          xv[u] = (ok && k0 + u < c1) ? *reinterpret_cast<const float4*>(X + (int64_t)(k0 + u) * sX + row * B + 4 * sub)
                                      : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (k0 + u >= c1) break;
          const float* Ck = sC + (int64_t)(k0 + u - c0) * B * B;
#pragma unroll
          for (int src = 0; src < LPR; ++src) {
            float v[4];
            v[0] = __shfl(xv[u].x, src, LPR);
            v[1] = __shfl(xv[u].y, src, LPR);
            v[2] = __shfl(xv[u].z, src, LPR);
            v[3] = __shfl(xv[u].w, src, LPR);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float* crow = Ck + (4 * src + q) * B + 4 * sub;
#pragma unroll
              for (int cc = 0; cc < 4; ++cc) acc[cc] += v[q] * crow[cc];
            }
          }
        }
      }
    }
    if (ok) {
      float4 o = make_float4(tb * acc[0], tb * acc[1], tb * acc[2], tb * acc[3]);
      if (Yin) {
        const float sc = wv ? wv[row] : (float)alpha;
        const float4 y = *reinterpret_cast<const float4*>(Yin + row * B + 4 * sub);
        o.x += sc * y.x;
        o.y += sc * y.y;
        o.z += sc * y.z;
        o.w += sc * y.w;
      }
      *reinterpret_cast<float4*>(Out + row * B + 4 * sub) = o;
    }
  }
}

// Out = beta sum_k X_k C_k + (wv ? wv : alpha) .* Yin for n x 16 FP32 blocks, as a
// tall-skinny product on the matrix cores (v_mfma_f32_16x16x4f32), optionally with the
// Gram Out^T Out accumulated in FP64 on the same registers (v_mfma_f64_16x16x4f64).
// A wave takes 16-row chunks.  Lane l loads 16 bytes of the chunk, row l % 16, columns
// 4 (l / 16) .. + 3; product step s uses the s-th of them as the A operand, i.e. the
// step runs over the columns {4 g + s : g = 0..3} of every X_k, and lane l supplies the
// matching B operand C_k[4 (l / 16) + s][l % 16] from a lane-ordered copy of C in LDS.
// Lane l then holds result rows 4 (l / 16) + v, column l % 16 (v = 0..3), which are
// also exactly its operands for the Gram: step v sums over rows {4 g + v}.  Rows past
// n load zeros and are not stored.  Out may alias X_k or Yin (a chunk is read whole
// before it is written).  The four waves' Grams are summed in LDS in a fixed order;
// each workgroup writes one 16 x 16 partial.
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int UPD_MFMA_MAXK = 48;

template <bool GRAM>
__global__ __launch_bounds__(256) void k_update_mfma16(int64_t n, const float* X, int64_t sX, int nblk,
                                                       const double* __restrict__ C, const float* Yin, double alpha,
                                                       const float* __restrict__ wv, double beta, float* Out,
                                                       double* __restrict__ partials,
                                                       const double* __restrict__ skip,
                                                       const double* __restrict__ skip_gram, ProjArgs pj) {
  if (skip && *skip != 0.0) return;  // identity update the caller elides
  extern __shared__ float4 sCl[];  // nblk x 64 lane-ordered operands (nblk KiB)
  __shared__ double red[256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  for (int e = threadIdx.x; e < nblk * 64; e += 256) {
    const int k = e >> 6, l = e & 63, gg = l >> 4, cc = l & 15;
    sCl[e] = make_float4((float)coef_at(C, pj, 16, k, 4 * gg, cc), (float)coef_at(C, pj, 16, k, 4 * gg + 1, cc),
                         (float)coef_at(C, pj, 16, k, 4 * gg + 2, cc), (float)coef_at(C, pj, 16, k, 4 * gg + 3, cc));
  }
  proj_outputs(pj, 16);
  __syncthreads();
  const bool gram = GRAM && !(skip_gram && *skip_gram != 0.0);
  const float tb = (float)beta, ta = (float)alpha;
  v4d gacc = {0.0, 0.0, 0.0, 0.0};
  const int64_t nchunks = (n + 15) / 16;
  const int64_t cstride = (int64_t)gridDim.x * 4;
  for (int64_t ch = (int64_t)blockIdx.x * 4 + wave; ch < nchunks; ch += cstride) {
    const int64_t r0 = ch * 16;
    const bool okA = r0 + c < n;
    const float* xa = X + (r0 + c) * 16 + 4 * g;
    v4f d = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < nblk; k0 += 4) {
      float4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        x[u] = (okA && k0 + u < nblk) ? *reinterpret_cast<const float4*>(xa + (int64_t)(k0 + u) * sX)
                                      : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (k0 + u >= nblk) break;
        const float4 bq = sCl[(k0 + u) * 64 + lane];
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].x, bq.x, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].y, bq.y, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].z, bq.z, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u].w, bq.w, d, 0, 0, 0);
      }
    }
    float o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = tb * d[v];
    if (Yin) {  // clamped loads, zero weight past n
      float yv[4], wq[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t row = min(r0 + 4 * g + v, n - 1);
        yv[v] = Yin[row * 16 + c];
        wq[v] = wv ? wv[row] : ta;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (r0 + 4 * g + v < n) o[v] += wq[v] * yv[v];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = r0 + 4 * g + v;
      if (row < n) Out[row * 16 + c] = o[v];
    }
    if (gram) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double ov = (double)o[v];
        gacc = __builtin_amdgcn_mfma_f64_16x16x4f64(ov, ov, gacc, 0, 0, 0);
      }
    }
  }
  if (!gram) return;  // uniform over the workgroup
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int idx = (4 * v + g) * 16 + c;  // FP64 16x16x4 output layout
        red[idx] = (w == 0 ? 0.0 : red[idx]) + gacc[v];
      }
    }
    __syncthreads();
  }
  partials[(int64_t)blockIdx.x * 256 + threadIdx.x] = red[threadIdx.x];
}

// The same for n x 32 FP32 blocks: the 32 x 32 product as 2 x 2 tiles of 16 on
// v_mfma_f32_16x16x4f32.  Lane l loads the 16 bytes at columns 16 h + 4 (l / 16)
// (h = 0, 1) of chunk row l % 16; product step (h, s) takes component s of half h as
// the A operand (the columns {16 h + 4 g + s : g = 0..3}) against the B operand
// C_k[16 h + 4 (l / 16) + s][16 t + l % 16] of output tile t, lane-ordered in LDS
// (4 KiB per block, at most UPD32_MAXK blocks per launch: longer combinations are
// chained launches that accumulate into Out).  Lane l holds result rows
// 4 (l / 16) + v of the columns l % 16 and 16 + l % 16; the optional Gram Out^T Out
// (FP64 matrix cores) takes its three distinct 16 x 16 tiles from the same registers.
// Each workgroup writes one full 32 x 32 partial.
constexpr int UPD32_MAXK = 12;

template <bool GRAM>
__global__ __launch_bounds__(256) void k_update_mfma32(int64_t n, const float* X, int64_t sX, int nblk,
                                                       const double* __restrict__ C, const float* Yin, double alpha,
                                                       const float* __restrict__ wv, double beta, float* Out,
                                                       double* __restrict__ partials,
                                                       const double* __restrict__ skip,
                                                       const double* __restrict__ skip_gram, ProjArgs pj) {
  if (skip && *skip != 0.0) return;  // identity update the caller elides
  extern __shared__ float4 sCl[];     // [block][tile t][half h][lane], nblk x 4 KiB
  __shared__ double red[3][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  for (int e = threadIdx.x; e < nblk * 256; e += 256) {
    const int k = e >> 8, th = (e >> 6) & 3, l = e & 63;
    const int t = th >> 1, h = th & 1, gg = l >> 4, cc = l & 15;
    const int r = 16 * h + 4 * gg, q = 16 * t + cc;
    sCl[e] = make_float4((float)coef_at(C, pj, 32, k, r, q), (float)coef_at(C, pj, 32, k, r + 1, q),
                         (float)coef_at(C, pj, 32, k, r + 2, q), (float)coef_at(C, pj, 32, k, r + 3, q));
  }
  proj_outputs(pj, 32);
  __syncthreads();
  const bool gram = GRAM && !(skip_gram && *skip_gram != 0.0);
  const float tb = (float)beta, ta = (float)alpha;
  v4d g00 = {0.0, 0.0, 0.0, 0.0}, g01 = g00, g11 = g00;
  const int64_t nchunks = (n + 15) / 16;
  const int64_t cstride = (int64_t)gridDim.x * 4;
  for (int64_t ch = (int64_t)blockIdx.x * 4 + wave; ch < nchunks; ch += cstride) {
    const int64_t r0 = ch * 16;
    const bool okA = r0 + c < n;
    const float* xa = X + (r0 + c) * 32 + 4 * g;
    v4f d0 = {0.f, 0.f, 0.f, 0.f}, d1 = d0;
    for (int k0 = 0; k0 < nblk; k0 += 4) {
      float4 x[4][2];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          x[u][h] = (okA && k0 + u < nblk) ? *reinterpret_cast<const float4*>(xa + (int64_t)(k0 + u) * sX + 16 * h)
                                           : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (k0 + u >= nblk) break;
        const float4* bk = sCl + (k0 + u) * 256 + lane;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 b0 = bk[h * 64], b1 = bk[128 + h * 64];
          d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].x, b0.x, d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].x, b1.x, d1, 0, 0, 0);
          d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].y, b0.y, d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].y, b1.y, d1, 0, 0, 0);
          d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].z, b0.z, d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].z, b1.z, d1, 0, 0, 0);
          d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].w, b0.w, d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][h].w, b1.w, d1, 0, 0, 0);
        }
      }
    }
    float o0[4], o1[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      o0[v] = tb * d0[v];
      o1[v] = tb * d1[v];
    }
    if (Yin) {  // clamped loads, zero weight past n
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t row = min(r0 + 4 * g + v, n - 1);
        const float y0 = Yin[row * 32 + c], y1 = Yin[row * 32 + 16 + c];
        const float wq = wv ? wv[row] : ta;
        if (r0 + 4 * g + v < n) {
          o0[v] += wq * y0;
          o1[v] += wq * y1;
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = r0 + 4 * g + v;
      if (row < n) {
        Out[row * 32 + c] = o0[v];
        Out[row * 32 + 16 + c] = o1[v];
      }
    }
    if (gram) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double a = (double)o0[v], b = (double)o1[v];
        g00 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, a, g00, 0, 0, 0);
        g01 = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, g01, 0, 0, 0);
        g11 = __builtin_amdgcn_mfma_f64_16x16x4f64(b, b, g11, 0, 0, 0);
      }
    }
  }
  if (!gram) return;  // uniform over the workgroup
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int idx = (4 * v + g) * 16 + c;  // FP64 16x16x4 output layout
        red[0][idx] = (w == 0 ? 0.0 : red[0][idx]) + g00[v];
        red[1][idx] = (w == 0 ? 0.0 : red[1][idx]) + g01[v];
        red[2][idx] = (w == 0 ? 0.0 : red[2][idx]) + g11[v];
      }
    }
    __syncthreads();
  }
  // the 32 x 32 partial: [[G00, G01], [G01^T, G11]]
  const int i = threadIdx.x >> 4, j = threadIdx.x & 15;
  double* P = partials + (int64_t)blockIdx.x * 1024;
  P[i * 32 + j] = red[0][threadIdx.x];
  P[i * 32 + 16 + j] = red[1][threadIdx.x];
  P[(16 + j) * 32 + i] = red[1][threadIdx.x];
  P[(16 + i) * 32 + 16 + j] = red[2][threadIdx.x];
}

// The same product for every other width b <= 64 and both precisions: a wave takes 16-row
// chunks, the 16 x (4 VW) A operand of one round is one VW-wide load per lane (row l % 16, columns
// VW (l / 16) ..; the round's step s sums over the columns {VW g + s : g}), NT 16-column
// output tiles, C lane-ordered in LDS as VW-wide vectors.  Columns past b load as zeros and are
// not stored, so a ragged width costs matrix-core slots but no extra bytes: the kernel is
// bound by its HBM traffic (X_k and Out once each).  The rows a lane holds of the result
// (FP32: 4 g + v, FP64: 4 v + g) are again the operands of the Gram.  Against the form with a row
// of B values per thread and C broadcast from LDS: FP32, 30 columns, 3 blocks of 100k rows
// 50.8 us -> 19.9 us with the Gram; FP64, 8 columns, 200k rows 20.2 us -> 13.6 us.
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  typedef v4f acc;
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int v) { return 4 * g + v; }
};
template <>
struct Mfma<double> {
  typedef v4d acc;
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int v) { return 4 * v + g; }
};

template <typename T, int VW>
struct __align__(sizeof(T) * VW) LaneVec {
  T v[VW];
};

// rounds of one block and LDS bytes of its coefficients
constexpr int mx_rounds(int b, int vw) { return (b + 4 * vw - 1) / (4 * vw); }
constexpr size_t mx_block_bytes(int b, int vw, int es) {
  return (size_t)mx_rounds(b, vw) * ((b + 15) / 16) * 64 * vw * es;
}

template <typename T, int VW, int NT, bool GRAM>
__global__ __launch_bounds__(256) void k_update_mx(int64_t n, int b, const T* X, int64_t sX, int nblk,
                                                   const double* __restrict__ C, const T* Yin, double alpha,
                                                   const T* __restrict__ wv, double beta, T* Out, int EB,
                                                   double* __restrict__ partials, const double* __restrict__ skip,
                                                   const double* __restrict__ skip_gram, ProjArgs pj) {
  if (skip && *skip != 0.0) return;  // identity update the caller elides
  typedef LaneVec<T, VW> V;
  typedef typename Mfma<T>::acc acc_t;
  extern __shared__ __align__(16) unsigned char smem[];
  V* sC = reinterpret_cast<V*>(smem);  // [block][round][tile][lane]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, c = lane & 15;
  const int KR = mx_rounds(b, VW), R = nblk * KR;
  for (int e = threadIdx.x; e < R * NT * 64; e += 256) {
    const int l = e & 63, t = (e >> 6) % NT, i = (e >> 6) / NT, k = i / KR, q = i - k * KR;
    const int col = 16 * t + (l & 15);
    V w;
#pragma unroll
    for (int s = 0; s < VW; ++s) {
      const int r = 4 * VW * q + VW * (l >> 4) + s;
      w.v[s] = r < b && col < b ? (T)coef_at(C, pj, b, k, r, col) : T(0);
    }
    sC[e] = w;
  }
  proj_outputs(pj, b);
  __syncthreads();
  const bool gram = GRAM && !(skip_gram && *skip_gram != 0.0);
  const T tb = (T)beta, ta = (T)alpha;
  constexpr int NP = NT * (NT + 1) / 2;  // tiles of the Gram's upper triangle
  v4d gacc[GRAM ? NP : 1];
  if constexpr (GRAM) {
#pragma unroll
    for (int p = 0; p < NP; ++p) gacc[p] = v4d{0.0, 0.0, 0.0, 0.0};
  }
  const int64_t nchunks = (n + 15) / 16;
  for (int64_t ch = (int64_t)blockIdx.x * 4 + wave; ch < nchunks; ch += (int64_t)gridDim.x * 4) {
    const int64_t r0 = ch * 16;
    const T* xa = X + (r0 + c) * b + VW * g;
    const bool rok = r0 + c < n;
    acc_t d[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) d[t] = acc_t{0, 0, 0, 0};
    constexpr int U = 4;  // rounds in flight
    int k = 0, q = 0;     // block and round of the next load
    for (int i0 = 0; i0 < R; i0 += U) {
      V x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ok = rok && i0 + u < R && 4 * VW * q + VW * g < b;
        if (ok) {
          x[u] = *reinterpret_cast<const V*>(xa + (int64_t)k * sX + 4 * VW * q);
        } else {
#pragma unroll
          for (int s = 0; s < VW; ++s) x[u].v[s] = T(0);
        }
        if (++q == KR) {
          q = 0;
          ++k;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + u >= R) break;
        const V* w = sC + (int64_t)(i0 + u) * NT * 64 + lane;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const V wt = w[t * 64];
#pragma unroll
          for (int s = 0; s < VW; ++s) d[t] = Mfma<T>::mul(x[u].v[s], wt.v[s], d[t]);
        }
      }
    }
    T o[NT][4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = r0 + Mfma<T>::row(g, v);
      const bool ok = row < n;
      const T wq = Yin && ok ? (wv ? wv[row] : ta) : T(0);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int col = 16 * t + c;
        o[t][v] = T(0);
        if (ok && col < b) {
          o[t][v] = tb * d[t][v];
          if (Yin) o[t][v] += wq * Yin[row * b + col];
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = r0 + Mfma<T>::row(g, v);
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (row < n && 16 * t + c < b) Out[row * b + 16 * t + c] = o[t][v];
    }
    if constexpr (GRAM) {
      if (gram) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          int p = 0;
#pragma unroll
          for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int j = i; j < NT; ++j, ++p)
              gacc[p] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)o[i][v], (double)o[j][v], gacc[p], 0, 0, 0);
        }
      }
    }
  }
  if constexpr (GRAM) {
    if (!gram) return;  // uniform over the workgroup
    __shared__ double red[256];
    double* P = partials + (int64_t)blockIdx.x * EB * EB;
    int p = 0;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = i; j < NT; ++j, ++p) {
        for (int w = 0; w < 4; ++w) {
          if (wave == w) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const int idx = (4 * v + g) * 16 + c;  // FP64 16x16x4 output layout
              red[idx] = (w == 0 ? 0.0 : red[idx]) + gacc[p][v];
            }
          }
          __syncthreads();
        }
        const int a = 16 * i + (threadIdx.x >> 4), e = 16 * j + (threadIdx.x & 15);
        if (a < EB && e < EB) {
          const double v = red[threadIdx.x];
          P[a * EB + e] = v;
          if (i != j) P[e * EB + a] = v;
        }
        __syncthreads();
      }
  }
}

template <typename T, int B>
struct RowVec {
  T v[B];
};

// Single-column blocks are plain vectors: rows are consecutive, so each lane moves 16
// contiguous bytes per load.  Dot products accumulate in FP64.
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  typedef float4 type;
  static constexpr int W = 4;
};
template <>
struct Vec16<double> {
  typedef double2 type;
  static constexpr int W = 2;
};

template <typename T>
__device__ __forceinline__ double vdot(const typename Vec16<T>::type& x, const typename Vec16<T>::type& y) {
  if constexpr (Vec16<T>::W == 4)
    return (double)x.x * (double)y.x + (double)x.y * (double)y.y + (double)x.z * (double)y.z +
           (double)x.w * (double)y.w;
  else
    return (double)x.x * (double)y.x + (double)x.y * (double)y.y;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

constexpr int VDOT_KB = 4;  // vectors X_k dotted with Y per workgroup

// partials[k * gridDim.x + blockIdx.x] = X_k . Y over this workgroup's rows, for
// k in [blockIdx.y * VDOT_KB, +VDOT_KB) and k < nblk.
template <typename T>
__global__ __launch_bounds__(256) void k_vdot(int64_t n, const T* __restrict__ X, int64_t sX, int nblk,
                                              const T* __restrict__ Y, double* __restrict__ partials,
                                              const double* __restrict__ skip) {
  if (skip && *skip != 0.0) return;
  typedef typename Vec16<T>::type V;
  constexpr int W = Vec16<T>::W;
  const int k0 = blockIdx.y * VDOT_KB;
  const int kn = min(VDOT_KB, nblk - k0);
  double acc[VDOT_KB] = {0.0, 0.0, 0.0, 0.0};
  const int64_t nv = n / W;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nv; i += (int64_t)gridDim.x * 256) {
    const V y = reinterpret_cast<const V*>(Y)[i];
#pragma unroll
    for (int kk = 0; kk < VDOT_KB; ++kk)
      if (kk < kn) acc[kk] += vdot<T>(reinterpret_cast<const V*>(X + (int64_t)(k0 + kk) * sX)[i], y);
  }
  if (blockIdx.x == 0) {  // rows past the last whole vector
    const int64_t r = nv * W + threadIdx.x;
    if (r < n) {
#pragma unroll
      for (int kk = 0; kk < VDOT_KB; ++kk)
        if (kk < kn) acc[kk] += (double)X[(int64_t)(k0 + kk) * sX + r] * (double)Y[r];
    }
  }
  __shared__ double red[4][VDOT_KB];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int kk = 0; kk < VDOT_KB; ++kk) {
    const double v = wave_sum(acc[kk]);
    if (lane == 0) red[wave][kk] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < kn)
    partials[(int64_t)(k0 + threadIdx.x) * gridDim.x + blockIdx.x] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

constexpr int VUPD_MAXK = 64;  // vectors combined by one update

// Out = (wv ? wv : alpha) .* Yin + beta * sum_k C[k] X_k on vectors (Out may alias X_k
// or Yin: every element is read and written by the same lane); with partials, the
// workgroup's part of Out . Out goes to partials[blockIdx.x].
template <typename T>
__global__ __launch_bounds__(256) void k_vupdate(int64_t n, const T* X, int64_t sX, int nblk,
                                                 const double* __restrict__ C, const T* Yin, double alpha,
                                                 const T* __restrict__ wv, double beta, T* Out,
                                                 double* __restrict__ partials, const double* __restrict__ skip, ProjArgs pj) {
  if (skip && *skip != 0.0) return;
  typedef typename Vec16<T>::type V;
  constexpr int W = Vec16<T>::W;
  __shared__ T sC[VUPD_MAXK];
  if ((int)threadIdx.x < nblk) sC[threadIdx.x] = (T)coef_at(C, pj, 1, threadIdx.x, 0, 0);
  proj_outputs(pj, 1);
  __syncthreads();
  const T tb = (T)beta, ta = (T)alpha;
  double dot = 0.0;
  const int64_t nv = n / W;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nv; i += (int64_t)gridDim.x * 256) {
    T acc[W];
#pragma unroll
    for (int l = 0; l < W; ++l) acc[l] = T(0);
    for (int k = 0; k < nblk; ++k) {
      const V x = reinterpret_cast<const V*>(X + (int64_t)k * sX)[i];
      const T c = sC[k];
      const T* xs = reinterpret_cast<const T*>(&x);
#pragma unroll
      for (int l = 0; l < W; ++l) acc[l] += xs[l] * c;
    }
    T o[W];
#pragma unroll
    for (int l = 0; l < W; ++l) o[l] = tb * acc[l];
    if (Yin) {
      const V y = reinterpret_cast<const V*>(Yin)[i];
      const T* ys = reinterpret_cast<const T*>(&y);
      if (wv) {
        const V w = reinterpret_cast<const V*>(wv)[i];
        const T* ws = reinterpret_cast<const T*>(&w);
#pragma unroll
        for (int l = 0; l < W; ++l) o[l] += ws[l] * ys[l];
      } else {
#pragma unroll
        for (int l = 0; l < W; ++l) o[l] += ta * ys[l];
      }
    }
    V ov;
    __builtin_memcpy(&ov, o, sizeof(V));
    reinterpret_cast<V*>(Out)[i] = ov;
    if (partials) {
#pragma unroll
      for (int l = 0; l < W; ++l) dot += (double)o[l] * (double)o[l];
    }
  }
  if (blockIdx.x == 0) {  // rows past the last whole vector
    const int64_t r = nv * W + threadIdx.x;
    if (r < n) {
      T acc = T(0);
      for (int k = 0; k < nblk; ++k) acc += X[(int64_t)k * sX + r] * sC[k];
      T o = tb * acc;
      if (Yin) o += (wv ? wv[r] : ta) * Yin[r];
      Out[r] = o;
      if (partials) dot += (double)o * (double)o;
    }
  }
  if (partials) {
    __shared__ double red[4];
    const double v = wave_sum(dot);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

// Out[r,:] = (wv ? wv[r] : alpha) * Yin[r,:] + beta * sum_k X_k[r,0:bx] C_k,  C_k = C[k*bx:(k+1)*bx, 0:by]
template <typename T, int B>
__global__ __launch_bounds__(256) void k_update(int64_t n, const T* X, int ldx, int64_t sX, int nblk,
                                                int bx, const double* __restrict__ C, const T* Yin, int ldy,
                                                double alpha, const T* __restrict__ wv, double beta, T* Out,
                                                int by, double* __restrict__ gram_partials, ProjArgs pj) {
  // rows of the result staged per chunk for the fused Gram (keeps LDS <= 64 KiB)
  constexpr int CHR = (256 * (B + 1) * (int)sizeof(T) <= 65536) ? 256 : 65536 / ((B + 1) * (int)sizeof(T)) / 64 * 64;
  __shared__ T sC[B * B];
  __shared__ T sO[CHR * (B + 1)];
  const int tid = threadIdx.x;
  const T tb = (T)beta;
  constexpr int E = B * B;
  constexpr int QE = E >= 256 ? E / 256 : 1;
  double gacc[QE];
#pragma unroll
  for (int q = 0; q < QE; ++q) gacc[q] = 0.0;
  constexpr int P = E >= 256 ? 1 : 256 / E;
  const int64_t ntiles = (n + 255) / 256;
  proj_outputs(pj, bx);
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int64_t row = t * 256 + tid;
    const bool ok = row < n;
    T acc[B];
#pragma unroll
    for (int j = 0; j < B; ++j) acc[j] = T(0);
    for (int k = 0; k < nblk; ++k) {
      __syncthreads();
      for (int e = tid; e < B * B; e += 256) {
        const int i = e / B, j = e % B;
        sC[e] = (i < bx && j < by) ? (T)(pj.nbv > 0 ? coef_at(C, pj, bx, k, i, j) : C[((int64_t)k * bx + i) * by + j])
                                   : T(0);
      }
      __syncthreads();
      if (ok) {
        const T* xr = X + (int64_t)k * sX + row * ldx;
        T xv[B];
#pragma unroll
        for (int i = 0; i < B; ++i) xv[i] = (i < bx) ? xr[i] : T(0);
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
          for (int j = 0; j < B; ++j) acc[j] += xv[i] * sC[i * B + j];
      }
    }
    if (ok) {
      const T sc = wv ? wv[row] : (T)alpha;
      T* orow = Out + row * ldy;
      const T* yrow = Yin ? Yin + row * ldy : nullptr;
#pragma unroll
      for (int j = 0; j < B; ++j) {
        if (j < by) {
          T o = tb * acc[j];
          if (yrow) o += sc * yrow[j];
          orow[j] = o;
          acc[j] = o;
        }
      }
    }
    if (gram_partials) {
      for (int c0 = 0; c0 < 256; c0 += CHR) {
        const int rows = (256 - c0) < CHR ? (256 - c0) : CHR;
        __syncthreads();
        if (tid >= c0 && tid < c0 + CHR) {
#pragma unroll
          for (int j = 0; j < B; ++j) sO[(tid - c0) * (B + 1) + j] = (ok && j < by) ? acc[j] : T(0);
        }
        __syncthreads();
        if constexpr (E >= 256) {
#pragma unroll
          for (int q = 0; q < QE; ++q) {
            const int e = tid + q * 256;
            const int i = e / B, j = e % B;
            double s = gacc[q];
            for (int r = 0; r < rows; ++r) s += (double)sO[r * (B + 1) + i] * (double)sO[r * (B + 1) + j];
            gacc[q] = s;
          }
        } else {
          const int e = tid % E, p = tid / E;
          if (p < P) {
            const int i = e / B, j = e % B;
            double s = gacc[0];
            for (int r = p; r < rows; r += P) s += (double)sO[r * (B + 1) + i] * (double)sO[r * (B + 1) + j];
            gacc[0] = s;
          }
        }
      }
    }
  }
  if (gram_partials) {
    double* out = gram_partials + (int64_t)blockIdx.x * E;
    if constexpr (E >= 256) {
#pragma unroll
      for (int q = 0; q < QE; ++q) out[tid + q * 256] = gacc[q];
    } else {
      __shared__ double sred[256];
      const int p = tid / E;
      __syncthreads();
      sred[tid] = (p < P) ? gacc[0] : 0.0;
      __syncthreads();
      if (tid < E) {
        double s = 0.0;
        for (int q = 0; q < P; ++q) s += sred[tid + q * E];
        out[tid] = s;
      }
    }
  }
}

// One projection step of block Lanczos (classical Gram-Schmidt against V_{j-1} and
// V_j).  P stacks nbv + 1 b x b blocks: [V_{j-1}^T W'; V_j^T W'; W'^T W'] (nbv = 2) or
// [V_j^T W'; W'^T W'] (nbv = 1).  Outputs: Aout = sym(V_j^T W') (the diagonal block of
// T); Cc = [-P1; -A; I] so that W = [V_{j-1} V_j W'] Cc is the projected block; ref =
// max_i (W'^T W')_ii, the block's scale before projection.  The projected block's
// Gram is then taken from W itself: forming it by Pythagoras from these inner
// products fails as soon as the basis loses orthogonality (converged Ritz vectors).
__global__ __launch_bounds__(256) void k_lanczos_proj(int b, int nbv, const double* __restrict__ P,
                                                     double* __restrict__ Aout, double* __restrict__ Cc, int64_t gs,
                                                     double* __restrict__ ref_out) {
  // one workgroup per graph of a batch: every matrix of graph g sits gs doubles further
  const int64_t go = (int64_t)blockIdx.x * gs;
  P += go;
  Aout += go;
  Cc += go;
  const int t = threadIdx.x;
  const int bb = b * b;
  const bool hasP1 = nbv == 2;
  const double* Aj = P + (size_t)(nbv - 1) * bb;
  const double* Gp = P + (size_t)nbv * bb;
  for (int e = t; e < bb; e += 256) {
    const int i = e / b, j = e % b;
    const double a = 0.5 * (Aj[i * b + j] + Aj[j * b + i]);
    Aout[e] = a;
    if (hasP1) Cc[e] = -P[e];
    Cc[(size_t)(nbv - 1) * bb + e] = -a;
    Cc[(size_t)nbv * bb + e] = i == j ? 1.0 : 0.0;
  }
  if (t < 64 && ref_out) {  // (one thread walking the diagonal waits b times for memory)
    double m = t < b ? fmax(0.0, Gp[t * b + t]) : 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if (t == 0) ref_out[go] = m;
  }
}

// Cholesky with deflation of the b x b matrix G (b <= B), one workgroup of NT threads:
// G = R^T R, a pivot at or below tol * ref gives a zero row of R and a zero column of Rinv.
// Bound: latency, one serial step per column.  The matrix stays in registers: thread
// (g, c) = (t / B, t % B) holds the entries (GR u + g, c), u < EPL, of G and of the unit
// lower factor's inverse E, which the same row operations build (Rinv = E^T / diag), so a
// step is one exchange of row k through LDS, the pivot's root, and EPL independent updates;
// there is no back substitution and no serial product for Bout = R Rprev.
// Measured (with the launch): 16 columns 14.1 us -> 7.3 us, 30 columns 47.7 -> 10.2, 32 columns
// 108 -> 20.0 (average over both CholQR passes of a step), against the form that kept G in LDS and walked R^{-1} and Bout one
// row per lane.
template <int NT>
__device__ __forceinline__ void chol_sync() {
  if constexpr (NT == 64) {  // one wave: LDS accesses stay in program order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// The step's last small matrices of one group of 16 columns: N_{j+1} = Rinv and the
// three-term coefficient N_j B_j^T of the next product.
template <int NT>
__device__ __forceinline__ void next_factors(const NextArgs& nx, const double* Rinv, const double* Bj, int64_t go) {
  for (int e = threadIdx.x; e < 256; e += NT) {
    const int i = e >> 4, j = e & 15;
    nx.Nnext[go + e] = Rinv[e];
    double c = 0.0;
    for (int k = 0; k < 16; ++k) c += nx.Ncur[go + i * 16 + k] * Bj[j * 16 + k];
    nx.Ct[go + e] = c;
  }
}

template <int B, int NT, int NF>
__global__ __launch_bounds__(NF) void k_chol(int b, const double* __restrict__ G, double tol,
                                             const double* __restrict__ Aref, const double* __restrict__ Bref,
                                             double* __restrict__ R, double* __restrict__ Rinv,
                                             const double* __restrict__ Rprev, double* __restrict__ Bout,
                                             int64_t gs, double* __restrict__ ref_out, const double* ref_in,
                                             double post_tol, double* skip_out, double skip_ratio,
                                             const double* skip_in, int dg, const double* dref,
                                             const double* __restrict__ parts, int nparts, int PB,
                                             int64_t pstride, NextArgs nx) {
  const int64_t go = (int64_t)blockIdx.x * gs;  // batch: graph g's matrices at +g gs
  if (ref_out) ref_out += go;
  if (ref_in) ref_in += go;
  if (skip_out) skip_out += go;
  if (skip_in) skip_in += go;
  const int t = threadIdx.x;
  G += go;
  if (Aref) Aref += go;
  if (Bref) Bref += go;
  if (R) R += go;
  Rinv += go;
  if (Rprev) Rprev += go;
  if (Bout) Bout += go;
  if (skip_in && *skip_in != 0.0) {
    // second pass not needed: identity factors, Bout = Rprev (the first pass's factor)
    for (int e = t; e < b * b; e += NF) {
      const double id = (e / b == e % b) ? 1.0 : 0.0;
      if (R) R[e] = id;
      Rinv[e] = id;
      if (Bout) Bout[e] = Rprev ? Rprev[e] : id;
    }
    if constexpr (NF > NT && B == 16) {
      if (nx.Nnext) next_factors<NF>(nx, nx.Ri1 + go, Rprev, go);
    }
    return;
  }
  if ((int)blockIdx.x == dg) {
    // A group of independent single-column processes (different operators side by
    // side): only the diagonal of G is meaningful.  Each column is factorised alone and
    // judged against its own scale (G_ii, A_ii^2 + B_ii^2, and for the later check the
    // diagonal of dref when given); one pass is exact, so no second pass is asked for.
    for (int e = t; e < b * b; e += NT) {
      if (R) R[e] = 0.0;
      Rinv[e] = 0.0;
      if (Bout) Bout[e] = 0.0;
    }
    __syncthreads();
    const double* dr = dref ? dref + go : nullptr;
    for (int i = t; i < b; i += NT) {
      const int d = i * b + i;
      const double g = G[d];
      double sref = g;
      if (Aref || Bref)
        sref = fmax(sref, (Aref ? Aref[d] * Aref[d] : 0.0) + (Bref ? Bref[d] * Bref[d] : 0.0));
      const bool keep = g > 0.0 && g > tol * sref;
      const double r = keep ? sqrt(g) : 0.0;
      double ri = keep ? 1.0 / r : 0.0;
      double bo = r * (Rprev ? Rprev[d] : 1.0);
      if (Bout && ref_in && post_tol > 0.0) {
        const double lim = post_tol * sqrt(fmax(dr ? dr[d] : ref_in[0], 0.0));
        if (fabs(bo) <= lim) {
          bo = 0.0;
          ri = 0.0;
        }
      }
      if (R) R[d] = r;
      Rinv[d] = ri;
      if (Bout) Bout[d] = bo;
    }
    if (t == 0) {
      if (ref_out) {
        double m = 0.0;
        for (int i = 0; i < b; ++i) m = fmax(m, G[i * b + i]);
        ref_out[0] = m;
      }
      if (skip_out) *skip_out = 1.0;
    }
    return;
  }
  // NF > NT: G is still in nparts partial sums of PB x PB entries, which all NF threads sum
  // (fixed order: entry e, phase p takes partials p, p + P, ..; then a tree over the phases)
  __shared__ double sG[NF > NT ? NF : 1];
  if constexpr (NF > NT) {
    const int E = PB * PB, P = NF / E, el = t % E, p = t / E;
    const double* src = parts + (int64_t)blockIdx.x * E + el;
    double u[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int q = p;
    for (; q + 7 * P < nparts; q += 8 * P) {
#pragma unroll
      for (int i = 0; i < 8; ++i) u[i] += src[(q + i * P) * pstride];
    }
    for (; q < nparts; q += P) u[0] += src[q * pstride];
    sG[t] = ((u[0] + u[1]) + (u[2] + u[3])) + ((u[4] + u[5]) + (u[6] + u[7]));
    __syncthreads();
    for (int h = P / 2; h > 0; h >>= 1) {
      if (p < h) sG[t] += sG[t + h * E];
      __syncthreads();
    }
    if (t >= NT) return;
  }
  auto gat = [&](int i, int j) { return NF > NT ? sG[i * PB + j] : G[i * b + j]; };
  constexpr int GR = NT / B, EPL = B / GR;
  static_assert(GR * EPL == B, "entries per thread");
  __shared__ double sR[B * B], sP[B * B];
  __shared__ double rowG[2][B], rowE[2][B];
  __shared__ double sRd[B], sBd[B];
  __shared__ double sref[NT / 64][2];
  const int c = t % B, g = t / B;
  double a[EPL], e[EPL];
#pragma unroll
  for (int u = 0; u < EPL; ++u) {
    const int i = GR * u + g;
    a[u] = (i < b && c < b) ? 0.5 * (gat(i, c) + gat(c, i)) : 0.0;
    e[u] = i == c ? 1.0 : 0.0;
  }
  if (Bout && Rprev) {
#pragma unroll
    for (int u = 0; u < EPL; ++u) {
      const int i = GR * u + g;
      sP[i * B + c] = (i < b && c < b) ? Rprev[i * b + c] : 0.0;
    }
  }
  // reference scale: max diagonal of G and ||Aref||_F^2 + ||Bref||_F^2 over b
  {
    double m = 0.0, fa = 0.0;
#pragma unroll
    for (int u = 0; u < EPL; ++u)
      if (GR * u + g == c) m = fmax(m, a[u]);
    if (Aref)
      for (int k = t; k < b * b; k += NT) fa += Aref[k] * Aref[k];
    if (Bref)
      for (int k = t; k < b * b; k += NT) fa += Bref[k] * Bref[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      m = fmax(m, __shfl_xor(m, off, 64));
      fa += __shfl_xor(fa, off, 64);
    }
    if ((t & 63) == 0) {
      sref[t >> 6][0] = m;
      sref[t >> 6][1] = fa;
    }
  }
  __syncthreads();
  double ref, thr;
  {
    double m = 0.0, fa = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      m = fmax(m, sref[w][0]);
      fa += sref[w][1];
    }
    ref = fmax(m, fa / b);
    thr = tol * ref;
    if (t == 0 && ref_out) ref_out[0] = ref;  // reference scale for a later check
  }
#pragma unroll
  for (int u0 = 0; u0 < EPL; ++u0) {
#pragma unroll 1
    for (int g0 = 0; g0 < GR; ++g0) {
      const int k = GR * u0 + g0, buf = k & 1;
      if (k >= b) break;
      if (g == g0) {
        rowG[buf][c] = a[u0];
        rowE[buf][c] = e[u0];
      }
      chol_sync<NT>();
      const double p = rowG[buf][k];
      const double gj = rowG[buf][c], ej = rowE[buf][c];
      const bool dk = !(p > thr) || !(p > 0.0);
      const double rkk = dk ? 0.0 : sqrt(p);
      const double irkk = dk ? 0.0 : 1.0 / rkk;
      const double ip = irkk * irkk;
#pragma unroll
      for (int u = u0; u < EPL; ++u) {
        const int i = GR * u + g;
        if (i > k) {
          const double m = rowG[buf][i] * ip;
          a[u] -= m * gj;
          e[u] -= m * ej;
        }
      }
      if (g == g0) {  // row k of R, and of R^{-T}
        a[u0] = c == k ? rkk : (c > k ? gj * irkk : 0.0);
        e[u0] = ej * irkk;
        sR[k * B + c] = a[u0];
        if (c == k) sRd[k] = rkk;
      }
    }
  }
  __syncthreads();
  if (R) {
#pragma unroll
    for (int u = 0; u < EPL; ++u) {
      const int i = GR * u + g;
      if (i < b && c < b) R[i * b + c] = a[u];
    }
  }
  if (Bout) {
    if (Rprev) {
#pragma unroll
      for (int u = 0; u < EPL; ++u) a[u] = 0.0;
      for (int k = 0; k < b; ++k) {
        const double q = sP[k * B + c];
#pragma unroll
        for (int u = 0; u < EPL; ++u) {
          const int i = GR * u + g;
          if (i <= k && k <= c) a[u] += sR[i * B + k] * q;  // both upper triangular
        }
      }
    }
#pragma unroll
    for (int u = 0; u < EPL; ++u)
      if (GR * u + g == c) sBd[c] = a[u];
    __syncthreads();
    // Bout is the R factor of the block as stored (R of its true Gram, or R2 R1 after a
    // second pass), so Bout_kk is the true norm of its k-th orthogonal component.
    // Components at the rounding level of the reference scale are dropped: column k of
    // Rinv and row k of Bout become zero, so the next basis block loses that column
    // instead of carrying normalised noise.
    if (ref_in && post_tol > 0.0) {
      const double lim = post_tol * sqrt(fmax(ref_in[0], 0.0));
#pragma unroll
      for (int u = 0; u < EPL; ++u) {
        const int i = GR * u + g;
        if (i < b && fabs(sBd[i]) <= lim) a[u] = e[u] = 0.0;
      }
      __syncthreads();
      if (t < b && fabs(sBd[t]) <= lim) sBd[t] = 0.0;
    }
#pragma unroll
    for (int u = 0; u < EPL; ++u) {
      const int i = GR * u + g;
      if (i < b && c < b) Bout[i * b + c] = c >= i ? a[u] : 0.0;
    }
  }
#pragma unroll
  for (int u = 0; u < EPL; ++u) {
    const int i = GR * u + g;
    if (i < b && c < b) Rinv[c * b + i] = c <= i ? e[u] : 0.0;
  }
  if constexpr (NF > NT && B == 16) {
    if (nx.Nnext) {
      __syncthreads();  // Rinv and Bout of all threads
      next_factors<NT>(nx, Rinv, Bout, go);
    }
  }
  // Is a second CholQR pass needed?  One pass with the Gram accumulated in FP64 leaves
  // the new block orthonormal to about u_64 kappa^2; kappa^2 is the ratio of the largest
  // to the smallest kept pivot.  skip_out = 1 when min / max >= skip_ratio.
  if (skip_out) {
    __syncthreads();
    if (t < 64) {
      double pmax = 0.0, pmin = INFINITY;
      if (t < b) {
        const double r = sRd[t];
        if (r > 0.0 && !(Bout && sBd[t] == 0.0)) pmax = pmin = r * r;
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        pmax = fmax(pmax, __shfl_xor(pmax, off, 64));
        pmin = fmin(pmin, __shfl_xor(pmin, off, 64));
      }
      if (t == 0) *skip_out = (pmax == 0.0 || pmin >= skip_ratio * pmax) ? 1.0 : 0.0;
    }
  }
}

__global__ void k_dadd(int count, const double* __restrict__ x, double* __restrict__ y) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) y[i] += x[i];
}
__global__ void k_dcopy(int count, const double* __restrict__ x, double* __restrict__ y) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) y[i] = x[i];
}

__global__ void k_dtranspose(int b, const double* __restrict__ x, double* __restrict__ y) {
  for (int e = threadIdx.x; e < b * b; e += blockDim.x) y[(e % b) * b + e / b] = x[e];
}

// One term of a Chebyshev series in a block tridiagonal T (K blocks of b x b, A_j and
// T_{j+1,j} = B_j): X0 <- T_k = two (al T X1 - be X1) - X0 with X1 = T_{k-1} and X0 = T_{k-2}
// ((K b) x b each; first: X0 is only written and two is 1), F += c T_k.  Workgroup (j, q) owns
// CHEB_ROWS rows of block row j; the three blocks of X1 it meets and its rows of T are staged in
// LDS.  A launch costs about as long as its work (a 1280 x 32 term: 9.2 us).
constexpr int CHEB_ROWS = 8;
__global__ __launch_bounds__(256) void k_cheb_step(int b, int K, const double* __restrict__ A,
                                                   const double* __restrict__ B, double al, double be, int first,
                                                   const double* __restrict__ X1, double* __restrict__ X0, double c,
                                                   double* __restrict__ F) {
  extern __shared__ double sh[];
  const int j = blockIdx.x, r0 = blockIdx.y * CHEB_ROWS, bb = b * b;
  double* sX = sh;           // 3 b x b
  double* sM = sh + 3 * bb;  // 3 CHEB_ROWS x b
  for (int e = threadIdx.x; e < 3 * bb; e += 256) {
    const int q = e / bb, jj = j - 1 + q;
    sX[e] = jj >= 0 && jj < K ? X1[(int64_t)jj * bb + (e - q * bb)] : 0.0;
  }
  for (int e = threadIdx.x; e < 3 * CHEB_ROWS * b; e += 256) {
    const int q = e / (CHEB_ROWS * b), w = e - q * CHEB_ROWS * b, r = r0 + w / b, k = w % b;
    double v = 0.0;
    if (r < b) {
      if (q == 1) v = A[(int64_t)j * bb + r * b + k];
      if (q == 0 && j > 0) v = B[(int64_t)(j - 1) * bb + r * b + k];
      if (q == 2 && j + 1 < K) v = B[(int64_t)j * bb + k * b + r];
    }
    sM[e] = v;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < CHEB_ROWS * b; e += 256) {
    const int r = r0 + e / b, col = e % b;
    if (r >= b) break;
    double s = 0.0;
    for (int q = 0; q < 3; ++q) {
      const double* M = sM + q * CHEB_ROWS * b + (r - r0) * b;
      const double* X = sX + q * bb + col;
      double s0 = 0.0, s1 = 0.0;
      int k = 0;
      for (; k + 1 < b; k += 2) {
        s0 += M[k] * X[k * b];
        s1 += M[k + 1] * X[(k + 1) * b];
      }
      if (k < b) s0 += M[k] * X[k * b];
      s += s0 + s1;
    }
    const int64_t at = (int64_t)j * bb + r * b + col;
    double v = al * s - be * sX[bb + r * b + col];
    if (!first) v = 2.0 * v - X0[at];
    X0[at] = v;
    F[at] += c * v;
  }
}

// X = E_1 R0, F = c X
__global__ void k_cheb_init(int count, int bb, const double* __restrict__ R0, double c, double* __restrict__ X,
                            double* __restrict__ F) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < count; e += gridDim.x * blockDim.x) {
    const double v = e < bb ? R0[e] : 0.0;
    X[e] = v;
    F[e] = c * v;
  }
}

template <typename T>
__global__ void k_fill(int64_t count, T value, T* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = value;
}

template <typename T>
__global__ void k_axpby_rows(int64_t n, int b, const T* __restrict__ w, const T* __restrict__ X, T beta,
                             const T* __restrict__ Y, T* __restrict__ Out) {
  const int64_t total = n * b;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / b;
    const T wr = w ? w[r] : T(1);
    Out[i] = wr * X[i] + beta * Y[i];
  }
}

template <typename T>
__global__ void k_degrees(int64_t n, const int32_t* __restrict__ rowptr, T* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (T)(rowptr[i + 1] - rowptr[i]);
}

// flags[0]: rowptr not monotone / out of range; [1]: column out of range;
// [2]: self loop; [3]: unsorted or duplicate column; [4]: missing reverse edge.
__global__ void k_validate(int64_t n, int64_t nnz, const int32_t* __restrict__ rowptr,
                           const int32_t* __restrict__ colidx, int32_t* __restrict__ flags) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const int64_t s = rowptr[r], e = rowptr[r + 1];
    if (s > e || s < 0 || e > nnz) {
      atomicOr(&flags[0], 1);
      continue;
    }
    for (int64_t k = s; k < e; ++k) {
      const int32_t c = colidx[k];
      if (c < 0 || c >= n) {
        atomicOr(&flags[1], 1);
        continue;
      }
      if (c == r) atomicOr(&flags[2], 1);
      if (k > s && colidx[k - 1] >= c) atomicOr(&flags[3], 1);
      // reverse edge by binary search in row c
      int64_t lo = rowptr[c], hi = rowptr[c + 1] - 1;
      if (lo < 0 || hi >= nnz) {
        atomicOr(&flags[0], 1);
        continue;
      }
      bool found = false;
      while (lo <= hi) {
        const int64_t mid = (lo + hi) >> 1;
        const int32_t v = colidx[mid];
        if (v == r) {
          found = true;
          break;
        }
        if (v < r) lo = mid + 1; else hi = mid - 1;
      }
      if (!found) atomicOr(&flags[4], 1);
    }
  }
}

// ------------------------------------------------------------ Philox4x32-10
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)M0 * c[0];
    const uint64_t p1 = (uint64_t)M1 * c[2];
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t n0 = hi1 ^ c[1] ^ k0;
    const uint32_t n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
    k0 += W0;
    k1 += W1;
  }
}

template <typename T>
__global__ void k_probes(int law, uint32_t k0, uint32_t k1, uint32_t stream, int64_t total, T* __restrict__ out) {
  const int64_t nq = (total + 3) / 4;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nq; q += (int64_t)gridDim.x * blockDim.x) {
    uint32_t c[4] = {(uint32_t)q, (uint32_t)((uint64_t)q >> 32), stream, 0u};
    philox4x32_10(c, k0, k1);
    double v[4];
    if (law == WL_PROBE_RADEMACHER) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (c[i] >> 31) ? -1.0 : 1.0;
    } else {
      const double two32i = 2.3283064365386963e-10;  // 2^-32
#pragma unroll
      for (int pr = 0; pr < 2; ++pr) {
        const double u1 = ((double)c[2 * pr] + 0.5) * two32i;
        const double u2 = ((double)c[2 * pr + 1] + 0.5) * two32i;
        const double rad = sqrt(-2.0 * log(u1));
        const double th = 6.283185307179586 * u2;
        v[2 * pr] = rad * cos(th);
        v[2 * pr + 1] = rad * sin(th);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t e = q * 4 + i;
      if (e < total) out[e] = (T)v[i];
    }
  }
}

// ------------------------------------------------------------ estimator rows
// s = sum_j Om_rj Y_rj, q = sum_j Om_rj^2 of row r by 16 neighbouring lanes (FP64 sums, the
// result in all of them): rows are read in consecutive pieces.  With one thread per row a
// wave touched 64 lines per load (512 K rows of 64: 1148 us; now 57 us).
template <typename T>
__device__ __forceinline__ void row_dots(int M, const T* __restrict__ o, const T* __restrict__ y, int sub, double* s,
                                         double* q) {
  double a = 0.0, b = 0.0;
  for (int j = sub; j < M; j += 16) {
    const double ov = (double)o[j];
    a += ov * (double)y[j];
    b += ov * ov;
  }
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
  }
  *s = a;
  *q = b;
}

template <typename T>
__global__ __launch_bounds__(256) void k_rowdot(int64_t n, int M, const T* __restrict__ Om, const T* __restrict__ Y,
                                                double* __restrict__ dot, double* __restrict__ sq, int accumulate) {
  const int sub = threadIdx.x & 15;
  for (int64_t r = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); r < n; r += (int64_t)gridDim.x * 16) {
    double s, q;
    row_dots<T>(M, Om + r * M, Y + r * M, sub, &s, &q);
    if (sub == 0) {
      dot[r] = s + (accumulate ? dot[r] : 0.0);
      sq[r] = q + (accumulate ? sq[r] : 0.0);
    }
  }
}

// Diagonal estimate from the accumulated row sums s_r = sum_j Omega_rj Y_rj and
// q_r = sum_j Omega_rj^2 over M probes (modes as in k_cv_finish).
template <typename T>
__global__ void k_sums_finish(int64_t n, int M, const double* __restrict__ dot, const double* __restrict__ sq,
                              const T* __restrict__ g, int mode, T* __restrict__ diag) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const double s = dot[r], q = sq[r];
    double d;
    if (mode == 1) {
      d = s / q;
    } else if (mode == 2) {
      const double gr = (double)g[r];
      d = gr + (s - gr * q) / M;
    } else {
      d = s / M;
    }
    diag[r] = (T)d;
  }
}

// mode 0: Hutchinson, 1: BKS, 2: control variate (Hutchinson law)
template <typename T>
__global__ __launch_bounds__(256) void k_cv_finish(int64_t n, int M, const T* __restrict__ Om,
                                                   const T* __restrict__ Y, const T* __restrict__ g, int mode,
                                                   T* __restrict__ diag) {
  const int sub = threadIdx.x & 15;
  for (int64_t r = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); r < n; r += (int64_t)gridDim.x * 16) {
    double s, q;
    row_dots<T>(M, Om + r * M, Y + r * M, sub, &s, &q);
    if (sub != 0) continue;
    double d;
    if (mode == 1) {
      d = s / q;
    } else if (mode == 2) {
      const double gr = (double)g[r];
      d = gr + (s - gr * q) / M;
    } else {
      d = s / M;
    }
    diag[r] = (T)d;
  }
}

// diag[r] = (y_r^T Q1 y_r + sum_j o_rj y_rj - y_r^T Q2 o_r) / M   (Q1, Q2 M x M, M <= 256)
template <typename T>
__global__ __launch_bounds__(256) void k_nys_diag(int64_t n, int M, const T* __restrict__ Om,
                                                  const T* __restrict__ Y, const double* __restrict__ Q1,
                                                  const double* __restrict__ Q2, T* __restrict__ diag) {
  extern __shared__ double sq[];  // Q1 then Q2 (only when 2*M*M*8 bytes fit)
  const bool staged = (int64_t)2 * M * M <= 8192;
  if (staged) {
    for (int e = threadIdx.x; e < M * M; e += blockDim.x) {
      sq[e] = Q1[e];
      sq[M * M + e] = Q2[e];
    }
    __syncthreads();
  }
  const double* q1 = staged ? sq : Q1;
  const double* q2 = staged ? sq + M * M : Q2;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    const T* o = Om + r * M;
    const T* y = Y + r * M;
    double tot = 0.0;
    for (int i = 0; i < M; ++i) {
      const double yi = (double)y[i];
      double a = 0.0, c = 0.0;
      for (int j = 0; j < M; ++j) {
        a += q1[i * M + j] * (double)y[j];
        c += q2[i * M + j] * (double)o[j];
      }
      tot += yi * (a - c) + (double)o[i] * yi;
    }
    diag[r] = (T)(tot / M);
  }
}

int grid_for(int64_t work, int per_block, int cap) {
  int64_t g = (work + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (int)g;
}

int fin_grid(int E) {
  const int EB = E < 16 ? E : 16;
  return (E + EB - 1) / EB;
}

// A Gram left in its partial sums for the factorisation that follows: where one workgroup
// of 1024 threads sums them in about the time of the launch it saves (up to 32768 values: 5
// columns of 5000 rows, 79 partials, 2.8 + 3.2 us in two launches -> 4.1 us; FP64, 8 columns
// of 200k rows, 512 partials, at the line, 4.6 + 3.2 -> 7.6), or, for a second pass that
// mostly is not needed at all, up to 131072 (1 MB through one CU: 33 us with the factorisation
// where it is needed).
// A Lanczos step is 8 launches so and was 11: 1.50 -> 1.31 ms for 30 steps of the first,
// 3.18 -> 3.14 ms for the second.
// Narrow blocks the same: 2 FP32 columns of 6000 nodes 1.35 -> 1.10 ms for 30 steps, FP64
// 2 columns of 35k nodes 1.44 -> 1.23.
bool defer_sum(GramParts* gp, const double* parts, int64_t nparts, int PB, const double* skip) {
  if (!gp || PB > 32 || nparts * PB * PB > (skip ? 131072 : 32768)) return false;
  gp->p = parts;
  gp->nparts = (int)nparts;
  gp->PB = PB;
  gp->stride = (int64_t)PB * PB;
  return true;
}

// blocks X_k that share a pass over Y: as many as the accumulators leave room for
template <typename T, int B>
void gram_mx(wl_ctx* ctx, int64_t n, const T* X, int ldx, int64_t sX, int nblk, const T* Y, int ldy, int bx, int by,
             int parts) {
  constexpr int NT = B <= 16 ? 1 : B / 16, NB = NT == 1 ? 3 : (NT == 2 ? 2 : 1);
  if (nblk == 1)
    hipLaunchKernelGGL((k_gram_mx<T, NT, 1>), dim3(parts, 1), dim3(256), 0, ctx->stream, n, X, ldx, sX, nblk, Y, ldy,
                       bx, by, B, ctx->partials.as<double>());
  else
    hipLaunchKernelGGL((k_gram_mx<T, NT, NB>), dim3(parts, (nblk + NB - 1) / NB), dim3(256), 0, ctx->stream, n, X,
                       ldx, sX, nblk, Y, ldy, bx, by, B, ctx->partials.as<double>());
}

// Partial sums per block that a Gram of nblk blocks leaves (gram_partials_bound plans by the
// same functions).  FP32 blocks of 16 to 64 columns: row sets of k_gram_mfma, a multiple of the 8
// XCDs; up to 1024 workgroups in all, and 256 per group of blocks (every row set writes one FP64
// partial per block, which for many wide blocks is a fair share of the blocks' own bytes: 20
// blocks of 32 columns, 262k rows, 168 MB at 1024 row sets beside 700 MB; 288 us -> 238, the
// reduction behind it 13.5 -> 6.4).
int64_t gram_row_sets(int64_t n, int B, int nblk) {
  const int64_t sets = ((n + 15) / 16 + 15) / 16;
  const int64_t groups = B >= 64 ? nblk : B == 32 || nblk == 2 ? (nblk + 1) / 2 : (nblk + 2) / 3;
  return (std::max<int64_t>(1, std::min(sets, std::max<int64_t>(256, 1024 / groups))) + 7) / 8 * 8;
}
// The other blocks: k_gram_mx from five columns on, a wave per 16-row chunk up to 256 workgroups,
// then four chunks per wave (5000 rows of 5: 9.0 us with four from the start, 5.5 us so); below,
// a 32-row tile each.  2^22 entries in all, between 32 and 512 per block.
int64_t gram_parts(int64_t n, int B, int nblk) {
  const int64_t cap = std::min<int64_t>(512, std::max<int64_t>(32, ((int64_t)1 << 22) / ((int64_t)B * B * nblk)));
  if (B < 8) return std::max<int64_t>(1, std::min((n + GRAM_TR - 1) / GRAM_TR, cap));
  int64_t parts = std::min(cap, std::max((n + 255) / 256, std::min<int64_t>((n + 63) / 64, 256)));
  if (parts > 8) parts = parts / 8 * 8;
  return std::max<int64_t>(1, parts);
}

template <int B>
wl_status gram_B(wl_ctx* ctx, int64_t n, const void* X, bool isf, int ldx, int64_t sX, int nblk, const void* Y,
                 int ldy, int bx, int by, double* out, const double* skip = nullptr, GramParts* gp = nullptr) {
  constexpr int E = B * B;
  if constexpr (B >= 16) {
    if (isf) {
      // matrix-core path, FP64 accumulation
      constexpr int NT = B / 16;
      const int64_t blocks = gram_row_sets(n, B, nblk);
      const int nparts = (int)blocks;  // one partial per row set and block
      WL_TRY(ctx->partials.ensure((size_t)nparts * nblk * E * sizeof(double)));
      double* pp = ctx->partials.as<double>();
      const float* Xf = (const float*)X;
      const float* Yf = (const float*)Y;
      if (NT >= 4 || nblk == 1) {
        hipLaunchKernelGGL((k_gram_mfma<NT, 1>), dim3((unsigned)(blocks * nblk)), dim3(256), 0, ctx->stream, n, Xf,
                           ldx, sX, nblk, Yf, ldy, bx, by, pp, skip, (int)blocks, nblk);
      } else if (nblk == 2 || NT == 2) {
        const int ny = (nblk + 1) / 2;
        hipLaunchKernelGGL((k_gram_mfma<NT, 2>), dim3((unsigned)(blocks * ny)), dim3(256), 0, ctx->stream, n, Xf,
                           ldx, sX, nblk, Yf, ldy, bx, by, pp, skip, (int)blocks, ny);
      } else {
        const int ny = (nblk + 2) / 3;
        hipLaunchKernelGGL((k_gram_mfma<NT, 3>), dim3((unsigned)(blocks * ny)), dim3(256), 0, ctx->stream, n, Xf,
                           ldx, sX, nblk, Yf, ldy, bx, by, pp, skip, (int)blocks, ny);
      }
      WL_HIP(hipGetLastError());
      hipLaunchKernelGGL(k_gram_finalize, dim3(fin_grid(E), nblk), dim3(256), 0, ctx->stream,
                         ctx->partials.as<double>(), nparts, B, bx, by, out, skip);
      WL_HIP(hipGetLastError());
      return WL_OK;
    }
  }
  if constexpr (B == 1) {
    const int W = isf ? 4 : 2;
    if (bx == 1 && by == 1 && ldx == 1 && ldy == 1 && sX % W == 0 &&
        ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Y)) & 15u) == 0) {
      int64_t parts = (n / W + 511) / 512;  // two vectors of 16 bytes per lane
      if (parts > 1024) parts = 1024;
      if (parts < 1) parts = 1;
      WL_TRY(ctx->partials.ensure((size_t)parts * nblk * sizeof(double)));
      const dim3 grid((unsigned)parts, (unsigned)((nblk + VDOT_KB - 1) / VDOT_KB));
      if (isf)
        hipLaunchKernelGGL(k_vdot<float>, grid, dim3(256), 0, ctx->stream, n, (const float*)X, sX, nblk,
                           (const float*)Y, ctx->partials.as<double>(), skip);
      else
        hipLaunchKernelGGL(k_vdot<double>, grid, dim3(256), 0, ctx->stream, n, (const double*)X, sX, nblk,
                           (const double*)Y, ctx->partials.as<double>(), skip);
      WL_HIP(hipGetLastError());
      hipLaunchKernelGGL(k_gram_finalize, dim3(1, nblk), dim3(256), 0, ctx->stream, ctx->partials.as<double>(),
                         (int)parts, 1, 1, 1, out, skip);
      WL_HIP(hipGetLastError());
      return WL_OK;
    }
  }
  const int64_t parts = gram_parts(n, B, nblk);
  if constexpr (B >= 8) {
    WL_TRY(ctx->partials.ensure((size_t)parts * nblk * E * sizeof(double)));
    if constexpr (B < 16) {  // (wider FP32 blocks have returned above)
      if (isf) gram_mx<float, B>(ctx, n, (const float*)X, ldx, sX, nblk, (const float*)Y, ldy, bx, by, (int)parts);
    }
    if (!isf)
      gram_mx<double, B>(ctx, n, (const double*)X, ldx, sX, nblk, (const double*)Y, ldy, bx, by, (int)parts);
    WL_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_gram_finalize, dim3(fin_grid(E), nblk), dim3(256), 0, ctx->stream,
                       ctx->partials.as<double>(), (int)parts, B, bx, by, out, skip);
    WL_HIP(hipGetLastError());
    return WL_OK;
  } else {
    WL_TRY(ctx->partials.ensure((size_t)parts * nblk * E * sizeof(double)));
    dim3 grid((unsigned)parts, nblk);
    hipLaunchKernelGGL(k_gram_partial<B>, grid, dim3(256), 0, ctx->stream, n,
                       isf ? (const float*)X : nullptr, isf ? nullptr : (const double*)X, ldx, sX,
                       isf ? (const float*)Y : nullptr, isf ? nullptr : (const double*)Y, ldy, bx, by,
                       ctx->partials.as<double>());
    WL_HIP(hipGetLastError());
    if (nblk == 1 && defer_sum(gp, ctx->partials.as<double>(), parts, B, nullptr)) return WL_OK;
    hipLaunchKernelGGL(k_gram_finalize, dim3(fin_grid(E), nblk), dim3(256), 0, ctx->stream,
                       ctx->partials.as<double>(), (int)parts, B, bx, by, out, nullptr);
    WL_HIP(hipGetLastError());
    return WL_OK;
  }
}

int pick_B(int b) {
  int B = 1;
  while (B < b) B <<= 1;
  return B;
}

// k_update_mx for blocks of b columns (rows of b values): *done = false where it does not
// apply.  Combinations longer than the LDS holds run as chained launches that accumulate
// into Out; where Out is one of the X_k they must fit one launch (up to 128 KiB instead of the
// 64 KiB that keep two workgroups on a CU).
template <typename T, int VW, int NT>
wl_status update_mx(wl_ctx* ctx, int64_t n, int b, const T* X, int64_t sX, int nblk, const double* C, const T* Yin,
                    double alpha, const T* wv, double beta, T* Out, double* gram_out, const double* skip,
                    const double* skip_gram, const ProjArgs& pj, GramParts* gp, bool* done) {
  const size_t bytes = mx_block_bytes(b, VW, sizeof(T));
  const uintptr_t xo = reinterpret_cast<uintptr_t>(X), oo = reinterpret_cast<uintptr_t>(Out);
  const bool alias = nblk > 0 && oo >= xo && oo < xo + ((uintptr_t)(nblk - 1) * sX + (uintptr_t)n * b) * sizeof(T);
  int kmax = (int)(65536 / bytes);
  if (nblk > kmax && (alias || kmax < 1)) {
    kmax = (int)(131072 / bytes);
    if (nblk > kmax && alias) return WL_OK;
  }
  if (pj.nbv > 0 && nblk > kmax) return WL_OK;  // its coefficients are staged by one launch
  *done = true;
  const int64_t nchunks = (n + 15) / 16;
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(gram_out ? 512 : 1024, (nchunks + 3) / 4));
  int EB = 1;
  while (EB < b) EB <<= 1;
  if (gram_out) WL_TRY(ctx->partials.ensure((size_t)grid * EB * EB * sizeof(double)));
  int k0 = 0;
  do {
    const int kb = std::min(kmax, nblk - k0);
    const bool first = k0 == 0, last = k0 + kb == nblk;
    const T* Xk = X + (int64_t)k0 * sX;
    const double* Ck = C + (int64_t)k0 * b * b;
    const T* Yk = first ? Yin : Out;
    const double ak = first ? alpha : 1.0;
    const T* wk = first ? wv : nullptr;
    if (last && gram_out)
      hipLaunchKernelGGL((k_update_mx<T, VW, NT, true>), dim3(grid), dim3(256), kb * bytes, ctx->stream, n, b, Xk, sX,
                         kb, Ck, Yk, ak, wk, beta, Out, EB, ctx->partials.as<double>(), skip, skip_gram, pj);
    else
      hipLaunchKernelGGL((k_update_mx<T, VW, NT, false>), dim3(grid), dim3(256), kb * bytes, ctx->stream, n, b, Xk,
                         sX, kb, Ck, Yk, ak, wk, beta, Out, EB, nullptr, skip, nullptr, pj);
    WL_HIP(hipGetLastError());
    k0 += kb;
  } while (k0 < nblk);
  if (gram_out && !defer_sum(gp, ctx->partials.as<double>(), grid, EB, skip_gram)) {
    hipLaunchKernelGGL(k_gram_finalize, dim3(fin_grid(EB * EB), 1), dim3(256), 0, ctx->stream,
                       ctx->partials.as<double>(), grid, EB, b, b, gram_out, skip_gram);
    WL_HIP(hipGetLastError());
  }
  return WL_OK;
}

template <typename T, int VW>
wl_status update_mx_nt(wl_ctx* ctx, int64_t n, int b, const T* X, int64_t sX, int nblk, const double* C, const T* Yin,
                       double alpha, const T* wv, double beta, T* Out, double* gram_out, const double* skip,
                       const double* skip_gram, const ProjArgs& pj, GramParts* gp, bool* done) {
  if (b <= 16)
    return update_mx<T, VW, 1>(ctx, n, b, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                             done);
  if (b <= 32)
    return update_mx<T, VW, 2>(ctx, n, b, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                             done);
  if (b <= 48)
    return update_mx<T, VW, 3>(ctx, n, b, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                             done);
  return update_mx<T, VW, 4>(ctx, n, b, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                             done);
}

// The widest loads that the width and the alignment of the blocks X_k allow (and that give
// every lane of a round columns: 8 FP32 columns are four 8-byte loads, not two of 16).
template <typename T>
wl_status update_mx_any(wl_ctx* ctx, int64_t n, int b, const T* X, int64_t sX, int nblk, const double* C,
                        const T* Yin, double alpha, const T* wv, double beta, T* Out, double* gram_out,
                        const double* skip, const double* skip_gram, const ProjArgs& pj, GramParts* gp,
                        bool* done) {
  *done = false;
  if (b < 5 || b > 64 || (skip && gram_out)) return WL_OK;
  const uintptr_t xo = reinterpret_cast<uintptr_t>(X);
  auto fits = [&](int vw) { return b % vw == 0 && sX % vw == 0 && xo % (vw * sizeof(T)) == 0; };
  if constexpr (sizeof(T) == 4) {
    if (b > 8 && fits(4))
      return update_mx_nt<T, 4>(ctx, n, b, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                             done);
  }
  if (fits(2))
    return update_mx_nt<T, 2>(ctx, n, b, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                             done);
  return update_mx_nt<T, 1>(ctx, n, b, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                             done);
}

template <typename T, int B>
wl_status update_B(wl_ctx* ctx, int64_t n, const T* X, int ldx, int64_t sX, int nblk, int bx, const double* C,
                   const T* Yin, int ldy, double alpha, const T* wv, double beta, T* Out, int by,
                   double* gram_out, const double* skip, const double* skip_gram, ProjArgs pj, GramParts* gp) {
  constexpr int E = B * B;
  if constexpr (sizeof(T) == 4 && B == 16) {
    const bool al = ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Out) |
                      reinterpret_cast<uintptr_t>(Yin)) & 15u) == 0 && (sX % 4) == 0;
    if (bx == 16 && by == 16 && ldx == 16 && ldy == 16 && al && nblk <= UPD_MFMA_MAXK && !(skip && gram_out)) {
      const int64_t nchunks = (n + 15) / 16;
      int64_t grid = (nchunks + 15) / 16;  // about four chunks per wave
      if (grid > 1024) grid = 1024;
      if (grid < 1) grid = 1;
      const size_t lds = (size_t)nblk * 64 * sizeof(float4);
      if (gram_out) {
        WL_TRY(ctx->partials.ensure((size_t)grid * 256 * sizeof(double)));
        hipLaunchKernelGGL(k_update_mfma16<true>, dim3((unsigned)grid), dim3(256), lds, ctx->stream, n,
                           (const float*)X, sX, nblk, C, (const float*)Yin, alpha, (const float*)wv, beta,
                           (float*)Out, ctx->partials.as<double>(), skip, skip_gram, pj);
        WL_HIP(hipGetLastError());
        if (!defer_sum(gp, ctx->partials.as<double>(), grid, 16, skip_gram)) {
          hipLaunchKernelGGL(k_gram_finalize, dim3(fin_grid(256), 1), dim3(256), 0, ctx->stream,
                             ctx->partials.as<double>(), (int)grid, 16, 16, 16, gram_out, skip_gram);
          WL_HIP(hipGetLastError());
        }
      } else {
        hipLaunchKernelGGL(k_update_mfma16<false>, dim3((unsigned)grid), dim3(256), lds, ctx->stream, n,
                           (const float*)X, sX, nblk, C, (const float*)Yin, alpha, (const float*)wv, beta,
                           (float*)Out, nullptr, skip, nullptr, pj);
        WL_HIP(hipGetLastError());
      }
      return WL_OK;
    }
  }
  if constexpr (sizeof(T) == 4 && B == 32) {
    const bool al = ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Out) |
                      reinterpret_cast<uintptr_t>(Yin)) & 15u) == 0 && (sX % 4) == 0;
    // chained launches overwrite Out before the later blocks are read: Out must not
    // be one of them
    const uintptr_t xo = reinterpret_cast<uintptr_t>(X), oo = reinterpret_cast<uintptr_t>(Out);
    const bool chain_alias = nblk > UPD32_MAXK && oo >= xo &&
                             oo < xo + ((uintptr_t)(nblk - 1) * (uintptr_t)sX + (uintptr_t)n * 32) * sizeof(float);
    if (bx == 32 && by == 32 && ldx == 32 && ldy == 32 && al && !(skip && gram_out) && !chain_alias &&
        (pj.nbv == 0 || nblk <= UPD32_MAXK)) {
      const int64_t nchunks = (n + 15) / 16;
      int64_t grid = (nchunks + 15) / 16;  // about four chunks per wave
      if (grid > (gram_out ? 512 : 1024)) grid = gram_out ? 512 : 1024;  // (partials: 8 KiB a workgroup)
      if (grid < 1) grid = 1;
      if (gram_out) WL_TRY(ctx->partials.ensure((size_t)grid * 1024 * sizeof(double)));
      for (int k0 = 0; k0 < nblk; k0 += UPD32_MAXK) {
        const int kb = std::min(UPD32_MAXK, nblk - k0);
        const bool first = k0 == 0, last = k0 + kb == nblk;
        const float* Xk = (const float*)X + (int64_t)k0 * sX;
        const float* Yk = first ? (const float*)Yin : (const float*)Out;
        const double ak = first ? alpha : 1.0;
        const float* wk = first ? (const float*)wv : nullptr;
        const size_t lds = (size_t)kb * 256 * sizeof(float4);
        if (last && gram_out) {
          hipLaunchKernelGGL(k_update_mfma32<true>, dim3((unsigned)grid), dim3(256), lds, ctx->stream, n, Xk, sX, kb,
                             C + (int64_t)k0 * 1024, Yk, ak, wk, beta, (float*)Out, ctx->partials.as<double>(), skip,
                             skip_gram, pj);
          WL_HIP(hipGetLastError());
          if (!defer_sum(gp, ctx->partials.as<double>(), grid, 32, skip_gram))
            hipLaunchKernelGGL(k_gram_finalize, dim3(fin_grid(1024), 1), dim3(256), 0, ctx->stream,
                             ctx->partials.as<double>(), (int)grid, 32, 32, 32, gram_out, skip_gram);
        } else {
          hipLaunchKernelGGL(k_update_mfma32<false>, dim3((unsigned)grid), dim3(256), lds, ctx->stream, n, Xk, sX, kb,
                             C + (int64_t)k0 * 1024, Yk, ak, wk, beta, (float*)Out, nullptr, skip, nullptr, pj);
        }
        WL_HIP(hipGetLastError());
      }
      return WL_OK;
    }
  }
  if constexpr (B >= 8) {
    if (bx == by && ldx == bx && ldy == by) {
      bool done = false;
      WL_TRY(update_mx_any<T>(ctx, n, bx, X, sX, nblk, C, Yin, alpha, wv, beta, Out, gram_out, skip, skip_gram, pj, gp,
                              &done));
      if (done) return WL_OK;
    }
  }
  if (pj.nbv > 0 && (bx != by || (B == 4 && nblk > 4))) {  // coefficients from memory
    WL_TRY(launch_lanczos_proj(ctx, bx, pj.nbv, pj.P, pj.Aout, const_cast<double*>(C), pj.ref, 1, 0));
    pj = ProjArgs();
  }
  if constexpr (sizeof(T) == 4 && B == 4) {
    const bool al = ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Out) |
                      reinterpret_cast<uintptr_t>(Yin)) & 15u) == 0 && (sX % 4) == 0;
    if (bx == B && by == B && ldx == B && ldy == B && al) {
      constexpr int RPT = 256 / (B / 4);
      int64_t ntiles = (n + RPT - 1) / RPT;
      const int grid = (int)(ntiles < 1 ? 1 : (ntiles > 8192 ? 8192 : ntiles));
      // C blocks staged per workgroup: all of them if they fit in 48 KB
      const int kc = std::max(1, std::min(nblk, 12288 / (B * B)));
      const size_t lds = (size_t)kc * B * B * sizeof(float);
      hipLaunchKernelGGL((k_update_f4<B>), dim3(grid), dim3(256), lds, ctx->stream, n, (const float*)X, sX, nblk,
                         kc, C, (const float*)Yin, alpha, (const float*)wv, beta, (float*)Out, skip, pj);
      WL_HIP(hipGetLastError());
      if (gram_out) return gram_B<B>(ctx, n, Out, true, B, 0, 1, Out, B, B, B, gram_out, skip_gram, gp);
      return WL_OK;
    }
  }
  if constexpr (B == 1) {
    constexpr int W = sizeof(T) == 4 ? 4 : 2;
    // (an update that may be skipped and also yields a Gram takes the general path)
    if (bx == 1 && by == 1 && ldx == 1 && ldy == 1 && nblk <= VUPD_MAXK && sX % W == 0 && !(skip && gram_out) &&
        ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Out) | reinterpret_cast<uintptr_t>(Yin) |
          reinterpret_cast<uintptr_t>(wv)) & 15u) == 0) {
      int64_t grid = (n / W + 1023) / 1024;
      if (grid > (gram_out ? 512 : 2048)) grid = gram_out ? 512 : 2048;
      if (grid < 1) grid = 1;
      double* parts = nullptr;
      if (gram_out) {
        WL_TRY(ctx->partials.ensure((size_t)grid * sizeof(double)));
        parts = ctx->partials.as<double>();
      }
      hipLaunchKernelGGL(k_vupdate<T>, dim3((unsigned)grid), dim3(256), 0, ctx->stream, n, X, sX, nblk, C, Yin,
                         alpha, wv, beta, Out, parts, skip, pj);
      WL_HIP(hipGetLastError());
      if (gram_out && !defer_sum(gp, parts, grid, 1, skip_gram)) {
        hipLaunchKernelGGL(k_gram_finalize, dim3(1, 1), dim3(256), 0, ctx->stream, parts, (int)grid, 1, 1, 1,
                           gram_out, skip_gram);
        WL_HIP(hipGetLastError());
      }
      return WL_OK;
    }
  }
  const int64_t ntiles = (n + 255) / 256;
  const int cap = gram_out ? 512 : 4096;
  const int grid = (int)(ntiles < cap ? (ntiles < 1 ? 1 : ntiles) : cap);
  double* parts = nullptr;
  if (gram_out) {
    WL_TRY(ctx->partials.ensure((size_t)grid * E * sizeof(double)));
    parts = ctx->partials.as<double>();
  }
  hipLaunchKernelGGL((k_update<T, B>), dim3(grid), dim3(256), 0, ctx->stream, n, X, ldx, sX, nblk, bx, C, Yin, ldy,
                     alpha, wv, beta, Out, by, parts, pj);
  WL_HIP(hipGetLastError());
  if (gram_out && !defer_sum(gp, parts, grid, B, nullptr)) {
    hipLaunchKernelGGL(k_gram_finalize, dim3(fin_grid(E), 1), dim3(256), 0, ctx->stream, parts, grid, B, by, by,
                       gram_out, nullptr);
    WL_HIP(hipGetLastError());
  }
  return WL_OK;
}

}  // namespace

template <typename T>
wl_status launch_gram(wl_ctx* ctx, int64_t n, const T* X, int bx, int64_t sX, int nblk, const T* Y, int by,
                      double* out) {
  WL_CHECK(bx >= 1 && bx <= 64 && by >= 1 && by <= 64 && nblk >= 1, WL_EINVAL, "gram: block sizes out of range");
  const bool isf = sizeof(T) == 4;
  const int B = pick_B(bx > by ? bx : by);
  switch (B) {
    case 1: return gram_B<1>(ctx, n, X, isf, bx, sX, nblk, Y, by, bx, by, out);
    case 2: return gram_B<2>(ctx, n, X, isf, bx, sX, nblk, Y, by, bx, by, out);
    case 4: return gram_B<4>(ctx, n, X, isf, bx, sX, nblk, Y, by, bx, by, out);
    case 8: return gram_B<8>(ctx, n, X, isf, bx, sX, nblk, Y, by, bx, by, out);
    case 16: return gram_B<16>(ctx, n, X, isf, bx, sX, nblk, Y, by, bx, by, out);
    case 32: return gram_B<32>(ctx, n, X, isf, bx, sX, nblk, Y, by, bx, by, out);
    default: return gram_B<64>(ctx, n, X, isf, bx, sX, nblk, Y, by, bx, by, out);
  }
}

template <typename T>
wl_status launch_update_skip(wl_ctx* ctx, int64_t n, const T* X, int bx, int64_t sX, int nblk, const double* C,
                             const T* Yin, double alpha, const T* wv, double beta, T* Out, int by, double* gram_out,
                             const double* skip, const double* skip_gram, const ProjArgs& pj, GramParts* gp) {
  WL_CHECK(bx >= 1 && bx <= 64 && by >= 1 && by <= 64, WL_EINVAL, "update: block sizes out of range");
  const int B = pick_B(bx > by ? bx : by);
  switch (B) {
    case 1: return update_B<T, 1>(ctx, n, X, bx, sX, nblk, bx, C, Yin, by, alpha, wv, beta, Out, by, gram_out,
                                                   skip, skip_gram, pj, gp);
    case 2: return update_B<T, 2>(ctx, n, X, bx, sX, nblk, bx, C, Yin, by, alpha, wv, beta, Out, by, gram_out,
                                                   skip, skip_gram, pj, gp);
    case 4: return update_B<T, 4>(ctx, n, X, bx, sX, nblk, bx, C, Yin, by, alpha, wv, beta, Out, by, gram_out,
                                                   skip, skip_gram, pj, gp);
    case 8: return update_B<T, 8>(ctx, n, X, bx, sX, nblk, bx, C, Yin, by, alpha, wv, beta, Out, by, gram_out,
                                                   skip, skip_gram, pj, gp);
    case 16: return update_B<T, 16>(ctx, n, X, bx, sX, nblk, bx, C, Yin, by, alpha, wv, beta, Out, by, gram_out,
                                                   skip, skip_gram, pj, gp);
    case 32: return update_B<T, 32>(ctx, n, X, bx, sX, nblk, bx, C, Yin, by, alpha, wv, beta, Out, by, gram_out,
                                                   skip, skip_gram, pj, gp);
    default: return update_B<T, 64>(ctx, n, X, bx, sX, nblk, bx, C, Yin, by, alpha, wv, beta, Out, by, gram_out,
                                                   skip, skip_gram, pj, gp);
  }
}

template <typename T>
wl_status launch_update(wl_ctx* ctx, int64_t n, const T* X, int bx, int64_t sX, int nblk, const double* C,
                        const T* Yin, double alpha, const T* wv, double beta, T* Out, int by, double* gram_out) {
  return launch_update_skip<T>(ctx, n, X, bx, sX, nblk, C, Yin, alpha, wv, beta, Out, by, gram_out, nullptr,
                               nullptr);
}

wl_status launch_lanczos_proj(wl_ctx* ctx, int b, int nbv, const double* P, double* Aout, double* Cc,
                              double* ref_out, int ngraphs, int64_t gs) {
  WL_CHECK(b >= 1 && b <= 64 && (nbv == 1 || nbv == 2) && ngraphs >= 1, WL_EINVAL,
           "lanczos projection: bad sizes");
  hipLaunchKernelGGL(k_lanczos_proj, dim3(ngraphs), dim3(256), 0, ctx->stream, b, nbv, P, Aout, Cc, gs, ref_out);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status launch_chol(wl_ctx* ctx, int b, const double* G, double tol, const double* Aref, const double* Bref,
                      double* R, double* Rinv, const double* Rprev, double* Bout, int ngraphs, int64_t gs,
                      double* ref_out, const double* ref_in, double post_tol, double* skip_out, double skip_ratio,
                      const double* skip_in, int dg, const double* dref, const GramParts* gp, const NextArgs& nx) {
  WL_CHECK(b >= 1 && b <= 64 && ngraphs >= 1, WL_EINVAL, "chol: b out of range");
  const bool sum = gp && gp->nparts > 0;
  WL_CHECK((!sum && !nx.Nnext) || (sum && b > gp->PB / 2 && b <= gp->PB && gp->PB <= 32 && (!nx.Nnext || b == 16)),
           WL_EINTERNAL,
           "chol: partial sums of another shape");
  auto run = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(ngraphs), dim3(threads), 0, ctx->stream, b, G, tol, Aref, Bref, R, Rinv, Rprev,
                       Bout, gs, ref_out, ref_in, post_tol, skip_out, skip_ratio, skip_in, dg, dref,
                       sum ? gp->p : nullptr, sum ? gp->nparts : 0, sum ? gp->PB : 0, sum ? gp->stride : 0, nx);
  };
  // the smallest size that holds the matrix, 16 entries per thread at most
  if (b <= 8)
    sum ? run(k_chol<8, 64, 1024>, 1024) : run(k_chol<8, 64, 64>, 64);
  else if (b <= 16)
    sum ? run(k_chol<16, 64, 1024>, 1024) : run(k_chol<16, 64, 64>, 64);
  else if (b <= 32)
    sum ? run(k_chol<32, 256, 1024>, 1024) : run(k_chol<32, 256, 256>, 256);
  else
    run(k_chol<64, 256, 256>, 256);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status launch_cheb(wl_ctx* ctx, int b, int K, const double* A, const double* B, const double* R0, double al,
                      double be, const std::vector<double>& c, double* X0, double* X1, double* F) {
  WL_CHECK(b >= 1 && b <= 64 && K >= 1 && c.size() >= 2, WL_EINVAL, "Chebyshev series: bad sizes");
  const int count = K * b * b;
  hipLaunchKernelGGL(k_cheb_init, dim3(grid_for(count, 256, 512)), dim3(256), 0, ctx->stream, count, b * b, R0, c[0],
                     X1, F);
  WL_HIP(hipGetLastError());
  const dim3 grid((unsigned)K, (unsigned)((b + CHEB_ROWS - 1) / CHEB_ROWS));
  const size_t lds = (size_t)3 * (b + CHEB_ROWS) * b * sizeof(double);
  for (size_t k = 1; k < c.size(); ++k) {
    hipLaunchKernelGGL(k_cheb_step, grid, dim3(256), lds, ctx->stream, b, K, A, B, al, be, k == 1 ? 1 : 0, X1, X0,
                       c[k], F);
    WL_HIP(hipGetLastError());
    std::swap(X0, X1);
  }
  return WL_OK;
}

wl_status launch_dadd(wl_ctx* ctx, int count, const double* x, double* y) {
  hipLaunchKernelGGL(k_dadd, dim3(grid_for(count, 256, 64)), dim3(256), 0, ctx->stream, count, x, y);
  WL_HIP(hipGetLastError());
  return WL_OK;
}
wl_status launch_dcopy(wl_ctx* ctx, int count, const double* x, double* y) {
  hipLaunchKernelGGL(k_dcopy, dim3(grid_for(count, 256, 64)), dim3(256), 0, ctx->stream, count, x, y);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status launch_dtranspose(wl_ctx* ctx, int b, const double* x, double* y) {
  hipLaunchKernelGGL(k_dtranspose, dim3(1), dim3(256), 0, ctx->stream, b, x, y);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_fill(wl_ctx* ctx, int64_t count, T value, T* out) {
  if (count <= 0) return WL_OK;
  hipLaunchKernelGGL((k_fill<T>), dim3(grid_for(count, 256, 8192)), dim3(256), 0, ctx->stream, count, value, out);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_axpby_rows(wl_ctx* ctx, int64_t n, int b, const T* w, const T* X, double beta, const T* Y,
                            T* Out) {
  if (n * b <= 0) return WL_OK;
  hipLaunchKernelGGL((k_axpby_rows<T>), dim3(grid_for(n * b, 256, 8192)), dim3(256), 0, ctx->stream, n, b, w, X,
                     (T)beta, Y, Out);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_degrees(wl_graph* g, T* out) {
  if (g->n == 0) return WL_OK;
  hipLaunchKernelGGL((k_degrees<T>), dim3(grid_for(g->n, 256, 8192)), dim3(256), 0, g->ctx->stream, g->n, g->rowptr,
                     out);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

wl_status launch_validate(wl_graph* g, int32_t* d_flags) {
  if (g->n == 0) return WL_OK;
  hipLaunchKernelGGL(k_validate, dim3(grid_for(g->n, 256, 8192)), dim3(256), 0, g->ctx->stream, g->n, g->nnz,
                     g->rowptr, g->colidx, d_flags);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_probes(wl_ctx* ctx, int law, uint64_t seed, uint32_t stream, int64_t n, int M, T* out) {
  const int64_t total = n * (int64_t)M;
  if (total <= 0) return WL_OK;
  hipLaunchKernelGGL((k_probes<T>), dim3(grid_for((total + 3) / 4, 256, 8192)), dim3(256), 0, ctx->stream, law,
                     (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32), stream, total, out);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_rowdot(wl_ctx* ctx, int64_t n, int M, const T* Om, const T* Y, double* dot, double* sq,
                        int accumulate) {
  hipLaunchKernelGGL((k_rowdot<T>), dim3(grid_for(n, 16, 8192)), dim3(256), 0, ctx->stream, n, M, Om, Y, dot, sq,
                     accumulate);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_sums_finish(wl_ctx* ctx, int64_t n, int M, const double* dot, const double* sq, const T* g,
                             int mode, T* diag) {
  hipLaunchKernelGGL((k_sums_finish<T>), dim3(grid_for(n, 256, 8192)), dim3(256), 0, ctx->stream, n, M, dot, sq, g,
                     mode, diag);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_cv_finish(wl_ctx* ctx, int64_t n, int M, const T* Om, const T* Y, const T* g, int mode, T* diag) {
  hipLaunchKernelGGL((k_cv_finish<T>), dim3(grid_for(n, 16, 8192)), dim3(256), 0, ctx->stream, n, M, Om, Y, g, mode,
                     diag);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

template <typename T>
wl_status launch_nys_diag(wl_ctx* ctx, int64_t n, int M, const T* Om, const T* Y, const double* Q1,
                          const double* Q2, T* diag) {
  const size_t lds = ((int64_t)2 * M * M <= 8192) ? (size_t)2 * M * M * sizeof(double) : 0;
  hipLaunchKernelGGL((k_nys_diag<T>), dim3(grid_for(n, 256, 8192)), dim3(256), lds, ctx->stream, n, M, Om, Y, Q1, Q2,
                     diag);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

size_t gram_partials_bound(int64_t n, int prec, int b, int nblk) {
  const int64_t B = pick_B(b), E = B * B;
  nblk = std::max(nblk, 1);
  int64_t doubles = 0;
  // matrix-core Gram (FP32, B >= 16): one partial per workgroup, at most 1024
  const int64_t mfma_parts = std::min<int64_t>(1024, std::max<int64_t>(1, ((n + 15) / 16 + 15) / 16));
  if (prec == WL_FP32 && B >= 16) doubles = std::max(doubles, mfma_parts * nblk * E);
  // single-column dot products: at most 1024 partials per block
  if (B == 1) doubles = std::max<int64_t>(doubles, 1024 * nblk);
  // general tiles: one partial per 32-row tile, at most clamp(2^22 / (E nblk), 32, 512)
  const int64_t ntiles = std::max<int64_t>(1, (n + GRAM_TR - 1) / GRAM_TR);
  const int64_t cap = std::min<int64_t>(512, std::max<int64_t>(32, ((int64_t)1 << 22) / (E * nblk)));
  doubles = std::max<int64_t>(doubles, std::min(ntiles, cap) * nblk * E);
  // the sums as taken, of every number of blocks up to nblk (their product is not monotone:
  // the caps round down and the row sets up to 8)
  for (int k = 1; k <= nblk; ++k)
    doubles = std::max(doubles, (prec == WL_FP32 && B >= 16 ? gram_row_sets(n, (int)B, k) : gram_parts(n, (int)B, k)) *
                                    k * E);
  return (size_t)doubles * sizeof(double);
}

size_t update_partials_bound(int64_t n, int prec, int b) {
  const int64_t B = pick_B(b), E = B * B;
  // matrix-core update with its Gram (FP32, 16 wide): one 256-value partial per workgroup
  const int64_t mfma_grid = std::min<int64_t>(1024, std::max<int64_t>(1, ((n + 15) / 16 + 15) / 16));
  int64_t doubles = (prec == WL_FP32 && B == 16) ? mfma_grid * 256 : 0;
  doubles = std::max<int64_t>(doubles, 512);  // single-column updates
  // general tiles with the Gram: one partial per 256-row tile, at most 512
  doubles = std::max<int64_t>(doubles, std::min<int64_t>(512, std::max<int64_t>(1, (n + 255) / 256)) * E);
  // updates that take a separate Gram of their output
  doubles = std::max<int64_t>(doubles, (int64_t)gram_partials_bound(n, prec, b, 1) / (int64_t)sizeof(double));
  return (size_t)doubles * sizeof(double);
}

#define WL_INST(T)                                                                                                   \
  template wl_status launch_gram<T>(wl_ctx*, int64_t, const T*, int, int64_t, int, const T*, int, double*);        \
  template wl_status launch_update<T>(wl_ctx*, int64_t, const T*, int, int64_t, int, const double*, const T*,      \
                                      double, const T*, double, T*, int, double*);                                 \
  template wl_status launch_update_skip<T>(wl_ctx*, int64_t, const T*, int, int64_t, int, const double*, const T*, \
                                           double, const T*, double, T*, int, double*, const double*,             \
                                           const double*, const ProjArgs&, GramParts*);                                                         \
  template wl_status launch_fill<T>(wl_ctx*, int64_t, T, T*);                                                      \
  template wl_status launch_axpby_rows<T>(wl_ctx*, int64_t, int, const T*, const T*, double, const T*, T*);       \
  template wl_status launch_degrees<T>(wl_graph*, T*);                                                              \
  template wl_status launch_probes<T>(wl_ctx*, int, uint64_t, uint32_t, int64_t, int, T*);                         \
  template wl_status launch_rowdot<T>(wl_ctx*, int64_t, int, const T*, const T*, double*, double*, int);           \
  template wl_status launch_sums_finish<T>(wl_ctx*, int64_t, int, const double*, const double*, const T*, int, T*); \
  template wl_status launch_cv_finish<T>(wl_ctx*, int64_t, int, const T*, const T*, const T*, int, T*);            \
  template wl_status launch_nys_diag<T>(wl_ctx*, int64_t, int, const T*, const T*, const double*, const double*,  \
                                        T*);
WL_INST(float)
WL_INST(double)
