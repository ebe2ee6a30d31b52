// Krylov evaluations of small graphs in one workgroup (gfx950).
//
// On a graph of a few thousand nodes a Lanczos step is a dozen launches of 2 to 5 us each for
// microseconds of work: the launches are the bound.  Here one workgroup of 1024 threads (16
// waves) runs a whole evaluation, or a whole orthogonalisation step, with barriers in place of
// launches, the graph (16-bit columns) and the gathered block in LDS, and the other vectors in
// registers:
//   * k_vec_lanczos: phi x of one column by K Lanczos steps on a A + (b0 + b1 D), the
//     tridiagonal solve and the recombination included;
//   * k_vec_orth: one fully reorthogonalised step for a vector W that another operator made;
//   * k_small_lanczos: the same steps for a block of two to four columns (the fused step of the
//     general driver: three-term subtraction, projection against the last one or two blocks,
//     CholQR2 with deflation; Gram matrices on the FP64 matrix cores) and T F = scale E_1 R0;
//   * k_small_series: the truncated series (eq. qrec), one workgroup per column.
// A row belongs to one thread, rows of more than SMALL_LONG neighbours to one wave.  A load that
// misses the CU takes about a microsecond here, a barrier a few hundred nanoseconds: what
// counts is the number of both per step (a first form with every vector in memory and
// eight lanes per row took 22 us per step at 1000 nodes).  No workgroup waits for another.
// Erdos-Renyi graph of 1000 nodes, FP64, one column: a resolvent product of 40 steps 1.63 ms ->
// 0.16 ms, walk degrees with L x and exp(-t L) u of 30 outer steps 52.9 -> 5.2 ms.
#include <algorithm>
#include <type_traits>

#include "wl_internal.h"

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int SMALL_T = 1024;         // threads
constexpr int SMALL_W = SMALL_T / 64;  // waves
constexpr int SMALL_B = 4;            // columns of a block
constexpr int SMALL_K = 256;          // steps k_vec_lanczos keeps scalars for
constexpr int64_t SMALL_BLOCK_VALUES = 5000;  // rows times columns of a block
typedef uint16_t idx_t;               // columns and row pointers in LDS

__device__ __forceinline__ double shfl(double v, int lane) { return __shfl(v, lane, 64); }

// out[(k b + i) b + j] = (X_k^T Y)_ij for k < nb (X_k = X + k sX, all n x b).  The nb b columns
// of the X_k are taken 16 at a time as A operands.  red: SMALL_W x 256 doubles.  Every
// thread of the workgroup calls; out is complete for all of them on return.
template <typename T>
__device__ void small_gram(int n, int b, const T* X, int64_t sX, int nb, const T* Y, double* red, double* out) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, c = lane & 15;
  const int cols = nb * b;
  const T* yp = Y + min(c, b - 1);
  for (int q = 0; q * 16 < cols; ++q) {
    const int col = min(16 * q + c, cols - 1), blk = col / b;
    const T* xp = X + blk * sX + (col - blk * b);
    const bool xok = 16 * q + c < cols, yok = c < b;
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int r0 = wave * 16; r0 < n; r0 += SMALL_W * 16) {
      double x[4], y[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int row = min(r0 + 4 * m + g, n - 1);
        x[m] = (double)xp[(int64_t)row * b];
        y[m] = (double)yp[(int64_t)row * b];
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const bool ok = r0 + 4 * m + g < n;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ok && xok ? x[m] : 0.0, ok && yok ? y[m] : 0.0, acc, 0, 0, 0);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave * 256 + (4 * v + g) * 16 + c] = acc[v];
    __syncthreads();
    if (t < 256) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < SMALL_W; ++w) s += red[w * 256 + t];
      const int i = 16 * q + (t >> 4), j = t & 15;
      if (i < cols && j < b) out[i * b + j] = s;
    }
    __syncthreads();
  }
}

// Cholesky with deflation of the b x b matrix sG by one wave (b <= 8; lane 8 i + c holds entry
// (i, c)), the inverse built by the same row operations: the rules of the general kernel.
// Bout = R Rprev (or R).  ref_in > 0 with post > 0: components of Bout at or below
// post sqrt(ref_in) are dropped.  Returns 1 when the kept pivots span at least ratio.
__device__ bool small_chol(int b, const double* sG, double thr, double* sRinv, const double* sRprev, double* sBout,
                           double ref_in, double post, double ratio) {
  const int lane = threadIdx.x & 63, i = lane >> 3, c = lane & 7;
  const bool in = i < b && c < b;
  double a = in ? 0.5 * (sG[i * b + c] + sG[c * b + i]) : 0.0, e = i == c ? 1.0 : 0.0;
  for (int k = 0; k < b; ++k) {
    const double p = shfl(a, 9 * k), gj = shfl(a, 8 * k + c), gi = shfl(a, 8 * k + i), ej = shfl(e, 8 * k + c);
    const bool dk = !(p > thr) || !(p > 0.0);
    const double rkk = dk ? 0.0 : sqrt(p), irkk = dk ? 0.0 : 1.0 / rkk;
    if (i > k) {
      const double m = gi * (irkk * irkk);
      a -= m * gj;
      e -= m * ej;
    } else if (i == k) {
      a = c == k ? rkk : (c > k ? gj * irkk : 0.0);
      e = ej * irkk;
    }
  }
  double bo = a;
  if (sRprev) {
    bo = 0.0;
    for (int k = 0; k < b; ++k) {
      const double r = shfl(a, 8 * i + k);
      if (i <= k && k <= c && c < b) bo += r * sRprev[k * b + c];
    }
  }
  if (ref_in > 0.0 && post > 0.0) {
    const double bd = shfl(bo, 9 * i);
    if (fabs(bd) <= post * sqrt(ref_in)) bo = e = 0.0;
  }
  if (in) {
    sRinv[c * b + i] = c <= i ? e : 0.0;
    sBout[i * b + c] = c >= i ? bo : 0.0;
  }
  const bool kept = in && i == c && a > 0.0 && bo != 0.0;
  double pmax = kept ? a * a : 0.0, pmin = kept ? a * a : INFINITY;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    pmax = fmax(pmax, __shfl_xor(pmax, off, 64));
    pmin = fmin(pmin, __shfl_xor(pmin, off, 64));
  }
  return pmax == 0.0 || pmin >= ratio * pmax;
}

__device__ double small_maxdiag(int b, const double* G) {
  const int lane = threadIdx.x & 63;
  double m = lane < b ? fmax(0.0, G[lane * b + lane]) : 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  return m;
}

// Entry (i, c) of M N^T or M N for 8 x 8 matrices held one entry per lane.
__device__ __forceinline__ double mul_nt(int b, double m, double n) {
  const int lane = threadIdx.x & 63, i = lane >> 3, c = lane & 7;
  double s = 0.0;
  for (int k = 0; k < b; ++k) s += shfl(m, 8 * i + k) * shfl(n, 8 * c + k);
  return s;
}
__device__ __forceinline__ double mul_nn(int b, double m, double n) {
  const int lane = threadIdx.x & 63, i = lane >> 3, c = lane & 7;
  double s = 0.0;
  for (int k = 0; k < b; ++k) s += shfl(m, 8 * i + k) * shfl(n, 8 * k + c);
  return s;
}
__device__ __forceinline__ double mul_tn(int b, double m, double n) {
  const int lane = threadIdx.x & 63, i = lane >> 3, c = lane & 7;
  double s = 0.0;
  for (int k = 0; k < b; ++k) s += shfl(m, 8 * k + i) * shfl(n, 8 * k + c);
  return s;
}

// F = scale T^{-1} E_1 R0 for the block tridiagonal T (diagonal blocks A_j, T_{j+1,j} = B_j) by
// block elimination in one wave; rows of T that are exactly zero (deflated basis columns)
// get a unit diagonal.  work: K blocks.  False where a pivot is not positive (or NaN).
__device__ bool small_solve(int b, int K, const double* A, const double* Bo, const double* R0, double scale,
                            double* work, double* F) {
  const int lane = threadIdx.x & 63, i = lane >> 3, c = lane & 7, bb = b * b;
  const bool in = i < b && c < b;
  const int at = in ? i * b + c : 0, tr = in ? c * b + i : 0;
  double y = in ? scale * R0[at] : 0.0, G = 0.0, Bp = 0.0;
  double An = in ? 0.5 * (A[at] + A[tr]) : 0.0;
  bool good = true;
  for (int j = 0; j < K; ++j) {
    double a = An;
    const bool more = j + 1 < K;
    const double Bj = in && more ? Bo[(int64_t)j * bb + at] : 0.0;
    const double Bjt = in && more ? Bo[(int64_t)j * bb + tr] : 0.0;
    An = in && more ? 0.5 * (A[(int64_t)(j + 1) * bb + at] + A[(int64_t)(j + 1) * bb + tr]) : 0.0;
    const unsigned long long nz = __ballot(a != 0.0 || Bp != 0.0 || Bjt != 0.0);
    if (i == c && i < b && ((nz >> (8 * i)) & 0xffull) == 0) a = 1.0;
    if (j > 0) a -= mul_nt(b, G, Bp);
    double e = i == c ? 1.0 : 0.0;
    for (int k = 0; k < b; ++k) {
      const double p = shfl(a, 9 * k), gj = shfl(a, 8 * k + c), gi = shfl(a, 8 * k + i), ej = shfl(e, 8 * k + c);
      good = good && p > 0.0;
      const double ir = 1.0 / sqrt(p);
      if (i > k) {
        const double m = gi * (ir * ir);
        a -= m * gj;
        e -= m * ej;
      } else if (i == k) {
        e = ej * ir;
      }
    }
    if (c > i) e = 0.0;
    const double P = mul_tn(b, e, e);  // S_j^{-1} = R^{-1} R^{-T}, e = R^{-T}
    const double z = mul_nn(b, P, y);
    if (in) F[(int64_t)j * bb + at] = z;
    if (more) {
      G = mul_nn(b, Bj, P);
      y = -mul_nn(b, G, y);
      if (in) work[(int64_t)j * bb + at] = G;
      Bp = Bj;
    }
  }
  double x = in ? F[(int64_t)(K - 1) * bb + at] : 0.0;
  double Gn = in && K > 1 ? work[(int64_t)(K - 2) * bb + at] : 0.0, Fn = in && K > 1 ? F[(int64_t)(K - 2) * bb + at] : 0.0;
  for (int j = K - 2; j >= 0; --j) {
    const double Gj = Gn, Fj = Fn;
    if (j > 0 && in) {
      Gn = work[(int64_t)(j - 1) * bb + at];
      Fn = F[(int64_t)(j - 1) * bb + at];
    }
    x = Fj - mul_tn(b, Gj, x);
    if (in) F[(int64_t)j * bb + at] = x;
  }
  return good;
}

// The graph in LDS: row pointers, columns, and the list of rows that take a wave.
struct LdsGraph {
  idx_t *rp, *ci, *longs;
  int n_long;
};

// Bytes of a staged graph (16-byte aligned).
__host__ __device__ inline size_t lds_graph_bytes(int64_t n, int64_t nnz) {
  return ((size_t)(n + 1 + nnz + n) * sizeof(idx_t) + 15) / 16 * 16;
}

template <int NT>
__device__ LdsGraph stage_graph(unsigned char* at, int n, const int32_t* __restrict__ rowptr,
                                const int32_t* __restrict__ colidx) {
  __shared__ int count;
  LdsGraph g;
  const int t = threadIdx.x, nnz = rowptr[n];
  g.rp = reinterpret_cast<idx_t*>(at);
  g.ci = g.rp + n + 1;
  g.longs = g.ci + nnz;
  if (t == 0) count = 0;
  __syncthreads();
  for (int r = t; r < n; r += NT) {
    const int s = rowptr[r], e = rowptr[r + 1];
    g.rp[r] = (idx_t)s;
    if (e - s > SMALL_LONG) g.longs[atomicAdd(&count, 1)] = (idx_t)r;  // (their order does not matter)
  }
  if (t == 0) g.rp[n] = (idx_t)nnz;
  for (int e = t; e < nnz; e += NT) g.ci[e] = (idx_t)colidx[e];
  __syncthreads();
  g.n_long = count;
  return g;
}

// acc = sum of the rows sV[j, 0:B] over the columns s + sub, s + sub + width, ... < e
template <typename T, int B>
__device__ __forceinline__ void gather_lds(const idx_t* ci, int s, int e, int sub, int width, const T* sV,
                                           T (&acc)[B]) {
#pragma unroll
  for (int c = 0; c < B; ++c) acc[c] = T(0);
  int k = s + sub;
  for (; k + 3 * width < e; k += 4 * width) {
    const int j0 = ci[k], j1 = ci[k + width], j2 = ci[k + 2 * width], j3 = ci[k + 3 * width];
#pragma unroll
    for (int c = 0; c < B; ++c)
      acc[c] = (((acc[c] + sV[j0 * B + c]) + sV[j1 * B + c]) + sV[j2 * B + c]) + sV[j3 * B + c];
  }
  for (; k < e; k += width) {
    const int j = ci[k];
#pragma unroll
    for (int c = 0; c < B; ++c) acc[c] += sV[j * B + c];
  }
}

// sL[r, :] = row sums of the long rows (a wave each); a barrier follows where there are any.
template <typename T, int B, int NT>
__device__ __forceinline__ void gather_long(const LdsGraph& g, const T* sV, T* sL) {
  if (g.n_long == 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int q = wave; q < g.n_long; q += NT / 64) {
    const int r = g.longs[q];
    T acc[B];
    gather_lds<T, B>(g.ci, g.rp[r], g.rp[r + 1], lane, 64, sV, acc);
#pragma unroll
    for (int c = 0; c < B; ++c) {
      for (int off = 32; off > 0; off >>= 1) acc[c] += __shfl_xor(acc[c], off, 64);
      if (lane == 0) sL[r * B + c] = acc[c];
    }
  }
  __syncthreads();
}

// v of the lane that a DPP control names (a register move; a shuffle goes through the LDS pipe).
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int2 h = __builtin_bit_cast(int2, v);
  int2 r;
  r.x = __builtin_amdgcn_update_dpp(0, h.x, CTRL, 0xf, 0xf, true);
  r.y = __builtin_amdgcn_update_dpp(0, h.y, CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, r);
}

// Sum over the 16 lanes of a row, in all of them: quad neighbours, quad pairs, then mirrored
// halves (each side already uniform).
__device__ __forceinline__ double row_sum(double v) {
  v += dpp<0xB1>(v);   // quad_perm 1,0,3,2
  v += dpp<0x4E>(v);   // quad_perm 2,3,0,1
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  return v;
}

__device__ __forceinline__ double wave_total(double v) {
  v = row_sum(v);
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

// Sums over a workgroup of NT threads of N doubles per thread, in a fixed order, in all threads.
// One barrier; red alternates between two halves (parity).
template <int NT, int N>
__device__ __forceinline__ void block_sums(double (&a)[N], double* red, int parity) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* h = red + parity * 3 * 16;
#pragma unroll
  for (int i = 0; i < N; ++i) a[i] = wave_total(a[i]);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) h[16 * i + wave] = a[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) a[i] = row_sum((lane & 15) < NT / 64 ? h[16 * i + (lane & 15)] : 0.0);
}

template <typename T>
struct SmallArgs {
  int n, b, K, reorth;
  const int32_t *rowptr, *colidx;
  double a, b0, b1;
  const T* X;
  T* basis;             // (K + 1) blocks
  double *A, *Bo, *R0;  // K, K, 1 blocks: the projected matrix
  double tol, post, ratio;
  double scale;  // > 0: solve T F = scale E_1 R0 (k_small_lanczos: into F, with `work` of K blocks)
  double *work, *F;
  const T *wv, *Xw;  // k_vec_lanczos: Y = V F, or wv (.) Xw - V F
  T* Y;
  int* done;  // host flag: 1 when F (Y) is valid
};

// One column; thread t owns the rows t, t + 1024, ..
template <typename T, int R, int NT>
__global__ __launch_bounds__(NT) void k_vec_lanczos(SmallArgs<T> p) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[2 * 3 * 16];
  __shared__ double sA[SMALL_K], sB[SMALL_K], sD[SMALL_K], sF[SMALL_K];
  __shared__ int good;
  const int t = threadIdx.x, n = p.n, K = p.K;
  auto total = [&](double x, int parity) {
    double a[1] = {x};
    block_sums<NT, 1>(a, red, parity);
    return a[0];
  };
  const LdsGraph g = stage_graph<NT>(smem, n, p.rowptr, p.colidx);
  T* sV = reinterpret_cast<T*>(smem + lds_graph_bytes(n, g.rp[n]));
  T* sL = sV + n;  // sums of the long rows
  int rs[R], re[R];
  T v[R], vp[R], dg[R];
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int r = t + q * NT;
    rs[q] = r < n ? g.rp[r] : 0;
    re[q] = r < n ? g.rp[r + 1] : 0;
    dg[q] = (T)(p.b0 + p.b1 * (double)(re[q] - rs[q]));
    vp[q] = T(0);
    v[q] = r < n ? p.X[r] : T(0);
    s += (double)v[q] * (double)v[q];
  }
  // V_0 R0 = x, normalised twice
  s = total(s, 0);
  const double ref = s;
  double r1 = s > p.tol * ref && s > 0.0 ? sqrt(s) : 0.0;
  T f = r1 > 0.0 ? (T)(1.0 / r1) : T(0);
  s = 0.0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    v[q] *= f;
    s += (double)v[q] * (double)v[q];
  }
  s = total(s, 1);
  const double r2 = s > p.tol * s && s > 0.0 ? sqrt(s) : 0.0;
  double R0 = r2 * r1;
  f = r2 > 0.0 ? (T)(1.0 / r2) : T(0);
  if (ref > 0.0 && fabs(R0) <= p.post * sqrt(ref)) {
    R0 = 0.0;
    f = T(0);
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int r = t + q * NT;
    v[q] *= f;
    if (r < n) p.basis[r] = sV[r] = v[q];
  }
  if (t == 0) p.R0[0] = R0;
  const T ca = (T)p.a;
  const bool diag = p.b0 != 0.0 || p.b1 != 0.0;
  double Bj = 0.0;
  for (int j = 0; j < K; ++j) {
    __syncthreads();  // sV holds V_j
    gather_long<T, 1, NT>(g, sV, sL);
    T w[R];
    double d[3] = {0.0, 0.0, 0.0};  // V_{j-1} . W, V_j . W, W . W
    const bool two = j > 0 && p.reorth >= 1;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      T acc[1];
      if (re[q] - rs[q] > SMALL_LONG)
        acc[0] = sL[t + q * NT];
      else
        gather_lds<T, 1>(g.ci, rs[q], re[q], 0, 1, sV, acc);
      T y = ca * acc[0];
      if (diag) y += dg[q] * v[q];
      if (j > 0) y -= vp[q] * (T)Bj;
      w[q] = t + q * NT < n ? y : T(0);
      d[0] += (double)vp[q] * (double)w[q];
      d[1] += (double)v[q] * (double)w[q];
      d[2] += (double)w[q] * (double)w[q];
    }
    block_sums<NT, 3>(d, red, 0);
    const T c1 = two ? (T)(-d[0]) : T(0), c2 = (T)(-d[1]);
    s = 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      T y = two ? vp[q] * c1 : T(0);
      y += v[q] * c2;
      w[q] = y + w[q];
      s += (double)w[q] * (double)w[q];
    }
    s = total(s, 1);
    r1 = s > p.tol * s && s > 0.0 ? sqrt(s) : 0.0;
    f = r1 > 0.0 ? (T)(1.0 / r1) : T(0);
    if (d[2] > 0.0 && r1 <= p.post * sqrt(d[2])) {
      r1 = 0.0;
      f = T(0);
    }
    Bj = r1;
    if (t == 0) {
      sA[j] = d[1];
      sB[j] = r1;
    }
    if (j + 1 == K) break;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = t + q * NT;
      vp[q] = v[q];
      v[q] = w[q] * f;
      if (r < n) p.basis[(int64_t)(j + 1) * n + r] = sV[r] = v[q];
    }
  }
  __syncthreads();
  for (int j = t; j < K; j += NT) {
    p.A[j] = sA[j];
    p.Bo[j] = sB[j];
  }
  if (t == 0) {
    // T F = scale E_1 R0 by elimination; rows of T that are exactly zero get a unit diagonal
    bool ok = p.scale > 0.0;
    double y = p.scale * R0, bp = 0.0, ip = 0.0;
    for (int j = 0; j < K && ok; ++j) {
      const double bj = j + 1 < K ? sB[j] : 0.0;
      double d = sA[j];
      if (d == 0.0 && bp == 0.0 && bj == 0.0) d = 1.0;
      const double l = bp * ip;
      if (j > 0) {
        d -= l * bp;
        y = -l * y;
      }
      ok = d > 0.0;
      ip = 1.0 / d;
      sD[j] = ip;
      sF[j] = y;
      bp = bj;
    }
    double x = 0.0;
    for (int j = K - 1; j >= 0 && ok; --j) {
      x = (sF[j] - (j + 1 < K ? sB[j] * x : 0.0)) * sD[j];
      sF[j] = x;
    }
    good = ok ? 1 : 0;
    *p.done = good;
    __threadfence_system();
  }
  __syncthreads();
  if (!good) return;
  T y[R];
#pragma unroll
  for (int q = 0; q < R; ++q) y[q] = T(0);
#pragma unroll 4
  for (int j = 0; j < K; ++j) {
    const T c = (T)sF[j];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = min(t + q * NT, n - 1);
      y[q] += p.basis[(int64_t)j * n + r] * c;
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int r = t + q * NT;
    if (r < n) p.Y[r] = p.wv ? p.wv[r] * p.Xw[r] - y[q] : y[q];
  }
}

// One step of the fully reorthogonalised process for a vector W made by another operator (the
// general driver's steps in one launch): W -= V_{j-1} B_{j-1}, A_j = V_j . W, W -= V_j A_j, a second
// pass against V_lo .. V_j, normalised twice with the post-check into V_{j+1}.
template <typename T>
struct OrthArgs {
  int n, j, lo, last;
  T* basis;  // slot 0
  const T* W;
  double *A, *Bo;
  double tol, post;
};

template <typename T, int R, int NT>
__global__ __launch_bounds__(NT) void k_vec_orth(OrthArgs<T> p) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* sW = reinterpret_cast<T*>(smem);  // n
  __shared__ double red[2 * 3 * 16];
  __shared__ T sP[SMALL_K + 1];
  __shared__ double slast;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, n = p.n, j = p.j;
  auto total = [&](double x, int parity) {
    double a[1] = {x};
    block_sums<NT, 1>(a, red, parity);
    return a[0];
  };
  const T* Vj = p.basis + (int64_t)j * n;
  const double Bp = j > 0 ? p.Bo[j - 1] : 0.0;
  T v[R], w[R];
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int r = min(t + q * NT, n - 1);
    const bool in = t + q * NT < n;
    v[q] = Vj[r];
    w[q] = p.W[r];
    if (j > 0) w[q] -= Vj[r - n] * (T)Bp;
    if (!in) v[q] = w[q] = T(0);
    s += (double)v[q] * (double)w[q];
  }
  double A = total(s, 0);
#pragma unroll
  for (int q = 0; q < R; ++q) {
    w[q] -= v[q] * (T)A;
    if (t + q * NT < n) sW[t + q * NT] = w[q];
  }
  __syncthreads();
  const int nb = j - p.lo + 1;
  const T* Vlo = p.basis + (int64_t)p.lo * n;
  for (int k = wave; k < nb; k += NT / 64) {
    double d = 0.0;
#pragma unroll 4
    for (int r = lane; r < n; r += 64) d += (double)Vlo[(int64_t)k * n + r] * (double)sW[r];
    d = wave_total(d);
    if (lane == 0) {
      sP[k] = (T)d;
      if (k == nb - 1) slast = d;
    }
  }
  __syncthreads();
  A += slast;
  T acc[R];
#pragma unroll
  for (int q = 0; q < R; ++q) acc[q] = T(0);
#pragma unroll 4
  for (int k = 0; k < nb; ++k) {
    const T c = sP[k];
#pragma unroll
    for (int q = 0; q < R; ++q) acc[q] += Vlo[(int64_t)k * n + min(t + q * NT, n - 1)] * c;
  }
  s = 0.0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    w[q] = t + q * NT < n ? w[q] - acc[q] : T(0);
    s += (double)w[q] * (double)w[q];
  }
  s = total(s, 1);
  const double ref = fmax(s, A * A + Bp * Bp);
  const double r1 = s > p.tol * ref && s > 0.0 ? sqrt(s) : 0.0;
  if (t == 0) p.A[j] = A;
  if (p.last) {
    if (t == 0) p.Bo[j] = r1;
    return;
  }
  T f = r1 > 0.0 ? (T)(1.0 / r1) : T(0);
  s = 0.0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    w[q] *= f;
    s += (double)w[q] * (double)w[q];
  }
  s = total(s, 0);
  const double r2 = s > p.tol * s && s > 0.0 ? sqrt(s) : 0.0;
  double B = r2 * r1;
  f = r2 > 0.0 ? (T)(1.0 / r2) : T(0);
  if (ref > 0.0 && B <= p.post * sqrt(ref)) {
    B = 0.0;
    f = T(0);
  }
  T* Vn = p.basis + (int64_t)(j + 1) * n;
#pragma unroll
  for (int q = 0; q < R; ++q)
    if (t + q * NT < n) Vn[t + q * NT] = w[q] * f;
  if (t == 0) p.Bo[j] = B;
}

// Small matrices of a block step in LDS.
struct SmallMats {
  double P[3 * SMALL_B * SMALL_B];
  double G[16], R1[16], Ri[16], B[16];
  double ref;
  int ok;
};

// A block of B columns.  V_j and the graph are in LDS, the blocks in memory (this CU's L2).
template <typename T, int B>
__global__ __launch_bounds__(SMALL_T) void k_small_lanczos(SmallArgs<T> p) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[SMALL_W * 256];
  __shared__ SmallMats m;
  __shared__ T sC[3 * B * B];
  constexpr int bb = B * B;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int n = p.n;
  const int64_t blk = (int64_t)n * B;
  const LdsGraph g = stage_graph<SMALL_T>(smem, n, p.rowptr, p.colidx);
  T* sV = reinterpret_cast<T*>(smem + lds_graph_bytes(n, g.rp[n]));  // n x B
  T* sL = sV + blk;                                                  // sums of the long rows
  T* basis = p.basis;
  // w times m.Ri into v and, for the next product, into LDS
  auto normalise = [&](const T* w, T* v) {
    for (int r = t; r < n; r += SMALL_T) {
      T x[B];
#pragma unroll
      for (int i = 0; i < B; ++i) x[i] = w[(int64_t)r * B + i];
#pragma unroll
      for (int c = 0; c < B; ++c) {
        T o = T(0);
#pragma unroll
        for (int i = 0; i < B; ++i) o += x[i] * (T)m.Ri[i * B + c];
        v[(int64_t)r * B + c] = sV[r * B + c] = o;
      }
    }
    __syncthreads();
  };
  // V_0 R0 = X by CholQR2
  small_gram<T>(n, B, p.X, 0, 1, p.X, red, m.G);
  if (wave == 0) {
    const double ref = small_maxdiag(B, m.G);
    small_chol(B, m.G, p.tol * ref, m.Ri, nullptr, m.R1, 0.0, 0.0, 0.0);
    if (lane == 0) m.ref = ref;
  }
  __syncthreads();
  normalise(p.X, basis);
  small_gram<T>(n, B, basis, 0, 1, basis, red, m.G);
  if (wave == 0) small_chol(B, m.G, p.tol * small_maxdiag(B, m.G), m.Ri, m.R1, m.B, m.ref, p.post, 0.0);
  __syncthreads();
  if (t < bb) p.R0[t] = m.B[t];
  normalise(basis, basis);
  const T ca = (T)p.a;
  const bool diag = p.b0 != 0.0 || p.b1 != 0.0;
  for (int j = 0; j < p.K; ++j) {
    const T* Vj = basis + j * blk;
    const T* Vp = j > 0 ? Vj - blk : nullptr;
    T* Wn = basis + (j + 1) * blk;
    gather_long<T, B, SMALL_T>(g, sV, sL);
    // product, diagonal term and three-term subtraction (m.B holds B_{j-1})
    for (int r = t; r < n; r += SMALL_T) {
      const int s = g.rp[r], e = g.rp[r + 1];
      T x[B], acc[B];
#pragma unroll
      for (int i = 0; i < B; ++i) x[i] = Vp ? Vp[(int64_t)r * B + i] : T(0);
      if (e - s > SMALL_LONG) {
#pragma unroll
        for (int c = 0; c < B; ++c) acc[c] = sL[r * B + c];
      } else {
        gather_lds<T, B>(g.ci, s, e, 0, 1, sV, acc);
      }
      const T dg = (T)(p.b0 + p.b1 * (double)(e - s));
#pragma unroll
      for (int c = 0; c < B; ++c) {
        T y = ca * acc[c];
        if (diag) y += dg * sV[r * B + c];
        if (Vp) {
#pragma unroll
          for (int i = 0; i < B; ++i) y -= x[i] * (T)m.B[c * B + i];
        }
        Wn[(int64_t)r * B + c] = y;
      }
    }
    __syncthreads();
    // projection against V_j (reorth 0), or against V_{j-1} too
    const int nbv = j > 0 && p.reorth >= 1 ? 2 : 1;
    const T* Vlo = nbv == 2 ? Vp : Vj;
    small_gram<T>(n, B, Vlo, blk, nbv + 1, Wn, red, m.P);
    if (wave == 0) {
      const double ref = small_maxdiag(B, m.P + nbv * bb);
      if (lane == 0) m.ref = ref;
    }
    if (t < bb) {
      const int i = t / B, c = t - i * B;
      const double* Aj = m.P + (nbv - 1) * bb;
      const double av = 0.5 * (Aj[i * B + c] + Aj[c * B + i]);
      p.A[(int64_t)j * bb + t] = av;
      if (nbv == 2) sC[t] = (T)(-m.P[t]);
      sC[(nbv - 1) * bb + t] = (T)(-av);
    }
    __syncthreads();
    for (int r = t; r < n; r += SMALL_T) {
      T acc[B];
#pragma unroll
      for (int c = 0; c < B; ++c) acc[c] = T(0);
      for (int k = 0; k < nbv; ++k) {
        const T* xr = Vlo + k * blk + (int64_t)r * B;
        T x[B];
#pragma unroll
        for (int i = 0; i < B; ++i) x[i] = xr[i];
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
          for (int c = 0; c < B; ++c) acc[c] += x[i] * sC[k * bb + i * B + c];
      }
#pragma unroll
      for (int c = 0; c < B; ++c) Wn[(int64_t)r * B + c] = acc[c] + Wn[(int64_t)r * B + c];
    }
    __syncthreads();
    small_gram<T>(n, B, Wn, 0, 1, Wn, red, m.G);
    if (wave == 0) {
      const bool ok = small_chol(B, m.G, p.tol * small_maxdiag(B, m.G), m.Ri, nullptr, m.R1, m.ref, p.post, p.ratio);
      if (lane == 0) m.ok = ok ? 1 : 0;
    }
    __syncthreads();
    if (j + 1 == p.K) {
      if (t < bb) p.Bo[(int64_t)j * bb + t] = m.R1[t];
      break;
    }
    normalise(Wn, Wn);
    if (!m.ok) {  // the second CholQR pass
      small_gram<T>(n, B, Wn, 0, 1, Wn, red, m.G);
      if (wave == 0) small_chol(B, m.G, p.tol * small_maxdiag(B, m.G), m.Ri, m.R1, m.B, 0.0, 0.0, 0.0);
      __syncthreads();
      normalise(Wn, Wn);
    } else {
      if (t < bb) m.B[t] = m.R1[t];
      __syncthreads();
    }
    if (t < bb) p.Bo[(int64_t)j * bb + t] = m.B[t];
  }
  __syncthreads();
  if (wave == 0) {
    const bool good = p.scale > 0.0 && small_solve(B, p.K, p.A, p.Bo, p.R0, p.scale, p.work, p.F);
    if (lane == 0) {
      *p.done = good ? 1 : 0;
      __threadfence_system();
    }
  }
}

// The truncated series for column blockIdx.x, with the recurrence and running sum of the general
// path: P_k = s A P_{k-1} + s^2 mu (mu - D) P_{k-2} (no mu^2 term at k = 2), S += omega_k P_k,
// finished into w (.) Xw - S where wv is given.  P_{k-2} and S are in registers.
template <typename T>
struct SeriesArgs {
  int n, b, K;
  const int32_t *rowptr, *colidx;
  double s, mu, ratio;  // ratio > 0: omega_k = ratio^k / k!, else 1
  const T *X, *wv, *Xw;
  T* Y;
};

template <typename T, int R>
__global__ __launch_bounds__(SMALL_T) void k_small_series(SeriesArgs<T> p) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = p.n, b = p.b, col = blockIdx.x, t = threadIdx.x;
  const LdsGraph g = stage_graph<SMALL_T>(smem, n, p.rowptr, p.colidx);
  T* src = reinterpret_cast<T*>(smem + lds_graph_bytes(n, g.rp[n]));  // P_{k-1}
  T* dst = src + n;                                                   // P_k
  T* sL = dst + n;                                                    // sums of the long rows
  int rs[R], re[R];
  T p0[R], p1[R], S[R];
  const T a = (T)p.s;
  const double c1 = -p.s * p.s * p.mu, c0 = p.s * p.s * p.mu * p.mu;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int r = t + q * SMALL_T;
    rs[q] = r < n ? g.rp[r] : 0;
    re[q] = r < n ? g.rp[r + 1] : 0;
    p0[q] = T(0);
    p1[q] = S[q] = r < n ? p.X[(int64_t)r * b + col] : T(0);
    if (r < n) src[r] = p1[q];
  }
  __syncthreads();
  double omega = 1.0;
  for (int k = 1; k <= p.K; ++k) {
    if (p.ratio > 0.0) omega *= p.ratio / k;
    const T w = (T)omega;
    gather_long<T, 1, SMALL_T>(g, src, sL);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = t + q * SMALL_T;
      T acc[1];
      if (re[q] - rs[q] > SMALL_LONG)
        acc[0] = sL[t + q * SMALL_T];
      else
        gather_lds<T, 1>(g.ci, rs[q], re[q], 0, 1, src, acc);
      T y = a * acc[0];
      if (k >= 2 && p.mu != 0.0) y += (T)((k == 2 ? 0.0 : c0) + c1 * (double)(re[q] - rs[q])) * p0[q];
      p0[q] = p1[q];
      p1[q] = y;
      S[q] += w * y;
      if (r < n) dst[r] = y;
    }
    __syncthreads();
    T* h = src;
    src = dst;
    dst = h;
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int r = t + q * SMALL_T;
    const int64_t o = (int64_t)r * b + col;
    if (r < n) p.Y[o] = p.wv ? p.wv[r] * p.Xw[o] - S[q] : S[q];
  }
}

// LDS of a staged graph and `vectors` vectors of n values, and whether 16-bit indices hold it.
size_t small_lds(const wl_graph* g, size_t es, int vectors) {
  return lds_graph_bytes(g->n, g->nnz) + (size_t)vectors * g->n * es;
}
bool small_graph(const wl_graph* g, size_t es, int vectors, size_t most) {
  return g->n >= 1 && g->n <= 4 * SMALL_T && g->nnz < 65536 && small_lds(g, es, vectors) <= most &&
         !g->ctx->profiling;
}

// (rows per thread, threads) of the single-vector kernels: two rows each before the waves grow
// beyond 8, because barriers and reductions cost by the wave and gathers want many of them
// (40 steps FP64, us, 8 / 4 waves: Erdos-Renyi 1000 nodes 159 / 189, Barabasi-Albert 1000 nodes
// 236 / 318).
template <typename F>
void small_rows(int64_t n, F f) {
  if (n <= 256)
    f(std::integral_constant<int, 1>(), std::integral_constant<int, 256>());
  else if (n <= 512)
    f(std::integral_constant<int, 1>(), std::integral_constant<int, 512>());
  else if (n <= 1024)
    f(std::integral_constant<int, 2>(), std::integral_constant<int, 512>());
  else if (n <= 2048)
    f(std::integral_constant<int, 2>(), std::integral_constant<int, 1024>());
  else
    f(std::integral_constant<int, 4>(), std::integral_constant<int, 1024>());
}

}  // namespace

// One column: up to 4096 nodes whose graph (16-bit indices) and vectors fit the LDS (40 steps,
// FP64, Erdos-Renyi 300 / 1000 / 4000 nodes 115 / 159 / 366 us against 1.4 to 1.6 ms of launches).  Two
// to four columns keep their blocks in memory and stop at 5000 values (2 columns of 2000 nodes
// 0.98 ms against 1.4 to 1.7; 4 of 1000 0.80).  Kernel statistics count products per launch, so
// profiling keeps the general path.  A row of more than SMALL_LONG neighbours is a wave's task of
// 0.7 us (one column), which 16 waves share; they may take about 20 us of a step for one column and
// 12 for blocks, whose rows take 0.45 (FP32) or 0.7 us (FP64) a column (30 steps, ms, small / general:
// 1000 nodes of degree 40, one column FP32 1.44 / 1.19; 500 of degree 50, one 0.83 / 1.21, four
// FP64 2.79 / 1.31).
bool small_lanczos_ok(const wl_graph* g, int prec, int b, int K, int reorth) {
  const size_t es = prec == WL_FP32 ? 4 : 8;
  if (g->ctx->h_flag == nullptr || reorth > 1) return false;
  if (b == 1) return K <= SMALL_K && g->small_long <= (es == 4 ? 500 : 400) && small_graph(g, es, 2, 148 * 1024);
  if (g->small_long * b * es > 1600) return false;
  return b <= SMALL_B && g->n * b <= SMALL_BLOCK_VALUES && small_graph(g, es, 2 * b, 120 * 1024);
}

template <typename T>
wl_status launch_small_lanczos(wl_graph* g, double a, double b0, double b1, const T* X, int b, int K, int reorth,
                               T* basis, double* S, double scale, double* F, const T* wv, const T* Xw, T* Y) {
  SmallLayout Ly{b, K, (size_t)b * b};
  SmallArgs<T> p;
  p.n = (int)g->n;
  p.b = b;
  p.K = K;
  p.reorth = reorth;
  p.rowptr = g->rowptr;
  p.colidx = g->colidx;
  p.a = a;
  p.b0 = b0;
  p.b1 = b1;
  p.X = X;
  p.basis = basis;
  p.A = S + Ly.A(0);
  p.Bo = S + Ly.B(0);
  p.R0 = S + Ly.R0();
  p.tol = defl_tol<T>();
  p.post = post_tol<T>();
  p.ratio = skip_ratio<T>();
  p.scale = scale;
  p.work = S + Ly.P();
  p.F = F;
  p.wv = wv;
  p.Xw = Xw;
  p.Y = Y;
  p.done = g->ctx->h_flag;
  *g->ctx->h_flag = 0;
  hipStream_t st = g->ctx->stream;
  const size_t lds = small_lds(g, sizeof(T), 2 * b);
  if (b == 1)
    small_rows(g->n, [&](auto r, auto nt) {
      hipLaunchKernelGGL((k_vec_lanczos<T, decltype(r)::value, decltype(nt)::value>), dim3(1),
                         dim3(decltype(nt)::value), lds, st, p);
    });
  else if (b == 2)
    hipLaunchKernelGGL((k_small_lanczos<T, 2>), dim3(1), dim3(SMALL_T), lds, st, p);
  else if (b == 3)
    hipLaunchKernelGGL((k_small_lanczos<T, 3>), dim3(1), dim3(SMALL_T), lds, st, p);
  else
    hipLaunchKernelGGL((k_small_lanczos<T, 4>), dim3(1), dim3(SMALL_T), lds, st, p);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

// One orthogonalisation step of a single vector: up to 4096 rows, and a basis that one CU reads
// twice in less than the step's 16 launches take (2 MiB at 64 bytes per cycle: 14 us).
bool small_orth_ok(const wl_graph* g, int prec, int b, int K) {
  const int64_t es = prec == WL_FP32 ? 4 : 8;
  return b == 1 && K < SMALL_K && g->n >= 1 && g->n <= 4 * SMALL_T && (K + 1) * g->n * es <= (2 << 20) &&
         !g->ctx->profiling;
}

template <typename T>
wl_status launch_small_orth(wl_graph* g, int K, int j, int lo, T* basis, const T* W, double* S) {
  SmallLayout Ly{1, K, 1};
  OrthArgs<T> p;
  p.n = (int)g->n;
  p.j = j;
  p.lo = lo;
  p.last = j + 1 == K;
  p.basis = basis;
  p.W = W;
  p.A = S + Ly.A(0);
  p.Bo = S + Ly.B(0);
  p.tol = defl_tol<T>();
  p.post = post_tol<T>();
  small_rows(g->n, [&](auto r, auto nt) {
    hipLaunchKernelGGL((k_vec_orth<T, decltype(r)::value, decltype(nt)::value>), dim3(1), dim3(decltype(nt)::value),
                       (size_t)g->n * sizeof(T), g->ctx->stream, p);
  });
  WL_HIP(hipGetLastError());
  return WL_OK;
}

// One workgroup per column, graph and three vectors in LDS; a step costs about 0.15 ns per entry
// against 3.4 us for a launch of the general kernel (40 steps, FP64: Erdos-Renyi 1000 nodes of degree
// 8, 74 us against 136; 2000 nodes, 130 against 136; Barabasi-Albert 1000 nodes of degree 10, 133 against
// 162; 2500 nodes, 290 against 185).  Rows of more than SMALL_LONG neighbours cost more: up to 80 of them
// in FP32, 40 in FP64 (30 steps, us: 100 nodes, 94 such rows, FP64 178 against 151; 300 nodes of degree
// 40 403 against 139; 500 nodes, 29 such rows, 130 against 137).
bool small_series_ok(const wl_graph* g, int prec, int K) {
  const size_t es = prec == WL_FP32 ? 4 : 8;
  return K >= 2 && g->n <= 2 * SMALL_T && g->nnz <= 12000 && g->small_long * es <= 320 &&
         small_graph(g, es, 3, 150 * 1024);
}

template <typename T>
wl_status launch_small_series(wl_graph* g, double s, double mu, double ratio, int K, const T* X, T* Y, int b,
                              const T* wv, const T* Xw) {
  SeriesArgs<T> p;
  p.n = (int)g->n;
  p.b = b;
  p.K = K;
  p.rowptr = g->rowptr;
  p.colidx = g->colidx;
  p.s = s;
  p.mu = mu;
  p.ratio = ratio;
  p.X = X;
  p.wv = wv;
  p.Xw = Xw;
  p.Y = Y;
  const size_t lds = small_lds(g, sizeof(T), 3);
  if (g->n <= SMALL_T)
    hipLaunchKernelGGL((k_small_series<T, 1>), dim3(b), dim3(SMALL_T), lds, g->ctx->stream, p);
  else
    hipLaunchKernelGGL((k_small_series<T, 2>), dim3(b), dim3(SMALL_T), lds, g->ctx->stream, p);
  WL_HIP(hipGetLastError());
  return WL_OK;
}

#define WL_INST_SMALL(T)                                                                                          \
  template wl_status launch_small_lanczos<T>(wl_graph*, double, double, double, const T*, int, int, int, T*,      \
                                             double*, double, double*, const T*, const T*, T*);                  \
  template wl_status launch_small_orth<T>(wl_graph*, int, int, int, T*, const T*, double*);                      \
  template wl_status launch_small_series<T>(wl_graph*, double, double, double, int, const T*, T*, int, const T*,  \
                                            const T*);
WL_INST_SMALL(float)
WL_INST_SMALL(double)
