// Banded J (the banded class of QRkit Section 4.4): row i of J holds w values at columns
// s_i .. s_i + w - 1 with s_i nondecreasing.  The QR of [J; sqrt(lam) D] is formed by
// Givens rotations (Section 2): R starts as the upper-triangular diag(sqrt(lam) d), and
// each row of J (with its b_i riding along as one more entry) is rotated into R in row
// order, one rotation per column of the row.  Because the starts are nondecreasing, the
// rows of R that a new row touches have no entries right of column s_i + w - 1, so R keeps
// upper bandwidth w - 1 and a w x w window of R (rows and columns s .. s + w - 1) is all
// that is live while row i is processed.
//
// This file holds the kernels shared by every width (J v, J^T r, adjoint entries), the dispatch
// (factor: banded_s.hpp; sweeps: banded_w.hpp up to w = 15, banded_s.hpp above), and run-time-width
// sweeps for the sizes that those do not take (offsets past 32 bits): one problem per 32 lanes.
// R is stored banded: row j holds R[j][j .. j + w - 1] (float or double), c is [N].
#include "qrk_device.hpp"
#include "qrk_banded.hpp"

namespace qrk {

template <int G, typename T>
__device__ __forceinline__ T gsum(T x) {
#pragma unroll
  for (int off = G / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, G);
  return x;
}

// lane l receives lane l - 1's value (the first lane keeps its own)
template <int G, typename T>
__device__ __forceinline__ T from_prev(T x) {
  return __shfl_up(x, 1, G);
}

// x = R^{-1} rhs for the banded R of every problem (backward sweep).
//   rhs: c (T, ADD = false, output set) or a float64 vector (ADD = true, output added).
template <typename T, int G, bool ADD>
__global__ void __launch_bounds__(256)
k_banded_bwd(int P, int64_t N, int w, const T* __restrict__ Rb, const T* __restrict__ cT,
             const double* __restrict__ rhs, double* __restrict__ out, int* __restrict__ status) {
  const int lane = threadIdx.x % G;
  const int64_t prob = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  if (prob >= P) return;
  const T* R = Rb + prob * N * w;
  double pw = 0.0;  // lane l holds x[j + l]
  double dmax = 0.0;
  bool bad = false, nonfinite = false;
  if (!ADD) {
    for (int64_t j = lane; j < N; j += G) dmax = fmax(dmax, fabs((double)R[j * w]));
    for (int off = G / 2; off >= 1; off >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, off, G));
  }
  for (int64_t j = N - 1; j >= 0; --j) {
    double part = (lane >= 1 && lane < w && j + lane < N) ? (double)R[j * w + lane] * pw : 0.0;
    part = gsum<G>(part);
    const double base = ADD ? rhs[prob * N + j] : (double)cT[prob * N + j];
    const double piv = (double)R[j * w];
    const double xj = (base - part) / piv;
    if (!ADD && is_finite(piv) && !(fabs(piv) > (double)N * Eps<T>::value * dmax)) bad = true;
    if (lane == 0) {
      if (ADD)
        out[prob * N + j] += xj;
      else
        out[prob * N + j] = xj;
      nonfinite |= !is_finite(xj);
    }
    if (lane == 0) pw = xj;
    pw = from_prev<G>(pw);
  }
  if (status) {
    if (bad) set_status(status, ST_SINGULAR);
    if (nonfinite) set_status(status, ST_NONFINITE);
  }
}

// y = R^{-T} g (forward sweep); g and y are float64 [P][N] (may alias).
template <typename T, int G>
__global__ void __launch_bounds__(256)
k_banded_fwd(int P, int64_t N, int w, const T* __restrict__ Rb, const double* g, double* y) {
  const int lane = threadIdx.x % G;
  const int64_t prob = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / G;
  if (prob >= P) return;
  const T* R = Rb + prob * N * w;
  double yw = 0.0;  // lane l holds y[j - l]
  for (int64_t j = 0; j < N; ++j) {
    double part = (lane >= 1 && lane < w && j - lane >= 0) ? (double)R[(j - lane) * w + lane] * yw : 0.0;
    part = gsum<G>(part);
    const double yj = (g[prob * N + j] - part) / (double)R[j * w];
    if (lane == 0) y[prob * N + j] = yj;
    if (lane == 0) yw = yj;
    yw = from_prev<G>(yw);
  }
}

// r = b - J v (float64), one row per lane: r [P][M].  With b == nullptr, r = J v.
template <typename T>
__global__ void __launch_bounds__(256)
k_banded_apply(int P, int64_t M, int64_t N, int w, const int32_t* __restrict__ row_start,
               const T* __restrict__ vals, const T* __restrict__ bvec, const double* __restrict__ v,
               double* __restrict__ r) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)P * M) return;
  const int64_t prob = t / M, i = t % M;
  int64_t si = row_start[prob * M + i];
  si = si < 0 ? 0 : (si > N - w ? N - w : si);
  const T* row = vals + (prob * M + i) * w;
  const double* vp = v + prob * N + si;
  double acc = 0.0;
  for (int l = 0; l < w; ++l) acc += (double)row[l] * vp[l];
  r[t] = bvec ? (double)bvec[t] - acc : acc;
}

// Row starts clamped to [0, N - w] (the same clamp as the factorisation's for valid input).
__device__ __forceinline__ int64_t band_start(const int32_t* rs, int64_t i, int64_t N, int w) {
  const int64_t s = rs[i];
  return s < 0 ? 0 : (s > N - w ? N - w : s);
}

// First-row table of every problem: fr[c] (c = 0 .. N) = the first row whose start is >= c,
// for nondecreasing starts.  Thread i (0 .. M) fills the columns after row i-1's start up to
// row i's start (thread M: up to N).  Starts out of order leave entries unset; the readers
// clamp what they read.
__global__ void __launch_bounds__(256)
k_band_first_row(int P, int64_t M, int64_t N, int w, const int32_t* __restrict__ row_start,
                 int32_t* __restrict__ fr) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)P * (M + 1)) return;
  const int64_t prob = t / (M + 1), i = t % (M + 1);
  const int32_t* rs = row_start + prob * M;
  int32_t* f = fr + prob * (N + 1);
  const int64_t c0 = i == 0 ? 0 : band_start(rs, i - 1, N, w) + 1;
  const int64_t c1 = i == M ? N : band_start(rs, i, N, w);
  for (int64_t c = c0; c <= c1; ++c) f[c] = (int32_t)i;
}

// g = J^T r - lam d^2 v (float64), TPC threads per column: column j of a problem collects the
// rows whose start lies in [j - w + 1, j], thread h of it rows h, h + TPC, ... of the range in order,
// and two threads' sums are added, so the result is deterministic.  The row ranges come from the
// first-row table.  A workgroup covers 256 / TPC consecutive columns of one problem: the starts,
// residuals and values of its rows (one contiguous range) are copied to LDS with coalesced
// loads, eight per thread in flight, and each column then reads only LDS; a range beyond the
// LDS capacity goes in chunks.  Bound by the loads in flight: with 256 columns and 53 KB of LDS a
// workgroup three fit a CU, with 128 five of twice the threads per column.  Two rows per column: 2,048
// problems of N = 2,048, w = 12 265 us with one thread, 207 with two.
//
// Columns of fewer than 8 values have no work for two threads, unless 256 columns a workgroup leave more of
// the last one empty (jt_thin).  Solves of two sweeps, one thread / two, one row per column: 2,000
// problems of N = 1,000 w = 1 394 / 410 us, w = 4 419 / 442, w = 7 454 / 463, w = 10 no difference; N = 300,
// w = 4 166 / 160.
inline bool jt_thin(int64_t M, int64_t N, int w) { return M * w < 8 * N && (N - 1) % 256 >= 128; }
template <typename T, int TPC>
__global__ void __launch_bounds__(256)
k_banded_jt(int P, int64_t M, int64_t N, int w, const int32_t* __restrict__ row_start, const int32_t* __restrict__ fr,
            const T* __restrict__ vals, const double* __restrict__ r, const double* __restrict__ d,
            const double* __restrict__ lamv, const double* __restrict__ v, double* __restrict__ g) {
  constexpr int COLS = 256 / TPC;
  constexpr int CAP = TPC == 1 ? 1024 : 576;                             // rows of a chunk
  constexpr int VCAP = (TPC == 1 ? 40960 : 24576) / (int)sizeof(T);      // and values
  __shared__ int32_t s_st[CAP];
  __shared__ double s_r[CAP];
  __shared__ T s_v[VCAP];
  const int64_t nb = (N + COLS - 1) / COLS;
  const int64_t wg = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;  // (a grid row holds fewer than 2^32 threads)
  const int64_t prob = wg / nb;
  if (prob >= P) return;
  const int64_t c0 = wg % nb * COLS;
  const int64_t j = c0 + threadIdx.x / TPC;
  const int half = threadIdx.x & (TPC - 1);
  const int32_t* rs = row_start + prob * M;
  const int32_t* f = fr + prob * (N + 1);
  const double* rp = r + prob * M;
  const T* V = vals + prob * M * w;
  auto entry = [&](int64_t c) -> int64_t { return f[c < 0 ? 0 : (c > N ? N : c)]; };
  auto clamp = [](int64_t i, int64_t lo, int64_t hi) -> int64_t { return i < lo ? lo : (i > hi ? hi : i); };
  const int64_t fa = entry(j - w + 1), fe = entry(j + 1);  // this column's rows, used when a chunk is staged
  const int64_t lo = clamp(entry(c0 - w + 1), 0, M);
  const int64_t hi = clamp(entry(c0 + COLS), lo, M);
  double acc = 0.0;
  const int64_t chunk = CAP < VCAP / w ? CAP : VCAP / w;
  for (int64_t cs = lo; cs < hi; cs += chunk) {
    const int64_t ce = cs + chunk < hi ? cs + chunk : hi;
    const int64_t n = ce - cs, nv = n * w;
    if (cs > lo) __syncthreads();  // every column is done with the chunk before
    const T* Vlo = V + cs * w;
    for (int64_t i0 = 0; i0 < nv; i0 += 256 * 8) {
      T buf[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t i = i0 + u * 256 + threadIdx.x;
        buf[u] = i < nv ? Vlo[i] : T(0);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t i = i0 + u * 256 + threadIdx.x;
        if (i < nv) s_v[i] = buf[u];
      }
    }
    for (int64_t i0 = 0; i0 < n; i0 += 256 * 4) {
      int32_t sb[4];
      double rb[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t i = i0 + u * 256 + threadIdx.x;
        sb[u] = i < n ? (int32_t)band_start(rs, cs + i, N, w) : 0;
        rb[u] = i < n ? rp[cs + i] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t i = i0 + u * 256 + threadIdx.x;
        if (i < n) {
          s_st[i] = sb[u];
          s_r[i] = rb[u];
        }
      }
    }
    __syncthreads();
    // this thread's rows of the chunk (every TPC-th one from a + half), a few per batch: their LDS reads
    // are independent, the sum keeps row order
    const int64_t a = clamp(fa, lo, hi), e = j < N ? clamp(fe, lo, hi) : a;
    const int64_t first = a + half, from = first < cs ? cs + ((cs - first) & (TPC - 1)) : first;
    const int i1 = (int)((e < ce ? e : ce) - cs);
    constexpr int U = 8 / TPC;
    for (int64_t ib = from - cs; ib < i1; ib += 8) {
      const int i0 = (int)ib;
      int kk[U];
      double rr[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + TPC * u < i1 ? i0 + TPC * u : i0;
        kk[u] = (int)(j - s_st[i]);
        rr[u] = s_r[i];
      }
      T vv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + TPC * u < i1 ? i0 + TPC * u : i0;
        const int k = kk[u] < 0 ? 0 : (kk[u] >= w ? w - 1 : kk[u]);
        vv[u] = s_v[i * w + k];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + TPC * u < i1 && kk[u] >= 0 && kk[u] < w) acc += (double)vv[u] * rr[u];
    }
  }
  if constexpr (TPC == 2) acc += __shfl_xor(acc, 1, kWave);
  if (half || j >= N) return;
  const int64_t t = prob * N + j;
  const double dj = d[t];
  g[t] = acc - lamv[prob] * dj * dj * v[t];
}

// Adjoint entries on the structural nonzeros: dvals[i][l] = r_i u_{s_i+l} - (J u)_i p_{s_i+l}.
template <typename T>
__global__ void __launch_bounds__(256)
k_banded_dvals(int P, int64_t M, int64_t N, int w, const int32_t* __restrict__ row_start,
               const double* __restrict__ r, const double* __restrict__ Ju, const double* __restrict__ u,
               const double* __restrict__ p, T* __restrict__ dvals) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)P * M * w) return;
  const int64_t row = t / w;
  const int l = (int)(t % w);
  const int64_t prob = row / M;
  int64_t si = row_start[row];
  si = si < 0 ? 0 : (si > N - w ? N - w : si);
  const int64_t col = prob * N + si + l;
  dvals[t] = (T)(r[row] * u[col] - Ju[row] * p[col]);
}

// ---------------------------------------------------------------------------------

template <typename T>
hipError_t launch_banded_givens(int P, int64_t M, int64_t N, int w, const int32_t* row_start,
                                const T* vals, const T* b, const double* d, const double* lam, T* Rb,
                                T* cb, double* binv, T* R16, int* status, hipStream_t st) {
  if (w < 1 || w > 31) return hipErrorInvalidValue;
  if (w <= 15)
    return launch_bgivens_s<T, 0>(P, M, N, w, row_start, vals, b, d, lam, Rb, cb, binv, R16, status, st);
  return launch_bgivens_s<T, 1>(P, M, N, w, row_start, vals, b, d, lam, Rb, cb, binv, nullptr, status, st);
}

template <typename T>
hipError_t launch_banded_backsub(int P, int64_t N, int w, const T* Rb, const T* R16, const double* binv, const T* cb,
                                 double* p, int* status, hipStream_t st) {
  if (R16) {
    return launch_bsweep_w<T>(0, P, N, w, R16, binv, cb, nullptr, p, status, st);
  } else if (bsweep_x_fits(N, w, sizeof(T))) {
    return launch_bsweep_x<T>(0, P, N, w, Rb, binv, cb, nullptr, p, status, st);
  } else {
    const int64_t threads = (int64_t)P * 32;
    hipLaunchKernelGGL((k_banded_bwd<T, 32, false>), dim3((threads + 255) / 256), dim3(256), 0, st, P, N, w,
                       Rb, cb, (const double*)nullptr, p, status);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_banded_solve_add(int P, int64_t N, int w, const T* Rb, const T* R16, const double* binv,
                                   const double* rhs, double* out, hipStream_t st) {
  if (R16) {
    return launch_bsweep_w<T>(1, P, N, w, R16, binv, nullptr, rhs, out, nullptr, st);
  } else if (bsweep_x_fits(N, w, sizeof(T))) {
    return launch_bsweep_x<T>(1, P, N, w, Rb, binv, nullptr, rhs, out, nullptr, st);
  } else {
    const int64_t threads = (int64_t)P * 32;
    hipLaunchKernelGGL((k_banded_bwd<T, 32, true>), dim3((threads + 255) / 256), dim3(256), 0, st, P, N, w,
                       Rb, (const T*)nullptr, rhs, out, (int*)nullptr);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_banded_fwd(int P, int64_t N, int w, const T* Rb, const T* R16, const double* binv, const double* g,
                             double* y, hipStream_t st) {
  if (R16) return launch_bsweep_w<T>(2, P, N, w, R16, binv, nullptr, g, y, nullptr, st);
  if (bsweep_x_fits(N, w, sizeof(T))) return launch_bsweep_x<T>(2, P, N, w, Rb, binv, nullptr, g, y, nullptr, st);
  const int64_t threads = (int64_t)P * 32;
  hipLaunchKernelGGL((k_banded_fwd<T, 32>), dim3((threads + 255) / 256), dim3(256), 0, st, P, N, w, Rb, g, y);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_banded_apply(int P, int64_t M, int64_t N, int w, const int32_t* row_start, const T* vals,
                               const T* b, const double* v, double* r, hipStream_t st) {
  const int64_t threads = (int64_t)P * M;
  if (threads == 0) return hipSuccess;
  if (w <= 15) return launch_bapply_w<T>(P, M, N, w, row_start, vals, b, v, r, st);
  hipLaunchKernelGGL((k_banded_apply<T>), dim3((threads + 255) / 256), dim3(256), 0, st, P, M, N, w, row_start,
                     vals, b, v, r);
  return hipGetLastError();
}

hipError_t launch_band_first_row(int P, int64_t M, int64_t N, int w, const int32_t* row_start, int32_t* fr,
                                 hipStream_t st) {
  const int64_t threads = (int64_t)P * (M + 1);
  hipLaunchKernelGGL(k_band_first_row, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, st, P, M, N, w,
                     row_start, fr);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_banded_jt(int P, int64_t M, int64_t N, int w, const int32_t* row_start, const int32_t* fr,
                            const T* vals, const double* r, const double* d, const double* lam, const double* v,
                            double* g, hipStream_t st) {
  const bool thin = jt_thin(M, N, w);
  const int cols = thin ? 256 : 128;
  const int64_t blocks = (int64_t)P * ((N + cols - 1) / cols);
  const int64_t gx = blocks < (1 << 22) ? blocks : 1 << 22;
  const dim3 grid((unsigned)gx, (unsigned)((blocks + gx - 1) / gx));
  if (thin)
    hipLaunchKernelGGL((k_banded_jt<T, 1>), grid, dim3(256), 0, st, P, M, N, w, row_start, fr, vals,
                       r, d, lam, v, g);
  else
    hipLaunchKernelGGL((k_banded_jt<T, 2>), grid, dim3(256), 0, st, P, M, N, w, row_start, fr, vals,
                       r, d, lam, v, g);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_banded_dvals(int P, int64_t M, int64_t N, int w, const int32_t* row_start, const double* r,
                               const double* Ju, const double* u, const double* p, T* dvals, hipStream_t st) {
  const int64_t threads = (int64_t)P * M * w;
  if (threads == 0) return hipSuccess;
  hipLaunchKernelGGL((k_banded_dvals<T>), dim3((threads + 255) / 256), dim3(256), 0, st, P, M, N, w, row_start,
                     r, Ju, u, p, dvals);
  return hipGetLastError();
}

#define QRK_BINST(T)                                                                                     \
  template hipError_t launch_banded_givens<T>(int, int64_t, int64_t, int, const int32_t*, const T*,        \
                                              const T*, const double*, const double*, T*, T*, double*, T*, int*, hipStream_t); \
  template hipError_t launch_banded_backsub<T>(int, int64_t, int, const T*, const T*, const double*, const T*, \
                                               double*, int*, hipStream_t);                               \
  template hipError_t launch_banded_solve_add<T>(int, int64_t, int, const T*, const T*, const double*,     \
                                                 const double*, double*, hipStream_t);                    \
  template hipError_t launch_banded_fwd<T>(int, int64_t, int, const T*, const T*, const double*,           \
                                           const double*, double*, hipStream_t);                          \
  template hipError_t launch_banded_apply<T>(int, int64_t, int64_t, int, const int32_t*, const T*,         \
                                             const T*, const double*, double*, hipStream_t);              \
  template hipError_t launch_banded_jt<T>(int, int64_t, int64_t, int, const int32_t*, const int32_t*, const T*, \
                                          const double*, const double*, const double*, const double*, double*, \
                                          hipStream_t);                                                   \
  template hipError_t launch_banded_dvals<T>(int, int64_t, int64_t, int, const int32_t*, const double*,    \
                                             const double*, const double*, const double*, T*, hipStream_t);
QRK_BINST(float)
QRK_BINST(double)
#undef QRK_BINST

}  // namespace qrk
