// Adjoint of the LM step through the stored factor (not in the paper; the derivation
// differentiates the paper's Eq. 1, (J^T J + lam D^2) p = J^T b):
//   M dp = dJ^T r + J^T db - J^T dJ p - dlam D^2 p - 2 lam D dD p,   r = b - J p,
// so for a loss with g = dL/dp and u = M^{-1} g = (R^T R)^{-1} g (two triangular solves):
//   dL/db = J u,  dL/dJ_ab = r_a u_b - (J u)_a p_b,  dL/dlam = -u^T D^2 p,
//   dL/dd_j = -2 lam u_j d_j p_j.
// The triangular solves run through the structured R of Section 4.2 exactly as in the
// refinement; this file holds the pieces that differ: the forward pass over the blocks
// with a given g, the row pass that writes the gradients on the structural nonzeros, and
// the vector terms.
#include "qrk_batch.hpp"
#include "qrk_device.hpp"
#include "qrk_launch.hpp"
#include "row_stream.hpp"

namespace qrk {

// y_i = R_i^{-T} g_i and per-workgroup partials of -sum_i S_i^T y_i (row stride kMaxDense).  A wave
// takes units of at most 64 / N consecutive blocks, fewer where there are too few blocks for the
// waves: lane k solves with block k while the unit's coupling rows (contiguous) are on their way,
// then the rows are streamed with a lane per column (RowStream).  One wave per block, as before,
// waited for three memory latencies per block: 10,000 blocks with 60 columns 14.0 -> 5.4 us.
template <typename T, int N, int CW>
__device__ __forceinline__ void adj_fwd_units(int64_t K, int nB, const T* __restrict__ Rblk,
                                              const T* __restrict__ Sc, const double* __restrict__ g,
                                              double* __restrict__ y, double* yv, int wv, int lane, double& t0,
                                              double& t1) {
  using S = RowStream<T, CW>;
  const int L = nB + 1;
  const int rg = lane / S::LN;
  const int64_t waves = (int64_t)gridDim.x * 4;
  const int64_t even = (K + waves - 1) / waves;
  constexpr int UMIN = 16 / N > 0 ? 16 / N : 1, UMAX = 64 / N;
  const int unit = even < UMIN ? UMIN : (even > UMAX ? UMAX : (int)even);
  for (int64_t b0 = ((int64_t)blockIdx.x * 4 + wv) * unit; b0 < K; b0 += waves * unit) {
    const int nb = K - b0 < unit ? (int)(K - b0) : unit;
    const int rows = nb * N;
    const __amdgpu_buffer_rsrc_t rsS =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(Sc + b0 * N * L), 0, 0x7fffffff, 0x00020000);
    StreamChunk<T, CW> va, vb;
    stream_load<T, CW>(va, rsS, 0, rows, L, nB, lane);
    const int64_t blk = b0 + (lane < nb ? lane : nb - 1);
    T Rb[N * N];
#pragma unroll
    for (int e = 0; e < N * N; ++e) Rb[e] = Rblk[blk * (N * N) + e];
    double yy[N];
#pragma unroll
    for (int i = 0; i < N; ++i) yy[i] = g[blk * N + i];
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int j = 0; j < i; ++j) yy[i] -= (double)Rb[j * N + i] * yy[j];
      yy[i] = yy[i] / (double)Rb[i * N + i];
    }
    if (lane < nb) {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        y[blk * N + c] = yy[c];
        yv[lane * N + c] = yy[c];
      }
    }
    yv[rows + lane] = 0.0;
    wave_lds_sync();
    auto coupling = [&](const StreamChunk<T, CW>& v, int s0) {
#pragma unroll
      for (int i = 0; i < S::NV; ++i) {
        const double yc = yv[s0 + i * S::RPL + rg];
        t0 -= (double)v[0][i] * yc;
        if constexpr (S::SL == 2) t1 -= (double)v[1][i] * yc;
      }
    };
    for (int s0 = 0;;) {
      if (s0 + S::CHR < rows) stream_load<T, CW>(vb, rsS, s0 + S::CHR, rows, L, nB, lane);
      coupling(va, s0);
      if ((s0 += S::CHR) >= rows) break;
      if (s0 + S::CHR < rows) stream_load<T, CW>(va, rsS, s0 + S::CHR, rows, L, nB, lane);
      coupling(vb, s0);
      if ((s0 += S::CHR) >= rows) break;
    }
    wave_lds_sync();  // the next unit overwrites yv
  }
}

template <typename T, int N>
__global__ void __launch_bounds__(256)
k_adj_fwd_blocks(int64_t K, int nB, const T* __restrict__ Rblk, const T* __restrict__ Sc,
                 const double* __restrict__ g, double* __restrict__ y, double* __restrict__ part) {
  __shared__ double yv_all[4][128];  // a unit's rows, zeros past them
  __shared__ double red[4][kMaxDense];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  double t0 = 0.0, t1 = 0.0;
  int rowstep = 64;
  stream_width(nB, [&](auto C) {
    constexpr int CW = decltype(C)::value;
    rowstep = RowStream<T, CW>::LN;
    adj_fwd_units<T, N, CW>(K, nB, Rblk, Sc, g, y, yv_all[wv], wv, lane, t0, t1);
  });
  red[wv][lane] = t0;
  red[wv][lane + 64] = t1;
  __syncthreads();
  for (int j = threadIdx.x; j < nB; j += blockDim.x) {
    double sum = 0.0;
    for (int w = 0; w < 4; ++w)
      for (int o = j; o < (j < 64 ? 64 : kMaxDense); o += rowstep) sum += red[w][o];
    part[(int64_t)blockIdx.x * kMaxDense + j] = sum;
  }
}

template <typename T>
hipError_t launch_adjoint_fwd_blocks(int64_t K, int n, int nB, const T* Rblk, const T* Sc, const double* g,
                                     double* y, double* part, int grid, hipStream_t st) {
  if (nB > 127) return hipErrorInvalidValue;
  switch (n) {
#define QRK_AF(NN)                                                                                              \
  case NN:                                                                                                     \
    hipLaunchKernelGGL((k_adj_fwd_blocks<T, NN>), dim3(grid), dim3(256), 0, st, K, nB, Rblk, Sc, g, y, part);   \
    break;
    QRK_AF(1) QRK_AF(2) QRK_AF(3) QRK_AF(4) QRK_AF(5) QRK_AF(6) QRK_AF(7) QRK_AF(8)
#undef QRK_AF
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// One wave per pack of whole blocks (at most 64 rows): r = b - J p and Ju = J u per row, dA = r u_i^T
// - Ju p_i^T and db = Ju with a lane per row, dB = r u_B^T - Ju p_B^T with a lane per column.  The
// pack's rows of B are streamed once (RowStream, the next chunk in flight): both row sums are folded
// from the same registers, and a chunk's rows of dB are written as soon as its r and Ju are known.
// Before, each lane walked its own row of B: a column of 64 rows per load, nB loads one after the
// other (120,000 rows of 60 columns 21.7 -> 17.6 us; B in and dB out alone take 12).
template <int N>
struct AdjRowsLds {
  double pv[64 * N], uv[64 * N];  // p_i and u_i of the pack's blocks
  double r[64], ju[64];           // first without, then with the dense part
};

template <typename T, int N, int CW>
__device__ __forceinline__ void adj_rows_packs(int64_t npacks, const int64_t* __restrict__ pack_blk, int nB,
                                               const int64_t* __restrict__ row_off, const T* __restrict__ A,
                                               const T* __restrict__ B, int64_t ldb, const T* __restrict__ bvec,
                                               const double* __restrict__ p, const double* __restrict__ u,
                                               int64_t Kn, T* __restrict__ dA, T* __restrict__ dB,
                                               T* __restrict__ db, AdjRowsLds<N>& lds, int wv, int lane) {
  using S = RowStream<T, CW>;
  const int rg = lane / S::LN, col = lane & (S::LN - 1);
  // with nB == 0 any unknown stands in for the dense part's (weight 0)
  const int64_t e0 = col < nB ? Kn + col : 0, e1 = col + 64 < nB ? Kn + col + 64 : 0;
  const double p0 = col < nB ? p[e0] : 0.0, u0 = col < nB ? u[e0] : 0.0;
  const double p1 = col + 64 < nB ? p[e1] : 0.0, u1 = col + 64 < nB ? u[e1] : 0.0;
  const int64_t waves = (int64_t)gridDim.x * 4;
  for (int64_t pk = (int64_t)blockIdx.x * 4 + wv; pk < npacks; pk += waves) {
    const int64_t b0 = pack_blk[pk];
    const int nb = (int)(pack_blk[pk + 1] - b0);
    const int64_t pr0 = row_off[b0];
    const int prows = (int)(row_off[b0 + nb] - pr0);
    if (prows == 0) continue;  // blocks without rows
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(nB > 0 ? B + pr0 * ldb : bvec + pr0), 0, 0x7fffffff, 0x00020000);
    StreamChunk<T, CW> va, vb;
    stream_load<T, CW>(va, rsB, 0, prows, (int)ldb, nB, lane);
    const int64_t row = pr0 + (lane < prows ? lane : prows - 1);
    T arow[N];
#pragma unroll
    for (int c = 0; c < N; ++c) arow[c] = A[row * N + c];
    const T bval = bvec[row];
    const int64_t blk = b0 + (lane < nb ? lane : nb - 1);
    const int lo = (int)(row_off[blk] - pr0);
    double pp[N], uu[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
      pp[c] = p[blk * N + c];
      uu[c] = u[blk * N + c];
    }
    if (lane < nb) {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        lds.pv[lane * N + c] = pp[c];
        lds.uv[lane * N + c] = uu[c];
      }
    }
    int rb = 0;  // the block of this lane's row: the last one that starts at or before it
    for (int k = 1; k < nb; ++k) rb += lane >= __builtin_amdgcn_readlane(lo, k) ? 1 : 0;
    if (lane >= prows) rb = nb - 1;
    wave_lds_sync();
    double ap = 0.0, au = 0.0;
#pragma unroll
    for (int c = 0; c < N; ++c) {
      pp[c] = lds.pv[rb * N + c];  // from here on the row's block's
      uu[c] = lds.uv[rb * N + c];
      ap += (double)arow[c] * pp[c];
      au += (double)arow[c] * uu[c];
    }
    lds.r[lane] = (double)bval - ap;
    lds.ju[lane] = au;
    wave_lds_sync();
    auto work = [&](const StreamChunk<T, CW>& v, int c0) {
      const int sr = c0 + S::sum_row(lane);  // < 64
      const double bp = stream_dot<T, CW>(v, p0, p1, lane);
      const double bu = stream_dot<T, CW>(v, u0, u1, lane);
      const double rv = lds.r[sr] - bp, jv = lds.ju[sr] + bu;
      wave_lds_sync();  // every lane of a row has read it before it is replaced
      lds.r[sr] = rv;
      lds.ju[sr] = jv;
      wave_lds_sync();
      if (dB) {
#pragma unroll
        for (int i = 0; i < S::NV; ++i) {
          const int r = c0 + i * S::RPL + rg;
          const double rr = lds.r[r], jj = lds.ju[r];
          T* out = dB + (pr0 + r) * ldb;
          if (r < prows && col < nB) out[col] = (T)(rr * u0 - jj * p0);
          if constexpr (S::SL == 2)
            if (r < prows && col + 64 < nB) out[col + 64] = (T)(rr * u1 - jj * p1);
        }
      }
    };
    for (int c0 = 0;;) {
      if (c0 + S::CHR < prows) stream_load<T, CW>(vb, rsB, c0 + S::CHR, prows, (int)ldb, nB, lane);
      work(va, c0);
      if ((c0 += S::CHR) >= prows) break;
      if (c0 + S::CHR < prows) stream_load<T, CW>(va, rsB, c0 + S::CHR, prows, (int)ldb, nB, lane);
      work(vb, c0);
      if ((c0 += S::CHR) >= prows) break;
    }
    if (lane < prows) {
      const double rv = lds.r[lane], jv = lds.ju[lane];
      if (dA) {
#pragma unroll
        for (int c = 0; c < N; ++c) dA[row * N + c] = (T)(rv * uu[c] - jv * pp[c]);
      }
      if (db) db[row] = (T)jv;
    }
    wave_lds_sync();  // the next pack overwrites the wave's LDS
  }
}

template <typename T, int N>
__global__ void __launch_bounds__(256)
k_adj_rows(int64_t npacks, const int64_t* __restrict__ pack_blk, int nB, const int64_t* __restrict__ row_off,
           const T* __restrict__ A, const T* __restrict__ B, int64_t ldb, const T* __restrict__ bvec,
           const double* __restrict__ p, const double* __restrict__ u, int64_t Kn, T* __restrict__ dA,
           T* __restrict__ dB, T* __restrict__ db) {
  __shared__ AdjRowsLds<N> lds_all[4];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  stream_width(nB, [&](auto C) {
    adj_rows_packs<T, N, decltype(C)::value>(npacks, pack_blk, nB, row_off, A, B, ldb, bvec, p, u, Kn, dA, dB, db,
                                             lds_all[wv], wv, lane);
  });
}

template <typename T>
hipError_t launch_adjoint_rows(int64_t npacks, const int64_t* pack_blk, int64_t K, int n, int nB,
                               const int64_t* row_off, const T* A, const T* B, int64_t ldb, const T* b,
                               const double* p, const double* u, T* dA, T* dB, T* db, int grid,
                               hipStream_t st) {
  if (nB > 127) return hipErrorInvalidValue;
  switch (n) {
#define QRK_AR(NN)                                                                                                 \
  case NN:                                                                                                        \
    hipLaunchKernelGGL((k_adj_rows<T, NN>), dim3(grid), dim3(256), 0, st, npacks, pack_blk, nB, row_off, A, B, ldb, \
                       b, p, u, K * n, dA, dB, db);                                                               \
    break;
    QRK_AR(1) QRK_AR(2) QRK_AR(3) QRK_AR(4) QRK_AR(5) QRK_AR(6) QRK_AR(7) QRK_AR(8)
#undef QRK_AR
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// dd and per-workgroup partials of -u^T D^2 p for every problem (problem = blockIdx.y).
__global__ void __launch_bounds__(256)
k_adj_vec(int64_t N, const double* __restrict__ u, const double* __restrict__ d,
          const double* __restrict__ p, double lam, double* __restrict__ dd, double* __restrict__ part) {
  __shared__ double red[256];
  const int64_t prob = blockIdx.y;
  double s = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < N; j += (int64_t)gridDim.x * 256) {
    const int64_t e = prob * N + j;
    const double t = u[e] * d[e] * p[e];
    s -= t * d[e];
    if (dd) dd[e] = -2.0 * lam * t;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off >= 1; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[prob * gridDim.x + blockIdx.x] = red[0];
}

// Sum of a problem's partials by one wave: lane l adds partials l, l + 64, ... in order, then the
// lanes are added in a fixed tree (one thread adding all of them: 7.2 us for 120 partials, now 2.6).
__global__ void __launch_bounds__(64) k_adj_vec_final(int nparts, const double* __restrict__ part,
                                                      double* __restrict__ dlam) {
  const int prob = blockIdx.x;
  double s = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < nparts; i += 64) s += part[(int64_t)prob * nparts + i];
  s = wave_allreduce_sum(s);
  if (threadIdx.x == 0) dlam[prob] = s;
}

hipError_t launch_adjoint_vec(int P, int64_t N, const double* u, const double* d, const double* p,
                              double lam, double* dd, double* dlam, double* part, hipStream_t st) {
  int grid = (int)((N + 255) / 256);
  const int cap = P > 0 ? 1024 / P : 1;
  if (grid > cap) grid = cap > 0 ? cap : 1;
  hipLaunchKernelGGL(k_adj_vec, dim3(grid, P), dim3(256), 0, st, N, u, d, p, lam, dd, part);
  if (dlam) hipLaunchKernelGGL(k_adj_vec_final, dim3(P), dim3(64), 0, st, grid, part, dlam);
  return hipGetLastError();
}

#define QRK_AINST(T)                                                                                     \
  template hipError_t launch_adjoint_fwd_blocks<T>(int64_t, int, int, const T*, const T*, const double*,   \
                                                   double*, double*, int, hipStream_t);                   \
  template hipError_t launch_adjoint_rows<T>(int64_t, const int64_t*, int64_t, int, int, const int64_t*,   \
                                             const T*, const T*, int64_t, const T*, const double*,         \
                                             const double*, T*, T*, T*, int, hipStream_t);
QRK_AINST(float)
QRK_AINST(double)
#undef QRK_AINST

}  // namespace qrk
