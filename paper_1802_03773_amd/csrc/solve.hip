// Back-substitution through the structured R of a horizontal concatenation
// (QRkit Section 4.2: R = [[blkdiag(R_i), S], [0, R_B]]) and corrected
// semi-normal-equation refinement of the step (Bjorck 1987):
//     r = b - J p,  g = J^T r - lam D^2 p   (float64),
//     R^T y = g,  R delta = y,  p <- p + delta.
// The two triangular solves run through the structure:
//     R_i^T y_i = g_i;   R_B^T y_B = g_B - sum_i S_i^T y_i;
//     R_B delta_B = y_B; R_i delta_i = y_i - S_i delta_B.
// Sums over blocks are deterministic: per-wave partials in registers, workgroup partials
// combined in a fixed order, then a fixed-order reduction of the workgroup partials.
// Every kernel serves a batch of independent problems (ProbDesc); a single problem is the
// batch of one.
#include "qrk_batch.hpp"
#include "qrk_device.hpp"
#include "qrk_launch.hpp"
#include "row_stream.hpp"

namespace qrk {

// ---------------------------------------------------------------------------------
// Dense triangle, one wave: forward (R_B^T y = g) and backward (R_B x = y) sweeps over the strict
// upper triangle of R_B, staged in LDS as doubles with an odd row stride.  Lane i holds rows i
// and i + 64 of the right-hand side.  NBP: nB rounded up to 32, 64, 96 or 128.
//
// A sweep is one chain of nB dependent steps, so its time is the latency of a step.  It goes by
// 16 x 16 blocks of the diagonal: the block's 16 right-hand sides, scaled by the reciprocal
// diagonal, sit in every 16-lane row of the wave, and a step is one FMA whose broadcast of the
// solved unknown is the instruction's own lane selection (a broadcast through scalar registers,
// a multiply and an FMA per step before).  The other rows then take the 16 solved unknowns off
// with FMAs that do not depend on each other.  Back-substitution of 121 columns 15.0 -> 8.3 us, of
// 91 columns 13.0 -> 7.6; refinement pass 2 (both sweeps and the sum of the partials) 28 -> 17.9
// and 24 -> 16.6.
// ---------------------------------------------------------------------------------
template <int NBP>
struct DenseTri {
  static constexpr int LS = NBP + 1;
  double r[NBP * LS];  // strict upper triangle, zeros elsewhere
  double dg[NBP];      // diagonal (1 past nB)
  double dinv[NBP];    // its reciprocals
};

// The triangle's elements of one thread of NT: loaded, then stored.  The loads are unconditional
// (element 0 stands for what is not in the triangle) and the values are selected when they are
// stored: a load under a condition is waited for before the next one is issued, one memory latency
// each (back-substitution of 121 columns: 11.0 us with conditional loads, 8.3 without).
template <typename T, int NBP, int NT>
struct StageDense {
  static constexpr int CW = NBP <= 32 ? 32 : (NBP <= 64 ? 64 : 128);  // threads along a row
  static constexpr int RS = NT / CW;                                   // rows per pass
  static constexpr int PER = (NBP + RS - 1) / RS;
  T buf[PER];
  __device__ __forceinline__ void load(const T* __restrict__ RB, int L, int nB, int tid) {
    const int c = tid & (CW - 1), r0 = tid / CW;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int r = r0 + u * RS;
      buf[u] = RB[(r <= c && c < nB) ? r * L + c : 0];
    }
  }
  __device__ __forceinline__ void store(DenseTri<NBP>& D, int nB, int tid) const {
    const int c = tid & (CW - 1), r0 = tid / CW;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int r = r0 + u * RS;
      if (c < NBP && r < NBP) {
        D.r[r * DenseTri<NBP>::LS + c] = r < c && c < nB ? (double)buf[u] : 0.0;
        if (r == c) D.dg[c] = c < nB ? (double)buf[u] : 1.0;
      }
    }
  }
};

// Reciprocals of the diagonal, by one wave.
template <int NBP>
__device__ __forceinline__ void dense_diag_inv(DenseTri<NBP>& D, int lane) {
  if (lane < NBP) D.dinv[lane] = 1.0 / D.dg[lane];
  if (NBP > 64 && lane + 64 < NBP) D.dinv[lane + 64] = 1.0 / D.dg[lane + 64];
  wave_lds_sync();
}

// The steps of a sweep inside a diagonal block: w += (lane K of the 16-lane row's w) r_K for K = 0 ..
// 14 (FWD) or 15 .. 1.  s_nop 1: a lane selection's source must not have been written by the VALU in
// the two preceding cycles, which the compiler does not track inside an asm statement.
#define QRK_SWEEP(OP, K) "s_nop 1\n\tv_fmac_f64_dpp %0, %0, " OP " row_newbcast:" #K " row_mask:0xf bank_mask:0xf\n\t"
template <bool FWD>
__device__ __forceinline__ void sweep_steps(double& w, const double (&r)[16]) {
  if constexpr (FWD)
    asm(QRK_SWEEP("%1", 0) QRK_SWEEP("%2", 1) QRK_SWEEP("%3", 2) QRK_SWEEP("%4", 3) QRK_SWEEP("%5", 4)
        QRK_SWEEP("%6", 5) QRK_SWEEP("%7", 6) QRK_SWEEP("%8", 7) QRK_SWEEP("%9", 8) QRK_SWEEP("%10", 9)
        QRK_SWEEP("%11", 10) QRK_SWEEP("%12", 11) QRK_SWEEP("%13", 12) QRK_SWEEP("%14", 13) QRK_SWEEP("%15", 14)
        : "+&v"(w)
        : "v"(r[0]), "v"(r[1]), "v"(r[2]), "v"(r[3]), "v"(r[4]), "v"(r[5]), "v"(r[6]), "v"(r[7]), "v"(r[8]),
          "v"(r[9]), "v"(r[10]), "v"(r[11]), "v"(r[12]), "v"(r[13]), "v"(r[14]));
  else
    asm(QRK_SWEEP("%15", 15) QRK_SWEEP("%14", 14) QRK_SWEEP("%13", 13) QRK_SWEEP("%12", 12) QRK_SWEEP("%11", 11)
        QRK_SWEEP("%10", 10) QRK_SWEEP("%9", 9) QRK_SWEEP("%8", 8) QRK_SWEEP("%7", 7) QRK_SWEEP("%6", 6)
        QRK_SWEEP("%5", 5) QRK_SWEEP("%4", 4) QRK_SWEEP("%3", 3) QRK_SWEEP("%2", 2) QRK_SWEEP("%1", 1)
        : "+&v"(w)
        : "v"(r[1]), "v"(r[2]), "v"(r[3]), "v"(r[4]), "v"(r[5]), "v"(r[6]), "v"(r[7]), "v"(r[8]), "v"(r[9]),
          "v"(r[10]), "v"(r[11]), "v"(r[12]), "v"(r[13]), "v"(r[14]), "v"(r[15]));
}
#undef QRK_SWEEP
// v + sum_K (lane K of the row's w) r_K, in two sums
template <int K>
__device__ __forceinline__ void sweep_take4(double& v, double& u, double w, double r0, double r1, double r2,
                                            double r3) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %2, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
      : "+&v"(v), "+&v"(u)
      : "v"(w), "v"(r0), "v"(r1), "v"(r2), "v"(r3), "n"(K), "n"(K + 1), "n"(K + 2), "n"(K + 3));
}
__device__ __forceinline__ double sweep_take(double v, double w, const double (&r)[16]) {
  double u = 0.0;
  sweep_take4<0>(v, u, w, r[0], r[1], r[2], r[3]);
  sweep_take4<4>(v, u, w, r[4], r[5], r[6], r[7]);
  sweep_take4<8>(v, u, w, r[8], r[9], r[10], r[11]);
  sweep_take4<12>(v, u, w, r[12], r[13], r[14], r[15]);
  return v + u;
}

// One sweep, in place: FWD y = R_B^{-T} g, else x = R_B^{-1} y; nblk diagonal blocks hold the nB
// rows.  A block's LDS reads (its own entries and those of the rows it feeds) are all issued before
// its steps, so they arrive while the steps run.  Rows that are solved keep their values: the
// triangle's other half is zeros.  The blocks are a loop, not unrolled: the code runs once per call,
// and a straight line of it waits on instruction fetch.
template <int NBP, bool FWD>
__device__ __forceinline__ void wave_sweep(const DenseTri<NBP>& D, int nblk, int lane, double& v0, double& v1) {
  constexpr int LS = DenseTri<NBP>::LS;
  const int c = lane & 15;
  const int i0 = lane < NBP ? lane : NBP - 1, i1 = lane + 64 < NBP ? lane + 64 : NBP - 1;
#pragma clang loop unroll(disable)
  for (int s = 0; s < nblk; ++s) {
    const int b = FWD ? s : nblk - 1 - s;
    const bool hi = NBP > 64 && b >= 4;
    const double* at = D.r + (FWD ? 16 * b * LS : 16 * b);  // entry (k, i) of the block: step k, row i
    const int sk = FWD ? LS : 1, si = FWD ? 1 : LS;
    double rd[16], r0[16], r1[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) rd[k] = at[k * sk + (16 * b + c) * si];
    const double dv = D.dinv[16 * b + c];
    const uint64_t u = __builtin_bit_cast(uint64_t, hi ? v1 : v0);
    const int from = ((b & 3) * 16 + c) * 4;  // every 16-lane row takes the block's right-hand sides
    const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(from, (int)(unsigned)u);
    const unsigned up = (unsigned)__builtin_amdgcn_ds_bpermute(from, (int)(unsigned)(u >> 32));
#pragma unroll
    for (int k = 0; k < 16; ++k) r0[k] = at[k * sk + i0 * si];
    if constexpr (NBP > 64)
#pragma unroll
      for (int k = 0; k < 16; ++k) r1[k] = at[k * sk + i1 * si];
    asm volatile("" ::: "memory");  // the reads above are issued before the steps
    double w = __builtin_bit_cast(double, ((uint64_t)up << 32) | lo) * dv;
#pragma unroll
    for (int k = 0; k < 16; ++k) rd[k] *= -dv;
    sweep_steps<FWD>(w, rd);
    const double wn = -w;
    v0 = sweep_take(v0, wn, r0);
    if constexpr (NBP > 64) v1 = sweep_take(v1, wn, r1);
    const bool mine = (lane >> 4) == (b & 3);
    v0 = mine && !hi ? w : v0;
    v1 = mine && hi ? w : v1;
  }
}

// ---------------------------------------------------------------------------------
// Dense part of the back-substitution: R_B p_B = c_B, one workgroup (one working wave)
// per problem.  c_B is column L-1 of R_B | c_B, or cext (laid out like p) when that is given.
// ---------------------------------------------------------------------------------
template <typename T, int NBP>
__global__ void __launch_bounds__(NBP <= 32 ? 256 : 1024)
k_backsub_dense(const ProbDesc* __restrict__ probs, int n, const T* __restrict__ RBall, double* __restrict__ p,
                int* __restrict__ status, const double* __restrict__ cext) {
  constexpr int NT = NBP <= 32 ? 256 : 1024;
  __shared__ DenseTri<NBP> D;
  const int pi = blockIdx.x;
  const ProbDesc& P = probs[pi];
  const int L = P.L, nB = P.nB;
  const int64_t off = P.noff + P.K * n;
  const T* RB = RBall + P.rboff;
  const int lane = threadIdx.x & 63;
  StageDense<T, NBP, NT> stage;
  stage.load(RB, L, nB, threadIdx.x);
  // c_B (row 0's when a lane has no row: R_B | c_B has L >= 1 rows and columns)
  double v0, v1;
  if (cext) {
    v0 = cext[nB > 0 ? off + (lane < nB ? lane : 0) : P.noff];
    v1 = cext[nB > 0 ? off + (lane + 64 < nB ? lane + 64 : 0) : P.noff];
  } else {
    const T c0 = RB[(lane < nB ? lane : 0) * L + nB], c1 = RB[(lane + 64 < nB ? lane + 64 : 0) * L + nB];
    v0 = (double)c0;
    v1 = (double)c1;
  }
  if (lane >= nB) v0 = 0.0;
  if (lane + 64 >= nB) v1 = 0.0;
  stage.store(D, nB, threadIdx.x);
  __syncthreads();
  if (threadIdx.x >= 64) return;
  // pivots against the largest one: each lane its own diagonal entries, then a wave maximum
  const double dg0 = lane < nB ? D.dg[lane] : 0.0;
  const double dg1 = lane + 64 < nB ? D.dg[lane + 64] : 0.0;
  dense_diag_inv<NBP>(D, lane);
  wave_sweep<NBP, false>(D, (nB + 15) >> 4, lane, v0, v1);
  const double dmax = wave_allreduce_max(fmax(fabs(dg0), fabs(dg1)));
  const double tol = (double)nB * Eps<T>::value * dmax;
  const bool bad = (lane < nB && is_finite(dg0) && !(fabs(dg0) > tol)) ||
                   (lane + 64 < nB && is_finite(dg1) && !(fabs(dg1) > tol));
  bool nonfinite = false;
  if (lane < nB) {
    p[off + lane] = v0;
    nonfinite |= !is_finite(v0);
  }
  if (lane + 64 < nB) {
    p[off + lane + 64] = v1;
    nonfinite |= !is_finite(v1);
  }
  if (bad) set_status(status + pi, ST_SINGULAR);
  if (nonfinite) set_status(status + pi, ST_NONFINITE);
}

// f(NBP) for the smallest triangle size that holds max_L - 1 coupled columns
template <typename F>
static void dense_size(int max_L, F&& f) {
  const int nB = max_L - 1;
  if (nB <= 32)
    f(std::integral_constant<int, 32>{});
  else if (nB <= 64)
    f(std::integral_constant<int, 64>{});
  else if (nB <= 96)
    f(std::integral_constant<int, 96>{});
  else
    f(std::integral_constant<int, 128>{});
}

template <typename T>
hipError_t launch_backsub_dense(const BatchView& bv, const T* RB, double* p, int* status, hipStream_t st,
                                const double* cext) {
  if (bv.max_L > kMaxDense) return hipErrorInvalidValue;
  dense_size(bv.max_L, [&](auto S) {
    constexpr int NBP = decltype(S)::value;
    hipLaunchKernelGGL((k_backsub_dense<T, NBP>), dim3(bv.P), dim3(NBP <= 32 ? 256 : 1024), 0, st, bv.probs, bv.n,
                       RB, p, status, cext);
  });
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Blocks: x_i (= | +=) R_i^{-1} (base_i - S_i v) for all blocks, v the dense-part vector of the
// block's problem.  A wave takes whole units of at most 64 / N consecutive blocks (at most 64
// coupling rows S|c, contiguous), fewer where the problem has too few blocks for its waves; the rows
// are streamed with the next chunk in flight, each row's dot with v is left in LDS, then lane k
// back-substitutes block k of the unit.
//   MODE 0 back-substitution: base_i = c_i (column nB of S|c, streamed with weight -1),
//                             v = p_B, p_i set, pivot and finiteness status;
//   MODE 1 refinement:        base_i = y_i, v = delta_B, p_i incremented;
//   MODE 2 adjoint:           base_i = y_i, v = u_B, u_i set;
//   MODE 3 back-substitution for a given c (laid out like p, in ybase): base_i = c_i,
//                             v = p_B, p_i set, pivot and finiteness status.
// ---------------------------------------------------------------------------------
template <typename T, int N, int MODE, int CW>
__device__ __forceinline__ void blocks_solve_units(const ProbDesc& P, int pi, const T* __restrict__ Rblk,
                                                   const T* __restrict__ Sc, const double* __restrict__ v,
                                                   const double* __restrict__ ybase, double* __restrict__ x,
                                                   int* __restrict__ status, double* rhs, int wv, int lane) {
  using S = RowStream<T, CW>;
  const int nB = P.nB, L = P.L;
  const int64_t koff = P.koff, noff = P.noff, soff = P.soff, K = P.K;
  const int ncol = MODE == 0 ? L : nB;
  const int col = lane & (S::LN - 1);
  double w0 = v[col < nB ? col : 0], w1 = 0.0;
  if (col >= nB) w0 = MODE == 0 && col == nB ? -1.0 : 0.0;
  if constexpr (S::SL == 2) {
    w1 = v[col + 64 < nB ? col + 64 : 0];
    if (col + 64 >= nB) w1 = MODE == 0 && col + 64 == nB ? -1.0 : 0.0;
  }
  const int64_t waves = (int64_t)P.nwg * 4;
  const int64_t even = (K + waves - 1) / waves;  // blocks of a wave
  constexpr int UMIN = 16 / N > 0 ? 16 / N : 1, UMAX = 64 / N;
  const int unit = even < UMIN ? UMIN : (even > UMAX ? UMAX : (int)even);
  for (int64_t lb0 = ((blockIdx.x - P.wg0) * 4 + wv) * (int64_t)unit; lb0 < K; lb0 += waves * unit) {
    const int nb = K - lb0 < unit ? (int)(K - lb0) : unit;
    const int rows = nb * N;
    const __amdgpu_buffer_rsrc_t rsS =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(Sc + soff + lb0 * N * L), 0, 0x7fffffff, 0x00020000);
    StreamChunk<T, CW> va, vb;
    stream_load<T, CW>(va, rsS, 0, rows, L, ncol, lane);
    // this lane's block (lanes < nb): R_i and the base values
    const int64_t lb = lb0 + (lane < nb ? lane : nb - 1), blk = koff + lb;
    T Rb[N * N];
#pragma unroll
    for (int e = 0; e < N * N; ++e) Rb[e] = Rblk[blk * (N * N) + e];
    double base[N], xold[N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
      base[c] = MODE == 0 ? 0.0 : (MODE == 3 ? ybase[noff + lb * N + c] : ybase[blk * N + c]);
      xold[c] = MODE == 1 ? x[noff + lb * N + c] : 0.0;
    }
    auto dots = [&](const StreamChunk<T, CW>& vv, int c0) {
      rhs[c0 + S::sum_row(lane)] = -stream_dot<T, CW>(vv, w0, w1, lane);  // -(S v) (mode 0: c - S p_B)
    };
    for (int c0 = 0;;) {
      if (c0 + S::CHR < rows) stream_load<T, CW>(vb, rsS, c0 + S::CHR, rows, L, ncol, lane);
      dots(va, c0);
      if ((c0 += S::CHR) >= rows) break;
      if (c0 + S::CHR < rows) stream_load<T, CW>(va, rsS, c0 + S::CHR, rows, L, ncol, lane);
      dots(vb, c0);
      if ((c0 += S::CHR) >= rows) break;
    }
    wave_lds_sync();
    if (lane < nb) {
      double out[N];
#pragma unroll
      for (int i = N - 1; i >= 0; --i) {
        double sacc = base[i] + rhs[lane * N + i];
#pragma unroll
        for (int j = i + 1; j < N; ++j) sacc -= (double)Rb[i * N + j] * out[j];
        out[i] = sacc / (double)Rb[i * N + i];
      }
      bool nonfinite = false;
      double* xo = x + noff + lb * N;
#pragma unroll
      for (int c = 0; c < N; ++c) {
        xo[c] = MODE == 1 ? xold[c] + out[c] : out[c];
        nonfinite |= !is_finite(out[c]);
      }
      if ((MODE == 0 || MODE == 3) && status) {
        double dmax = 0.0;
#pragma unroll
        for (int c = 0; c < N; ++c) dmax = fmax(dmax, fabs((double)Rb[c * N + c]));
        bool bad = false;
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const double piv = (double)Rb[c * N + c];
          if (is_finite(piv) && !(fabs(piv) > (double)N * Eps<T>::value * dmax)) bad = true;
        }
        if (bad) set_status(status + pi, ST_SINGULAR);
        if (nonfinite) set_status(status + pi, ST_NONFINITE);
      }
    }
    wave_lds_sync();  // the next unit overwrites rhs
  }
}

template <typename T, int N, int MODE>
__global__ void __launch_bounds__(256)
k_blocks_solve_n(const ProbDesc* __restrict__ probs, const int32_t* __restrict__ wg_prob,
                 const T* __restrict__ Rblk, const T* __restrict__ Sc,
                 const double* __restrict__ vbuf, const double* __restrict__ ybase, double* __restrict__ x,
                 int* __restrict__ status) {
  __shared__ double rhs_all[4][128];  // a unit's rows, rounded up to whole chunks
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int pi = wg_prob[blockIdx.x];
  const ProbDesc& P = probs[pi];
  // with nB == 0 the dense vector may be empty: any element stands in (weight 0)
  const double* v = MODE == 1 ? vbuf + (int64_t)pi * kMaxDense : vbuf + P.noff + (P.nB > 0 ? P.K * N : 0);
  stream_width(MODE == 0 ? P.L : P.nB, [&](auto C) {
    blocks_solve_units<T, N, MODE, decltype(C)::value>(P, pi, Rblk, Sc, v, ybase, x, status, rhs_all[wv], wv, lane);
  });
}

template <typename T, int MODE>
static hipError_t launch_blocks_solve(const BatchView& bv, const T* Rblk, const T* Sc, const double* vbuf,
                                      const double* ybase, double* x, int* status, hipStream_t st) {
  if (bv.max_L > kMaxDense) return hipErrorInvalidValue;
  switch (bv.n) {
#define QRK_BS(NN)                                                                                          \
  case NN:                                                                                                  \
    hipLaunchKernelGGL((k_blocks_solve_n<T, NN, MODE>), dim3(bv.nwg), dim3(256), 0, st, bv.probs, bv.wg_prob, \
                       Rblk, Sc, vbuf, ybase, x, status);                                                  \
    break;
    QRK_BS(1) QRK_BS(2) QRK_BS(3) QRK_BS(4) QRK_BS(5) QRK_BS(6) QRK_BS(7) QRK_BS(8)
#undef QRK_BS
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_backsub_blocks(const BatchView& bv, const T* Rblk, const T* Sc, double* p, int* status,
                                 hipStream_t st, const double* cext) {
  if (cext) return launch_blocks_solve<T, 3>(bv, Rblk, Sc, p, cext, p, status, st);
  return launch_blocks_solve<T, 0>(bv, Rblk, Sc, p, nullptr, p, status, st);
}

template <typename T>
hipError_t launch_refine_blocks(const BatchView& bv, const T* Rblk, const T* Sc, const double* y,
                                const double* delta_B, double* p, hipStream_t st) {
  return launch_blocks_solve<T, 1>(bv, Rblk, Sc, delta_B, y, p, nullptr, st);
}

template <typename T>
hipError_t launch_adjoint_blocks(const BatchView& bv, const T* Rblk, const T* Sc, const double* y, double* u,
                                 hipStream_t st) {
  return launch_blocks_solve<T, 2>(bv, Rblk, Sc, u, y, u, nullptr, st);
}

// ---------------------------------------------------------------------------------
// Refinement pass 1: one wave per pack of whole blocks (at most 64 rows).
//   r = b - A_i p_i - B p_B;  g_i = A_i^T r - lam d_i^2 p_i;  y_i = R_i^{-T} g_i;
//   per-workgroup partial of  B^T r - sum_i S_i^T y_i.
// b - A_i p_i and A_i's products with r go with a lane per row of the pack, A_i^T r with a lane per
// (block, unknown), the triangular solves with a lane per block.  The pack's rows of B are streamed
// once (RowStream), the next chunk in flight while one is worked on: B p_B by folding, B^T r from
// the same registers with a lane per column.  Every sum runs in a fixed order, so the partials are
// deterministic.
// Workgroup w serves problem wg_prob[w] only; its packs are that problem's packs
// lw*4 + wave, lw*4 + wave + 4*nwg, ... (lw = w - wg0), its partial goes to part[w].
// CAM: the coupled columns are cameras of ldb columns (nB = ncam * ldb); B holds each row's ldb
// values and cam[row] its camera (outside [0, ncam): none), so a streamed row is zero outside its
// camera's columns.
// ---------------------------------------------------------------------------------
template <int N>
struct Pass1Lds {
  double pg[64 * N + 64];  // p_i of the pack's blocks, then A_i^T r, then y (0 past the last block)
  double prod[64 * N];     // A_row * r per pack row
  double base[64];         // b - A_i p_i
  double rr[64];           // r
  int lo[65];              // first row of every block of the pack
};

template <typename T, int N, bool CAM, int CW>
__device__ __forceinline__ void pass1_packs(const ProbDesc& P, const int64_t* __restrict__ pack_blk,
                                            const int64_t* __restrict__ row_off, const T* __restrict__ A,
                                            const T* __restrict__ B, const int32_t* __restrict__ cam,
                                            const T* __restrict__ bvec, const double* __restrict__ d, double lam,
                                            const T* __restrict__ Rblk, const T* __restrict__ Sc,
                                            const double* __restrict__ p, double* __restrict__ y, Pass1Lds<N>& lds,
                                            int wv, int lane, double& t0, double& t1) {
  using S = RowStream<T, CW>;
  const int nB = P.nB, L = P.L;
  const int64_t koff = P.koff, noff = P.noff, moff = P.moff, soff = P.soff;
  const int ldb = nB > 0 ? (int)P.ldb : 0;
  const uint32_t ncam = CAM ? (uint32_t)(nB / ldb) : 0u;
  const int g = lane / S::LN, col = lane & (S::LN - 1);
  const double* pBv = p + noff + (nB > 0 ? P.K * N : 0);
  double w0 = pBv[col < nB ? col : 0], w1 = 0.0;
  if (col >= nB) w0 = 0.0;
  if constexpr (S::SL == 2) {
    w1 = pBv[col + 64 < nB ? col + 64 : 0];
    if (col + 64 >= nB) w1 = 0.0;
  }
  const int64_t lw = blockIdx.x - P.wg0;
  const int64_t pend = P.pack0 + P.npacks;
  for (int64_t pk = P.pack0 + lw * 4 + wv; pk < pend; pk += (int64_t)P.nwg * 4) {
    const int64_t b0 = pack_blk[pk];
    const int nb = (int)(pack_blk[pk + 1] - b0);
    const int64_t pr0 = row_off[b0];
    const int prows = (int)(row_off[b0 + nb] - pr0);
    // with nB == 0 there may be no B at all: every column is out of range then, nothing is read
    const T* Bbase = nB > 0 ? B + P.boff + (pr0 - moff) * ldb : bvec + pr0;
    const __amdgpu_buffer_rsrc_t rsB =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(Bbase), 0, 0x7fffffff, 0x00020000);
    const int64_t grow = pr0 + (lane < prows ? lane : prows - 1);  // this lane's row (if prows > 0)
    int camv = 0;
    auto load = [&](StreamChunk<T, CW>& v, int c0) {
      if constexpr (CAM) {
        static_assert(S::RPL == 1, "a camera row takes the whole wave");
#pragma unroll
        for (int i = 0; i < S::NV; ++i) {
          const int row = c0 + i < prows ? c0 + i : prows - 1;
          const int cr = __builtin_amdgcn_readlane(camv, row);
          const int cb = (uint32_t)cr < ncam ? cr * ldb : 1 << 20;
          const uint32_t k0 = (uint32_t)(lane - cb), k1 = (uint32_t)(lane + 64 - cb);
          const uint32_t so = (uint32_t)(row * ldb) * (uint32_t)sizeof(T);
          v[0][i] = buf_ld_row<T>(rsB, k0 < (uint32_t)ldb ? k0 * (uint32_t)sizeof(T) : kNoColumn, so);
          if constexpr (S::SL == 2)
            v[1][i] = buf_ld_row<T>(rsB, k1 < (uint32_t)ldb ? k1 * (uint32_t)sizeof(T) : kNoColumn, so);
        }
      } else {
        stream_load<T, CW>(v, rsB, c0, prows, ldb, nB, lane);
      }
    };
    StreamChunk<T, CW> va, vb;
    T arow[N] = {}, bval = T(0);
    if (prows > 0) {  // a pack of blocks without rows has none to read
      if constexpr (CAM) camv = cam[grow];
      load(va, 0);
#pragma unroll
      for (int c = 0; c < N; ++c) arow[c] = A[grow * N + c];
      bval = bvec[grow];
    }
    // this lane's block (lanes < nb)
    const int64_t blk = b0 + (lane < nb ? lane : nb - 1);
    const int64_t lb = blk - koff;
    const int lo = (int)(row_off[blk] - pr0);
    double dd[N], pp[N];
    T Rb[N * N];
#pragma unroll
    for (int c = 0; c < N; ++c) {
      dd[c] = d[noff + lb * N + c];
      pp[c] = p[noff + lb * N + c];
    }
#pragma unroll
    for (int e = 0; e < N * N; ++e) Rb[e] = Rblk[blk * (N * N) + e];
    if (lane < nb) {
#pragma unroll
      for (int c = 0; c < N; ++c) lds.pg[lane * N + c] = pp[c];
      lds.lo[lane] = lo;
    }
    if (lane == 0) lds.lo[nb] = prows;
    int rb = 0;  // the block of this lane's row: the last one that starts at or before it
    for (int k = 1; k < nb; ++k) rb += lane >= __builtin_amdgcn_readlane(lo, k) ? 1 : 0;
    if (lane >= prows) rb = nb - 1;
    wave_lds_sync();
    {
      double dot = 0.0;
#pragma unroll
      for (int c = 0; c < N; ++c) dot += (double)arow[c] * lds.pg[rb * N + c];
      lds.base[lane] = (double)bval - dot;
    }
    wave_lds_sync();
    auto work = [&](const StreamChunk<T, CW>& v, int c0) {
      const double acc = stream_dot<T, CW>(v, w0, w1, lane);
      const int row = c0 + S::sum_row(lane);  // < 64: a chunk does not pass the pack's 64 rows
      const double bs = lds.base[row];
      lds.rr[row] = row < prows ? bs - acc : 0.0;
      wave_lds_sync();
#pragma unroll
      for (int i = 0; i < S::NV; ++i) {
        const double rv = lds.rr[c0 + i * S::RPL + g];
        t0 += (double)second_use<(N > 5)>(v[0][i]) * rv;
        if constexpr (S::SL == 2) t1 += (double)second_use<(N > 5)>(v[1][i]) * rv;
      }
    };
    for (int c0 = 0; c0 < prows;) {
      if (c0 + S::CHR < prows) load(vb, c0 + S::CHR);
      work(va, c0);
      if ((c0 += S::CHR) >= prows) break;
      if (c0 + S::CHR < prows) load(va, c0 + S::CHR);
      work(vb, c0);
      c0 += S::CHR;
    }
    // the coupling rows of the pack are contiguous: their first chunk travels during the solves
    const int rs = nb * N;
    const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(Sc + soff + (b0 - koff) * N * L), 0, 0x7fffffff, 0x00020000);
    stream_load<T, CW>(va, rsS, 0, rs, L, nB, lane);
    if (lane < prows) {
      const double rv = lds.rr[lane];
#pragma unroll
      for (int c = 0; c < N; ++c) lds.prod[lane * N + c] = (double)arow[c] * rv;
    }
    wave_lds_sync();
    for (int e = lane; e < rs; e += 64) {  // (A_i^T r)_c, rows in order, eight reads in flight
      const int k = e / N, c = e - k * N;
      const int r1 = lds.lo[k + 1];
      double sum = 0.0;
      for (int r = lds.lo[k]; r < r1; r += 8) {
        double q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = lds.prod[(r + u < r1 ? r + u : r1 - 1) * N + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += r + u < r1 ? q[u] : 0.0;
      }
      lds.pg[e] = sum;
    }
    wave_lds_sync();
    if (lane < nb) {  // R_i^T y = A_i^T r - lam d_i^2 p_i (R_i upper triangular, row-major)
      double yy[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        double sacc = lds.pg[lane * N + i] - lam * dd[i] * dd[i] * pp[i];
#pragma unroll
        for (int j = 0; j < i; ++j) sacc -= (double)Rb[j * N + i] * yy[j];
        yy[i] = sacc / (double)Rb[i * N + i];
      }
#pragma unroll
      for (int c = 0; c < N; ++c) {
        y[blk * N + c] = yy[c];
        lds.pg[lane * N + c] = yy[c];
      }
    }
    lds.pg[rs + lane] = 0.0;
    wave_lds_sync();
    auto coupling = [&](const StreamChunk<T, CW>& v, int s0) {
#pragma unroll
      for (int i = 0; i < S::NV; ++i) {
        const double yc = lds.pg[s0 + i * S::RPL + g];
        t0 -= (double)v[0][i] * yc;
        if constexpr (S::SL == 2) t1 -= (double)v[1][i] * yc;
      }
    };
    for (int s0 = 0;;) {
      if (s0 + S::CHR < rs) stream_load<T, CW>(vb, rsS, s0 + S::CHR, rs, L, nB, lane);
      coupling(va, s0);
      if ((s0 += S::CHR) >= rs) break;
      if (s0 + S::CHR < rs) stream_load<T, CW>(va, rsS, s0 + S::CHR, rs, L, nB, lane);
      coupling(vb, s0);
      if ((s0 += S::CHR) >= rs) break;
    }
    wave_lds_sync();  // the next pack overwrites the wave's LDS
  }
}

template <typename T, int N, bool CAM>
__global__ void __launch_bounds__(256)
k_refine_pass1(const ProbDesc* __restrict__ probs, const int32_t* __restrict__ wg_prob,
               const int64_t* __restrict__ pack_blk, const int64_t* __restrict__ row_off,
               const T* __restrict__ A, const T* __restrict__ B, const int32_t* __restrict__ cam,
               const T* __restrict__ bvec,
               const double* __restrict__ d, const double* __restrict__ lamv, const T* __restrict__ Rblk,
               const T* __restrict__ Sc, const double* __restrict__ p, double* __restrict__ y,
               double* __restrict__ part) {
  __shared__ Pass1Lds<N> lds_all[4];
  __shared__ double red[4][kMaxDense];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int pi = wg_prob[blockIdx.x];
  const ProbDesc& P = probs[pi];
  const int nB = P.nB;
  const double lam = lamv[pi];
  double t0 = 0.0, t1 = 0.0;  // partial B^T r - S^T y of the lane's columns (and rows of a load)
  int rowstep = 64;           // lanes per row
  stream_width(CAM && nB <= 32 ? 64 : nB, [&](auto C) {
    constexpr int CW = CAM && decltype(C)::value < 64 ? 64 : decltype(C)::value;
    rowstep = RowStream<T, CW>::LN;
    pass1_packs<T, N, CAM, CW>(P, pack_blk, row_off, A, B, cam, bvec, d, lam, Rblk, Sc, p, y, lds_all[wv], wv, lane,
                               t0, t1);
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
hipError_t launch_refine_residual(const BatchView& bv, const T* A, const T* B, const int32_t* cam, const T* b,
                                  const double* d, const T* Rblk, const T* Sc, const double* p, double* y,
                                  double* part, hipStream_t st) {
  if (bv.max_L > kMaxDense) return hipErrorInvalidValue;
  switch (bv.n) {
#define QRK_P1(NN)                                                                                           \
  case NN:                                                                                                   \
    if (cam)                                                                                                 \
      hipLaunchKernelGGL((k_refine_pass1<T, NN, true>), dim3(bv.nwg), dim3(256), 0, st, bv.probs, bv.wg_prob, \
                         bv.pack_blk, bv.row_off, A, B, cam, b, d, bv.lam, Rblk, Sc, p, y, part);           \
    else                                                                                                     \
      hipLaunchKernelGGL((k_refine_pass1<T, NN, false>), dim3(bv.nwg), dim3(256), 0, st, bv.probs,           \
                         bv.wg_prob, bv.pack_blk, bv.row_off, A, B, cam, b, d, bv.lam, Rblk, Sc, p, y, part); \
    break;
    QRK_P1(1) QRK_P1(2) QRK_P1(3) QRK_P1(4) QRK_P1(5) QRK_P1(6) QRK_P1(7) QRK_P1(8)
#undef QRK_P1
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------
// Refinement pass 2 (one workgroup per problem): g_B = sum of the problem's workgroup
// partials (fixed order) - lam d_B^2 p_B, then y_B = R_B^{-T} g_B and delta_B = R_B^{-1} y_B
// by one wave; p_B += delta_B.
// ADJ = false: refinement (delta_B -> delta[pi * kMaxDense ..]).
// ADJ = true : adjoint (rhs = g_B + sum of partials; the solution -> u_B in out, laid out
//              like p; p untouched).
// ---------------------------------------------------------------------------------
template <typename T, bool ADJ, int NBP>
__global__ void __launch_bounds__(1024)
k_refine_dense(const ProbDesc* __restrict__ probs, int n, const double* __restrict__ part,
               const T* __restrict__ RBall, const double* __restrict__ dvec, const double* __restrict__ lamv,
               double* __restrict__ p, double* __restrict__ out, const double* __restrict__ gvec) {
  using Stage = StageDense<T, NBP, 1024>;
  constexpr int CW = Stage::CW, G = 1024 / CW;
  __shared__ DenseTri<NBP> D;
  __shared__ double acc[G][CW];
  const int pi = blockIdx.x;
  const ProbDesc& P = probs[pi];
  const int nB = P.nB, L = P.L;
  const int64_t off = P.noff + P.K * n;
  const double* pp = part + (int64_t)P.wg0 * kMaxDense;
  const int nparts = P.nwg;
  const int t = threadIdx.x;
  const int lane = t & 63;
  const bool on0 = lane < nB, on1 = lane + 64 < nB;
  Stage stage;
  stage.load(RBall + P.rboff, L, nB, t);
  // the first wave's part of the right-hand side and of p_B
  // (an unknown of the problem stands in where a lane has none; N >= 1)
  const int64_t e0 = on0 ? off + lane : P.noff, e1 = on1 ? off + lane + 64 : P.noff;
  const double* dsrc = ADJ ? gvec : dvec;
  const double d0 = dsrc[e0], d1 = dsrc[e1];
  const double p0 = ADJ ? 0.0 : p[e0], p1 = ADJ ? 0.0 : p[e1];
  const double lam = ADJ ? 0.0 : lamv[pi];
  // partials of group q: w = q, q + G, ...; loaded up to 32 at a time so the loads overlap, then
  // added in order
  const int j = t & (CW - 1), q = t / CW;
  double s = 0.0;
  if (j < nB) {
    for (int w0 = q; w0 < nparts; w0 += G * 32) {
      double buf[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) {
        const int w = w0 + G * u;
        buf[u] = pp[(int64_t)(w < nparts ? w : q) * kMaxDense + j];
      }
#pragma unroll
      for (int u = 0; u < 32; ++u) s += w0 + G * u < nparts ? buf[u] : 0.0;
    }
  }
  acc[q][j] = s;
  stage.store(D, nB, t);
  __syncthreads();
  if (t >= 64) return;
  double g0 = 0.0, g1 = 0.0;
#pragma unroll
  for (int k = 0; k < G; ++k) {
    g0 += acc[k][lane & (CW - 1)];
    if (CW > 64) g1 += acc[k][(lane + 64) & (CW - 1)];
  }
  double v0 = 0.0, v1 = 0.0;
  if (on0) v0 = ADJ ? d0 + g0 : g0 - lam * d0 * d0 * p0;
  if (on1) v1 = ADJ ? d1 + g1 : g1 - lam * d1 * d1 * p1;
  const int nblk = (nB + 15) >> 4;
  dense_diag_inv<NBP>(D, lane);
  wave_sweep<NBP, true>(D, nblk, lane, v0, v1);
  wave_sweep<NBP, false>(D, nblk, lane, v0, v1);
  double* o = ADJ ? out + off : out + (int64_t)pi * kMaxDense;
  if (on0) {
    o[lane] = v0;
    if (!ADJ) p[off + lane] = p0 + v0;
  }
  if (on1) {
    o[lane + 64] = v1;
    if (!ADJ) p[off + lane + 64] = p1 + v1;
  }
}

template <typename T>
hipError_t launch_refine_dense(const BatchView& bv, const double* part, const T* RB, const double* dvec,
                               double* p, double* delta_B, hipStream_t st) {
  if (bv.max_L > kMaxDense) return hipErrorInvalidValue;
  dense_size(bv.max_L, [&](auto S) {
    hipLaunchKernelGGL((k_refine_dense<T, false, decltype(S)::value>), dim3(bv.P), dim3(1024), 0, st, bv.probs, bv.n,
                       part, RB, dvec, bv.lam, p, delta_B, (const double*)nullptr);
  });
  return hipGetLastError();
}

template <typename T>
hipError_t launch_adjoint_dense(const BatchView& bv, const double* part, const T* RB, const double* g, double* u,
                                hipStream_t st) {
  if (bv.max_L > kMaxDense) return hipErrorInvalidValue;
  dense_size(bv.max_L, [&](auto S) {
    hipLaunchKernelGGL((k_refine_dense<T, true, decltype(S)::value>), dim3(bv.P), dim3(1024), 0, st, bv.probs, bv.n,
                       part, RB, (const double*)nullptr, bv.lam, (double*)nullptr, u, g);
  });
  return hipGetLastError();
}

#define QRK_INST(T)                                                                                      \
  template hipError_t launch_backsub_dense<T>(const BatchView&, const T*, double*, int*, hipStream_t,      \
                                              const double*);                                            \
  template hipError_t launch_backsub_blocks<T>(const BatchView&, const T*, const T*, double*, int*,        \
                                               hipStream_t, const double*);                              \
  template hipError_t launch_refine_residual<T>(const BatchView&, const T*, const T*, const int32_t*,       \
                                                const T*, const double*, const T*, const T*, const double*, \
                                                double*, double*, hipStream_t);                          \
  template hipError_t launch_refine_dense<T>(const BatchView&, const double*, const T*, const double*,     \
                                             double*, double*, hipStream_t);                             \
  template hipError_t launch_refine_blocks<T>(const BatchView&, const T*, const T*, const double*,         \
                                              const double*, double*, hipStream_t);                      \
  template hipError_t launch_adjoint_blocks<T>(const BatchView&, const T*, const T*, const double*, double*, \
                                               hipStream_t);                                             \
  template hipError_t launch_adjoint_dense<T>(const BatchView&, const double*, const T*, const double*,     \
                                              double*, hipStream_t);
QRK_INST(float)
QRK_INST(double)
#undef QRK_INST

}  // namespace qrk
