// Tall-skinny QR of the reduced dense rows in float64 on the gfx950 matrix cores (QRkit
// Section 4.2, the factorisation Q'R' = qr(Q_1^perp^T A_2)), for a batch of problems with the
// same number of 16-column blocks at once.
//
// Organisation (that of the float32 path, tsqr_mfma.hpp and tsqr_tree.hpp): every wave is a leaf
// that streams a contiguous range of one problem's rows, a tile of 16 NRB rows at a time, into
// its own running triangle; the leaf triangles are then merged pairwise in a second launch, one
// wave per inner node of every problem's tree, pipelined over column blocks.  Merging a tile is
// blocked Householder with the compact WY form: 16-column panels on the VALU, the trailing
// products on v_mfma_f64_16x16x4_f64.
//
// What bounds it: one column of a panel is a dependency chain (Gram row, sum over the wave's
// rows, reciprocal square root, update), and the VALU issues its two passes over the tile at one
// wave per SIMD (the tile and the triangle fill the register file); the matrix cores are busy
// for about a quarter of a tile's time and HBM is idle.  Taller tiles spread the chain over more
// rows, so each width takes the tallest tile that the registers hold (leaf_tile_rows_f64).
// Measured against the kernel before it (a thread per column, a barrier per column, eight
// triangles merged per level): 120,000 rows x 61 columns 2,798 -> 157 us (leaves 66, tree 91;
// 0.9 GFLOP), 800 x 25 240 -> 48 us.
//
// Register layout of a 16 x 16 block M (the accumulator layout of the float64 product): lane l,
// component v holds M[4 v + (l >> 4)][l & 15].  Component v of a tile block is then the operand of
// the v-th 4-row slice of X_P^T X_q as it stands.
#pragma once

#include "qrk_batch.hpp"
#include "qrk_device.hpp"

namespace qrk {

typedef double d4 __attribute__((ext_vector_type(4)));

// Rows per leaf tile and, for the wide dense parts, the block rows of the running triangle that
// stay in registers (the later ones live in the wave's LDS: a panel reads and writes only its own
// block row).  Registers per lane: 8 (NRB NCB + blocks of the triangle), about 100 more for the
// panel; LDS per wave: 2 KiB per triangle block and the staging of T and W.
constexpr int leaf_tile_rows_f64(int ncb) {
  return ncb <= 4 ? 128 : (ncb == 5 ? 96 : (ncb == 6 ? 64 : (ncb == 7 ? 48 : 32)));
}
constexpr int leaf_reg_rows_f64(int ncb) {
  return ncb <= 3 ? ncb : (ncb == 4 ? 0 : (ncb == 5 ? 1 : (ncb == 7 ? 2 : 3)));
}

constexpr int kF64Ld = 17;                    // row stride of a 16 x 16 block staged in LDS
constexpr int kF64Blk = 16 * kF64Ld;          // doubles of a staged block
constexpr int kF64Stage = kF64Blk + 16;       // T and the column scales; the blocks of W follow

template <int NCB>
struct Tri64 {
  static constexpr int count = NCB * (NCB + 1) / 2;
  static constexpr int idx(int p, int q) { return p * NCB - (p * (p - 1)) / 2 + (q - p); }
  static constexpr int slot = count * 256;  // doubles of a stored triangle (lane-major blocks)
};

// Broadcast lane J of every 16-lane row to the whole row.
template <int J>
__device__ __forceinline__ double row_bcast64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x150 + J, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x150 + J, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

// acc += b(x) x over a 4-row block, and x += b(x) f, with the broadcast as the FMA's DPP modifier
// (row_newbcast is the one DPP control of 64-bit instructions).  s_nop 1: a DPP source must not
// have been written by the VALU in the two preceding cycles, which the compiler does not track
// across an asm statement; inside a group no DPP source is a result of the group.
template <int J>
__device__ __forceinline__ void gram4_64(double& p0, double& p1, const d4& x) {
  asm volatile("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %2 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %3, %3 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, %4, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %5, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
      : "+v"(p0), "+v"(p1)
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "n"(J));
}
template <int J>
__device__ __forceinline__ void axpy4_64(d4& x, double f) {
  double x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
  asm volatile("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %0, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %1, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %3, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
      : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3)
      : "v"(f), "n"(J));
  x = d4{x0, x1, x2, x3};
}

// Sum over the wave's four 16-lane rows, the same bits in every lane (the permlane swaps of
// sum_rows4 in tsqr_mfma.hpp, on the two halves of a double).
__device__ __forceinline__ double sum_rows4_64(double x) {
  uint64_t u = __builtin_bit_cast(uint64_t, x);
  auto a = __builtin_amdgcn_permlane16_swap((unsigned)u, opaque_copy((unsigned)u), false, false);
  auto b = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), opaque_copy((unsigned)(u >> 32)), false, false);
  x = __builtin_bit_cast(double, ((uint64_t)(unsigned)b[0] << 32) | (unsigned)a[0]) +
      __builtin_bit_cast(double, ((uint64_t)(unsigned)b[1] << 32) | (unsigned)a[1]);
  u = __builtin_bit_cast(uint64_t, x);
  auto e = __builtin_amdgcn_permlane32_swap((unsigned)u, opaque_copy((unsigned)u), false, false);
  auto f = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), opaque_copy((unsigned)(u >> 32)), false, false);
  return __builtin_bit_cast(double, ((uint64_t)(unsigned)f[0] << 32) | (unsigned)e[0]) +
         __builtin_bit_cast(double, ((uint64_t)(unsigned)f[1] << 32) | (unsigned)e[1]);
}
__device__ __forceinline__ double read_lane64(double x, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Lane (g, c) receives lane (G, c)'s x (a fetch through the LDS crossbar; every lane active).
template <int G>
__device__ __forceinline__ double rows_from64(double x, int c) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute((G * 16 + c) * 4, (int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_ds_bpermute((G * 16 + c) * 4, (int)(unsigned)(u >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// sqrt(q) and 1 / sqrt(q) for q > 0 (a subnormal one too: 1 / sqrt(q) < 2^538): the hardware estimate
// (about 24 bits) and two Goldschmidt steps, then one correction of the root.  1 / t: the estimate and
// two Newton steps.
__device__ __forceinline__ void sqrt_rsqrt64(double q, double& root, double& inv) {
  const double y = __builtin_amdgcn_rsq(q);
  double s = q * y, h = 0.5 * y;
  double r = fma(-s, h, 0.5);
  s = fma(s, r, s);
  h = fma(h, r, h);
  r = fma(-s, h, 0.5);
  s = fma(s, r, s);
  h = fma(h, r, h);
  root = fma(fma(-s, s, q), h, s);
  inv = h + h;
}
__device__ __forceinline__ double rcp64(double t) {
  double y = __builtin_amdgcn_rcp(t);
  y = fma(y, fma(-t, y, 1.0), y);
  return fma(y, fma(-t, y, 1.0), y);
}

// Householder factorisation of one 16-column panel [Rd; X[0..RBN-1]] with the compact-WY factor T
// built alongside: the steps and signs of panel_factor in tsqr_mfma.hpp.  A zero squared column norm
// gives the identity reflector (a subnormal one reflects, to the digits that it has); NaN takes
// the reflection, so that it reaches R.  Column 0 reads tile values that the matrix cores may have just written,
// so its passes are compiler-generated code (which tracks that hazard), the others the fused groups.
// ONLY: the panel is the whole matrix, of ncol <= 16 columns: the columns past them are left alone and
// T is not built, since there is nothing to apply it to (90,000 rows, one column: factor 78 -> 41 us,
// and 46 with the kernel before the matrix cores, which worked column by column).
template <int RBN, bool ONLY = false>
__device__ __forceinline__ void panel_factor64(d4& Rd, d4 (&X)[RBN], double (&trow)[16], double& sc, int lane,
                                               int ncol = 16) {
  const int g = lane >> 4;
  const int c = lane & 15;
  sc = 0.0;
  static_for<0, 16>([&](auto JJ) {
    constexpr int j = decltype(JJ)::value;
    if (ONLY && j >= ncol) return;
    const double rrow = rows_from64<(j & 3)>(Rd[j >> 2], c);  // R's row j in every row of the wave
    double p0 = 0.0, p1 = 0.0;
    if constexpr (j == 0) {
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (v & 1)
            p1 = fma(row_bcast64<j>(X[rb][v]), X[rb][v], p1);
          else
            p0 = fma(row_bcast64<j>(X[rb][v]), X[rb][v], p0);
        }
    } else {
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb) gram4_64<j>(p0, p1, X[rb]);
    }
    const double gram = sum_rows4_64(p0 + p1);  // x_j^T x_c
    const double sigma = row_bcast64<j>(gram);
    const double alpha = read_lane64(Rd[j >> 2], (j & 3) * 16 + j);
    const bool refl = !(sigma == 0.0);
    double nrm, rinv;
    sqrt_rsqrt64(fma(alpha, alpha, sigma), nrm, rinv);
    const double bneg = alpha >= 0.0 ? -nrm : nrm;
    const double beta = refl ? bneg : alpha;
    const double tau = refl ? (bneg - alpha) * (alpha >= 0.0 ? -rinv : rinv) : 0.0;
    const double scale = refl ? rcp64(alpha - bneg) : 0.0;
    const double pd = fma(gram, scale, rrow);  // R[j][c] + w_j^T x_c
    const double s = tau * pd;
    const double nf = (c > j) ? -scale * s : 0.0;
    if constexpr (j == 0) {
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) X[rb][v] = fma(row_bcast64<j>(X[rb][v]), nf, X[rb][v]);
    } else {
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb) axpy4_64<j>(X[rb], nf);
    }
    if (g == (j & 3)) Rd[j >> 2] = (c > j) ? Rd[j >> 2] - s : (c == j ? beta : Rd[j >> 2]);
    if constexpr (ONLY) return;
    const double gk = sc * pd;  // at lane k < j: w_k^T w_j
    double t = 0.0;
    static_for<0, j>([&](auto KK) {
      constexpr int k = decltype(KK)::value;
      t = fma(trow[k], row_bcast64<k>(gk), t);
    });
    trow[j] = (c < j) ? -tau * t : (c == j ? tau : 0.0);
    if (c == j) sc = scale;
    // T's column is done before the next column's passes start (volatile asm statements keep
    // their order): left to the scheduler, the recurrences of all 16 columns sink to the end of
    // the panel and hold about 170 more registers, which spilled at every width from 4 blocks on
    asm volatile("" : "+v"(trow[j]));
  });
}

__device__ __forceinline__ d4 mfma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// A factored panel in LDS at `keep`: T (row stride kF64Ld), the 16 column scales and the raw
// reflector columns W, RBN blocks of 16 x 16.
template <int RBN>
__device__ __forceinline__ void panel_keep64(double* __restrict__ keep, const double (&trow)[16], double sc,
                                             const d4 (&X)[RBN], int lane) {
  const int g = lane >> 4;
  const int c = lane & 15;
  if (g == 0) {
#pragma unroll
    for (int k = 0; k < 16; ++k) keep[c * kF64Ld + k] = trow[k];
    keep[kF64Blk + c] = sc;
  }
#pragma unroll
  for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) keep[kF64Stage + rb * kF64Blk + (4 * v + g) * kF64Ld + c] = X[rb][v];
  wave_lds_sync();
}

// The operands of a kept panel's application: T and the scales in the accumulator layout, and
// -W transposed.
template <int RBN>
struct Wy64 {
  d4 Td, srow;
  d4 Wt[RBN];
  __device__ __forceinline__ void load(const double* __restrict__ keep, int lane) {
    const int g = lane >> 4;
    const int c = lane & 15;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      Td[v] = keep[(4 * v + g) * kF64Ld + c];
      srow[v] = keep[kF64Blk + 4 * v + g];
    }
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v) Wt[rb][v] = -keep[kF64Stage + rb * kF64Blk + c * kF64Ld + 4 * v + g];
  }
  // Z = Rq + diag(s) Y;  Z' = T^T Z;  Rq -= Z';  returns diag(s) Z'
  __device__ __forceinline__ d4 small(d4& Rq, const d4& Y) const {
    const d4 Z = Rq + srow * Y;
    d4 Zp = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int v = 0; v < 4; ++v) Zp = mfma64(Td[v], Z[v], Zp);
    Rq -= Zp;
    return srow * Zp;
  }
};

// Merge the dense tile X (NRB block rows, L columns) into the running triangle R; the block rows from RL on
// are in LDS at rl (block t at (t - first) * 256, lane-major).
template <int NCB, int NRB, int RL>
__device__ __forceinline__ void merge_tile64(d4 (&R)[Tri64<NCB>::count], d4 (&X)[NRB][NCB], double* __restrict__ lds,
                                             double* __restrict__ rl, int lane, int L) {
  constexpr int first = Tri64<NCB>::idx(RL, RL);
  auto tri = [&](int t) -> d4* { return reinterpret_cast<d4*>(rl + (t - first) * 256 + lane * 4); };
  static_for<0, NCB>([&](auto PP) {
    constexpr int P = decltype(PP)::value;
    constexpr int rp = Tri64<NCB>::idx(P, P);
    double trow[16], sc;
    d4 Xp[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) Xp[rb] = X[rb][P];
    if constexpr (P < RL) {
      panel_factor64<NRB, NCB == 1>(R[rp], Xp, trow, sc, lane, L);
    } else {
      d4 Rd = *tri(rp);
      panel_factor64<NRB, NCB == 1>(Rd, Xp, trow, sc, lane, L);
      *tri(rp) = Rd;
    }
    if constexpr (P + 1 < NCB) {
      panel_keep64<NRB>(lds, trow, sc, Xp, lane);
      Wy64<NRB> wy;
      wy.load(lds, lane);
      wave_lds_sync();
      static_for<P + 1, NCB>([&](auto QQ) {
        // one column block's products at a time (interleaved, they spill)
        __builtin_amdgcn_sched_barrier(0);
        constexpr int q = decltype(QQ)::value;
        constexpr int rq = Tri64<NCB>::idx(P, q);
        d4 Y0 = {0.0, 0.0, 0.0, 0.0}, Y1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (v & 1)
              Y1 = mfma64(Xp[rb][v], X[rb][q][v], Y1);
            else
              Y0 = mfma64(Xp[rb][v], X[rb][q][v], Y0);
          }
        d4 Zs;
        if constexpr (P < RL) {
          Zs = wy.small(R[rq], Y0 + Y1);
        } else {
          d4 Rq = *tri(rq);
          Zs = wy.small(Rq, Y0 + Y1);
          *tri(rq) = Rq;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb) X[rb][q] = mfma64(wy.Wt[rb][v], Zs[v], X[rb][q]);
      });
    }
  });
}

// Leaves of the problems with NCB column blocks: wave w is global leaf leaf_begin + w, leaf li of
// problem p, and streams rows [li * rows_per_leaf, ...) of the problem's reduced rows (leaf 0
// starts from diag(sqrt(lam_p) d_B)).  Its triangle goes to the problem's slot li, or, when the
// problem has one leaf, row-major to R_B | c_B.
template <int NCB>
__global__ void __launch_bounds__(256)
k_tsqr64_leaf(int leaf_begin, int nleaves_cls, const int32_t* __restrict__ leaf_prob,
              const int32_t* __restrict__ leaf_idx, const ProbDesc* __restrict__ probs, int n,
              const double* __restrict__ Red, const double* __restrict__ d, const double* __restrict__ lamv,
              double* __restrict__ slots, double* __restrict__ RBall) {
  constexpr int NRB = leaf_tile_rows_f64(NCB) / 16;
  constexpr int RL = leaf_reg_rows_f64(NCB);
  constexpr int NT = Tri64<NCB>::count;
  constexpr int first = Tri64<NCB>::idx(RL, RL);
  constexpr int KT = 16 * NRB;
  __shared__ double stage_all[4][kF64Stage + NRB * kF64Blk];
  __shared__ double rl_all[4][NT > first ? (NT - first) * 256 : 1];
  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  const int wl = blockIdx.x * 4 + wv;
  if (wl >= nleaves_cls) return;
  const int pi = leaf_prob[leaf_begin + wl], leaf = leaf_idx[leaf_begin + wl];
  double* rl = rl_all[wv];
  const ProbDesc& P = probs[pi];
  const double* Xg = Red + P.redoff;
  const int64_t ldx = P.ldr;
  const int L = P.L;
  const int g = lane >> 4;
  const int c = lane & 15;

  d4 R[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) R[t] = d4{0.0, 0.0, 0.0, 0.0};
  if (leaf == 0) {
    const double* dB = d + P.noff + P.K * n;
    const double sqrt_lam = sqrt(lamv[pi]);
    static_for<0, NCB>([&](auto QQ) {
      constexpr int Q = decltype(QQ)::value;
      const int col = 16 * Q + c;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (4 * v + g == c && col < L - 1) R[Tri64<NCB>::idx(Q, Q)][v] = sqrt_lam * dB[col];
    });
  }
#pragma unroll
  for (int t = first; t < NT; ++t) *reinterpret_cast<d4*>(rl + (t - first) * 256 + lane * 4) = R[t];

  const int64_t r0 = (int64_t)leaf * P.rows_per_leaf;
  const int64_t r1 = r0 + P.rows_per_leaf < P.M ? r0 + P.rows_per_leaf : P.M;
  for (int64_t t = r0; t < r1; t += KT) {
    d4 X[NRB][NCB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int q = 0; q < NCB; ++q) {
        const int col = 16 * q + c;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t row = t + rb * 16 + 4 * v + g;
          X[rb][q][v] = (row < r1 && col < L) ? __builtin_nontemporal_load(Xg + row * ldx + col) : 0.0;
        }
      }
    __builtin_amdgcn_sched_barrier(0);
    merge_tile64<NCB, NRB, RL>(R, X, stage_all[wv], rl, lane, L);
  }
#pragma unroll
  for (int t = first; t < NT; ++t) R[t] = *reinterpret_cast<const d4*>(rl + (t - first) * 256 + lane * 4);

  if (P.leaves > 1) {
    double* dst = slots + P.slot0 + (int64_t)leaf * Tri64<NCB>::slot;
#pragma unroll
    for (int t = 0; t < NT; ++t) *reinterpret_cast<d4*>(dst + t * 256 + lane * 4) = R[t];
    return;
  }
  double* Rout = RBall + P.rboff;
  static_for<0, NCB>([&](auto PP) {
    constexpr int Q = decltype(PP)::value;
    static_for<0, NCB>([&](auto QQ) {
      constexpr int q = decltype(QQ)::value;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * Q + 4 * v + g;
        const int col = 16 * q + c;
        double val = 0.0;
        if constexpr (q >= Q) val = (col >= row) ? R[Tri64<NCB>::idx(Q, q)][v] : 0.0;
        if (row < L && col < L) Rout[(int64_t)row * L + col] = val;
      }
    });
  });
}

// ---- merge tree -------------------------------------------------------------------------------
// Kept panels of a node in LDS: panel p has p + 1 blocks of W.
template <int NCB>
struct TreeKeep64 {
  static constexpr int off(int p) { return p * kF64Stage + kF64Blk * (p * (p + 1) / 2); }
  static constexpr int total = NCB > 1 ? off(NCB - 1) : 1;  // the last panel is applied to nothing
};
// Nodes (waves) per workgroup: as many as the kept panels (20 KiB per wave at 4 column blocks,
// 75 KiB at 8) leave room for in 160 KiB of LDS, at most four.
constexpr int tree_waves_f64(int ncb) { return ncb <= 5 ? 4 : (ncb == 6 ? 3 : 2); }

// Published blocks move with device-coherent accesses (sc1), as in tsqr_tree.hpp: the producer
// waits for its stores before the flag, the consumer reads past the per-XCD L2.
typedef unsigned u4 __attribute__((ext_vector_type(4)));
constexpr int kCoherent64 = 16;
__device__ __forceinline__ void tree_store64(double* dst, const d4& v, int lane) {
  const auto rs = __builtin_amdgcn_make_buffer_rsrc(dst, 0, 2048, 0x00020000);
  const uint64_t a = __builtin_bit_cast(uint64_t, (double)v[0]), b = __builtin_bit_cast(uint64_t, (double)v[1]);
  const uint64_t e = __builtin_bit_cast(uint64_t, (double)v[2]), f = __builtin_bit_cast(uint64_t, (double)v[3]);
  const u4 lo = {(unsigned)a, (unsigned)(a >> 32), (unsigned)b, (unsigned)(b >> 32)};
  const u4 hi = {(unsigned)e, (unsigned)(e >> 32), (unsigned)f, (unsigned)(f >> 32)};
  __builtin_amdgcn_raw_buffer_store_b128(lo, rs, lane * 32, 0, kCoherent64);
  __builtin_amdgcn_raw_buffer_store_b128(hi, rs, lane * 32 + 16, 0, kCoherent64);
}
__device__ __forceinline__ d4 tree_load64(const double* src, int lane) {
  const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(src), 0, 2048, 0x00020000);
  const u4 lo = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 32, 0, kCoherent64);
  const u4 hi = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 32 + 16, 0, kCoherent64);
  d4 r;
  r[0] = __builtin_bit_cast(double, ((uint64_t)lo[1] << 32) | lo[0]);
  r[1] = __builtin_bit_cast(double, ((uint64_t)lo[3] << 32) | lo[2]);
  r[2] = __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | hi[0]);
  r[3] = __builtin_bit_cast(double, ((uint64_t)hi[3] << 32) | hi[2]);
  return r;
}
// One wave per inner node of the trees of every problem with NCB column blocks, an entry each of the
// tables from node_begin on: node node_idx of problem node_prob with children node_l / node_r (>= 0 a
// node of the same problem, < 0 its leaf -1 - r).  The entries are in level order over all the
// problems and workgroups take them as they start (tree_first_entry), so a node's children are
// leaves (the launch before) or entries of waves that have started.  Every wait is bounded all the
// same; a timeout sets the problem's ST_STALL bit and the wave still publishes every block.  Leaf
// triangles are at the problem's slots 0 .. leaves - 1, node outputs at slots leaves + node;
// flags[(node NCB + q) 2 + k] at the problem's ctr0 (cleared by the factor call's first launch): k = 0
// the blocks above the diagonal of column block q, 1 its diagonal block.
template <int NCB>
__global__ void __launch_bounds__(64 * tree_waves_f64(NCB))
k_tsqr64_tree(int node_begin, int nnodes, const int32_t* __restrict__ node_prob, const int32_t* __restrict__ node_idx,
              const int32_t* __restrict__ node_l, const int32_t* __restrict__ node_r,
              const ProbDesc* __restrict__ probs, double* slots, int* flags, int* ticket, double* __restrict__ RBall,
              int* status) {
  constexpr int WPG = tree_waves_f64(NCB);
  __shared__ double keep_all[WPG][TreeKeep64<NCB>::total];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int entry = tree_first_entry<WPG>(ticket) + wv;
  if (entry >= nnodes) return;
  const int pi = node_prob[node_begin + entry];
  const int node = node_idx[node_begin + entry];
  const int lref = node_l[node_begin + entry], rref = node_r[node_begin + entry];
  const ProbDesc& P = probs[pi];
  const int L = P.L;
  const int nleaves = P.leaves;
  constexpr int SLOT = Tri64<NCB>::slot;
  double* pslots = slots + P.slot0;
  int* pflags = flags + P.ctr0;
  const double* lsrc = pslots + (int64_t)(lref >= 0 ? nleaves + lref : -1 - lref) * SLOT;
  const double* rsrc = pslots + (int64_t)(rref >= 0 ? nleaves + rref : -1 - rref) * SLOT;
  double* out = pslots + (int64_t)(nleaves + node) * SLOT;
  const bool root = node == nleaves - 2;
  double* keep = keep_all[wv];
  const int g = lane >> 4;
  const int c = lane & 15;
  bool stalled = false;
  d4 a[NCB];  // column block q: R part (left child), block rows 0..q
  d4 x[NCB];  // column block q: tile (right child), block rows 0..q
  auto load_blocks = [&](int p, int q, d4& av, d4& xv) {
    const double* ls = lsrc + Tri64<NCB>::idx(p, q) * 256;
    const double* rs = rsrc + Tri64<NCB>::idx(p, q) * 256;
    av = lref >= 0 ? tree_load64(ls, lane) : *reinterpret_cast<const d4*>(ls + lane * 4);
    xv = rref >= 0 ? tree_load64(rs, lane) : *reinterpret_cast<const d4*>(rs + lane * 4);
  };
  auto publish = [&](int q, int k) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0)
      __hip_atomic_store(pflags + ((int64_t)node * NCB + q) * 2 + k, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // the children's flags (a leaf child counts as published: the other child's flags stand in)
  const bool inner = lref >= 0 || rref >= 0;
  const int* fl = pflags + (int64_t)(lref >= 0 ? lref : rref) * NCB * 2;
  const int* fr = pflags + (int64_t)(rref >= 0 ? rref : lref) * NCB * 2;
  int seen = inner ? tree_look(fl, fr, 0, lane) : 1;
  auto wait_children = [&](int q, int k) {
    if (!stalled && inner) stalled = !tree_wait(seen, fl, fr, q, k, lane);
    asm volatile("" ::: "memory");  // the block's loads stay after the flags were seen
  };
  static_for<0, NCB>([&](auto QQ) {
    constexpr int q = decltype(QQ)::value;
    bool have_diag = false;
    if constexpr (q > 0) {
      // above the diagonal: panels 0..q-1 applied, then published (the diagonal block is loaded here
      // too when it is there already)
      wait_children(q, 0);
      have_diag = stalled || tree_seen(seen, 1);
#pragma unroll
      for (int p = 0; p < q; ++p) load_blocks(p, q, a[p], x[p]);
      if (have_diag)
        load_blocks(q, q, a[q], x[q]);
      else
        seen = tree_look(fl, fr, q, lane);
      static_for<0, q>([&](auto PP) {
        constexpr int p = decltype(PP)::value;
        const double* kp = keep + TreeKeep64<NCB>::off(p);
        Wy64<p + 1> wy;
        wy.load(kp, lane);
        d4 Y0 = {0.0, 0.0, 0.0, 0.0}, Y1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int rb = 0; rb <= p; ++rb)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double w = kp[kF64Stage + rb * kF64Blk + (4 * v + g) * kF64Ld + c];
            if (v & 1)
              Y1 = mfma64(w, x[rb][v], Y1);
            else
              Y0 = mfma64(w, x[rb][v], Y0);
          }
        const d4 Zs = wy.small(a[p], Y0 + Y1);
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int rb = 0; rb <= p; ++rb) x[rb] = mfma64(wy.Wt[rb][v], Zs[v], x[rb]);
      });
      if (!root) {
#pragma unroll
        for (int p = 0; p < q; ++p) tree_store64(out + Tri64<NCB>::idx(p, q) * 256, a[p], lane);
        publish(q, 0);
      }
    }
    // the diagonal block: panel q factored, then published
    if (!have_diag) {
      wait_children(q, 1);
      load_blocks(q, q, a[q], x[q]);
    }
    if (q + 1 < NCB && inner) seen = tree_look(fl, fr, q + 1, lane);
    {
      double trow[16], sc;
      d4 Xp[q + 1];
#pragma unroll
      for (int rb = 0; rb <= q; ++rb) Xp[rb] = x[rb];
      panel_factor64<q + 1, NCB == 1>(a[q], Xp, trow, sc, lane, L);
      if constexpr (q + 1 < NCB) panel_keep64<q + 1>(keep + TreeKeep64<NCB>::off(q), trow, sc, Xp, lane);
    }
    if (root) {
      // column block q of R_B | c_B, row-major L x L (zeros below the diagonal)
      double* Rout = RBall + P.rboff;
      static_for<0, NCB>([&](auto PR) {
        constexpr int p = decltype(PR)::value;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 16 * p + 4 * v + g;
          const int col = 16 * q + c;
          double val = 0.0;
          if constexpr (p < q) val = a[p][v];
          if constexpr (p == q) val = (col >= row) ? a[p][v] : 0.0;
          if (row < L && col < L) Rout[(int64_t)row * L + col] = val;
        }
      });
    } else {
      tree_store64(out + Tri64<NCB>::idx(q, q) * 256, a[q], lane);
      publish(q, 1);
    }
  });
  if (stalled) set_status(status + pi, ST_STALL);
}

template <int NCB>
hipError_t launch_tsqr64_leaf_n(int leaf_begin, int count, const int32_t* leaf_prob, const int32_t* leaf_idx,
                                const ProbDesc* probs, int n, const double* Red, const double* d, const double* lam,
                                double* slots, double* RB, hipStream_t st);
template <int NCB>
hipError_t launch_tsqr64_tree_n(int node_begin, int count, const int32_t* node_prob, const int32_t* node_idx,
                                const int32_t* node_l, const int32_t* node_r, const ProbDesc* probs, double* slots,
                                int* flags, int* ticket, double* RB, int* status, hipStream_t st);

// The launches of one column-block count (one translation unit each, tsqr_f64_<N>.hip).
#define QRK_TSQR64_INST(NCB)                                                                                     \
  template <>                                                                                                    \
  hipError_t launch_tsqr64_leaf_n<NCB>(int leaf_begin, int count, const int32_t* leaf_prob,                      \
                                       const int32_t* leaf_idx, const ProbDesc* probs, int n, const double* Red, \
                                       const double* d, const double* lam, double* slots, double* RB,            \
                                       hipStream_t st) {                                                         \
    hipLaunchKernelGGL((k_tsqr64_leaf<NCB>), dim3((unsigned)((count + 3) / 4)), dim3(256), 0, st, leaf_begin,    \
                       count, leaf_prob, leaf_idx, probs, n, Red, d, lam, slots, RB);                            \
    return hipGetLastError();                                                                                    \
  }                                                                                                              \
  template <>                                                                                                    \
  hipError_t launch_tsqr64_tree_n<NCB>(int node_begin, int count, const int32_t* node_prob,                      \
                                       const int32_t* node_idx, const int32_t* node_l, const int32_t* node_r,    \
                                       const ProbDesc* probs, double* slots, int* flags, int* ticket,            \
                                       double* RB, int* status, hipStream_t st) {                                \
    constexpr int W = tree_waves_f64(NCB);                                                                       \
    hipLaunchKernelGGL((k_tsqr64_tree<NCB>), dim3((unsigned)((count + W - 1) / W)), dim3(64 * W), 0, st,         \
                       node_begin, count, node_prob, node_idx, node_l, node_r, probs, slots, flags, ticket, RB,  \
                       status);                                                                                  \
    return hipGetLastError();                                                                                    \
  }

}  // namespace qrk
