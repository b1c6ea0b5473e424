// Streams of rows through registers, shared by the solve kernels and the adjoint.
#pragma once

#include "qrk_device.hpp"

namespace qrk {

// ---------------------------------------------------------------------------------
// Rows of a pack (B's or S|c's) streamed through registers.  A row of at most CW columns (16, 32,
// 64 or 128, chosen per problem) takes min(CW, 64) lanes, so one load moves RPL = 1, 2 or 4 whole
// rows and a chunk of NV loads CHR = NV RPL rows: narrow dense parts use all lanes of a load.
// Lane (g, col): column col (and col + 64 at CW = 128) of rows i RPL + g.
//
// Row sums (B p_B, S v): every lane multiplies its values by its columns' entries, and the NV sums
// are folded across the lanes of a row in halving steps: a step adds two lanes' values for one half
// of the rows in one of the lanes and for the other half in the other, so NV values cost NV - 1
// folds, and each lane ends with one row's sum.  (Before, the chunk went through LDS transposed
// and each row was summed by four lanes: 128 columns of p_B per lane, 64 registers, held one wave
// less per SIMD.)  All sums run in a fixed order.  Bound: instruction issue and, in large problems, the
// stream itself.  Refinement pass 1 of 50,000 blocks of 12 x 3 with 91 columns 71 -> 54 us (4.0 -> 5.3
// TB/s of A, B, b and S|c), of 128 ragged problems with 6, 30 or 90 columns 1,670 -> 1,006 us; block solves there 275 -> 91
// us (units of 64 / n blocks instead of packs of 64 rows, and one load for up to four rows).
// ---------------------------------------------------------------------------------
template <typename T, int CW>
struct RowStream {
  static constexpr int LN = CW < 64 ? CW : 64;  // lanes of a row
  static constexpr int RPL = 64 / LN;
  static constexpr int NV = sizeof(T) == 4 ? 16 : 8;
  static constexpr int SL = CW > 64 ? 2 : 1;
  static constexpr int CHR = NV * RPL;
  // row of a chunk whose sum the lane holds after fold_rows
  static __device__ __forceinline__ int sum_row(int lane) {
    return ((lane & (LN - 1)) / (LN / NV)) * RPL + lane / LN;
  }
};

template <typename T, int CW>
using StreamChunk = T[RowStream<T, CW>::SL][RowStream<T, CW>::NV];

// Raw buffer load of one element: the descriptor holds the wave-uniform base, the row offset is the
// scalar offset and the lane's column (and row of the load) the vector offset.  Word 3 is the gfx9
// raw-buffer format; the record count only bounds the range check, and every offset used stays
// inside the rows of the pack, or is kNoColumn, which the range check answers with zero.
constexpr uint32_t kNoColumn = 0x80000000u;
template <typename T>
__device__ __forceinline__ T buf_ld_row(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff, (int)soff, 0));
}

// Loads one chunk (rows c0 .. of `rows` rows of stride ld, ncol columns); rows past the last one
// re-read it.
template <typename T, int CW>
__device__ __forceinline__ void stream_load(StreamChunk<T, CW>& v,
                                            __amdgpu_buffer_rsrc_t rs, int c0, int rows, int ld, int ncol, int lane) {
  using S = RowStream<T, CW>;
  const int g = lane / S::LN, col = lane & (S::LN - 1);
  const int lastg = (rows - 1) / S::RPL * S::RPL;  // first row of the last load that holds a row
  const int gl = lastg + g < rows ? g : rows - 1 - lastg;
  const uint32_t full = (uint32_t)(g * ld + col) * (uint32_t)sizeof(T);
  const uint32_t last = (uint32_t)(gl * ld + col) * (uint32_t)sizeof(T);
  const uint32_t o0 = col < ncol ? full : kNoColumn, l0 = col < ncol ? last : kNoColumn;
  const uint32_t o1 = col + 64 < ncol ? full + 64u * sizeof(T) : kNoColumn;
#pragma unroll
  for (int i = 0; i < S::NV; ++i) {
    const int r = c0 + i * S::RPL;
    const int rc = r < lastg ? r : lastg;
    const uint32_t so = (uint32_t)(rc * ld) * (uint32_t)sizeof(T);
    v[0][i] = buf_ld_row<T>(rs, S::RPL > 1 && r >= lastg ? l0 : o0, so);
    if constexpr (S::SL == 2) v[1][i] = buf_ld_row<T>(rs, o1, so);
  }
}

__device__ __forceinline__ double mk_double(unsigned lo, unsigned hi) {
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int CTRL, int BANK>
__device__ __forceinline__ double dpp_into(double old, double x) {
  const uint64_t o = __builtin_bit_cast(uint64_t, old), v = __builtin_bit_cast(uint64_t, x);
  const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)o, (int)(unsigned)v, CTRL, 0xF, BANK, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(o >> 32), (int)(unsigned)(v >> 32), CTRL, 0xF, BANK, false);
  return mk_double((unsigned)lo, (unsigned)hi);
}
// x, which with FRESH the compiler cannot identify with x: a chunk is then converted to double anew
// for its second use, else the converted values (twice the registers) are kept from the first.  Kept
// they cost registers up to the two waves per SIMD that pass 1's grid fills, and save conversions:
// n = 3, 91 columns, 50,000 blocks 54.0 us kept, 57.2 fresh; from n = 6 on they would leave one wave.
template <bool FRESH, typename T>
__device__ __forceinline__ T second_use(T x) {
  if constexpr (FRESH) asm("" : "+v"(x));
  return x;
}
// Fold step ST (lanes l and l ^ 32, 16, 15, 7, 2, 1): lanes with the step's bit clear (5, 4, 3, 2,
// 1, 0) return a's sum over the pair, the others b's.
template <int ST>
__device__ __forceinline__ double fold2(double a, double b, int lane) {
  const uint64_t ua = __builtin_bit_cast(uint64_t, a), ub = __builtin_bit_cast(uint64_t, b);
  if constexpr (ST == 0) {
    auto x = __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false);
    auto y = __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    return mk_double(x[0], y[0]) + mk_double(x[1], y[1]);
  } else if constexpr (ST == 1) {
    auto x = __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
    auto y = __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    return mk_double(x[0], y[0]) + mk_double(x[1], y[1]);
  } else if constexpr (ST == 2 || ST == 3) {
    constexpr int ctrl = ST == 2 ? 0x140 : 0x141;   // row_mirror, row_half_mirror
    constexpr int hi = ST == 2 ? 0xC : 0xA;         // banks with bit 3 (bit 2) of the lane set
    const double t = dpp_into<ctrl, hi>(dpp_into<ctrl, 0xF ^ hi>(a, a), b);
    const double k = dpp_into<0xE4, hi>(a, b);      // quad_perm identity
    return k + t;
  } else {
    constexpr int ctrl = ST == 4 ? 0x4E : 0xB1;     // quad_perm xor 2, xor 1
    const bool up = lane & (ST == 4 ? 2 : 1);
    const double send = up ? a : b, k = up ? b : a;
    return k + dpp_into<ctrl, 0xF>(send, send);
  }
}
template <int ST>
__device__ __forceinline__ double fold1(double a) {
  if constexpr (ST <= 1) {
    const uint64_t u = __builtin_bit_cast(uint64_t, a);
    return fold2<ST>(a, mk_double(opaque_copy((unsigned)u), opaque_copy((unsigned)(u >> 32))), 0);
  } else {
    constexpr int ctrl = ST == 2 ? 0x140 : (ST == 3 ? 0x141 : (ST == 4 ? 0x4E : 0xB1));
    return a + dpp_into<ctrl, 0xF>(a, a);
  }
}
template <int ST, int M, int NV>
__device__ __forceinline__ void fold_steps(double (&s)[NV], int lane) {
  if constexpr (ST <= 5) {
    if constexpr (M > 1) {
#pragma unroll
      for (int i = 0; i < M / 2; ++i) s[i] = fold2<ST>(s[i], s[i + M / 2], lane);
      fold_steps<ST + 1, M / 2, NV>(s, lane);
    } else {
      s[0] = fold1<ST>(s[0]);
      fold_steps<ST + 1, 1, NV>(s, lane);
    }
  }
}
// Sum of row RowStream::sum_row(lane) of a chunk over its columns, w0 / w1 the lane's columns'
// factors.
template <typename T, int CW>
__device__ __forceinline__ double stream_dot(const StreamChunk<T, CW>& v, double w0,
                                             double w1, int lane) {
  using S = RowStream<T, CW>;
  double s[S::NV];
#pragma unroll
  for (int i = 0; i < S::NV; ++i) {
    s[i] = (double)v[0][i] * w0;
    if constexpr (S::SL == 2) s[i] += (double)v[1][i] * w1;
  }
  fold_steps<S::LN == 64 ? 0 : (S::LN == 32 ? 1 : 2), S::NV, S::NV>(s, lane);
  return s[0];
}

// f(CW) for ncol columns
template <typename F>
__device__ __forceinline__ void stream_width(int ncol, F&& f) {
  if (ncol <= 16)
    f(std::integral_constant<int, 16>{});
  else if (ncol <= 32)
    f(std::integral_constant<int, 32>{});
  else if (ncol <= 64)
    f(std::integral_constant<int, 64>{});
  else
    f(std::integral_constant<int, 128>{});
}

}  // namespace qrk
