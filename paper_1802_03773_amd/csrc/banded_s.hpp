// Banded Givens QR as a ring of lanes, one row of R per lane (the banded class of QRkit Section
// 4.4, rotations of Section 2), for every band width W = 1 .. 31, and the triangular sweeps for
// 16 <= w <= 31.
//
// What is computed: R starts as diag(sqrt(lam) d) and every row of J (its b_i riding along) is
// rotated into R in row order, one rotation per column of the row, as in every version before.
//
// Organisation (the linear systolic array of Gentleman and Kung 1981).  Lane j mod RING of a
// problem's group holds row j of R: R[j][j .. j + W - 1] and c_j.  A row x of J with start s enters
// at lane s and moves to the next lane at every step, so at a step every lane rotates the row that
// it holds with its own row of R, all lanes in the same instructions; a row leaves the last of its
// W lanes with nothing left.  The row is held relative to the lane's column, so that a move is a
// DPP ring rotation and a renaming of registers.  At every step a group either enters its next
// row (when that row starts at the current column s) or retires row s of R and moves s on; a row
// entered a step later than the one before it always finds that one a lane ahead.  M + N steps in
// all, whatever the starts.  Live rows of R are s .. s + W - 1, so a ring of RING >= W lanes holds
// them: 16 lanes (four problems per wave) up to W = 16, a whole wave above.
//
// What bounds it: the issue of one wave, about 4 W + 50 instructions a step; rows wait in LDS (chunks
// loaded one chunk ahead of the one in use, the next row read a step ahead), and so do retired rows,
// so a step waits for no memory.  The kernels before it kept a problem's rows in a dependency chain
// of rotations (one row, or two of equal start, in flight).  Factor, float32, two rows per column:
// 50 problems of N = 1001, w = 24: 9.10 -> 1.21 ms; 2,048 of N = 2,048: w = 4 1.90 -> 1.56, w = 12
// 2.58 -> 2.19, w = 15 2.90 -> 2.28 ms; 8,192 of N = 1,024, w = 12: 2.25 -> 1.36 ms; float64, 64 of
// N = 1,024: w = 12 2.28 -> 1.22, w = 31 13.3 -> 2.0 ms.  Doing a step's other columns during the next
// step's chain (software pipelining) was 3 to 8% slower: the issue, not the chain, is full.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qrk_banded.hpp"
#include "qrk_device.hpp"

namespace qrk {

// One move of the ring: every lane takes the values of the lane before it (lane 0 those of the
// last), or, where `mask` is set, its `in`.  Move and select are one instruction (v_cndmask with a
// DPP source).  s_nop 1: a DPP source must not have been written by the VALU in the two cycles
// before, which the compiler does not track into an asm statement.
template <int RING>
__device__ __forceinline__ void bs_move1(uint32_t& y, uint32_t in, uint64_t mask) {
  if constexpr (RING == 16)
    asm("s_mov_b64 vcc, %2\n\ts_nop 1\n\tv_cndmask_b32_dpp %0, %0, %1, vcc row_ror:1 row_mask:0xf bank_mask:0xf"
        : "+v"(y) : "v"(in), "s"(mask) : "vcc");
  else
    asm("s_mov_b64 vcc, %2\n\ts_nop 1\n\tv_cndmask_b32_dpp %0, %0, %1, vcc wave_ror:1 row_mask:0xf bank_mask:0xf"
        : "+v"(y) : "v"(in), "s"(mask) : "vcc");
}
template <int RING>
__device__ __forceinline__ void bs_move8(uint32_t (&y)[8], const uint32_t (&in)[8], uint64_t mask) {
#define QRK_BS_MOVE8(ROT)                                                                        \
  asm("s_mov_b64 vcc, %16\n\ts_nop 1\n\t"                                                        \
      "v_cndmask_b32_dpp %0, %0, %8, vcc " ROT " row_mask:0xf bank_mask:0xf\n\t"                 \
      "v_cndmask_b32_dpp %1, %1, %9, vcc " ROT " row_mask:0xf bank_mask:0xf\n\t"                 \
      "v_cndmask_b32_dpp %2, %2, %10, vcc " ROT " row_mask:0xf bank_mask:0xf\n\t"                \
      "v_cndmask_b32_dpp %3, %3, %11, vcc " ROT " row_mask:0xf bank_mask:0xf\n\t"                \
      "v_cndmask_b32_dpp %4, %4, %12, vcc " ROT " row_mask:0xf bank_mask:0xf\n\t"                \
      "v_cndmask_b32_dpp %5, %5, %13, vcc " ROT " row_mask:0xf bank_mask:0xf\n\t"                \
      "v_cndmask_b32_dpp %6, %6, %14, vcc " ROT " row_mask:0xf bank_mask:0xf\n\t"                \
      "v_cndmask_b32_dpp %7, %7, %15, vcc " ROT " row_mask:0xf bank_mask:0xf"                     \
      : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]), "+v"(y[4]), "+v"(y[5]), "+v"(y[6]), "+v"(y[7]) \
      : "v"(in[0]), "v"(in[1]), "v"(in[2]), "v"(in[3]), "v"(in[4]), "v"(in[5]), "v"(in[6]), "v"(in[7]), \
        "s"(mask)                                                                                \
      : "vcc")
  if constexpr (RING == 16)
    QRK_BS_MOVE8("row_ror:1");
  else
    QRK_BS_MOVE8("wave_ror:1");
#undef QRK_BS_MOVE8
}
// N values at once: as 32-bit words, eight words a block.
template <int RING, typename T, int N>
__device__ __forceinline__ void bs_move(T (&y)[N], const T (&in)[N], uint64_t mask) {
  constexpr int K = (int)sizeof(T) / 4;
  uint32_t w[N * K], v[N * K];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if constexpr (K == 1) {
      w[i] = __builtin_bit_cast(uint32_t, y[i]);
      v[i] = __builtin_bit_cast(uint32_t, in[i]);
    } else {
      const uint64_t a = __builtin_bit_cast(uint64_t, y[i]), b = __builtin_bit_cast(uint64_t, in[i]);
      w[2 * i] = (uint32_t)a;
      w[2 * i + 1] = (uint32_t)(a >> 32);
      v[2 * i] = (uint32_t)b;
      v[2 * i + 1] = (uint32_t)(b >> 32);
    }
  }
#pragma unroll
  for (int i = 0; i + 7 < N * K; i += 8) {
    uint32_t p[8] = {w[i], w[i + 1], w[i + 2], w[i + 3], w[i + 4], w[i + 5], w[i + 6], w[i + 7]};
    const uint32_t q[8] = {v[i], v[i + 1], v[i + 2], v[i + 3], v[i + 4], v[i + 5], v[i + 6], v[i + 7]};
    bs_move8<RING>(p, q, mask);
#pragma unroll
    for (int k = 0; k < 8; ++k) w[i + k] = p[k];
  }
#pragma unroll
  for (int i = N * K / 8 * 8; i < N * K; ++i) bs_move1<RING>(w[i], v[i], mask);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if constexpr (K == 1)
      y[i] = __builtin_bit_cast(T, w[i]);
    else
      y[i] = __builtin_bit_cast(T, ((uint64_t)w[2 * i + 1] << 32) | w[2 * i]);
  }
}

// 1 / sqrt(q) for normal q > 0, the hardware estimate (1 ulp in float32, about 24 bits in float64)
// with one and two Newton steps.
__device__ __forceinline__ float bs_rsqrt(float q) {
  const float y = __builtin_amdgcn_rsqf(q);
  return fmaf(0.5f * y, fmaf(-q * y, y, 1.f), y);
}
__device__ __forceinline__ double bs_rsqrt(double q) {
  double y = __builtin_amdgcn_rsq(q);
  y = fma(0.5 * y, fma(-q * y, y, 1.0), y);
  return fma(0.5 * y, fma(-q * y, y, 1.0), y);
}
__device__ __forceinline__ float bs_rcp(float t) {
  const float y = __builtin_amdgcn_rcpf(t);
  return fmaf(y, fmaf(-t, y, 1.f), y);
}
__device__ __forceinline__ double bs_rcp(double t) {
  double y = __builtin_amdgcn_rcp(t);
  y = fma(y, fma(-t, y, 1.0), y);
  return fma(y, fma(-t, y, 1.0), y);
}
template <typename T>
struct BsBits;
template <>
struct BsBits<float> {
  typedef uint32_t type;
};
template <>
struct BsBits<double> {
  typedef uint64_t type;
};
// The smallest normal number; twice its root, from which on a pivot keeps every squared norm normal; and
// the power of two by which a rotation's two inputs are multiplied when the sum of their squares is
// not: no square overflows or is subnormal then.
template <typename T>
struct BsTiny;
template <>
struct BsTiny<float> {
  static constexpr float value = 0x1p-126f;
  static constexpr float pivot = 0x1p-62f;
  static constexpr float up = 0x1p100f;
};
template <>
struct BsTiny<double> {
  static constexpr double value = 0x1p-1022;
  static constexpr double pivot = 0x1p-510;
  static constexpr double up = 0x1p700;
};

// c - a b into a register of its own: the row moves down one register at every step, and with the
// two-address form that the compiler prefers each move is a copy.
__device__ __forceinline__ float bs_fnma(float a, float b, float c) {
  float d;
  asm("v_fma_f32 %0, -%1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ double bs_fnma(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, -%1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// Four problems a wave up to W = 15.  A wave of one problem has scalar control and slightly shorter
// steps (W = 16, 50 problems of N = 1001: 0.96 ms against 1.06 on 16 lanes), but from a wave for each
// SIMD on it is the slower one (1,024 problems of N = 1,024, w = 12: 1.21 against 1.02 ms).
constexpr int bs_ring(int w) { return w <= 15 ? 16 : 64; }

template <typename T, int W>
struct BsShape {
  static constexpr int RING = bs_ring(W);
  static constexpr int GROUPS = 64 / RING;                     // problems per wave
  static constexpr int C = 32 * 4 / (int)sizeof(T);            // rows per chunk
  static constexpr int V = 16 / (int)sizeof(T);                // values per 16-byte LDS access
  static constexpr int WP = (W + 2 + V - 1) / V * V;           // row slot: W values, b, the start
  static constexpr int LOADS = (C * W + RING - 1) / RING;      // values of a chunk per lane
};

// Output as the other banded factorisations: band R [P][N][W], c [P][N], reciprocal pivots
// [P][N] and, when R16 is given (W <= 15), the sweep copy [P][N][16].
template <typename T, int W>
__global__ void __launch_bounds__(64)
k_bgivens_s(int P, int64_t M, int64_t N, const int32_t* __restrict__ row_start, const T* __restrict__ vals,
            const T* __restrict__ bvec, const double* __restrict__ d, const double* __restrict__ lam,
            T* __restrict__ Rb, T* __restrict__ cb, double* __restrict__ binv, T* __restrict__ R16,
            int* __restrict__ status) {
  using Sh = BsShape<T, W>;
  constexpr int RING = Sh::RING, C = Sh::C, WP = Sh::WP, V = Sh::V, LOADS = Sh::LOADS;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  // per group two chunks of rows; 16 words between the groups' banks, so that their reads of a
  // row do not collide
  constexpr int GST = 2 * C * WP + 64 / (int)sizeof(T);
  constexpr int WR = (W + V - 1) / V * V;           // slot of a retired row
  constexpr int GRT = RING * WR + 64 / (int)sizeof(T);
  __shared__ __align__(16) T rows_all[Sh::GROUPS * GST];
  __shared__ __align__(16) T done_all[Sh::GROUPS * GRT];
  const int lane = threadIdx.x & (RING - 1);
  const int grp = (threadIdx.x & 63) / RING;
  const int64_t prob = (int64_t)blockIdx.x * Sh::GROUPS + grp;
  if (prob >= P) return;
  T* rows = rows_all + grp * GST;
  T* done = done_all + grp * GRT;
  const double sl = sqrt(lam[prob]);
  const int32_t* rs = row_start + prob * M;
  const T* Vp = vals + prob * M * W;
  const T* bb = bvec + prob * M;
  const double* dd = d + prob * N;
  T* R = Rb + prob * N * W;
  T* cc = cb + prob * N;
  double* iv = binv + prob * N;
  T* S16 = (W <= 15 && R16) ? R16 + prob * N * 16 : nullptr;
  const int smax = (int)(N - W < 0x7fffffff ? N - W : 0x7fffffff);

  // ---- rows of J: chunk k is rows C k .. C k + C - 1, in LDS buffer k & 1 ---------------------
  constexpr int HEADS = (C + RING - 1) / RING;
  T pv[LOADS], pb[HEADS];
  int32_t ps[HEADS];
  auto fetch = [&](int64_t k) {  // chunk k into registers
    const int64_t i0 = k * C;
    const int64_t left = (M - i0) * W;  // values from here to the problem's last
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      const int e = lane + u * RING;
      pv[u] = (e < C * W && e < left) ? Vp[i0 * W + e] : T(0);
    }
#pragma unroll
    for (int u = 0; u < HEADS; ++u) {
      const bool in = lane + u * RING < C && i0 + lane + u * RING < M;
      pb[u] = in ? bb[i0 + lane + u * RING] : T(0);
      ps[u] = in ? rs[i0 + lane + u * RING] : 0;
    }
  };
  // Registers into chunk k's buffer.  The starts are clamped to the largest one before them and to
  // N - W (a scan over the chunk; a start that changes is bad input), and the slots past the last
  // row start nowhere.
  bool bad = false;
  int last = 0;
  auto stage = [&](int64_t k) {
    T* dst = rows + (int)(k & 1) * (C * WP);
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      const int e = lane + u * RING;
      if (e < C * W) dst[e / W * WP + e % W] = pv[u];
    }
#pragma unroll
    for (int u = 0; u < HEADS; ++u) {
      const int slot = lane + u * RING;
      const bool in = slot < C && k * C + slot < M;
      int st = in ? ps[u] : 0;
#pragma unroll
      for (int off = 1; off < RING; off <<= 1) {
        const int o = __shfl_up(st, off, RING);
        st = lane >= off && o > st ? o : st;
      }
      st = st > last ? st : last;
      st = st < smax ? st : smax;
      last = __shfl(st, RING - 1, RING);
      bad = bad || (in && st != ps[u]);
      if (slot < C) {
        dst[slot * WP + W] = pb[u];
        *reinterpret_cast<int32_t*>(dst + slot * WP + W + 1) = in ? st : -1;
      }
    }
  };
  // Wide bands: do all pivots start high enough for every squared norm to be normal (they only grow)?
  // Else (no damping, or tiny values) each step looks at its norms.
  bool low = false;
  if constexpr (W > 15) {
    for (int64_t j = lane; j < N; j += RING) low = low || (T)(sl * fabs(dd[j])) < BsTiny<T>::pivot;
    low = __ballot(low) != 0;
  }
  fetch(0);
  stage(0);
  fetch(1);
  stage(1);
  fetch(2);
  wave_lds_sync();

  // ---- state: the current column s, the next row (in chunk kc) and its start ------------------
  T Rw[W], Rc = T(0);  // this lane's row of R
  T x[W + 1];          // the row of J it holds and its b (in x[W]), relative to the lane's column
  T xin[W + 1];        // the next row and its b
#pragma unroll
  for (int l = 0; l < W; ++l) Rw[l] = T(0);
#pragma unroll
  for (int l = 0; l <= W; ++l) x[l] = T(0);
  uint32_t s = 0;
  int64_t kc = 0;
  int ic = 0;  // slot of the next row among the two chunks' (it wraps)
  int sn = 0;
  auto read_next = [&]() {  // exactly the values used: a wait for others would come early
    const T* src = rows + ic * WP;
    constexpr int FULL = (W + 2) / V;
#pragma unroll
    for (int u = 0; u < FULL; ++u) {
      const vec q = *reinterpret_cast<const vec*>(src + u * V);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if (u * V + v <= W)
          xin[u * V + v] = q[v];
        else
          sn = (int)__builtin_bit_cast(typename BsBits<T>::type, (T)q[v]);
      }
    }
#pragma unroll
    for (int e = FULL * V; e <= W; ++e) xin[e] = src[e];
    if constexpr (FULL * V <= W + 1) sn = *reinterpret_cast<const int32_t*>(src + W + 1);
  };
  // damping values of the lanes' next rows: block s / RING of columns is current, the lanes that
  // retire in it take their row of the next block (past the last column the last one's, so that no
  // lane divides by zero).  Their size: the rotation needs pivots >= 0, and a row's sign is free; taken
  // after the conversion: taken at the load, every block waits for its load (300 problems of 807 columns,
  // W = 18: 916 us against 893 in float32, 1,347 against 1,308 in float64).
  auto load_d = [&](int64_t col) -> double { return dd[col < N ? col : N - 1]; };
  Rw[0] = fabs((T)(sl * load_d(lane)));
  T dnext = fabs((T)(sl * load_d((int64_t)RING + lane)));
  double dload = load_d((int64_t)2 * RING + lane);  // converted when it is needed
  T piv = T(1), pc = T(0);  // pivot and c of the row this lane retired in this block
  read_next();

  // Retired rows wait in LDS (one slot per lane) until their block of RING columns is done, and go
  // out together: contiguous stores, and no store is in flight when a chunk of rows is waited for
  // (the counter of outstanding loads also counts stores).
  auto flush = [&](int64_t col0, int count) {
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < W; ++u) {
      const int e = lane + u * RING;
      if (e < count * W) R[col0 * W + e] = done[e / W * WR + e % W];
    }
    if constexpr (W <= 15) {
      if (S16) {
#pragma unroll
        for (int u = 0; u < RING; ++u)
          if (u < count) S16[(col0 + u) * 16 + lane] = (lane >= 1 && lane < W) ? done[u * WR + lane] : T(0);
      }
    }
    if (lane < count) {
      iv[col0 + lane] = 1.0 / (double)piv;
      cc[col0 + lane] = pc;
    }
    wave_lds_sync();
  };

  const int64_t steps = M + N;
  for (int64_t t = 0; t < steps; ++t) {
    // the rows move on, and a group's next one enters if it starts at the current column;
    // otherwise the current column's row of R is final (one problem per wave: scalar state)
    const uint32_t next = (uint32_t)(RING == 64 ? __builtin_amdgcn_readfirstlane(sn) : sn);
    const uint64_t enter_mask = __ballot(next == s), mine_mask = __ballot((s & (RING - 1)) == (uint32_t)lane);
    const uint64_t retire_mask = mine_mask & ~enter_mask;
    const bool enter = __builtin_amdgcn_inverse_ballot_w64(enter_mask);
    bs_move<RING>(x, xin, enter_mask & mine_mask);
    ic += enter ? 1 : 0;
    s += enter ? 0u : 1u;
    if (__builtin_amdgcn_inverse_ballot_w64(retire_mask)) {  // row s - 1 of R
#pragma unroll
      for (int l = 0; l < W; ++l) done[lane * WR + l] = Rw[l];
      piv = Rw[0];
      pc = Rc;
      Rw[0] = dnext;
      Rc = T(0);
#pragma unroll
      for (int l = 1; l < W; ++l) Rw[l] = T(0);
    }
    // rarely: a chunk of rows used up, or a block of RING columns retired (its last lane's row)
    const uint64_t chunk_mask = __ballot((ic & (C - 1)) == 0) & enter_mask;
    const uint64_t last_lanes = RING == 64 ? 1ull << 63 : 0x8000800080008000ull;
    if (__builtin_expect((chunk_mask | (retire_mask & last_lanes)) != 0, 0)) {
      if (__builtin_amdgcn_inverse_ballot_w64(chunk_mask)) {
        // on to the next chunk (staged); the one after it into the buffer of the one before
        ++kc;
        ic &= 2 * C - 1;
        stage(kc + 1);
        fetch(kc + 2);
        wave_lds_sync();
      }
      if (!enter && (s & (RING - 1)) == 0) {
        flush((int64_t)s - RING, RING);
        dnext = fabs((T)(sl * dload));
        dload = load_d((int64_t)s + 2 * RING + lane);
      }
    }
    read_next();
    asm volatile("" ::: "memory");  // the reads are issued here, not sunk to the next step's use
    // Every lane rotates its two rows.  With cs = a / r, sn = x_0 / r and tn = sn / (1 + cs) = x_0 / (r
    // + a), the rotation (R, x) -> (cs R + sn x, cs x - sn R) is three shears, three FMAs a column:
    // u = R + tn x, x' = x - sn u, R' = u + tn x'.  a >= 0, so tn <= 1.  Lanes whose row is spent or
    // not there (x_0 = 0) keep both.  Up to W = 15 a squared norm below the smallest normal number
    // rotates nothing (NaN does).  Above, sn and tn come from a and x_0 scaled up then, which changes
    // neither; looking for such lanes at every step cost 8%, so only problems that can have them do.
    T a = Rw[0], x0 = x[0];
    T q = fma(x0, x0, a * a);
    if constexpr (W <= 15) {
      const bool none = q < BsTiny<T>::value;
      x0 = none ? T(0) : x0;
      q = none ? BsTiny<T>::value : q;
    } else if (__builtin_expect(low, 0)) {
      const T up = q < BsTiny<T>::value ? BsTiny<T>::up : T(1);
      a *= up;
      x0 *= up;
      q = fma(x0, x0, a * a);
      q = q < BsTiny<T>::value ? BsTiny<T>::value : q;  // a = x_0 = 0
    }
    const T inv = bs_rsqrt(q);
    const T sn_ = x0 * inv;
    const T tn = x0 * bs_rcp(fma(q, inv, a));
    Rw[0] = fma(tn, W <= 15 ? x0 : x[0], Rw[0]);  // a + x_0^2 / (r + a) = r
#pragma unroll
    for (int l = 1; l < W; ++l) {
      const T u = fma(tn, x[l], Rw[l]);
      x[l - 1] = bs_fnma(sn_, u, x[l]);
      Rw[l] = fma(tn, x[l - 1], u);
    }
    x[W - 1] = T(0);
    const T u = fma(tn, x[W], Rc);
    x[W] = fma(-sn_, u, x[W]);
    Rc = fma(tn, x[W], u);
  }
  flush(N / RING * RING, (int)(N % RING));  // the last, partial block of columns
  if (bad) set_status(status, ST_BADINPUT);
}

// Banded triangular sweep for 16 <= w <= 31, one unknown per step, one problem per wave (what and
// how: k_bsweep_w in banded_w.hpp, with 32 lanes and the band itself in place of its padded copy).
//   BWD:  x = R^{-1} rhs, rows N-1 .. 0;  !BWD: y = R^{-T} rhs, rows 0 .. N-1.
// Lane c (mod 32) accumulates the pending sum of the unknowns of steps t = c (mod 32); the unknown
// of a step is read from its lane into scalar registers and every lane adds it times its coupling.
// Couplings are buffer loads two chunks of 32 steps ahead: lanes not coupled to a step point past
// the band, and rows before the first lie past it as unsigned offsets, so both read zero (bands
// under 2^30 bytes, bsweep_x_fits).  Bound by the chain of a step (FMA, lane read, FMA).
template <typename T, bool BWD, bool ADD, bool RHS_T, bool CHECK>
__global__ void __launch_bounds__(64)
k_bsweep_x(int64_t N, int w, const T* __restrict__ Rb, const double* __restrict__ binv, const T* __restrict__ rhsT,
           const double* rhsD, double* out, int* __restrict__ status) {
  constexpr int C = 32;
  constexpr int D = 2;
  constexpr uint32_t kPast = 0x80000000u;
  const int lane = threadIdx.x & 31;
  const int64_t prob = blockIdx.x;
  const double* iv = binv + prob * N;
  const T* rt = RHS_T ? rhsT + prob * N : nullptr;
  const double* rd = RHS_T ? nullptr : rhsD + prob * N;
  double* o = out + prob * N;
  const int row_bytes = w * (int)sizeof(T);
  const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(Rb + prob * N * w), 0, (int)(N * row_bytes),
                                                    0x00020000);
  uint32_t voff[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int l = (lane - c) & 31;
    const int64_t row = BWD ? N - 1 - c - l : c;
    voff[c] = (l >= 1 && l < w) ? (uint32_t)(int32_t)(row * row_bytes + l * (int)sizeof(T)) : kPast;
  }
  struct Chunk {
    T cr[C];
    double ivv, bvv, outv;
  };
  auto load_chunk = [&](int64_t t0, Chunk& k) {
    if (t0 >= N) return;
    const uint32_t step = (uint32_t)(int32_t)((BWD ? -t0 : t0) * row_bytes);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if constexpr (sizeof(T) == 4)
        k.cr[c] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(voff[c] + step), 0, 0));
      else
        k.cr[c] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(voff[c] + step), 0, 0));
    }
    const int64_t tl = t0 + lane < N ? t0 + lane : N - 1;  // clamped past the end: the value is not used
    const int64_t j = BWD ? N - 1 - tl : tl;
    k.ivv = iv[j];
    k.bvv = RHS_T ? (double)rt[j] : rd[j];
    k.outv = ADD ? o[j] : 0.0;
  };
  Chunk ring[D];
#pragma unroll
  for (int b = 0; b < D; ++b) load_chunk((int64_t)b * C, ring[b]);
  double acc = 0.0;
  double amin = __builtin_inf(), amax = 0.0;  // extreme |1 / pivot| seen by this lane
  bool nonfinite = false;
  for (int64_t T0 = 0; T0 < N; T0 += (int64_t)C * D) {
    static_for<0, D>([&](auto BB) {
      constexpr int b = decltype(BB)::value;
      const int64_t t0 = T0 + (int64_t)b * C;
      if (t0 >= N) return;
      Chunk& k = ring[b];
      const double bi = k.bvv * k.ivv;
      double xs = 0.0;  // lane c: the unknown of step t0 + c
      static_for<0, C>([&](auto CC) {
        constexpr int c = decltype(CC)::value;
        const double x = fma(-acc, k.ivv, bi);  // meaningful in lane c
        if (lane == c) xs = x;
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, c);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), c);
        const double xb = __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
        acc = lane == c ? 0.0 : acc;
        acc = fma((double)k.cr[c], xb, acc);
      });
      const int64_t t = t0 + lane;
      if (t < N && threadIdx.x < 32) {
        if (CHECK) {
          const double a = fabs(k.ivv);
          if (!is_finite(xs)) nonfinite = true;
          if (a == a) {
            amin = fmin(amin, a);
            amax = fmax(amax, a);
          }
        }
        const int64_t j = BWD ? N - 1 - t : t;
        o[j] = ADD ? k.outv + xs : xs;
      }
      load_chunk(t0 + (int64_t)C * D, k);  // refill this slot with the chunk D ahead
    });
  }
  if (CHECK && status) {
    // |pivot| = 1 / |1 / pivot|: flag a pivot at most N eps times the largest one
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) {
      amin = fmin(amin, __shfl_xor(amin, off, 32));
      amax = fmax(amax, __shfl_xor(amax, off, 32));
    }
    const double pmax = 1.0 / amin, pmin = 1.0 / amax;
    const bool sing = amax > 0.0 && is_finite(pmin) && pmin <= (double)N * Eps<T>::value * pmax;
    if (threadIdx.x == 0 && sing) set_status(status, ST_SINGULAR);
    if (nonfinite) set_status(status, ST_NONFINITE);
  }
}

// Launchers: bands LO .. HI - 1 in one translation unit.
template <typename T, int W>
hipError_t launch_bgivens_s_w(int P, int64_t M, int64_t N, const int32_t* row_start, const T* vals, const T* b,
                              const double* d, const double* lam, T* Rb, T* cb, double* binv, T* R16, int* status,
                              hipStream_t st) {
  constexpr int G = BsShape<T, W>::GROUPS;
  if (N > 0xfffffff0ll) return hipErrorInvalidValue;  // columns are counted in 32 bits
  hipLaunchKernelGGL((k_bgivens_s<T, W>), dim3((unsigned)((P + G - 1) / G)), dim3(64), 0, st, P, M, N, row_start, vals,
                     b, d, lam, Rb, cb, binv, R16, status);
  return hipGetLastError();
}
template <typename T, int LO, int HI>
hipError_t launch_bgivens_s_range(int P, int64_t M, int64_t N, int w, const int32_t* row_start, const T* vals,
                                  const T* b, const double* d, const double* lam, T* Rb, T* cb, double* binv, T* R16,
                                  int* status, hipStream_t st) {
  if constexpr (LO < HI) {
    if (w == LO)
      return launch_bgivens_s_w<T, LO>(P, M, N, row_start, vals, b, d, lam, Rb, cb, binv, R16, status, st);
    return launch_bgivens_s_range<T, LO + 1, HI>(P, M, N, w, row_start, vals, b, d, lam, Rb, cb, binv, R16, status,
                                                 st);
  } else {
    return hipErrorInvalidValue;
  }
}

// kind 0: p = R^{-1} c (checked);  1: out += R^{-1} rhs;  2: y = R^{-T} rhs
template <typename T>
hipError_t launch_bsweep_x_t(int kind, int P, int64_t N, int w, const T* Rb, const double* binv, const T* rhsT,
                             const double* rhsD, double* out, int* status, hipStream_t st) {
  if (!bsweep_x_fits(N, w, sizeof(T))) return hipErrorInvalidValue;
  const dim3 grid((unsigned)P), blk(64);
  if (kind == 0)
    hipLaunchKernelGGL((k_bsweep_x<T, true, false, true, true>), grid, blk, 0, st, N, w, Rb, binv, rhsT,
                       (const double*)nullptr, out, status);
  else if (kind == 1)
    hipLaunchKernelGGL((k_bsweep_x<T, true, true, false, false>), grid, blk, 0, st, N, w, Rb, binv, (const T*)nullptr,
                       rhsD, out, (int*)nullptr);
  else
    hipLaunchKernelGGL((k_bsweep_x<T, false, false, false, false>), grid, blk, 0, st, N, w, Rb, binv,
                       (const T*)nullptr, rhsD, out, (int*)nullptr);
  return hipGetLastError();
}

// The instantiations of one type and half of the bands (a translation unit each).
#define QRK_BS_INST(T, HALF, LO, HI)                                                                              \
  template <>                                                                                                     \
  hipError_t launch_bgivens_s<T, HALF>(int P, int64_t M, int64_t N, int w, const int32_t* row_start, const T* vals, \
                                       const T* b, const double* d, const double* lam, T* Rb, T* cb, double* binv, \
                                       T* R16, int* status, hipStream_t st) {                                     \
    return launch_bgivens_s_range<T, LO, HI>(P, M, N, w, row_start, vals, b, d, lam, Rb, cb, binv, R16, status, st); \
  }

}  // namespace qrk
