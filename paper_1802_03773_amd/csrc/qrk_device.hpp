// Device-side helpers shared by the qrkit HIP kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "qrk_batch.hpp"

namespace qrk {

// Status bits recorded in the handle's device status word.
enum : int {
  ST_SINGULAR = 1,
  ST_NONFINITE = 2,
  ST_BADINPUT = 4,
  ST_STALL = 8,  // a dense-part merge did not see its inputs within its wait bound
  ST_NOTCONVERGED = 16,  // qrk_solve_tol used all its sweeps above the requested tolerance
};

constexpr int kWave = 64;

// Compile-time loop: f(std::integral_constant<int, I>) for I in [I0, N).
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Make LDS writes of one lane visible to the other lanes of the same wave.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T>
__device__ __forceinline__ T wave_allreduce_sum(T v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

template <typename T>
__device__ __forceinline__ T wave_allreduce_max(T v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off, kWave));
  return v;
}

template <typename T>
__device__ __forceinline__ bool is_finite(T x) {
  return __builtin_isfinite(x);
}

template <typename T>
struct Eps;
template <>
struct Eps<float> {
  static constexpr double value = 5.9604644775390625e-08;  // 2^-24
};
template <>
struct Eps<double> {
  static constexpr double value = 1.1102230246251565e-16;  // 2^-53
};

// The first per-block QR launch's clearing and lambda store (BqrPrologue), by the NT threads
// of workgroup 0.
template <int NT>
__device__ __forceinline__ void bqr_prologue(const BqrPrologue& pro) {
  if (blockIdx.x != 0) return;
  for (int64_t i = threadIdx.x; i < pro.n0; i += NT) pro.z0[i] = 0;
  for (int64_t i = threadIdx.x; i < pro.n1; i += NT) pro.z1[i] = 0;
  if (threadIdx.x == 0 && pro.lam_out) *pro.lam_out = pro.lam_val;
}

// A copy of x that the compiler cannot identify with x (an empty asm on a register;
// no memory is touched).  The permlane swaps need two distinct operands.
__device__ __forceinline__ unsigned opaque_copy(unsigned x) {
  unsigned y = x;
  asm volatile("" : "+v"(y));
  return y;
}

// First node entry of a workgroup of a pipelined merge tree (WPG waves, an entry each; entries in
// level order): workgroups are numbered as they start, by a counter, not by block index.  A node waits
// for lower entries only, so whatever a wave waits for belongs to a workgroup that has started and
// keeps its compute unit: the lowest unfinished entry never waits for a workgroup still to be placed.
// Block indices do not give that.  The XCDs place their shares of a grid each at its own pace, so with
// two such launches on two streams the waiting nodes of each could hold one XCD against the other's
// children.  The count costs a memory round trip, about 1 us a launch.
template <int WPG>
__device__ __forceinline__ int tree_first_entry(int* ticket) {
  if (gridDim.x == 1) return 0;  // the workgroup is placed as a whole
  __shared__ int first;
  if (threadIdx.x == 0) first = atomicAdd(ticket, 1);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(first) * WPG;
}

// Flags between the nodes of a pipelined merge tree: flag 2 q + k of a node says that part k (0: above
// the diagonal, 1: the diagonal block) of its column block q is published.  A look reads both parts'
// flags of both children (fa, fb) in one device-scope load, a lane each, so a round trip to memory
// answers all four; it is issued before the work that comes ahead of the wait, which then usually finds
// the answer there.
__device__ __forceinline__ int tree_look(const int* fa, const int* fb, int q, int lane) {
  return __hip_atomic_load(((lane & 1) ? fb : fa) + 2 * q + ((lane >> 1) & 1), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}
// Part k published by both children, as of the look v?
__device__ __forceinline__ bool tree_seen(int v, int k) {
  return (__builtin_amdgcn_ballot_w64(v == 0) & (k ? 0xccccccccccccccccull : 0x3333333333333333ull)) == 0;
}
// Wait (bounded) until it is; false on timeout.
__device__ __forceinline__ bool tree_wait(int& v, const int* fa, const int* fb, int q, int k, int lane) {
#pragma clang loop unroll(disable)
  for (int it = 0; it < (1 << 21); ++it) {
    if (tree_seen(v, k)) return true;
    __builtin_amdgcn_s_sleep(1);
    v = tree_look(fa, fb, q, lane);
  }
  return false;
}

__device__ __forceinline__ void set_status(int* status, int bits) {
  if (status) atomicOr(status, bits);
}

}  // namespace qrk
