// Device helpers shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "job.hpp"

namespace bires {

// Block -> job: starts[0..nj] are the first block of each job (starts[nj] =
// grid size); returns the largest j with starts[j] <= b (uniform, scalar).
// The job j of block b: starts[j] <= b < starts[j + 1] (nj + 1 prefix
// entries; jobs without blocks repeat an entry).  With the launch's block
// count `total`, the guess b nj / total is the answer whenever the jobs have
// equal block counts, and two independent loads confirm it; otherwise (or
// with total = 0) a binary search, whose dependent loads cost a round trip
// to L2 each.
__device__ __forceinline__ int find_job(const int* __restrict__ starts, int nj, int b, int total = 0) {
  if (total > 0) {
    const int g = min((int)(((unsigned long long)b * (unsigned)nj) / (unsigned)total), nj - 1);
    if (starts[g] <= b && b < starts[g + 1]) return g;
  }
  int lo = 0, hi = nj;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (starts[mid] <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Global-memory view of a pointer the host guarantees to be device memory:
// loads through it compile to global (not flat) loads, which do not share
// the LDS wait counter.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(1))) T* gmem(const T* p) {
  return (const __attribute__((address_space(1))) T*)p;
}

// Lane of the calling thread in its wave.  The device functions that one wave
// runs index with it, so that a block of several waves (the persistent
// launch) can give each wave a task of its own.
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

// Synchronisation of the threads that run a device function together: the
// whole block, or (WAVE) one wave of it.  A wave's LDS accesses complete in
// order, so the wave needs no barrier; the fences keep the compiler from
// moving memory accesses across the point.
template <bool WAVE>
__device__ __forceinline__ void group_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// a b + c with 32-bit a, b (one v_mad_u64_u32).  Inline assembly keeps a as a
// single 32-bit register where the compiler would keep a zero-extended pair.
// SB: b is wave-uniform and held in a scalar register (the residues read
// through the scalar cache).
template <bool SB = false>
__device__ __forceinline__ uint64_t mad_u64_u32(uint32_t a, uint32_t b, uint64_t c) {
  uint64_t d;
  uint64_t carry;
  if constexpr (SB)
    asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(d), "=s"(carry) : "v"(a), "s"(b), "v"(c));
  else
    asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(d), "=s"(carry) : "v"(a), "v"(b), "v"(c));
  return d;
}

// Exact sums of products of residues in 96 bits: 64-bit partial sums (up to
// eight products of residues, below 8 p^2 < 2^64) added with a carry word.
struct Acc96 {
  uint64_t lo = 0;
  uint32_t hi = 0;
  __device__ void add(uint64_t s) {
    lo += s;
    hi += lo < s ? 1u : 0u;
  }
};

// S R^{-1} mod p for S = hi 2^64 + lo with hi < 2^32 - 4 (here hi <= 2):
// REDC(lo_lo + hi R^2) = lo_lo R^{-1} + hi R, and lo_hi R R^{-1} = lo_hi.
// The REDC argument is below p 2^32, so its result is below 2p.
__device__ __forceinline__ uint32_t fold96(const Acc96& S, const ModP& q) {
  const uint64_t t = (uint64_t)S.hi * q.r2 + (uint32_t)S.lo;
  return madd(redc(t, q.p, q.pinv), reduce32((uint32_t)(S.lo >> 32), q.p), q.p);
}

// The four balanced base-256 digits of the symmetric representative v of
// x mod p, packed little-endian into one word.  Adding 128 at each of the
// three low digit positions makes those digits d_s + 128 in [0, 255] (plain
// base 256), with the top digit (|d_3| <= 64) left in the top byte; flipping
// bit 7 of the three low bytes subtracts the 128 again in int8 terms.
__device__ __forceinline__ uint32_t digits4(uint32_t x, uint32_t p) {
  const uint32_t v = x > (p >> 1) ? x - p : x;
  return (v + 0x808080u) ^ 0x808080u;
}

// Workgroups are dispatched to the 8 XCDs round-robin in blockIdx order, and
// each XCD has its own L2.  This bijection of [0, nb) gives XCD x the
// contiguous logical range [x q + min(x, r), ...) of q + (x < r) blocks
// (q = nb / 8, r = nb % 8), so the blocks of one (job, prime), which share
// that prime's residues, run on one XCD and share its L2.
__device__ __forceinline__ int xcd_block(int b, int nb) {
  const int q = nb >> 3, r = nb & 7, x = b & 7;
  return x * q + min(x, r) + (b >> 3);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 4 x 4 byte transpose: word s of the result holds byte s of d0..d3 in order.
__device__ __forceinline__ u32x4 byte_planes(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3) {
  const uint32_t a01 = __builtin_amdgcn_perm(d1, d0, 0x05010400u), a23 = __builtin_amdgcn_perm(d3, d2, 0x05010400u);
  const uint32_t b01 = __builtin_amdgcn_perm(d1, d0, 0x07030602u), b23 = __builtin_amdgcn_perm(d3, d2, 0x07030602u);
  return (u32x4){__builtin_amdgcn_perm(a23, a01, 0x05040100u), __builtin_amdgcn_perm(a23, a01, 0x07060302u),
                 __builtin_amdgcn_perm(b23, b01, 0x05040100u), __builtin_amdgcn_perm(b23, b01, 0x07060302u)};
}

// Montgomery form of evaluation point pt of prime k: the tables' 2^pt when
// the launch interpolates on the geometric nodes, else pt itself.
__device__ __forceinline__ uint32_t eval_point(const TablesDev& tab, int k, int pt, const ModP& q) {
  return tab.qpow ? tab.qpow[(size_t)k * tab.geo_D + pt] : to_mont((uint32_t)pt, q);
}

typedef int im_v4i __attribute__((ext_vector_type(4)));
typedef int im_v16i __attribute__((ext_vector_type(16)));

// Byte offset of element (row, idx) of a digit plane of the matrix-core
// interpolation with Kp = padded contraction length, in operand order: 1 KiB
// blocks per (32-row tile, 32-wide step), lane l of an operand holding row
// l % 32 and contraction indices 16 (l / 32) + 0..15.
__device__ __forceinline__ size_t im_off(int row, int idx, int Kp) {
  const int rt = row >> 5, r = row & 31, ks = idx >> 5, g = (idx >> 4) & 1, b = idx & 15;
  return ((((size_t)rt * (Kp >> 5) + ks) * 64) + r + 32 * g) * 16 + b;
}

// The value v = R(a) mod p_k (plain residue) of point a of job J: into vals,
// or for a job of the matrix-core interpolation group straight into the
// group's four digit planes of prime k (column ycol), which the
// interpolation reads as its right operand.  Those planes are not cleared:
// columns past the group only reach output columns that are not written,
// and points in [D, Dp) meet zero entries of the inverse Vandermonde planes.
// (A call, not inlined: the register allocation of the evaluation kernels'
// loops stays that of a single store.)
static __device__ __noinline__ void put_planes(int8_t* yp, int ycol, int ynp, int ydp, int k, int a, uint32_t v, uint32_t p) {
  const size_t plane = (size_t)ynp * ydp;
  int8_t* base = yp + (size_t)k * 4 * plane + im_off(ycol, a, ydp);
  const uint32_t d = digits4(v, p);
#pragma unroll
  for (int s = 0; s < 4; ++s) base[s * plane] = (int8_t)(d >> (8 * s));
}

__device__ __forceinline__ void put_value(const JobDev& J, int k, int a, uint32_t v, uint32_t p) {
  if (J.yp)
    put_planes(J.yp, J.ycol, J.ynp, J.ydp, k, a, v, p);
  else
    J.vals[(size_t)k * J.D + a] = v;
}

}  // namespace bires
