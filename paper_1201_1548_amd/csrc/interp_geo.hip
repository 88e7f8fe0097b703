// (d) interpolation per prime on the nodes x_i = 2^i, i = 0..D-1 (distinct modulo
// every table prime: the order of 2 exceeds MAX_POINTS for all of them).
//
// On a geometric sequence both halves of Newton's interpolation are the same
// triangular convolution.  With u_i = prod_{m=1}^{i} (2^m - 1) and
// C(i) = i (i - 1) / 2,
//   prod_{j<=k, j!=i} (x_i - x_j) = (-1)^{k-i} 2^{C(k) - C(k-i)} u_i u_{k-i},
// so the divided differences are c_k = 2^{-C(k)} sum_{i<=k} a_i b_{k-i} with
//   a_i = v_i / u_i,   b_j = (-1)^j 2^{C(j)} / u_j,
// and by the q-binomial theorem prod_{t<k} (x - 2^t) =
// sum_j u_k / (u_j u_{k-j}) (-1)^{k-j} 2^{C(k-j)} x^j, so the coefficients are
//   p_j = (1 / u_j) sum_{k>=j} e_k b_{k-j},   e_k = c_k u_k:
// the same convolution with b, read from the top down.  b, 1 / u_i and
// u_k 2^{-C(k)} depend on the prime only, not on D.
//
// The convolution runs on the int8 matrix cores.  Cut the output index into
// 16 c + s: for a tile of 16 columns c (256 outputs) and a window of 64 inputs
// per column,
//   out[16 c + s] = sum_w sum_{kk<64} A_w[s][kk] x[16 c - 48 - 64 w + kk],
//   A_w[s][kk] = b[s + 48 + 64 w - kk]   (zero for negative indices),
// a v_mfma_i32_16x16x64_i8 per window and pair of digits (balanced base-256
// digits of the symmetric representatives, four per residue, products of
// equal weight u = s + t in one of seven accumulators).  The right operand of
// a column is 16 contiguous bytes per lane of a digit plane in LDS; the left
// operands (Toeplitz blocks of b) are expanded once per prime into operand
// order (k_geo_tables).  Tile R needs the windows w < 4 (R + 1).
//
// What bounds it: 16 matrix products per window (about 272 cycles of a SIMD)
// against 4 KiB of left operand from L2, so a wave works on two column tiles
// at once where it can (the tiles R and nt - 1 - R, which also evens out the
// triangle): each left operand is then used 32 times.
//
// Measured against the per-(job, prime) kernel on the nodes 0..D-1 (a VALU
// convolution and a Horner recurrence over D / 32 blocks with a barrier each):
// one degree-40 discriminant (D = 1561, 55 primes) 194 -> 22 us, one degree-64
// resultant (D = 4097, 573 primes) 2604 -> 187 us, 3800 arrangement pairs
// (D 17..901) 5026 -> 895 us, 64 serving requests (D up to 4097) 5085 -> 500 us.
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "job.hpp"
#include "kernels.hpp"

namespace bires {

// Tables of prime k (blockIdx.x) for indices below Dc (a multiple of 256, at
// most MAX_POINTS): 2^i, 1 / u_i and u_i 2^{-C(i)} (Montgomery form), and the
// Toeplitz operands of b: window w, digit plane s at 1 KiB blocks 4 w + s,
// lane l holding row l % 16 and contraction indices 16 (l / 16) + 0..15.
// Thread t computes the entries of its contiguous 1/256 of the range; a block
// scan joins the partial products u.
__global__ __launch_bounds__(256) void k_geo_tables(const ModP* primes, int Dc, uint32_t* qpow, uint32_t* invu,
                                                    uint32_t* wt, int8_t* A) {
  extern __shared__ __align__(16) uint32_t lds[];
  uint32_t* dig = lds;        // [Dc] digit words of b
  uint32_t* tot = lds + Dc;   // [256] inclusive products of the threads' ranges
  const int k = blockIdx.x, t = threadIdx.x, ch = Dc >> 8, i0 = t * ch;
  const ModP q = primes[k];
  const uint32_t two = madd(q.one, q.one, q.p), half = to_mont((q.p + 1u) >> 1, q);
  qpow += (size_t)k * Dc;
  invu += (size_t)k * Dc;
  wt += (size_t)k * Dc;
  A += (size_t)k * Dc * 64;
  const uint32_t x0 = mpow(two, (uint32_t)i0, q);
  uint32_t x = x0, loc = q.one;
  for (int i = i0; i < i0 + ch; ++i) {
    if (i) loc = mmul(loc, msub(x, q.one, q.p), q);
    x = madd(x, x, q.p);
  }
  tot[t] = loc;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {
    const uint32_t v = t >= o ? mmul(tot[t - o], tot[t], q) : tot[t];
    __syncthreads();
    tot[t] = v;
    __syncthreads();
  }
  uint32_t u = t ? tot[t - 1] : q.one;
  uint32_t y = mpow(half, (uint32_t)i0, q);  // 2^{-i}
  uint32_t c = mpow(half, (uint32_t)i0 * (uint32_t)(i0 - 1) / 2u, q);  // 2^{-C(i)}; C(0) = 0: 0 * (2^32 - 1) / 2 = 0
  x = x0;
  for (int i = i0; i < i0 + ch; ++i) {
    if (i) u = mmul(u, msub(x, q.one, q.p), q);
    qpow[i] = x;
    wt[i] = mmul(u, c, q);
    c = mmul(c, y, q);
    y = mmul(y, half, q);
    x = madd(x, x, q.p);
  }
  // backward: 1 / u_i, b_i
  const int i1 = i0 + ch - 1;
  uint32_t inv = minv(u, q);
  x = mpow(two, (uint32_t)i1, q);
  y = mpow(half, (uint32_t)(i1 > 0 ? i1 - 1 : 0), q);  // 2^{-(i-1)}
  uint32_t d = i1 > 0 ? mpow(two, (uint32_t)i1 * (uint32_t)(i1 - 1) / 2u, q) : q.one;  // 2^{C(i)}
  for (int i = i1; i >= i0; --i) {
    invu[i] = inv;
    uint32_t b = mmul(d, inv, q);
    if (i & 1) b = mneg(b, q.p);
    dig[i] = digits4(from_mont(b, q), q.p);
    if (i) {
      inv = mmul(inv, msub(x, q.one, q.p), q);
      d = mmul(d, y, q);
    }
    x = mmul(x, half, q);
    y = madd(y, y, q.p);
  }
  __syncthreads();
  for (int e = t; e < Dc; e += 256) {
    const int w = e >> 6, l = e & 63, s = l & 15, g = l >> 4;
    uint32_t pl[4][4];
#pragma unroll
    for (int b4 = 0; b4 < 4; ++b4) {
      uint32_t dw[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int idx = s + 48 + 64 * w - 16 * g - (4 * b4 + j);
        dw[j] = idx >= 0 ? dig[idx] : 0u;
      }
      const u32x4 v = byte_planes(dw[0], dw[1], dw[2], dw[3]);
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) pl[s4][b4] = v[s4];
    }
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4)
      *(u32x4*)(A + (size_t)(4 * w + s4) * 1024 + 16 * l) = (u32x4){pl[s4][0], pl[s4][1], pl[s4][2], pl[s4][3]};
  }
}

namespace {

typedef __attribute__((address_space(1))) const im_v4i g_v4i;

// The four left operand planes of window w (lane's 16 bytes each).
__device__ __forceinline__ void geo_load_a(im_v4i (&a)[4], const __attribute__((address_space(1))) int8_t* A, int w) {
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = *(g_v4i*)(A + ((size_t)w * 4 + s) * 1024);
}

__device__ __forceinline__ void geo_load_b(im_v4i (&b)[4], const int8_t* x, int PS) {
#pragma unroll
  for (int s = 0; s < 4; ++s) b[s] = *(const im_v4i*)(x + s * PS);
}

// digit s of b against digit t of x into class s + t
__device__ __forceinline__ void geo_products(im_v4i (&G)[7], const im_v4i (&a)[4], const im_v4i (&b)[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int t = 0; t < 4; ++t) G[s + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[s], b[t], G[s + t], 0, 0, 0);
}

// sum_u G_u 256^u mod p for accumulator element j (plain residue).  With
// D <= 8192 the class sums satisfy sum_u |G_u| <= 16 D 2^14 <= 2^31, so
// |sum_u G_u w_u| < 2^31 p for the Montgomery forms w_u < p of 256^u; adding
// p 2^32 leaves a value in (0, 2 p 2^32), where redc gives one below 2p.
__device__ __forceinline__ uint32_t geo_value(const im_v4i (&G)[7], int j, const uint32_t (&wu)[7], const ModP& q) {
  int64_t acc = (int64_t)q.p << 32;
#pragma unroll
  for (int u = 0; u < 7; ++u) acc += (int64_t)G[u][j] * (int64_t)(int32_t)wu[u];
  const uint32_t v = redc((uint64_t)acc, q.p, q.pinv);
  return umin32(v, v - q.p);
}

}  // namespace

// One block of TW waves per (job, prime).  LDS: two sets of four digit planes
// of PS = 256 (nt + 1) bytes (256 zero bytes, then nt = ceil(D / 256) tiles).
// PAIR: a wave takes the tile pair (nt - 1 - pr, pr); without it one tile.
// The left operand of the next window, with several waves of the next two, is on its
// way (a window lasts 272 or 544 cycles, a miss in the L2, which does not hold the
// tables of all primes at work, longer).  Two waves per SIMD at least: with the
// default of one the compiler keeps the sums in accumulation registers and
// copies them out and back in every window (84 copies to 32 products: 301 instead
// of 187 us for D = 4097 and 573 primes).
template <int TW, bool PAIR>
__global__ __launch_bounds__(64 * TW) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_interp_geo(
    const JobDev* jobs, const int* starts, int nj, TablesDev tab) {
  constexpr int AHEAD = TW == 1 ? 1 : 2;
  extern __shared__ __align__(16) int8_t geo_lds[];
  const int job = find_job(starts, nj, blockIdx.x, gridDim.x);
  const JobDev& J = jobs[job];
  const int k = blockIdx.x - starts[job], D = J.D, nt = (D + 255) >> 8, PS = 256 * (nt + 1), Dr = 256 * nt;
  const int tid = threadIdx.x, l = tid & 63, wv = TW == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = l & 15, g = l >> 4;
  const ModP q = tab.primes[k];
  const uint32_t* iu = tab.geo_invu + (size_t)k * tab.geo_D;
  const uint32_t* wt = tab.geo_w + (size_t)k * tab.geo_D;
  const __attribute__((address_space(1))) int8_t* At = gmem(tab.geo_A) + (size_t)k * tab.geo_D * 64 + 16 * l;
  const uint32_t* v = J.vals + (size_t)k * D;
  int8_t* X[2] = {geo_lds, geo_lds + 4 * PS};
  // zeros below index 0 of every plane (one dword per lane of the first wave and plane)
  if (tid < 64) {
#pragma unroll
    for (int s = 0; s < 8; ++s) *(uint32_t*)(geo_lds + s * PS + 4 * tid) = 0u;
  }
  // a_i = v_i / u_i as digits, four consecutive elements per thread
  for (int i0 = 4 * tid; i0 < Dr; i0 += 256 * TW) {
    const u32x4 f = *(const u32x4*)(iu + i0);
    uint32_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + j;
      const uint32_t x = v[min(i, D - 1)];
      d[j] = i < D ? digits4(mmul(x, f[j], q), q.p) : 0u;
    }
    const u32x4 pl = byte_planes(d[0], d[1], d[2], d[3]);
#pragma unroll
    for (int s = 0; s < 4; ++s) *(uint32_t*)(X[0] + s * PS + 256 + i0) = pl[s];
  }
  uint32_t wu[7];  // Montgomery forms of 256^u
  wu[0] = q.one;
  const uint32_t m256 = to_mont(256u, q);
#pragma unroll
  for (int u = 1; u < 7; ++u) wu[u] = mmul(wu[u - 1], m256, q);
  uint32_t* out = J.coefs + (size_t)k * D;
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    group_sync<TW == 1>();
    // windows that can hold a non-zero product: b indices below D (the second
    // pass reads e from the top down, behind Dr - D zeros)
    const int nwin = pass ? (D + 14) / 64 + 1 : (D - 1) / 64 + 1;
    // outputs of one tile: rows 4 g + j of column c16
    auto finish = [&](const im_v4i(&G)[7], int R) {
      const int o0 = 256 * R + 16 * c16 + 4 * g;
      uint32_t y[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = geo_value(G, j, wu, q);
      if (pass == 0) {
        const u32x4 f = *(const u32x4*)(wt + o0);
        uint32_t d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) d[j] = o0 + j < D ? digits4(mmul(y[j], f[j], q), q.p) : 0u;
        const u32x4 pl = byte_planes(d[3], d[2], d[1], d[0]);  // e_k at index Dr - 1 - k
#pragma unroll
        for (int s = 0; s < 4; ++s) *(uint32_t*)(X[1] + s * PS + 256 + Dr - 4 - o0) = pl[s];
      } else {
        const int j0 = Dr - 4 - o0;  // output o0 + j is coefficient j0 + 3 - j
        const u32x4 f = *(const u32x4*)(iu + j0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j0 + 3 - j < D) out[j0 + 3 - j] = mmul(y[j], f[3 - j], q);
      }
    };
    for (int pr = wv; pr < (PAIR ? (nt + 1) >> 1 : nt); pr += TW) {
      const int hi = nt - 1 - pr, lo = pr;
      const bool two = PAIR && lo < hi;
      const int Wh = min(4 * (hi + 1), nwin), Wl = two ? min(4 * (lo + 1), nwin) : 0;
      const int8_t* xh = X[pass] + 256 + 256 * hi + 16 * c16 + 16 * g - 48;
      const int8_t* xl = X[pass] + 256 + 256 * lo + 16 * c16 + 16 * g - 48;
      im_v4i Gh[7], Gl[PAIR ? 7 : 1];
#pragma unroll
      for (int u = 0; u < 7; ++u) Gh[u] = (im_v4i){0, 0, 0, 0};
      im_v4i a[AHEAD + 1][4], b[4];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) geo_load_a(a[i], At, min(i, Wh - 1));
      auto next = [&](int w) {
        geo_load_a(a[AHEAD], At, min(w + AHEAD, Wh - 1));
      };
      auto shift = [&] {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
#pragma unroll
          for (int s = 0; s < 4; ++s) a[i][s] = a[i + 1][s];
      };
      int w = 0;
      if constexpr (PAIR) {
#pragma unroll
        for (int u = 0; u < 7; ++u) Gl[u] = (im_v4i){0, 0, 0, 0};
        for (; w < Wl; ++w) {
          next(w);
          im_v4i c[4];
          geo_load_b(b, xh - 64 * w, PS);
          geo_load_b(c, xl - 64 * w, PS);
          geo_products(Gh, a[0], b);
          geo_products(Gl, a[0], c);
          shift();
        }
      }
      for (; w < Wh; ++w) {
        next(w);
        geo_load_b(b, xh - 64 * w, PS);
        geo_products(Gh, a[0], b);
        shift();
      }
      finish(Gh, hi);
      if constexpr (PAIR) {
        if (two) finish(Gl, lo);
      }
    }
  }
}

size_t geo_table_bytes(int Dc, int P) { return (size_t)P * Dc * (3 * sizeof(uint32_t) + 64); }

void launch_geo_tables(const ModP* primes, int Dc, int P, uint32_t* qpow, uint32_t* invu, uint32_t* wt, int8_t* A,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_geo_tables, dim3(P), dim3(256), (size_t)(Dc + 256) * sizeof(uint32_t), s, primes, Dc, qpow,
                     invu, wt, A);
}

int geo_class(int D) { return D <= 256 ? 0 : D <= 512 ? 1 : D <= 1024 ? 2 : 3; }

void launch_interp_geo(int cls, const JobDev* jobs, const int* starts, int nj, int nblocks, int max_points,
                       TablesDev tab, hipStream_t s) {
  const size_t lds = (size_t)8 * 256 * ((max_points + 255) / 256 + 1);
#define BIRES_GEO(TW, PAIR) \
  hipLaunchKernelGGL((k_interp_geo<TW, PAIR>), dim3(nblocks), dim3(64 * TW), lds, s, jobs, starts, nj, tab)
  switch (cls) {
    case 0: BIRES_GEO(1, false); break;
    case 1: BIRES_GEO(1, true); break;
    case 2: BIRES_GEO(2, true); break;
    default: BIRES_GEO(4, true); break;
  }
#undef BIRES_GEO
}

}  // namespace bires
