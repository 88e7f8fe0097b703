// (a8) gcds over F_p: the modular gcd per prime (Section 5.1, "Computing gcds
// in Z[x]", step (b)) and the degree chain of the N^- / N^+ test (Section 3.2.2).
//
// Euclid's algorithm on a pair of degree n takes about n dependent steps, and a
// block that updates all coefficients in every step spends its time in
// barriers and LDS round trips (0.9 us per step at n = 1560, 1.39 ms for the
// pair (R, R') of a degree-40 curve).  A step only depends on the leading
// coefficients, so here one wave runs up to 31 steps on the top 64
// coefficients of the pair, one per lane, in registers (lane shifts by DPP,
// no barrier), and carries the 2 x 2 matrix of polynomials that takes the pair
// to the one 31 steps later along in two more registers.  The other waves then
// apply the matrix of the previous round to the whole pair - a 32-tap
// convolution, one reduction per coefficient instead of one per step - while
// the first computes the next matrix from the top of the new pair, which it
// forms by itself.  Degrees below 63 finish on the one wave.  Steps that are
// not normal (degree gaps) are divisions with remainder in rounds of 32
// quotient coefficients, found by one wave and applied by all.
// 512 threads: seven waves apply a matrix in less time than the one wave takes
// for its 31 steps (about 70 instructions each, one dependent chain), which
// is what a round now waits for; that wave runs at a raised priority.
// Measured for a degree-1560 pair: k_gcd_p, 115 primes, 1393 -> 265 us; with a
// common factor of degree 200 and the two exact divisions 1090 -> 280 us;
// k_fiber_chain (two chains, one block each) 2525 -> 259 us.
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "job.hpp"
#include "kernels.hpp"

namespace bires {

namespace {

constexpr int GB = 512;     // threads per block
constexpr int TAPS = 32;    // matrix taps, quotient coefficients per round
constexpr int PAD = 36;     // zero words below index 0 of the double-buffered arrays

struct GcdShared {
  uint32_t M[2][TAPS][4];  // [buffer][power of y]: A' = M0 X + M1 Y, B' = M2 X + M3 Y
  uint32_t q[2][TAPS];     // quotient coefficients of a round (two divisions side by side)
  int steps, a, b;
};

// lane i receives lane i + 1 (0 in lane 63) / lane i - 1 (0 in lane 0)
__device__ __forceinline__ uint32_t lane_down(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t lane_up(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t lane_of(uint32_t x, int l) { return __builtin_amdgcn_readlane(x, l); }

// One normal step (A of degree deg B + 1) on top-aligned lanes as two
// eliminations: T = lb A - a0 y B, R = lb T - t0 B, with lb and an0 = p - a0 the scalar
// multipliers, and tn0 = p - t0 for the caller.  (Its three-product form R = l2 A +
// (l1 y + n2) B has a shorter chain in the lanes, but computes its three
// constants in scalar registers: 36 more instructions on a wave that waits for
// each of them.)
__device__ __forceinline__ uint32_t step_rem(uint32_t A, uint32_t B, uint32_t lb, uint32_t an0, uint32_t& tn0,
                                             const ModP& q) {
  const uint32_t B1 = lane_down(B);
  const uint32_t T = mdot2(lb, lane_down(A), an0, B1, q);
  tn0 = mneg_factor(lane_of(T, 0), q.p);
  return mdot2(lb, lane_down(T), tn0, B1, q);
}

// Up to 31 normal steps of a wave on the top 64 coefficients A, B (lane i: the
// coefficient i below the leading one).  Every step loses two lanes of the
// window at its low end: after 31 the remainder still has two.  Stops before
// a step whose remainder's leading coefficient vanishes.  The matrix starts as
// the identity: lanes 0..31 hold the powers of y of the entries that multiply
// X, lanes 32..63 of those that multiply Y (of degree below 31, so the shift by
// one power never crosses the halves).
__device__ __forceinline__ int window_steps(const uint32_t A0, const uint32_t B0, uint32_t (*M)[4], const ModP& q) {
  const int l = lane_id();
  int s = TAPS - 1;
  for (;;) {
    uint32_t A = A0, B = B0, MA = l == 0 ? q.one : 0u, MB = l == 32 ? q.one : 0u;
    // a vanishing leading coefficient is one chance in 2^25 per round and does
    // no harm here: the steps run without a branch, and if there was one the
    // steps before it are run again
    int zero = TAPS;
    uint32_t an0 = mneg_factor(lane_of(A, 0), q.p), lb = lane_of(B, 0);
#pragma unroll 2
    for (int i = 0; i < s; ++i) {
      uint32_t tn0;
      const uint32_t R = step_rem(A, B, lb, an0, tn0, q);
      const uint32_t MR = mdot2(lb, mdot2(lb, MA, an0, lane_up(MB), q), tn0, MB, q);
      an0 = mneg_factor(lb, q.p);
      lb = lane_of(R, 0);
      if (lb == 0u) zero = min(zero, i);
      A = B;
      B = R;
      MA = MB;
      MB = MR;
    }
    if (zero == TAPS) {
      M[l & 31][l >> 5] = MA;
      M[l & 31][2 + (l >> 5)] = MB;
      return s;
    }
    s = zero;
  }
}

// X2 <- M0 X + M1 Y (degree an), Y2 <- M2 X + M3 Y (degree an - 1) for the taps
// below nt, by nthr threads: four consecutive coefficients of both per
// thread, sliding windows of X and Y in registers (sixteen multiply-adds per
// two words read and one broadcast of the taps).
__device__ __forceinline__ void apply_matrix(const uint32_t* X, const uint32_t* Y, uint32_t* X2, uint32_t* Y2,
                                             const uint32_t (*M)[4], int nt, int an, int tid, int nthr, const ModP& q) {
  for (int t0 = 4 * tid; t0 <= an; t0 += 4 * nthr) {
    uint32_t x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      x[u] = X[t0 + u];
      y[u] = Y[t0 + u];
    }
    Acc96 A[4], B[4];
    for (int i0 = 0; i0 < nt; i0 += 4) {
      uint64_t sa[4] = {0, 0, 0, 0}, sb[4] = {0, 0, 0, 0};
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int i = i0 + g;
        const u32x4 m = *(const u32x4*)M[i];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          sa[u] = mad_u64_u32(x[u], m.x, sa[u]);
          sa[u] = mad_u64_u32(y[u], m.y, sa[u]);
          sb[u] = mad_u64_u32(x[u], m.z, sb[u]);
          sb[u] = mad_u64_u32(y[u], m.w, sb[u]);
        }
        // eight products of residues stay below 2^64
        x[3] = x[2], x[2] = x[1], x[1] = x[0], x[0] = X[t0 - i - 1];
        y[3] = y[2], y[2] = y[1], y[1] = y[0], y[0] = Y[t0 - i - 1];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        A[u].add(sa[u]);
        B[u].add(sb[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (t0 + u <= an) X2[t0 + u] = fold96(A[u], q);
      if (t0 + u < an) Y2[t0 + u] = fold96(B[u], q);
    }
  }
}

// The top 64 coefficients of the same two polynomials, one per lane.
__device__ __forceinline__ void apply_top(const uint32_t* X, const uint32_t* Y, const uint32_t (*M)[4], int nt, int an,
                                          uint32_t& Aw, uint32_t& Bw, const ModP& q) {
  const int t = an - lane_id();
  uint32_t x = X[t], y = Y[t];
  Acc96 A, B;
  for (int i0 = 0; i0 < nt; i0 += 4) {
    uint64_t sa = 0, sb = 0;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int i = i0 + g;
      const u32x4 m = *(const u32x4*)M[i];
      sa = mad_u64_u32(x, m.x, sa);
      sa = mad_u64_u32(y, m.y, sa);
      x = X[t - i - 1];
      y = Y[t - i - 1];
      sb = mad_u64_u32(x, m.z, sb);  // B' one degree lower: the same words one tap later
      sb = mad_u64_u32(y, m.w, sb);
    }
    A.add(sa);
    B.add(sb);
  }
  Aw = fold96(A, q);
  Bw = fold96(B, q);
}

// X <- X mod Y in place (degrees a >= b >= 1, inv = 1 / lc(Y)) by the nthr
// threads tid of a team, in `rounds` rounds of 32 quotient coefficients (both
// teams of a block must take the same number, at least their own
// ceil((a - b + 1) / 32)).  qb: the team's 32 words of LDS.  out: where the
// quotient goes, times scl (null: dropped).
__device__ __forceinline__ void team_mod(uint32_t* X, int a, const uint32_t* Y, int b, uint32_t inv, bool monic,
                                         uint32_t* qb, uint32_t* out, uint32_t scl, int tid, int nthr, int rounds,
                                         const ModP& q) {
  for (int r = 0; r < rounds; ++r) {
    const int n = min(TAPS, a - b + 1);  // quotient coefficients of this round (0 or less: none left)
    if (tid < 64 && n > 0) {
      const int l = tid;
      uint32_t x = a - l >= 0 ? X[a - l] : 0u, y = lane_down(b - l >= 0 ? Y[b - l] : 0u), qv = 0u;
      for (int j = 0; j < n; ++j) {
        uint32_t c = lane_of(x, 0);
        if (!monic) c = mmul(c, inv, q);
        if (l == j) qv = c;
        x = msub(lane_down(x), mmul(c, y, q), q.p);
      }
      if (l < TAPS) qb[l] = qv;
      if (out && l < n) out[a - b - l] = mmul(qv, scl, q);
    }
    __syncthreads();
    if (n > 0) {
      const int s = a - b, top = a - n;
      // X_t -= sum_j q_j Y_{t - s + j}; zero contributions below s - n + 1
      for (int t0 = (max(0, s - n + 1) & ~3) + 4 * tid; t0 <= top; t0 += 4 * nthr) {
        uint32_t y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = t0 + u - s;
          y[u] = i >= 0 ? Y[min(i, b)] : 0u;
        }
        Acc96 A[4];
        for (int j0 = 0; j0 < n; j0 += 4) {
          uint64_t sm[4] = {0, 0, 0, 0};
          const u32x4 c = *(const u32x4*)(qb + j0);
#pragma unroll
          for (int g = 0; g < 4; ++g) {
#pragma unroll
            for (int u = 0; u < 4; ++u) sm[u] = mad_u64_u32(y[u], c[g], sm[u]);
            const int i = t0 + 4 + j0 + g - s;
            y[0] = y[1], y[1] = y[2], y[2] = y[3], y[3] = i >= 0 ? Y[min(i, b)] : 0u;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) A[u].add(sm[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (t0 + u <= top) X[t0 + u] = msub(X[t0 + u], fold96(A[u], q), q.p);
      }
      a -= n;
    }
    __syncthreads();
  }
}

// Zero words below index 0 of a double-buffered array.
__device__ __forceinline__ void clear_pad(uint32_t* X) {
  if (threadIdx.x < PAD) X[-1 - (int)threadIdx.x] = 0u;
}

// Euclid's algorithm over F_p on X (degree a) and Y (degree b) in LDS, run by
// the whole block, without inverses on normal steps: each changes the
// remainder only by a unit factor, so the last non-zero remainder is an
// associate of the gcd.  Leading coefficients must be non-zero.  Returns the
// gcd's degree d, with an associate of the gcd in Y[0..d] (the pointers are
// swapped as the roles alternate; every array needs max(a, b) + 4 words).
// X2, Y2: second buffers for the rounds of 31 steps (null: none, every step
// is a division), all four arrays then with PAD zero words below index 0.
__device__ int block_gcd_fp(uint32_t*& X, uint32_t*& Y, uint32_t*& X2, uint32_t*& Y2, int a, int b, GcdShared& sh,
                            const ModP& q) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = lane_id();
  auto swap = [](uint32_t*& u, uint32_t*& v) {
    uint32_t* t = u;
    u = v;
    v = t;
  };
  if (a < b) {
    swap(X, Y);
    const int t = a;
    a = b;
    b = t;
  }
  if (X2) {
    clear_pad(X);
    clear_pad(Y);
    clear_pad(X2);
    clear_pad(Y2);
  }
  __syncthreads();
  // the first wave's chain of steps is what a round waits for
  if (wave == 0) __builtin_amdgcn_s_setprio(3);
  for (;;) {
    if (b == 0) return 0;  // a non-zero constant divides both
    if (a == b + 1 && X2 && b >= 63) {
      if (wave == 0) {
        const int s = window_steps(X[a - l], Y[b - l], sh.M[0], q);
        if (l == 0) sh.steps = s;
      }
      __syncthreads();
      int cur = 0, s = sh.steps;
      while (s > 0) {
        const int an = a - s, nt = (s + 4) & ~3;  // taps 0..s
        if (wave == 0) {
          int sn = 0;
          if (an >= 64) {
            uint32_t Aw, Bw;
            apply_top(X, Y, sh.M[cur], nt, an, Aw, Bw, q);
            sn = window_steps(Aw, Bw, sh.M[1 - cur], q);
          }
          if (l == 0) sh.a = sn;
        } else {
          apply_matrix(X, Y, X2, Y2, sh.M[cur], nt, an, tid - 64, GB - 64, q);
        }
        __syncthreads();
        s = sh.a;
        swap(X, X2);
        swap(Y, Y2);
        a = an;
        b = an - 1;
        cur ^= 1;
        __syncthreads();  // sh.a is read before the next round writes it
      }
      if (b < 63) continue;
    } else if (a == b + 1 && b <= 62) {
      // the whole pair fits the lanes of one wave
      if (wave == 0) {
        uint32_t A = l <= a ? X[a - l] : 0u, B = l <= b ? Y[b - l] : 0u;
        int bb = b;
        while (bb >= 1) {
          uint32_t tn0;
          const uint32_t R = step_rem(A, B, lane_of(B, 0), mneg_factor(lane_of(A, 0), q.p), tn0, q);
          if (lane_of(R, 0) == 0u) break;
          A = B;
          B = R;
          --bb;
        }
        if (l <= bb + 1) X[bb + 1 - l] = A;
        if (l <= bb) Y[bb - l] = B;
        if (l == 0) sh.b = bb;
      }
      __syncthreads();
      b = sh.b;
      a = b + 1;
      __syncthreads();
      if (b == 0) return 0;
    }
    // a degree gap, or a remainder whose leading coefficient vanishes
    team_mod(X, a, Y, b, minv(Y[b], q), false, sh.q[0], nullptr, 0u, tid, GB, (a - b + TAPS) / TAPS, q);
    // the remainder's degree; every thread has read X before any returns (the
    // caller may write X at once)
    int c = X[b - 1] ? b - 1 : -1;
    __syncthreads();
    if (c < 0) {
      if (tid == 0) sh.a = -1;
      __syncthreads();
      for (int i = tid; i < b - 1; i += GB)
        if (X[i]) c = i;
      if (c >= 0) atomicMax(&sh.a, c);
      __syncthreads();
      c = sh.a;
      __syncthreads();
    }
    if (c < 0) return b;
    swap(X, Y);
    a = b;
    b = c;
    __syncthreads();
  }
}

}  // namespace

// One block per prime.  The gcd is made monic with one inverse; then the two
// halves of the block divide a and b exactly by it.  Outputs are scaled for
// the integer reconstruction: beta g, (lc a / beta) a/g, (lc b / beta) b/g,
// whose images multiply to lc(a) a and lc(b) b.
__global__ __launch_bounds__(GB) void k_gcd_p(GcdDev G, TablesDev tab) {
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ __align__(16) GcdShared sh;
  __shared__ int bad_any;
  const int k = blockIdx.x;
  const ModP q = tab.primes[k];
  const int da = G.da, db = G.db;
  const int ld = (max(da, db) + 4 + PAD + 3) & ~3;
  const int mn = min(da, db);
  uint32_t* X = lds + PAD;
  uint32_t* Y = X + ld;
  uint32_t* X2 = Y + ld;
  uint32_t* Y2 = X2 + ld;
  const int tid = threadIdx.x;
  const uint32_t* ra = G.res_a + (size_t)k * (da + 1);
  const uint32_t* rb = G.res_b + (size_t)k * (db + 1);
  if (ra[da] == 0u || rb[db] == 0u) {
    if (tid == 0) G.gdeg[k] = -2;
    return;
  }
  if (tid == 0) bad_any = 0;
  for (int i = tid; i <= da; i += GB) X[i] = ra[i];
  for (int i = tid; i <= db; i += GB) Y[i] = rb[i];
  __syncthreads();
  const int d = block_gcd_fp(X, Y, X2, Y2, da, db, sh, q);
  const uint32_t beta = G.sc[3 * k], sa = G.sc[3 * k + 1], sb = G.sc[3 * k + 2];
  uint32_t* F = G.F + (size_t)k * (mn + 1);
  uint32_t* qa = G.QA + (size_t)k * (da + 1);
  uint32_t* qb = G.QB + (size_t)k * (db + 1);
  if (d == 0) {  // coprime: the cofactors are a and b
    for (int i = tid; i <= mn; i += GB) F[i] = i ? 0u : mmul(q.one, beta, q);
    for (int i = tid; i <= da; i += GB) qa[i] = mmul(ra[i], sa, q);
    for (int i = tid; i <= db; i += GB) qb[i] = mmul(rb[i], sb, q);
    if (tid == 0) G.gdeg[k] = 0;
    return;
  }
  // monic gcd (Montgomery form) in X2, then a in X and b in Y2 as work arrays
  const uint32_t inv = minv(Y[d], q);
  for (int i = tid; i <= d; i += GB) X2[i] = mmul(Y[i], inv, q);
  for (int i = tid; i <= da; i += GB) X[i] = ra[i];
  for (int i = tid; i <= db; i += GB) Y2[i] = rb[i];
  __syncthreads();
  for (int i = tid; i <= mn; i += GB) F[i] = i <= d ? mmul(X2[i], beta, q) : 0u;
  const int team = tid / (GB / 2);
  const int dn = team ? db : da;
  uint32_t* W = team ? Y2 : X;
  uint32_t* out = team ? qb : qa;
  const int tt = tid - team * (GB / 2);
  const int rounds = (max(da, db) - d + TAPS) / TAPS;
  team_mod(W, dn, X2, d, q.one, true, sh.q[team], out, team ? sb : sa, tt, GB / 2, rounds, q);
  bool bad = false;
  for (int i = tt; i < d; i += GB / 2) bad |= W[i] != 0u;
  for (int i = dn - d + 1 + tt; i <= dn; i += GB / 2) out[i] = 0u;
  if (__ballot(bad) != 0ull && lane_id() == 0) atomicOr(&bad_any, 1);
  __syncthreads();
  if (tid == 0) G.gdeg[k] = bad_any ? -3 : d;
}

// ---------------------------------------------------------------------------
// The degree chain of the N^- / N^+ test (Section 3.2.2) over F_p, two blocks:
//   block 0: S_0 = R* mod p, S_i = gcd(S_{i-1}, sr_i) (i >= 1, until S_i is constant);
//   block 1: deg gcd(R^inf, Q) = the degrees of the gcds removed from Q by
//   H <- H / gcd(H, R*) until that gcd is constant.
// Inputs in Montgomery form or plain as stated; every gcd is block_gcd_fp.

// Degree of v[0..n) (-1 for zero), computed by the block.
__device__ int block_degree(const uint32_t* v, int n, int* red) {
  int top = -1;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    if (v[i] != 0u) top = i;
  __syncthreads();
  if (threadIdx.x == 0) *red = -1;
  __syncthreads();
  if (top >= 0) atomicMax(red, top);
  __syncthreads();
  const int d = *red;
  __syncthreads();
  return d;
}

// dbl: the LDS holds the second buffers of block_gcd_fp (five arrays, else three).
__global__ __launch_bounds__(GB) void k_fiber_chain(ChainDev C, int dbl, TablesDev tab) {
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ __align__(16) GcdShared sh;
  __shared__ int red;
  const ModP q = tab.primes[0];
  const int tid = threadIdx.x;
  const int mx = max(max(C.dr + 1, C.D), C.Dq);
  const int ld = (mx + 3 + PAD + 3) & ~3;
  uint32_t* S = lds + PAD;  // block 0: the current S_i; block 1: H = Q / (removed gcds)
  uint32_t* X = S + ld;
  uint32_t* Y = X + ld;
  uint32_t* X2 = dbl ? Y + ld : nullptr;
  uint32_t* Y2 = dbl ? X2 + ld : nullptr;
  if (blockIdx.x == 0) {
    for (int i = tid; i <= C.dr; i += GB) S[i] = C.rstar[i];
    int ds = block_degree(S, C.dr + 1, &red);
    if (tid == 0) C.out[0] = ds;
    int i = 1;
    for (; i < C.K && ds >= 1; ++i) {
      const uint32_t* sr = C.srs + (size_t)i * C.D;
      for (int t = tid; t < C.D; t += GB) Y[t] = to_mont(sr[t], q);
      const int db = block_degree(Y, C.D, &red);
      if (db >= 0) {  // gcd(S, 0) = S
        for (int t = tid; t <= ds; t += GB) X[t] = S[t];
        __syncthreads();
        const int d = block_gcd_fp(X, Y, X2, Y2, ds, db, sh, q);
        __syncthreads();
        for (int t = tid; t <= d; t += GB) S[t] = Y[t];
        ds = d;
        __syncthreads();
      }
      if (tid == 0) C.out[i] = ds;
    }
    for (; i < C.K; ++i)
      if (tid == 0) C.out[i] = 0;
    return;
  }
  // the common part of R and Q with Q's multiplicities
  for (int t = tid; t <= C.dr; t += GB) Y[t] = C.rstar[t];
  const int d0 = block_degree(Y, C.dr + 1, &red);
  for (int t = tid; t < C.Dq; t += GB) S[t] = to_mont(C.qpol[t], q);
  int dh = block_degree(S, C.Dq, &red);
  int total = 0;
  while (dh >= 1 && d0 >= 1) {
    for (int t = tid; t <= dh; t += GB) X[t] = S[t];
    for (int t = tid; t <= d0; t += GB) Y[t] = C.rstar[t];
    __syncthreads();
    const int d = block_gcd_fp(X, Y, X2, Y2, dh, d0, sh, q);
    __syncthreads();
    if (d == 0) break;
    total += d;
    // H <- H / G (G = Y[0..d]); the quotient goes to X
    team_mod(S, dh, Y, d, minv(Y[d], q), false, sh.q[0], X, q.one, tid, GB, (dh - d + TAPS) / TAPS, q);
    dh -= d;
    for (int t = tid; t <= dh; t += GB) S[t] = X[t];
    __syncthreads();
  }
  if (tid == 0) {
    C.out[C.K] = total;
    C.out[C.K + 1] = dh < 0 ? 1 : 0;
  }
}

static size_t chain_words(int dr, int D, int Dq) {
  int mx = dr + 1 > D ? dr + 1 : D;
  if (Dq > mx) mx = Dq;
  return (size_t)((mx + 3 + PAD + 3) & ~3);
}

size_t fiber_chain_lds_bytes(int dr, int D, int Dq) {
  return (3 * chain_words(dr, D, Dq) + PAD) * sizeof(uint32_t) + sizeof(GcdShared) + 64;
}

void launch_fiber_chain(const ChainDev& C, size_t lds_per_block, TablesDev tab, hipStream_t s) {
  const size_t n = chain_words(C.dr, C.D, C.Dq);
  size_t lds = (5 * n + PAD) * sizeof(uint32_t);
  const int dbl = lds + sizeof(GcdShared) + 64 <= lds_per_block;
  if (!dbl) lds = (3 * n + PAD) * sizeof(uint32_t);
  hipLaunchKernelGGL(k_fiber_chain, dim3(2), dim3(GB), lds, s, C, dbl, tab);
}

size_t gcd_lds_bytes(int da, int db) {
  const int mx = da > db ? da : db;
  return ((size_t)4 * ((mx + 4 + PAD + 3) & ~3) + PAD) * sizeof(uint32_t);
}

void launch_gcd_p(const GcdDev& g, TablesDev tab, hipStream_t s) {
  hipLaunchKernelGGL(k_gcd_p, dim3(g.P), dim3(GB), gcd_lds_bytes(g.da, g.db), s, g, tab);
}

}  // namespace bires
