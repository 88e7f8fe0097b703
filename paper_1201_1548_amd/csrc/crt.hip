// (e) the explicit CRT for any prime count whose operands fit in LDS (in
// practice up to 630 primes; k_crt_mfma in kernels.hip keeps the
// small counts, whose left operands fit in registers), and its tables.
//
// The formula is k_crt_mfma's: with M = prod p_k, y_k the symmetric
// representative of x_k (M / p_k)^{-1} mod p_k and t the integer nearest to
// sum y_k / p_k, the coefficient is X - t M, X = sum_k y_k M / p_k, and X is a
// product [rows x 4P] x [4P x byte columns] of balanced base-256 digits with
// |S_c| <= P (3 * 128 + 64) 128 < 2^31.
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "job.hpp"
#include "kernels.hpp"

namespace bires {

// ---------------------------------------------------------------------------
// Tables of a prime count P (layout of crt_operand_offset): w_k, the digits of
// the M / p_k, the words of M, the right operand in operand order.

// One thread per prime: M / p_k by exact division from the low limb up (each
// quotient word is the remaining low word times p^{-1} mod 2^32), each word
// stored as its four balanced base-256 digits: adding 0x80 at every byte with
// the carries of the whole number and flipping those bits again. M / p_k <
// 2^(32 LM - 30), so nothing is carried out of the top word.  The words of M
// come from the table of radix products.
__global__ __launch_bounds__(64) void k_crt_rows(TablesDev tab, int P, int LM, uint32_t* buf) {
  const int k = blockIdx.x * 64 + threadIdx.x;
  const uint32_t* M = tab.pi + (size_t)P * (P + 1) / 2;
  if (blockIdx.x == 0)
    for (int l = threadIdx.x; l < LM; l += 64) buf[(size_t)P + (size_t)P * LM + l] = M[l];
  if (k >= P) return;
  const uint32_t p = tab.primes[k].p, pin = 0u - tab.primes[k].pinv;
  uint32_t* row = buf + (size_t)P + (size_t)k * LM;
  uint32_t borrow = 0u;
  uint64_t c = 0;
  for (int l = 0; l < LM; ++l) {
    const uint32_t m = M[l], t = m - borrow, qd = t * pin;
    borrow = (uint32_t)(((uint64_t)qd * p) >> 32) + (m < borrow ? 1u : 0u);
    c += (uint64_t)qd + 0x80808080u;
    row[l] = (uint32_t)c ^ 0x80808080u;
    c >>= 32;
  }
}

// One wave per prime: w_k = ((M / p_k) mod p_k)^{-1} from the product of the
// differences p_j - p_k, j != k (the table's primes differ by less than 2^30).
__global__ __launch_bounds__(64) void k_crt_weights(TablesDev tab, int P, uint32_t* buf) {
  const int k = blockIdx.x, l = threadIdx.x;
  const ModP q = tab.primes[k];
  uint32_t r = q.one;
  for (int j = l; j < P; j += 64) {
    const uint32_t pj = tab.primes[j].p;
    if (j != k) r = mmul(r, to_mont(pj > q.p ? pj - q.p : pj, q), q);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) r = mmul(r, __shfl_xor(r, o), q);
  const uint32_t w = minv(r, q);
  if (l == 0) buf[k] = w;
}

// One 1 KiB operand block per wave: column tile blockIdx.x, step blockIdx.y;
// lane L = x + 32 g holds column 32 ct + x, indices 32 ks + 16 g + 0..15 =
// (prime, digit s) with entry digit (column - s) of M / p_k.
__global__ __launch_bounds__(64) void k_crt_operand(int P, int LM, uint32_t* buf, size_t off) {
  const int ct = blockIdx.x, ks = blockIdx.y, nks = gridDim.y, L = threadIdx.x;
  const int col = 32 * ct + (L & 31);
  u32x4 v = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int k = 8 * ks + 4 * (L >> 5) + j;
    const uint8_t* e = (const uint8_t*)(buf + (size_t)P + (size_t)min(k, P - 1) * LM);
    uint32_t x = 0u;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int c = col - s;
      if (c >= 0 && c < 4 * LM && k < P) x |= (uint32_t)e[c] << (8 * s);
    }
    v[j] = x;
  }
  *(u32x4*)(buf + off + ((size_t)ct * nks + ks) * 256 + 4 * L) = v;
}

// B's word offset, its column tiles and steps, and the words of the buffer.
static size_t operand_offset(int P, int LM) { return ((size_t)P + (size_t)P * LM + LM + 3) & ~(size_t)3; }
static int column_tiles(int LM) { return (4 * LM + 4 + 31) / 32; }

size_t crt_table_words(int P, int LM) { return operand_offset(P, LM) + (size_t)column_tiles(LM) * ((P + 7) / 8) * 256; }

void launch_crt_tables(TablesDev tab, int P, int LM, uint32_t* buf, hipStream_t s) {
  hipLaunchKernelGGL(k_crt_rows, dim3((P + 63) / 64), dim3(64), 0, s, tab, P, LM, buf);
  hipLaunchKernelGGL(k_crt_weights, dim3(P), dim3(64), 0, s, tab, P, buf);
  hipLaunchKernelGGL(k_crt_operand, dim3(column_tiles(LM), (P + 7) / 8), dim3(64), 0, s, P, LM, buf,
                     operand_offset(P, LM));
}

// ---------------------------------------------------------------------------
// One block of eight waves per 32 coefficients of a job.
//   1. All threads form the digit words of the 32 rows' y_k straight into the
//      left operand blocks in LDS (4 bytes per prime and row) and the fp64
//      partial sums of y_k / p_k.
//   2. Wave w takes the column tiles w, w + 8, ...: a chain of
//      v_mfma_i32_32x32x32_i8 over the steps with the right operand from L2, the
//      tile through LDS, and lane x + 32 h folds row x's 16 byte columns of
//      half h into four limbs of X - t M with carry 0 coming in.  Limbs go to the
//      output row; the carry out of each four-limb segment, its lowest limb
//      and whether the other three are all zeros go to LDS.
//   3. One lane per row adds each segment's carry into the next one's lowest
//      limb; a carry that leaves that limb (about one in 2^12) ripples through
//      the other three.
// Every tile is independent until 3, so the eight waves share the columns of
// a row; a serial carry chain over all columns in one wave would leave most of
// the chip idle at a few thousand rows.  Bound: the right operand's traffic
// from L2, 16 P LM bytes per block.  Measured against Garner's digits, limb sums
// and carries (a wave's chain of P^2 / 2 products per coefficient): 573 primes
// and 4097 coefficients (one degree-64 resultant) 2290 -> 143 us; 64 serving
// requests 4550 -> 520 us with the small counts' launches; the three
// polynomials of a degree-1560 gcd over 150 primes 308 -> 55 us.
namespace {
constexpr int CBW = 8;          // waves per block
constexpr int CB_TAIL = 20;     // limbs at and above the output's limb count kept for the range check
struct CbLayout {
  int KS, NCT, NS, ld;          // steps, column tiles, segments, stride of the segment records
  size_t a, t, cr, l0, fl, fs, tq, ms, tail, bytes;
};
__host__ __device__ inline CbLayout cb_layout(int P, int LM) {
  CbLayout c;
  c.KS = (P + 7) >> 3;
  c.NCT = (4 * LM + 4 + 31) >> 5;
  c.NS = 2 * c.NCT;
  c.ld = c.NS | 1;
  size_t o = 0;
  c.a = o, o += (size_t)c.KS * 1024;
  c.t = o, o += (size_t)CBW * 32 * 33 * 4;
  c.fs = c.t;  // the partial sums are done with before the tiles are written
  c.cr = o, o += (size_t)32 * c.ld * 4;
  c.l0 = o, o += (size_t)32 * c.ld * 4;
  c.ms = o, o += (size_t)8 * c.NCT * 4;
  c.tq = o, o += 32 * 4;
  c.tail = o, o += (size_t)32 * CB_TAIL * 4;
  c.fl = o, o += (size_t)32 * c.ld;
  c.bytes = (o + 15) & ~(size_t)15;
  return c;
}
}  // namespace

__global__ __launch_bounds__(64 * CBW) void k_crt_big(const JobDev* jobs, const int* starts, int nj, TablesDev tab) {
  extern __shared__ __align__(16) uint8_t cb_lds[];
  const int job = find_job(starts, nj, blockIdx.x, gridDim.x);
  const JobDev& J = jobs[job];
  const int P = J.P, D = J.D, Lc = J.Lcap, LM = J.crt_LM;
  const CbLayout cl = cb_layout(P, LM);
  const int KS = cl.KS, NCT = cl.NCT, NS = cl.NS, ld = cl.ld;
  const int tid = threadIdx.x, l = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bj = blockIdx.x - starts[job], c0 = bj * 32;
  uint32_t* A = (uint32_t*)(cb_lds + cl.a);
  int32_t* T = (int32_t*)(cb_lds + cl.t) + wv * 32 * 33;
  double* fs = (double*)(cb_lds + cl.fs);
  int32_t* cr = (int32_t*)(cb_lds + cl.cr);
  uint32_t* l0 = (uint32_t*)(cb_lds + cl.l0);
  uint8_t* fl = cb_lds + cl.fl;
  int32_t* tq = (int32_t*)(cb_lds + cl.tq);
  uint32_t* Ms = (uint32_t*)(cb_lds + cl.ms);
  uint32_t* tail = (uint32_t*)(cb_lds + cl.tail);
  const uint32_t* Mw = J.crt + P + (size_t)P * LM;
  const __attribute__((address_space(1))) uint32_t* Bt =
      gmem(J.crt) + (((size_t)P + (size_t)P * LM + LM + 3) & ~(size_t)3) + 4 * l;
  {
    // this block's share of the zero coefficients above the job's last block
    const int nbj = (min(D, J.degcap + 1) + 31) / 32, cz = nbj * 32;
    if (cz <= J.degcap) {
      const long long nw = (long long)(J.degcap + 1 - cz) * Lc, share = (nw + nbj - 1) / nbj;
      const long long w0 = bj * share, w1 = min(nw, w0 + share);
      uint32_t* dst = J.out + (size_t)cz * Lc;
      for (long long i = w0 + tid; i < w1; i += 64 * CBW) dst[i] = 0u;
    }
  }
  for (int w = tid; w < 8 * NCT; w += 64 * CBW) Ms[w] = w < LM ? Mw[w] : 0u;
  {
    const int x = tid & 31, kg = tid >> 5;
    const bool rv = c0 + x < D;
    const uint32_t* col = J.coefs + min(c0 + x, D - 1);
    double f = 0.0;
#pragma unroll 4
    for (int k = kg; k < 8 * KS; k += 2 * CBW) {
      const int kc = min(k, P - 1);
      const uint32_t p = tab.primes[kc].p, pinv = tab.primes[kc].pinv;
      const uint32_t y = redc((uint64_t)col[(size_t)kc * D] * J.crt[kc], p, pinv);
      const bool live = rv && k < P;
      const int32_t ys = y > (p >> 1) ? (int32_t)(y - p) : (int32_t)y;
      f = fma((double)(live ? ys : 0), tab.inv_p[kc], f);
      A[(k >> 3) * 256 + (x + 32 * ((k >> 2) & 1)) * 4 + (k & 3)] = live ? digits4(y, p) : 0u;
    }
    fs[kg * 32 + x] = f;
  }
  __syncthreads();
  if (tid < 32) {
    double f = 0.0;
    for (int g = 0; g < 2 * CBW; ++g) f += fs[g * 32 + tid];
    tq[tid] = (int32_t)floor(f + 0.5);  // |t| <= P / 2
  }
  __syncthreads();
  const int Lt = Lc & ~3;  // first limb of the segment that holds the output's end
  {
    const int row = l & 31, h = l >> 5;
    const int64_t t = tq[row];
    const bool live = c0 + row <= J.degcap;
    uint32_t* orow = J.out + (size_t)(c0 + row) * Lc;
    // Every wave starts its chains at another step: in step with each other the
    // waves of all blocks would ask the same few channels of the L2 for the same
    // lines (a step is 1 KiB, the channels repeat every 4 KiB): 252 us instead of 143
    // for 573 primes and 4097 coefficients.
    const int k0 = (int)((unsigned)(wv * 9 + bj * 5) % (unsigned)KS);
    for (int ct = wv; ct < NCT; ct += CBW) {
      im_v16i acc = {0};
      const __attribute__((address_space(1))) uint32_t* Bc = Bt + (size_t)ct * KS * 256;
#pragma unroll 8
      for (int i = 0; i < KS; ++i) {
        const int ks = i + k0 < KS ? i + k0 : i + k0 - KS;
        const im_v4i a = *(const im_v4i*)(A + ks * 256 + 4 * l);
        const im_v4i b = *(const __attribute__((address_space(1))) im_v4i*)(Bc + (size_t)ks * 256);
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, acc, 0, 0, 0);
      }
      // accumulator register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
#pragma unroll
      for (int r = 0; r < 16; ++r) T[(8 * (r >> 2) + 4 * h + (r & 3)) * 33 + row] = acc[r];
      group_sync<true>();
      const int32_t* tr = T + row * 33 + 16 * h;
      const int seg = 2 * ct + h;
      int64_t carry = 0;
      uint32_t limb[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int64_t v = carry + tr[4 * w] + ((int64_t)tr[4 * w + 1] << 8) + ((int64_t)tr[4 * w + 2] << 16) +
                          ((int64_t)tr[4 * w + 3] << 24) - t * (int64_t)Ms[4 * seg + w];
        limb[w] = (uint32_t)v;
        carry = v >> 32;
      }
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const int L = 4 * seg + w;
        if (live && L < Lc) orow[L] = limb[w];
        if (L >= Lt && L - Lt < CB_TAIL) tail[row * CB_TAIL + L - Lt] = limb[w];
      }
      cr[row * ld + seg] = (int32_t)carry;  // |S_c| 2^24 / 2^32 and t M's share: below 2^27
      l0[row * ld + seg] = limb[0];
      fl[row * ld + seg] = (limb[1] | limb[2] | limb[3]) == 0u;
      group_sync<true>();
    }
  }
  __syncthreads();
  bool nz = false;
  if (tid < 32 && c0 + tid <= J.degcap) {
    const int row = tid;
    uint32_t* orow = J.out + (size_t)(c0 + row) * Lc;
    uint32_t* trow = tail + row * CB_TAIL;
    auto get = [&](int L) { return L < Lc ? orow[L] : trow[L - Lt]; };
    auto put = [&](int L, uint32_t v) {
      if (L < Lc) orow[L] = v;
      if (L >= Lt && L - Lt < CB_TAIL) trow[L - Lt] = v;
    };
    int64_t c = 0;  // carry into the segment
    for (int s = 0; s < NS; ++s) {
      const uint32_t low = l0[row * ld + s];
      const int64_t v = c + (int64_t)(uint64_t)low;
      const uint32_t nl = (uint32_t)v;
      int64_t up = v >> 32;
      if (nl != low) put(4 * s, nl);
      if (up == 0) {
        nz |= nl != 0u || !fl[row * ld + s];
      } else {
        nz |= nl != 0u;
        for (int w = 1; w < 4; ++w) {
          if (4 * s + w - Lt >= CB_TAIL) break;  // (not reached: see the host's check)
          const int64_t u = up + (int64_t)(uint64_t)get(4 * s + w);
          put(4 * s + w, (uint32_t)u);
          nz |= (uint32_t)u != 0u;
          up = u >> 32;
        }
      }
      c = up + cr[row * ld + s];
    }
    // the number fits when everything above the output's limbs is its sign
    const uint32_t ext = c < 0 ? 0xFFFFFFFFu : 0u;
    bool bad = c != 0 && c != -1;
    const int top = min(Lc, 4 * NS);
    for (int L = Lc; L < 4 * NS; ++L) bad |= L - Lt >= CB_TAIL || trow[L - Lt] != ext;
    bad |= (get(top - 1) >> 31) != (ext >> 31);
    nz |= ext != 0u && Lc > 4 * NS;
    tq[row] = (int32_t)ext;
    if (bad && c0 + row < D) atomicOr(J.err, 1);
  }
  if (wv == 0) {
    const uint64_t any = __ballot(nz);
    if (any && l == 0) atomicMax(J.deg_out, c0 + 63 - __clzll((long long)any));
  }
  __syncthreads();
  // limbs above the last byte column
  const int nx = Lc - 4 * NS, nr = min(32, J.degcap + 1 - c0);
  for (int i = tid; nx > 0 && i < nr * nx; i += 64 * CBW) {
    const int r = i / nx;
    J.out[(size_t)(c0 + r) * Lc + 4 * NS + (i - r * nx)] = (uint32_t)tq[r];
  }
}

size_t crt_big_lds_bytes(int P, int LM) { return cb_layout(P, LM).bytes; }

// The range check keeps CB_TAIL limbs from the end of the output row on.
bool crt_big_limbs_ok(int LM, int lcap) { return 8 * column_tiles(LM) - (lcap & ~3) <= CB_TAIL; }

bool crt_fits(int P, int LM, int lcap, size_t lds_per_block) {
  const int c = crt_class(P);
  return c >= 0 && (c != CRT_BIG || (crt_big_lds_bytes(P, LM) <= lds_per_block && crt_big_limbs_ok(LM, lcap)));
}

void launch_crt_big(const JobDev* jobs, const int* starts, int nj, int nblocks, size_t lds, TablesDev tab,
                    hipStream_t s) {
  hipLaunchKernelGGL(k_crt_big, dim3(nblocks), dim3(64 * CBW), lds, s, jobs, starts, nj, tab);
}

}  // namespace bires
