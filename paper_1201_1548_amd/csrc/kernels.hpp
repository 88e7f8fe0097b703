// Launchers of the HIP kernels in kernels.hip (host-callable, no HIP types
// beyond hipStream_t and the plain structs of job.hpp).
#pragma once
#include <hip/hip_runtime.h>

#include "job.hpp"

namespace bires {

// Planning statistics of one limb rectangle: out[3*j + {0,1,2}] =
// (x-degree of row j or -1, max bit length of |c| in the row, non-zero count).
struct ScanTask {
  const uint32_t* limbs;
  int32_t rows, ld, L;
  int32_t* out;
};

// waves: the largest scan_waves of the tasks
int scan_waves(int rows, int ld, int L);
void launch_scan(const ScanTask* tasks, const int4* bmap, int nblocks, int waves, hipStream_t s);
// Issue-rate probe: kind 0..5 = v_add_u32, v_min_u32, v_mul_lo_u32,
// v_mad_u64_u32, v_fma_f64 (16 chains per lane), v_mfma_i32_32x32x32_i8
// (16 products per round over 4 accumulators); `iters` rounds; out holds
// blocks * 256 words.
void launch_issue_rate(int kind, uint32_t* out, int blocks, int iters, hipStream_t s);
// Sets *flag (not cleared here) when got[0..n) and want[0..n) differ.
void launch_stats_check(const int32_t* got, const int32_t* want, long long n, int* flag, hipStream_t s);
// dst[0..words) = src_mapped[0..words): src_mapped is the device mapping of
// pinned host memory (hipHostGetDevicePointer).
void launch_upload(const uint32_t* src_mapped, uint32_t* dst, long long words, hipStream_t s);
void launch_transpose(const uint32_t* src, uint32_t* dst, int rows, int cols, int L, hipStream_t s);
// Job launchers: starts[0..nj] hold the first block of each job (starts[nj] = nblocks).
// Blocks per job: reduce ceil(Tf/64)+ceil(Tg/64); eval_elim P*ceil(D/64);
// interp P; mrc D; limbs_sum ceil(D*Lacc/256); limbs_carry ceil((degcap+1)/64).
void launch_reduce(const JobDev* jobs, const int* starts, int nj, int nblocks, int max_primes, TablesDev tab,
                   hipStream_t s);
int eval_elim_block();
// Residue rows are stored at a stride rounded up to a multiple of 4 words so
// the evaluation reads them as aligned 16-byte groups.
inline int pad4(int ld) { return (ld + 3) & ~3; }
// max_words: max over jobs of m+n+2; max_res: max over jobs of Tf+Tg (padded).
size_t eval_elim_lds_bytes(int words, int res);
void launch_eval_elim(const JobDev* jobs, const int* starts, int nj, int nblocks, int max_words, int max_res,
                      TablesDev tab, hipStream_t s);
// Evaluation + elimination with both coefficient arrays in registers (ee.hip):
// the register capacity C (24, 32, 48 or 68) for a job of degrees m, n in the
// eliminated variable, or 0 when the job needs the LDS kernel (min(m, n) = 0
// or max(m, n) >= 68).  launch_eval_elim_rg runs the blocks of jobs with that
// capacity, whose residues are digit words (JobDev::dig) followed by at least
// EE_SLACK_BYTES of workspace, then recomputes with the LDS kernel (max_words:
// max over jobs of m + n + 2) the blocks that leave the uniform normal case.
// fb_count: one device int, zero before the launch; fb_queue: nblocks ints of
// workspace.
constexpr size_t EE_SLACK_BYTES = 512;
int eval_elim_rg_capacity(int m, int n);
// Whether a job of capacity 24 is better left to the general kernel (row: the
// coefficients of its longest row; instances: points times primes of the call).
bool eval_elim_light(int m, int n, int row, long long instances);
void launch_eval_elim_rg(int C, const JobDev* jobs, const int* starts, int nj, int nblocks, int max_words,
                         int* fb_count, int* fb_queue, TablesDev tab, hipStream_t s);
// TablesDev::pow_planes for blocks < nb and primes < P on tab's nodes.
size_t pow_planes_bytes(int nb, int P);
void launch_pow_planes(TablesDev tab, int nb, int P, int8_t* out, hipStream_t s);
// The recomputation of launch_eval_elim_rg's queued blocks by at most max_blocks.
void launch_eval_elim_fb(const JobDev* jobs, const int* starts, int nj, int nblocks, int max_blocks, int max_words,
                         const int* fb_count, const int* fb_queue, TablesDev tab, hipStream_t s);
// Evaluation + elimination by the Schur algorithm on the displacement
// generators, one wave (block of 64) per (prime, point) instance: P * D blocks
// per job; rows per lane NR = schur_rows_per_lane(m, n) (0: the job cannot
// use it: min(m, n) = 0 or m + n > 128); max_words: max over jobs of m + n + 2.
int schur_rows_per_lane(int m, int n);
// fallbacks: one device int counting the instances recomputed by Euclid.
void launch_schur(int NR, const JobDev* jobs, const int* starts, int nj, int nblocks, int max_words, int* fallbacks,
                  TablesDev tab, hipStream_t s);
// Interpolation of one (job, prime) per block.  W, Q: the block tables of
// launch_interp_tables for tab_blocks blocks (null: computed in the kernel).
void launch_interp(const JobDev* jobs, const int* starts, int nj, int nblocks, int max_points, TablesDev tab,
                   const uint32_t* W, const uint32_t* Q, int tab_blocks, hipStream_t s);
// Newton-to-monomial block tables for `blocks` 32-node blocks (enough for
// max_points nodes: interp_table_blocks) and the first `primes` primes:
// interp_table_words words, W at 0 and Q at *q_offset.
int interp_table_blocks(int max_points);
size_t interp_table_words(int blocks, int primes, size_t* q_offset);
void launch_interp_tables(int blocks, int primes, TablesDev tab, uint32_t* W, uint32_t* Q, hipStream_t s);
size_t interp_lds_words(int D);
// Interpolation on the geometric nodes 2^i (interp_geo.hip): the tables of P
// primes for Dc indices (a multiple of 256; geo_table_bytes in all), and one
// block per (job, prime) of the jobs of one class (geo_class of D); the jobs'
// values are those at the nodes tab.qpow and tab.geo_D covers max_points.
size_t geo_table_bytes(int Dc, int P);
void launch_geo_tables(const ModP* primes, int Dc, int P, uint32_t* qpow, uint32_t* invu, uint32_t* wt, int8_t* A,
                       hipStream_t s);
constexpr int GEO_CLASSES = 4;
int geo_class(int D);
void launch_interp_geo(int cls, const JobDev* jobs, const int* starts, int nj, int nblocks, int max_points,
                       TablesDev tab, hipStream_t s);
// Interpolation of N jobs sharing D and P (gco[n] the coefs of job n of the
// group) as int8 matrix-core products with V^{-1}: Ap = vinv_bytes(Dp, P)
// bytes built by launch_vinv (Dp = D rounded up to 32); Yp = 4 Np Dp P bytes
// (Np = N rounded up to 32) holding the jobs' values as digit planes, which
// the evaluation kernels write (JobDev::yp).  Writes the jobs' coefs.
size_t vinv_bytes(int Dp, int P);
void launch_vinv(int D, int Dp, int P, TablesDev tab, int8_t* Ap, hipStream_t s);
void launch_interp_mfma(uint32_t* const* gco, int N, int D, int P, const int8_t* Ap, const int8_t* Yp, TablesDev tab,
                        hipStream_t s);
void launch_invfact(const ModP* primes, int K, uint32_t* invfact, int dmax, hipStream_t s);
// Garner digits: one wave per coefficient, D blocks per job.
void launch_mrc(const JobDev* jobs, const int* starts, int nj, int nblocks, int max_primes, TablesDev tab,
                hipStream_t s);
// Explicit CRT straight to limbs on the matrix cores (k_crt_mfma): one wave
// per rows = crt_rows_per_block(max primes) output coefficients,
// ceil(min(D, degcap + 1) / rows) blocks per job, which also write the job's
// zero coefficients above them up to degcap; needs at most
// CRT_SMALL_PRIMES, the jobs' crt tables (launch_crt_tables) and
// crt_lds_bytes(max output limbs, max primes) within the LDS per block.
// Classes of prime counts: 0..5 one instance of k_crt_mfma each (counts up to
// crt_class_primes(c)), CRT_BIG k_crt_big; crt_class gives -1 above
// CRT_MAX_PRIMES.
constexpr int CRT_SMALL_PRIMES = 128, CRT_MAX_PRIMES = 1024, CRT_BIG = 6, CRT_CLASSES = 7;
int crt_class(int primes);
int crt_class_primes(int cls);
// k_crt_big: blocks of 32 coefficients, LDS crt_big_lds_bytes(P, LM) (the
// largest of the launch), output rows with crt_big_limbs_ok.
size_t crt_big_lds_bytes(int P, int LM);
bool crt_big_limbs_ok(int LM, int lcap);
// Whether the kernel of P's class takes a job of P primes (a modulus of LM limbs)
// with output rows of lcap limbs; of the small classes the launch's LDS remains
// to be checked.  No tables are needed for the answer, and none should be
// built before it.
bool crt_fits(int P, int LM, int lcap, size_t lds_per_block);
void launch_crt_big(const JobDev* jobs, const int* starts, int nj, int nblocks, size_t lds, TablesDev tab,
                    hipStream_t s);
// Explicit CRT constants of the first P primes, M = prod_{k<P} p_k: one
// buffer of crt_table_words(P, LM) words [w (P) | digit rows (P x LM) | M (LM) |
// pad to 4 words | B] with w[k] the Montgomery form of ((M / p_k) mod p_k)^{-1}
// mod p_k, LM the limbs of M and row k the balanced base-256 digits of M / p_k
// (4 per word).  B is the int8 operand of the matrix-core CRT: entry
// (k, s; c) = digit c - s of M / p_k (zero outside 0..4 LM - 1) for
// contraction index 4 k + s and byte column c, in operand order: for column
// tile ct (32 columns) and contraction step ks (32 indices, 8 primes) one 1 KiB
// block whose lane x + 32 g holds column 32 ct + x, indices 32 ks + 16 g + 0..15.
size_t crt_table_words(int P, int LM);
void launch_crt_tables(TablesDev tab, int P, int LM, uint32_t* buf, hipStream_t s);
size_t crt_lds_bytes(int max_lcap, int max_primes);
size_t crt_lds_bytes_rows(int max_lcap, int max_primes, int rows);
// the CRT's LDS strides: limb rows (sld) and prime constants (cps)
int crt_row_stride(int max_lcap);
int crt_const_stride(int max_primes);
int crt_rows_per_block(int max_primes);
void launch_crt(const JobDev* jobs, const int* starts, int nj, int nblocks, int max_primes, int max_lcap,
                TablesDev tab, hipStream_t s);
void launch_limbs_sum(const JobDev* jobs, const int* starts, int nj, int nblocks, TablesDev tab, hipStream_t s);
// Persistent fused launch (see FusedPlan), blocks of 256 threads: C the
// register Euclid's capacity (fused_capacity: 24, 32, or 0 for the LDS
// kernel only), KS = fused_crt_steps(max primes); blocks of one CU at once
// for this LDS size (0 on a runtime error).  The matrix-core interpolation
// takes fused_interp_lds_bytes per block (64 x 32 blocks of C), the CRT
// crt_lds_bytes_rows(.., 32) per wave.
int fused_capacity(int rg_capacity);
int fused_crt_steps(int max_primes);
int fused_blocks_per_cu(int C, int KS, size_t lds_bytes);
size_t fused_interp_lds_bytes();
void launch_fused(int C, int KS, const FusedPlan& F, size_t lds_bytes, int blocks, TablesDev tab, hipStream_t s);
// Principal subresultant coefficients modulo prime index 0 of tab (the caller
// shifts the table to its prime): one lane per point a < J.D, J.m and J.n the
// formal degrees; writes sr_i(a) (plain) to num[i * D + a] for i < K, with
// den ([K][D]) as workspace.
size_t psc_lds_bytes(int m, int n);
// J.dig = psc_registers(m, n): in registers (ee.hip; fallback: one int per 64
// points), the blocks it leaves and all others with the arrays in LDS.
bool psc_registers(int m, int n);
void launch_psc(const JobDev& J, TablesDev tab, uint32_t* num, uint32_t* den, int K, int* fallback, hipStream_t s);
void launch_psc_ee(const JobDev& J, TablesDev tab, uint32_t* out, int K, int* fallback, hipStream_t s);
// The N^- / N^+ degree chain over prime index 0 of tab, two blocks (the second
// buffers of the gcds only where lds_per_block has room for them).
size_t fiber_chain_lds_bytes(int dr, int D, int Dq);
void launch_fiber_chain(const ChainDev& C, size_t lds_per_block, TablesDev tab, hipStream_t s);
size_t gcd_lds_bytes(int da, int db);
void launch_gcd_p(const GcdDev& g, TablesDev tab, hipStream_t s);
void launch_gather_rows(const uint32_t* src, int ld, const int* idx, int rows, int n, uint32_t* dst, hipStream_t s);
// max_lcap: the largest Lcap of the jobs in the launch.
void launch_limbs_carry(const JobDev* jobs, const int* starts, int nj, int nblocks, int max_lcap, hipStream_t s);

}  // namespace bires
