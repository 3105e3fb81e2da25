// Host-side launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "gemm_plan.h"

namespace dy {

enum DType { F32 = 0, BF16 = 1 };

// A list of token rows living on the device.  idx == nullptr means the identity (row j = token j);
// count == nullptr means exactly `cap` rows.  The device count is clamped to cap by every kernel.
struct Rows {
  const int32_t *idx;
  const int32_t *count;
  int32_t cap;
};

// K splits of a raw GEMM result: the rows below tail_from hold n partial sums each, the rows from
// tail_from on (a short last row tile in tiles of another shape) n_tail.  The split stride is the number of
// rows that exist times the row length.  dev: the plan was made on the device, which left
// {n, tail_from, n_tail, done_to} there (mm::PlanWord); the members are then ignored.
struct Splits {
  int n = 1, tail_from = 0x7fffffff, n_tail = 1;
  int done_to = 0;  // rows below it were finished by the GEMM's own epilogue (down projection, q|k|v); at most the list's capacity
  const int32_t *dev = nullptr;
  __host__ __device__ int of(int j) const { return j < tail_from ? n : n_tail; }
};

// The plan of a GEMM whose rows the device counts, to be made by a row kernel ahead of it (plan_gemm_*): a workgroup of
// that kernel prices the candidates while the others take their rows, and the GEMM reads words.  words == nullptr: no such job.
struct PlanMaker {
  mm::PlanArgs args;
  Rows rows;
  int32_t *words = nullptr;
  bool finishes = false;  // the GEMM finishes the rows whose K is not split
};
// ... and what the launcher of that GEMM keeps of its choice
struct PlanJob {
  PlanMaker make;
  mm::GemmPlan full;       // raw results: the plan of a full list, where it was looked at
  bool finishing = false;  // raw results: the kernel that can finish rows is taken
  bool sums = false;       // down projection: a kernel for split sums follows
};

// Candidates of the approximate update of a sequence (bf16, head_dim 128): up to a fifth of its tokens their keys and
// value residuals lie one after the other, and the normalisers come from a sweep over all keys; from there on the
// residuals lie by token, zero elsewhere, and every key meets them, which needs no sweep.  The step without its FFN half in
// one form and the other, 32 heads, us: 8 x 1024 tokens, 10 / 15 / 20 / 25 / 50 / 100 % candidates 575 617 647 678 870 1258
// against 588 625 646 676 834 1157; 2 x 513 tokens 140 144 150 153 171 232 against 141 144 149 151 166 221; a window of
// 512 of 2048 positions, 1 / 7.5 / 12.5 / 25 % of the sequence 153 165 174 194 against 159 168 175 192.  The line is decided
// per sequence, on the device.
__host__ __device__ inline bool compact_form(int candidates, int L) { return candidates <= L / 5; }
// Row of candidate r (entry j of its list, which has `cap` entries at most) among the [B*L] rows of both forms.  Inside the
// sequence's rows whatever the offsets say.
struct CandidateRow { int row; bool compact; };
__device__ __forceinline__ CandidateRow candidate_row(const int32_t *offsets, int cap, int L, int r, int j) {
  const int b = r / L, lo = min(offsets[b], cap);
  const bool compact = compact_form(min(offsets[b + 1], cap) - lo, L);
  return CandidateRow{compact ? b * L + min(max(j - lo, 0), L - 1) : r, compact};
}
enum DvLayout { DV_NONE, DV_BY_TOKEN, DV_BY_ENTRY, DV_BY_SEQUENCE };

// Where q|k|v (or q alone: no key-value heads) of a row go once they are finished: bias, rotary embedding of q and k by the
// table entry of position (row_j mod L), q at q[j] (q[row_j] when q_by_token), k and v at row_j of the caches.
// rope_tab: [max_seq, dh/2, 2] fp32 (cos, sin).  dh is 64 or 128.
struct QkvOut {
  void *q = nullptr, *k = nullptr, *v = nullptr;
  const void *bq = nullptr, *bk = nullptr, *bv = nullptr;
  const float *tab = nullptr;
  int H = 0, Hkv = 0, dh = 0, L = 0, q_by_token = 0;
  size_t tokens = 0;  // of all sequences
};

// ---- row kernels (HBM-bound) ------------------------------------------------------------------
// out[j,:] (by_token: out[row_j,:]) = RMSNorm(x[row_j,:]) * gain            x: [T,d] T-typed, out: [cap,d] ([T,d]) T-typed
void launch_gather_rmsnorm(DType t, const void *x, const void *gain, Rows rows, int d, float eps,
                           void *out, int by_token, const PlanMaker &job, hipStream_t s);
// The GEMMs leave fp32 "raw" results part[z][j][n] (z = K split, j = position in the row list); the
// finalize kernels below sum the splits and apply the fused tail of the step, one workgroup per row.
//
// What the approximate step keeps of its candidates beside the caches (a kernel of its own: with these in the kernel of
// every step, q of 8192 rows took 55 instead of 42 us):
//   dv        v - v_cache of the rows before the merge, at row_j (DV_BY_TOKEN), at j (DV_BY_ENTRY) or at their candidate_row
//             by `offsets` (DV_BY_SEQUENCE; not for the rows at positions below entry_lo)
//   k         nullptr, or a copy of the rotated k rows at the same places (DV_BY_SEQUENCE: in the compact form only)
//   entry_of  [T]: entry_of[row_j] = j + 1, the map from a token to its list entry, written for the rows at positions
//             >= entry_lo of their sequence only
struct CandidateOut {
  void *dv, *k;
  DvLayout layout;
  const int32_t *offsets;
  int32_t *entry_of;
  int entry_lo;
};
// q/k/v: sum of splits, then as QkvOut says, for the rows from splits.done_to on
void launch_qkv_finalize(DType t, const float *part, Splits splits, Rows rows, const QkvOut &out, const CandidateOut *cand,
                         hipStream_t s);
// out-projection (bf16): h[j] = x[row_j] + sum of splits (fp32 [cap,d]); f[j] = RMSNorm(h[j]) * gain
void launch_oproj_finalize(const float *part, Splits splits, const void *x,
                           const void *gain, Rows rows, int d, float eps, float *h, void *f,
                           const PlanMaker &job0, const PlanMaker &job1, hipStream_t s);
// down projection (bf16) after a K split: out_cache[row_j] = h[j] + sum of splits, for the rows from
// splits.done_to on (the rows below it were written by the GEMM's own epilogue)
void launch_down_finalize(const float *part, Splits splits, const float *h,
                          Rows rows, int d, void *out_cache, hipStream_t s);
// cosine of c_new[j] vs c_cache[row_j], flag = cos < tau, optional commit of the new row.
void launch_saliency(DType t, const void *c_new, void *c_cache, Rows rows, int D, float tau,
                     float *cos_out, uint8_t *flag_out, int commit, hipStream_t s);
// stable compaction over up to 1024 chained workgroups; out_offsets[b] = #selected tokens with id < b*L.
// scan: compact_scan_words() device ints, all zero before the launch; the kernel leaves them zero.
// Launches that share `scan` must not overlap.
void launch_compact(const uint8_t *flag, Rows rows, int B, int L, int32_t *out_idx,
                    int32_t *out_offsets, int out_cap, int32_t *status, int32_t *scan, hipStream_t s);
constexpr int COMPACT_SCAN_WORDS = 2 + 1024;
inline int compact_scan_words() { return COMPACT_SCAN_WORDS; }

// The cosine test from per-head sums, then the same compaction: entry j of `rows` has
// cos = sum_h p[j][h][0] / (max(sqrt(sum_h p[j][h][1]), 1e-8) * max(sqrt(sum_h p[j][h][2]), 1e-8)),
// flag = cos < tau; cos_out[j] and flag_out[j] are written, the flagged tokens compacted as by
// launch_compact.  cos_part: [cap, H, 4] fp32.
void launch_cos_compact(const float *cos_part, int H, float tau, float *cos_out, uint8_t *flag_out, Rows rows,
                        int B, int L, int32_t *out_idx, int32_t *out_offsets, int out_cap, int32_t *status,
                        int32_t *scan, hipStream_t s);

// The union of two lists (any order; ids outside [0, B*L) and positions below pos_lo ignored; a list with
// cap 0 is none) in one launch: flags of all tokens to flag_out, the flagged tokens compacted as by
// launch_compact.  B*L <= MERGE_TOKENS: every workgroup of 256 tokens reads both lists.  Against the four
// launches this replaces (clear, mark twice, compact: 15.8 us): two lists of 80 entries 8.3 us; two full ones
// 14.6 us at 8192 tokens, 40.7 us at 32768.  Every workgroup reads both lists whole, so the time grows with their
// length: the line is the largest of the measured sizes at which even full lists gain.  Short lists, which are the
// usual ones, would gain beyond it.
void launch_merge_compact(Rows a, Rows b, int pos_lo, uint8_t *flag_out, int B, int L, int32_t *out_idx,
                          int32_t *out_offsets, int out_cap, int32_t *status, int32_t *scan, hipStream_t s);
constexpr int MERGE_TOKENS = 8192;

// ---- attention ---------------------------------------------------------------------------------
struct AttnArgs {
  const void *q;        // [cap, H, dh] T-typed; with q_by_token: [T, H, dh], row of query j = rows.idx[j]
  int q_by_token;
  const void *k, *v;    // [B, L, Hkv, dh] T-typed; with key_offsets: compact rows [*, Hkv, dh]
  const int32_t *key_offsets;  // nullptr, or [B+1]: the keys of sequence b are rows [key_offsets[b],
                               // key_offsets[b+1]) of k / v, at most key_cap rows (a split past a sequence's last
                               // key writes nothing)
  int key_cap;
  const void *norm_k;   // nullptr, or (bf16, head_dim 128, with key_offsets) [B, L, Hkv, dh]: the context update of Alg. 4.
                        // k and v are laid out by sequence then (candidate_row): where compact_form holds the rows are
                        // divided by the sum over all of these keys, of which the compact ones are a part; elsewhere v
                        // has a row for every one of these keys.  `splits` and `chunk` cut all L keys
  float *lse_out;       // nullptr, or [T, H]: the merge kernels store log(sum exp) of every merged row here
  Rows rows;            // token ids of the query rows (idx may be nullptr = identity)
  const int32_t *offsets;  // [B+1] per-sequence offsets into rows, or nullptr = every sequence has L rows
  int B, L, H, Hkv, dh;
  int splits;           // key range split into this many parts (>= 1), none of them empty
  int chunk;            // keys per split (multiple of the key tile); split s covers [s*chunk, min(L,(s+1)*chunk))
  int bq;               // query rows per workgroup the plan chose (bf16: 128 or 64; fp32: 16)
  int partial;          // 1: leave partials even for a single split (a finalize kernel follows)
  float *part_o;        // [splits, cap, H*dh] fp32 un-normalised partial outputs
  float *part_ml;       // [splits, cap, H, 2] fp32 (running max in natural-log units, running sum)
  void *out;            // [cap, H*dh] T-typed (unused when partials are left)
  // Fused commit (bf16, head_dim 128, one key split; null otherwise): the attention kernel itself
  // normalises its rows, rounds them to the storage type, reads the cached context row of the query's
  // token (rows.idx, or the identity), overwrites it with the new one, and leaves the three sums the
  // cosine needs -- <new, old>, |new|^2, |old|^2 over the head's dh columns -- in cos_part[j][h][0..2]
  // (fp32, [cap, H, 4]); no partial output is written.
  void *c_commit;       // [T, H*dh] T-typed context cache
  float *cos_part;
};
// attention rows; merges the splits into a.out unless a.partial is set
void launch_attention(DType t, const AttnArgs &a, hipStream_t s);
// exact rows (a) and the context update of Alg. 4 (b: norm_k) in one launch, where both are bf16 with head_dim 128, one key split
// and the same query tile: returns whether they were launched
bool launch_attention_both(const AttnArgs &a, const AttnArgs &b, hipStream_t s);
// merge of the attention partials of a call that left them (a.partial) into a.out (and a.lse_out)
void launch_attn_combine(DType t, const AttnArgs &a, hipStream_t s);
// merge of the attention partials fused with the saliency test and the context commit:
// new = merged row (rounded to T), cos against c_cache[row_j], flag = cos < tau, c_cache[row_j] = new.
// The workgroup that finishes last also compacts the flags into (out_idx, out_offsets) like
// launch_compact; `counter` is a zero-initialised device word the kernel leaves at zero.
void launch_attn_finalize(DType t, const AttnArgs &a, void *c_cache, float tau, float *cos_out,
                          uint8_t *flag_out, int32_t *out_idx, int32_t *out_offsets, int out_cap,
                          int32_t *status, int32_t *counter, hipStream_t s);
// Chooses the query tile, the number of key splits and the keys per split for a call (host);
// rows_per_seq = expected query rows per sequence (capacity / B for a row list, L for a dense step);
// grouped_heads = query heads per KV head.
void attention_plan(DType t, int B, int L, int H, int dh, int cap, int rows_per_seq, size_t part_elems,
                    AttnArgs *a, int grouped_heads);

// ---- GEMMs  C[m,n] = sum_k A[m,k] * W[n,k]  (W [N,K]: row-major for fp32, 32-row panels for bf16) --
struct GemmA {
  const void *a;        // T-typed, row stride lda
  const int32_t *gather;  // nullptr, or row j of the GEMM reads a[gather[j], :]
  int lda;
  // rows of the buffer `a` points to when `gather` is set (without it the row list's capacity bounds
  // the rows read); 0 = unknown.  Kernels that address the operand with 32-bit offsets need it.
  size_t a_rows = 0;
};
// Up to three weight matrices stacked along N (q | k | v); the bf16 kernels look the matrix up per
// tile row, so a column tile may span two of them.
struct WSeg {
  const void *w[3];
  int n_end[3];  // exclusive end column of each segment; N = n_end[2]
};
inline WSeg wseg_one(const void *w, int N) {
  WSeg s;
  s.w[0] = s.w[1] = s.w[2] = w;
  s.n_end[0] = s.n_end[1] = s.n_end[2] = N;
  return s;
}
// raw GEMM: part[z][j][n] = sum over K split z of A[j,:] * W[n,:] (fp32, split stride rows*N);
// returns the numbers of splits used (>= 1), chosen from the rows that exist, N and K (on the device, in
// the PLAN_WORDS words `plan`, when their number is known there alone).
// job: made by plan_gemm_raw of the same arguments and done by a row kernel since, or empty (the GEMM plans for itself).
// qkv: where the results go in the end.  The GEMM may finish rows itself (those below Splits::done_to, which have no raw
// result then); the row kernel finishes the others.  Without a table (raw_beside) it only says which q|k|v the result goes with.
PlanJob plan_gemm_raw(DType t, GemmA A, Rows rows, int K, WSeg seg, size_t part_elems, int32_t *plan, const QkvOut &qkv);
Splits launch_gemm_raw(DType t, GemmA A, Rows rows, int K, WSeg seg, float *part, size_t part_elems,
                       int32_t *plan, const PlanJob &job, const QkvOut &qkv, hipStream_t s);
inline QkvOut raw_beside(int H, int Hkv, int dh, size_t tokens) { return QkvOut{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, H, Hkv, dh, 0, 0, tokens}; }
// up (bf16): act[j,:] = silu(A w_gate^T) * (A w_up^T), out [cap, N]; here and below A[j,:] = a[j,:], rows of K elements
// job: made by plan_gemm_swiglu of the same rows, K and N and done by a row kernel since
PlanJob plan_gemm_swiglu(Rows rows, int K, int N, int32_t *plan);
void launch_gemm_swiglu(const void *a, Rows rows, int K, int N, const void *w_gate,
                        const void *w_up, void *act, const PlanJob &job, hipStream_t s);
// down: out_cache[row_j,:] = h[j,:] + A[j,:] * w_down^T, T-typed scatter into [T, N]; `scratch`
// holds K-split partials when K is split; job: as for launch_gemm_swiglu.
PlanJob plan_gemm_down(DType t, Rows rows, int K, int N, size_t scratch_elems, int32_t *plan);
void launch_gemm_down(DType t, const void *a, Rows rows, int K, int N, const void *w_down, const float *h,
                      void *out_cache, float *scratch, size_t scratch_elems, const PlanJob &job, hipStream_t s);

// fp32: the same steps without row kernels between them.  K is never split, so a GEMM finishes its rows, and each takes its
// operand's RMSNorm along.
// q|k|v of RMSNorm(x[row_j,:]) * gain, or without a gain of x[j,:], finished as QkvOut says.  x is read while results are written:
// none of them may lie in its rows.
void launch_qkv_f32(const void *x, const void *gain, float eps, Rows rows, int K, WSeg seg, const QkvOut &out, hipStream_t s);
// h[j,:] = x[row_j,:] + A[j,:] * wo^T
void launch_oproj_f32(GemmA A, Rows rows, int K, int N, const void *wo, const void *x, float *h, hipStream_t s);
// act[j,:] = silu(n w_gate^T) * (n w_up^T) of n = RMSNorm(h[j,:]) * gain
void launch_swiglu_f32(const float *h, const void *gain, float eps, Rows rows, int K, int N, const void *w_gate,
                       const void *w_up, void *act, hipStream_t s);

// row-major [n_out, n_in] (2-byte elements; n_out % 32 == 0, n_in % 64 == 0) -> weight panels of the bf16 GEMMs
void launch_pack_weight(const void *src, int n_out, int n_in, void *dst, hipStream_t s);
void launch_fill_i32(int32_t *p, int32_t v, int n, hipStream_t s);

// ---- approximate (column-sparse) context update of the non-salient rows  [Sec. 3.3; Alg. 3, Alg. 4]
// pos[row_j] = j + 1 for the candidates among the step's tokens (written by the k|v finalize kernel of
// the step through its entry_of argument, consumed and zeroed by launch_saliency_approx; pos is zero
// elsewhere, before and after a step)
// For every entry j of the window `win` (token r = win.idx[j], or j): new context = c_sal[pos[r]-1]
// where pos[r] != 0, else c_cache[r] + residual (rounded to T); cosine against the cached row, commit;
// cos_out[r] (may be nullptr), flag_out[j] = cos < tau.  The residual is dc[j], or (cached != nullptr)
// sum over the key splits s of part_o[s][j] * exp(m_s - lse[r, h]) from the partials of an attention
// pass over the compact candidate keys (cached->key_offsets) -- the normalisers are NOT recomputed.
// Every pos entry that is read non-zero is set back to zero, and so is the residual row of that token where the
// residuals lie by sequence (residuals.dv).
struct Residuals {
  void *dv = nullptr;  // [T, dkv] T-typed, rows by candidate_row of the list entry
  const int32_t *offsets = nullptr;
  int cap = 0, L = 0, dkv = 0;
};
void launch_saliency_approx(DType t, Rows win, int D, const void *c_sal, const void *dc, int32_t *pos,
                            void *c_cache, float tau, float *cos_out, uint8_t *flag_out,
                            const AttnArgs *cached, const float *lse, int L, Residuals residuals, hipStream_t s);
// idx/off := the tokens at positions [lo, L) of each of the B sequences, as an index list
void launch_make_window(int B, int L, int lo, int32_t *idx, int32_t *off, hipStream_t s);
// flag[r] = 1 for every token r < T of the list whose position in its sequence is >= lo
void launch_mark_flags(Rows rows, int T, int L, int lo, uint8_t *flag, hipStream_t s);
// dv[row_j, :] = 0 for the rows of the list
void launch_clear_rows(DType t, Rows rows, void *dv, int dkv, hipStream_t s);

}  // namespace dy
