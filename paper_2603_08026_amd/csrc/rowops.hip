// Row-wise kernels of the sparse layer step: gather + RMSNorm, rotary embedding + K/V merge,
// cosine saliency (+ context commit), stream compaction.  All are HBM-bound: one workgroup walks
// one token row with 16-byte loads, reductions in fp32.
#include <algorithm>
#include <type_traits>
#include "common.h"
#include "compact.h"
#include "kernels.h"

namespace dy {

namespace {

constexpr int RB = 1024;  // threads per row workgroup: a row of up to 16384 elements in one pass
constexpr int KEEP = 4;   // 16-byte vectors a thread keeps in registers between the two passes of a row

__device__ __forceinline__ int row_count(const Rows &rows) {
  return rows.count ? min(*rows.count, rows.cap) : rows.cap;
}

// Four neighbouring elements, loaded and stored as one word
template <typename T> struct Vec4;
template <> struct Vec4<float> {
  float4 raw;
  __device__ __forceinline__ float get(int i) const { return (&raw.x)[i]; }
  __device__ __forceinline__ void set(int i, float v) { (&raw.x)[i] = v; }
};
template <> struct Vec4<bf16_t> {
  uint2 raw;
  __device__ __forceinline__ float get(int i) const {
    const uint32_t w = (&raw.x)[i >> 1];
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
  __device__ __forceinline__ void set(int i, float v) {
    const uint32_t b = f2bf(v);
    uint32_t &w = (&raw.x)[i >> 1];
    w = (i & 1) ? ((w & 0x0000ffffu) | (b << 16)) : ((w & 0xffff0000u) | b);
  }
};
template <typename T> __device__ __forceinline__ Vec4<T> ld4(const T *p) {
  Vec4<T> v;
  v.raw = *reinterpret_cast<const decltype(v.raw) *>(p);
  return v;
}
template <typename T> __device__ __forceinline__ void st4(T *p, const Vec4<T> &v) { *reinterpret_cast<decltype(v.raw) *>(p) = v.raw; }

// How many rows exist and the splits of a GEMM's result.  Where the device has planned, both are read at once (the plan's words with one
// load: the count is on the device then); one after the other they are up to five round trips at the head of a kernel.  1942 rows of 4096,
// with row_ahead, us: down projection's sums 19.5 -> 18.8, out-projection's tail 21.3 -> 20.6, norm 9.8 -> 9.5; 1137 of 3584 14.7 -> 14.2.
struct RowsAndSplits {
  int n;
  Splits sp;
};
__device__ __forceinline__ RowsAndSplits rows_and_splits(const Rows &rows, const Splits &splits) {
  RowsAndSplits r{0, splits};
  if (splits.dev) {
    const int4 w = *reinterpret_cast<const int4 *>(splits.dev);
    const int n = *rows.count;
    r.sp.n = w.x; r.sp.tail_from = w.y; r.sp.n_tail = w.z; r.sp.done_to = w.w;
    r.n = min(n, rows.cap);
  } else {
    r.n = row_count(rows);
  }
  return r;
}
// Row id of entry j, which need not exist: asked for beside the count
__device__ __forceinline__ int row_ahead(const Rows &rows, int j) { return rows.idx && j < rows.cap ? rows.idx[j] : j; }

// The first workgroups of a row kernel, one for every job, make plans instead of taking rows (all NT threads, a multiple of four waves).  The
// GEMM behind needs its plan as soon as it starts and would take 1.7 us to make it; here that happens beside the rows.  Hidden 4096,
// steps of 410 listed rows 292.5 -> 287.4 us, of 2064 795 -> 790, loop of 8 x 1024 tokens 1991 -> 1966; 28 over 4 heads, 1137 rows equal.
// Beside few rows the plans are what ends last: the out-projection's tail 6.8 -> 7.7 at 330 rows and 6.9 -> 8.1 at 410 (14.2 -> 14.7 at 1137,
// 21.2 -> 20.4 at 2064), which gate|up and the down projection then gain twice over.
template <int NT> __device__ __forceinline__ void make_plan(const PlanMaker &job) {
  __shared__ uint32_t lds[2 * NT / WAVE];  // eight words for four waves, which all make the same plan
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const mm::GemmPlan p = mm::plan_on_device(job.args, row_count(job.rows), wave % 4, lds + 8 * (wave / 4));
  if (threadIdx.x == 0) mm::store_plan(p, job.finishes, job.words);
}

// ---- gather + RMSNorm  [Alg. 3: layernorm(x) restricted to the salient rows] -------------------
// NT threads per row: 256 when the row fits KEEP vectors per thread (more rows in flight per CU and a
// four-wave reduction), else RB.
// JOB: with a plan to make (in the kernel without, for rows whose plan is made on the host, its code and registers would be for nothing).
// NV: vectors a thread keeps, two (rows of up to 4096 bf16 elements) or four.
template <typename T, int NT, bool JOB, int NV>
__global__ __launch_bounds__(NT, 8) void k_gather_rmsnorm(const T *__restrict__ x,
                                                        const T *__restrict__ gain, Rows rows, int d,
                                                        float eps, T *__restrict__ out, int by_token, PlanMaker job) {
  __shared__ float red[NT / WAVE];
  constexpr int N = Vec16<T>::N;
  constexpr int first = JOB ? 1 : 0;
  if constexpr (JOB) {
    if (blockIdx.x == 0) {
      make_plan<NT>(job);
      return;
    }
  }
  const int nv = d / N;
  int j = blockIdx.x - first, r = row_ahead(rows, j);
  const int n = row_count(rows);
  // A row is a chain of round trips (count, id, row, sum), so what can be asked for ahead is: both of a thread's vectors of the row at once
  // (an index past the end reads the last vector again; a branch around a load waits for it), and the gain.  Four of each
  // would not leave the registers for eight waves a SIMD.  Hidden 4096, us: 20480 rows 57 -> 50, 8192 27.6 -> 24.5, 1942 10.6 -> 9.8.
  constexpr bool AHEAD = NV <= 2;
  Vec16<T> g[NV];
#pragma unroll
  for (int it = 0; it < NV; ++it)
    if (AHEAD && it * NT < nv) g[it] = ld16(gain + min((int)threadIdx.x + it * NT, nv - 1) * N);  // (uniform branch)
  for (; j < n; j += gridDim.x - first, r = row_ahead(rows, j)) {
    const T *xr = x + (size_t)r * d;
    float ss = 0.f;
    Vec16<T> keep[NV];
#pragma unroll
    for (int it = 0; it < NV; ++it)
      if (AHEAD && it * NT < nv) keep[it] = ld16(xr + min((int)threadIdx.x + it * NT, nv - 1) * N);
#pragma unroll
    for (int it = 0; it < NV; ++it)
      if ((int)threadIdx.x + it * NT < nv) {
        if (!AHEAD) keep[it] = ld16(xr + (threadIdx.x + it * NT) * N);
#pragma unroll
        for (int i = 0; i < N; ++i) ss += keep[it].get(i) * keep[it].get(i);
      }
    ss = block_sum<NT>(ss, red);
    const float sc = 1.0f / sqrtf(ss / (float)d + eps);
    T *orow = out + (size_t)(by_token ? r : j) * d;
#pragma unroll
    for (int it = 0; it < NV; ++it) {
      const int v = threadIdx.x + it * NT;
      if (v < nv) {
        const Vec16<T> gv = AHEAD ? g[it] : ld16(gain + v * N);
        Vec16<T> o;
#pragma unroll
        for (int i = 0; i < N; ++i) o.set(i, keep[it].get(i) * sc * gv.get(i));
        st16(orow + v * N, o);
      }
    }
  }
}

// ---- out-projection tail  [Alg. 3: x <- layernorm(out_proj(C)), with the residual] ---------------
// h[j] = x[row_j] + sum_z part[z][j] (kept in fp32 for the second residual), f[j] = RMSNorm(h[j]) * gain
// JOBS: with plans to make
template <bool JOBS>
__global__ __launch_bounds__(RB) void k_oproj_finalize(const float *__restrict__ part, Splits splits_of,
                                                        const bf16_t *__restrict__ x,
                                                        const bf16_t *__restrict__ gain, Rows rows, int d,
                                                        float eps, float *__restrict__ h,
                                                        bf16_t *__restrict__ f, PlanMaker job0, PlanMaker job1) {
  __shared__ float red[RB / WAVE];
  const int first = JOBS ? (job0.words ? 1 : 0) + (job1.words ? 1 : 0) : 0;
  if constexpr (JOBS) {
    if ((int)blockIdx.x < first) {
      // (a selected job would be copied to scratch memory)
      if (blockIdx.x == 0 && job0.words) make_plan<RB>(job0);
      else make_plan<RB>(job1);
      return;
    }
  }
  int j = blockIdx.x - first, r = row_ahead(rows, j);
  const auto [n, sp] = rows_and_splits(rows, splits_of);
  const int nv = d / 4;
  const size_t split_stride = (size_t)n * d;
  for (; j < n; j += gridDim.x - first, r = row_ahead(rows, j)) {
    const int splits = sp.of(j);
    const bf16_t *xr = x + (size_t)r * d;
    float *hr = h + (size_t)j * d;
    float ss = 0.f;
    float4 keep[KEEP];
#pragma unroll
    for (int it = 0; it < KEEP; ++it) {
      const int v = threadIdx.x + it * RB;
      if (v < nv) {
        float4 a = *reinterpret_cast<const float4 *>(part + (size_t)j * d + v * 4);
        for (int z = 1; z < splits; ++z) {
          const float4 b = *reinterpret_cast<const float4 *>(part + z * split_stride + (size_t)j * d + v * 4);
          a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
        }
        a.x += to_f<bf16_t>(xr[v * 4 + 0]); a.y += to_f<bf16_t>(xr[v * 4 + 1]);
        a.z += to_f<bf16_t>(xr[v * 4 + 2]); a.w += to_f<bf16_t>(xr[v * 4 + 3]);
        *reinterpret_cast<float4 *>(hr + v * 4) = a;
        ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
        keep[it] = a;
      }
    }
    ss = block_sum<RB>(ss, red);
    const float sc = 1.0f / sqrtf(ss / (float)d + eps);
    bf16_t *fr = f + (size_t)j * d;
#pragma unroll
    for (int it = 0; it < KEEP; ++it) {
      const int v = threadIdx.x + it * RB;
      if (v < nv) {
        const float4 a = keep[it];
        const bf16_t *g = gain + v * 4;
        fr[v * 4 + 0] = from_f<bf16_t>(a.x * sc * to_f<bf16_t>(g[0]));
        fr[v * 4 + 1] = from_f<bf16_t>(a.y * sc * to_f<bf16_t>(g[1]));
        fr[v * 4 + 2] = from_f<bf16_t>(a.z * sc * to_f<bf16_t>(g[2]));
        fr[v * 4 + 3] = from_f<bf16_t>(a.w * sc * to_f<bf16_t>(g[3]));
      }
    }
  }
}

// ---- down-projection tail after a K split  [Alg. 3: FFN second half + cache commit] ---------------
__global__ __launch_bounds__(RB) void k_down_finalize(const float *__restrict__ part, Splits splits_of,
                                                       const float *__restrict__ h,
                                                       Rows rows, int d, bf16_t *__restrict__ out) {
  const auto [n, sp] = rows_and_splits(rows, splits_of);
  const int nv = d / 4;
  const size_t split_stride = (size_t)n * d;
  for (int j = sp.done_to + blockIdx.x; j < n; j += gridDim.x) {
    const int r = rows.idx ? rows.idx[j] : j;
    const int splits = sp.of(j);
    bf16_t *orow = out + (size_t)r * d;
    for (int v = threadIdx.x; v < nv; v += RB) {
      float4 a = *reinterpret_cast<const float4 *>(h + (size_t)j * d + v * 4);
      for (int z = 0; z < splits; ++z) {
        const float4 b = *reinterpret_cast<const float4 *>(part + z * split_stride + (size_t)j * d + v * 4);
        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
      }
      orow[v * 4 + 0] = from_f<bf16_t>(a.x); orow[v * 4 + 1] = from_f<bf16_t>(a.y);
      orow[v * 4 + 2] = from_f<bf16_t>(a.z); orow[v * 4 + 3] = from_f<bf16_t>(a.w);
    }
  }
}

// ---- q/k/v tail: bias + rotary embedding + K/V merge  [Alg. 3: K[idx] <- k_proj(x[idx]), same V] --
// Half-split pairing: element p of a head couples with element p + dh/2, rotated by the angle
// pos * theta^(-2p/dh); the table holds (cos, sin) per (pos, p).  A thread handles 4 neighbouring
// pairs of one head (two float4 of the raw result, two float4 of the table), stored four elements at a time.  Bound by the
// HBM where the rows are many, by the two workgroups that a CU holds where they are a few hundred: the form without candidates
// keeps to 96 scalar registers, the most with which a SIMD's 800 hold eight waves.  (The v sums two splits at a
// time took 106, and with them one workgroup a CU.)  Rows of a list with room for 8192, elements stored one at a time / v sums in
// pairs, one workgroup a CU / as here, us: 12288 columns 330 rows 10.4 / 9.1 / 8.9, 1024 15.7 / 15.2 / 14.7, 4096 65.5 / 51.6 / 51.2;
// 4608 columns 512 rows 6.9 / 7.0 / 5.9, 768 8.9 / 9.4 / 7.9, 2048 12.5 / 12.8 / 11.2.  Candidates (330 rows of 8192 columns) 12.3 /
// 11.8 / 11.1.
// DV: with what the approximate step keeps of its candidates (CandidateOut).
template <typename T, DvLayout DV>
__global__ __launch_bounds__(RB) void k_qkv_finalize(const float *__restrict__ part, Splits splits_of,
                                                      const float *__restrict__ tab,
                                                      Rows rows, int L, int H, int Hkv, int dh,
                                                      const T *__restrict__ bq, const T *__restrict__ bk,
                                                      const T *__restrict__ bv, T *__restrict__ q_out,
                                                      T *__restrict__ kc, T *__restrict__ vc,
                                                      int q_by_token, T *__restrict__ dv_out, T *__restrict__ k_out,
                                                      const int32_t *__restrict__ cand_offsets,
                                                      int32_t *__restrict__ entry_of, int entry_lo) {
  const auto [n, sp] = rows_and_splits(rows, splits_of);
  const int half = dh / 2, dq = H * dh, dkv = Hkv * dh, ld = dq + 2 * dkv;
  const int per_head = half / 4;  // items of 4 pairs per head
  const int qk_items = (H + Hkv) * per_head, v_items = dkv / 4;
  const size_t split_stride = (size_t)n * ld;
  for (int j = sp.done_to + blockIdx.x; j < n; j += gridDim.x) {
    const int r = rows.idx ? rows.idx[j] : j;
    const int splits = sp.of(j);
    const int pos = r % L;
    // token -> its list entry (0 = not in the list), for the tokens at positions >= entry_lo only
    if (DV != DV_NONE && threadIdx.x == 0 && pos >= entry_lo) entry_of[r] = j + 1;
    int cand_row = DV == DV_BY_TOKEN ? r : j;
    bool dv_here = DV != DV_NONE, k_here = DV == DV_BY_ENTRY;
    if constexpr (DV == DV_BY_SEQUENCE) {  // (a residual is put back to zero by the token's entry in entry_of)
      const CandidateRow c = candidate_row(cand_offsets, rows.cap, L, r, j);
      cand_row = c.row;
      dv_here = pos >= entry_lo;
      k_here = c.compact;
    }
    const float *src = part + (size_t)j * ld;
    const float *t = tab + (size_t)pos * half * 2;
    for (int it = threadIdx.x; it < qk_items + v_items; it += RB) {
      if (it < qk_items) {
        const int head = it / per_head, p4 = (it % per_head) * 4;
        const bool isq = head < H;
        const int hh = isq ? head : head - H;
        const int c0 = hh * dh + p4;              // column inside q or k
        const int s0 = (isq ? 0 : dq) + c0;       // column inside the raw row
        const float4 t0 = *reinterpret_cast<const float4 *>(t + 2 * p4);      // cos0 sin0 cos1 sin1
        const float4 t1 = *reinterpret_cast<const float4 *>(t + 2 * p4 + 4);  // cos2 sin2 cos3 sin3
        float4 x1 = *reinterpret_cast<const float4 *>(src + s0);
        float4 x2 = *reinterpret_cast<const float4 *>(src + s0 + half);
        for (int z = 1; z < splits; ++z) {
          const float4 y1 = *reinterpret_cast<const float4 *>(src + z * split_stride + s0);
          const float4 y2 = *reinterpret_cast<const float4 *>(src + z * split_stride + s0 + half);
          x1.x += y1.x; x1.y += y1.y; x1.z += y1.z; x1.w += y1.w;
          x2.x += y2.x; x2.y += y2.y; x2.z += y2.z; x2.w += y2.w;
        }
        const T *b = isq ? bq : bk;
        if (b) {
          x1.x += to_f<T>(b[c0]); x1.y += to_f<T>(b[c0 + 1]); x1.z += to_f<T>(b[c0 + 2]); x1.w += to_f<T>(b[c0 + 3]);
          x2.x += to_f<T>(b[c0 + half]); x2.y += to_f<T>(b[c0 + half + 1]);
          x2.z += to_f<T>(b[c0 + half + 2]); x2.w += to_f<T>(b[c0 + half + 3]);
        }
        T *dst = isq ? q_out + (size_t)(q_by_token ? r : j) * dq : kc + (size_t)r * dkv;
        const float a1[4] = {x1.x, x1.y, x1.z, x1.w}, a2[4] = {x2.x, x2.y, x2.z, x2.w};
        const float co[4] = {t0.x, t0.z, t1.x, t1.z}, si[4] = {t0.y, t0.w, t1.y, t1.w};
        Vec4<T> lo4, hi4;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          lo4.set(u, rotated(a1[u], co[u], -(a2[u] * si[u])));
          hi4.set(u, rotated(a2[u], co[u], a1[u] * si[u]));
        }
        st4(dst + c0, lo4);
        st4(dst + c0 + half, hi4);
        if (k_here && !isq) {
          T *ks = k_out + (size_t)cand_row * dkv;
          st4(ks + c0, lo4);
          st4(ks + c0 + half, hi4);
        }
      } else {
        const int c0 = (it - qk_items) * 4;
        float4 x = *reinterpret_cast<const float4 *>(src + dq + dkv + c0);
        for (int z = 1; z < splits; ++z) {
          const float4 y = *reinterpret_cast<const float4 *>(src + z * split_stride + dq + dkv + c0);
          x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
        }
        if (bv) {
          x.x += to_f<T>(bv[c0]); x.y += to_f<T>(bv[c0 + 1]); x.z += to_f<T>(bv[c0 + 2]); x.w += to_f<T>(bv[c0 + 3]);
        }
        T *vrow = vc + (size_t)r * dkv + c0;
        Vec4<T> v;
        v.set(0, x.x); v.set(1, x.y); v.set(2, x.z); v.set(3, x.w);
        if (dv_here) {  // residual of the stored values, before the merge overwrites the cached row
          const Vec4<T> old = ld4(vrow);
          Vec4<T> dv;
#pragma unroll
          for (int u = 0; u < 4; ++u) dv.set(u, v.get(u) - old.get(u));
          st4(dv_out + (size_t)cand_row * dkv + c0, dv);
        }
        st4(vrow, v);
      }
    }
  }
}

// ---- temporal cosine similarity + salient test (+ commit)  [Sec. 3.1, Sec. 3.2] ----------------
// s = <a,b> / (max(|a|,1e-8) max(|b|,1e-8)), flag = s < tau.  The old cache row b is read before
// the same thread overwrites the same elements with a.
// A row per workgroup: many small workgroups keep the loads of a CU in flight, a thread's four at a time (all of them up to 4096 bf16 or
// 2048 fp32 columns).  HBM-bound where the rows are many: 32768 rows of 4096 bf16 columns (537 MB), compaction included, 96.5 -> 84.7
// us, most of it by loads that leave the L2 alone; 7500 rows of 3584 24.3 -> 22.5; up to 30 MB equal.
constexpr int SAL_NT = 256;

template <typename T>
__global__ __launch_bounds__(SAL_NT) void k_saliency(const T *__restrict__ c_new, T *c_cache, Rows rows,
                                                      int D, float tau, float *__restrict__ cos_out,
                                                      uint8_t *__restrict__ flag_out, int commit) {
  __shared__ float red[3 * SAL_NT / WAVE];
  constexpr int N = Vec16<T>::N, AHEAD = 2;
  const int n = row_count(rows), nv = D / N;
  for (int j = blockIdx.x; j < n; j += gridDim.x) {
    const int r = rows.idx ? rows.idx[j] : j;
    const T *a = c_new + (size_t)j * D;
    T *b = c_cache + (size_t)r * D;
    float dot = 0.f, na = 0.f, nb = 0.f;
    for (int v0 = threadIdx.x; v0 < nv; v0 += AHEAD * SAL_NT) {
      Vec16<T> va[AHEAD], vb[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (v0 + u * SAL_NT < nv) {
          va[u] = ld16_once(a + (v0 + u * SAL_NT) * N);
          vb[u] = ld16_once(b + (v0 + u * SAL_NT) * N);
        }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        if (v0 + u * SAL_NT < nv) {
#pragma unroll
          for (int i = 0; i < N; ++i) {
            const float fa = va[u].get(i), fb = vb[u].get(i);
            dot += fa * fb;
            na += fa * fa;
            nb += fb * fb;
          }
          if (commit) st16(b + (v0 + u * SAL_NT) * N, va[u]);
        }
    }
    block_sum3<SAL_NT>(dot, na, nb, red);
    if (threadIdx.x == 0) {
      const float s = dot / (fmaxf(sqrtf(na), 1e-8f) * fmaxf(sqrtf(nb), 1e-8f));
      if (cos_out) cos_out[j] = s;
      flag_out[j] = (s < tau) ? 1 : 0;
    }
  }
}

// ---- stream compaction as a kernel of its own ------------------------------------------------------
// Workgroup i takes entries [i*chunk, (i+1)*chunk) of the list.  It counts its flagged entries,
// publishes the count, adds up the counts of the chunks before it, and then places its own entries.
// scan (COMPACT_SCAN_WORDS ints, all zero before and after a launch): [0] a ticket counter that numbers the
// workgroups in the order they start, [1] finished workgroups, [2 + i] 1 + count of chunk i once
// published.  Every workgroup publishes BEFORE it waits, and it only waits for tickets lower than its
// own, whose workgroups are already running: every wait ends.  The workgroup that finishes last puts
// the words back to zero for the next launch.  Launches that share `scan` must not overlap.
// FROM_PARTS: the flags do not exist yet; eight lanes together first take the cosine of an entry from
// the per-head sums the attention kernel left (cos_part [n, H, 4]: <new, old>, |new|^2, |old|^2), write
// cos_out and the flag, and then the workgroup counts and places the flags it wrote itself.  (A thread per entry read 16
// bytes of 64 rows at a time; with 64 entries a workgroup instead of 256 and the flags kept in registers, 330 entries in a list of
// 8192 take 7.3 instead of 10.0 us, 2064 take 8.7 instead of 10.9.  A launch and four dependent round trips are left.)
// FROM_LISTS: the flags do not exist yet either; a workgroup marks the tokens of its own chunk that are in
// one of two lists (any order, ids outside [0, B*L) and positions below pos_lo ignored) and goes on with
// the flags it wrote itself.  Every workgroup reads both lists, so this is for a moderate number of tokens.
struct ListPair {
  Rows a, b;  // count == nullptr and cap == 0: no such list
  uint8_t *flag_out;
  int pos_lo;
};
enum CompactFrom { FROM_FLAGS, FROM_COS, FROM_LISTS };
struct CosParts {
  const float *part;
  float *cos_out;
  uint8_t *flag_out;
  int H;
  float tau;
};

template <CompactFrom FROM>
__global__ __launch_bounds__(CB) void k_compact(const uint8_t *__restrict__ flag, Rows rows, int B, int L,
                                                 int chunk, int32_t *out_idx, int32_t *out_off, int out_cap,
                                                 int32_t *status, int overflow_code, int32_t *scan, CosParts cp, ListPair lp) {
  constexpr bool FROM_PARTS = FROM == FROM_COS;
  uint8_t *const own_flags = FROM == FROM_LISTS ? lp.flag_out : cp.flag_out;
  __shared__ int wave_cnt[CB / WAVE];
  __shared__ uint8_t mark[FROM == FROM_FLAGS ? 1 : CB];
  __shared__ int s_bid, s_last;
  const int tid = threadIdx.x, lane = tid % WAVE, w = tid / WAVE;
  const int n = row_count(rows);
  const int G = gridDim.x;
  if (tid == 0) s_bid = __hip_atomic_fetch_add(scan, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const int bid = s_bid;
  const int lo = min(n, bid * chunk), hi = min(n, lo + chunk);
  // FROM_PARTS: a chunk of one sweep stays in registers: its flags, tokens and the sequences before them are there when the
  // counts of the chunks before it arrive.  (The others are quicker with the flags read again: 8192 flags 5.4 against 6.4 us,
  // the union of two lists 7.7 against 8.1 us.)
  const bool one_sweep = FROM_PARTS && chunk <= CB;
  bool f = false;
  int row = 0, sprev = -1;
  if (one_sweep && lo + tid < hi) {
    const int j = lo + tid;
    row = rows.idx ? rows.idx[j] : j;
    if (j > 0) sprev = seq_of(rows.idx ? rows.idx[j - 1] : j - 1, B, L);
  }
  int mine = 0;  // wave-uniform
  for (int start = lo; start < hi; start += CB) {
    const int j = start + tid;
    f = false;
    if constexpr (FROM == FROM_LISTS) {
      mark[tid] = 0;
      __syncthreads();
      auto mark_list = [&](const Rows &l) {
        const int m = row_count(l);
        for (int i = tid; i < m; i += CB) {
          const int r = l.idx[i];
          if (r >= start && r < min(hi, start + CB) && r % L >= lp.pos_lo) mark[r - start] = 1;
        }
      };
      mark_list(lp.a);
      mark_list(lp.b);
      __syncthreads();
      if (j < hi) {
        f = mark[tid] != 0;
        lp.flag_out[j] = f ? 1 : 0;
      }
    } else if constexpr (FROM_PARTS) {
      constexpr int LANES = 8, AHEAD = 4;  // lanes per entry, loads in flight per lane
      const int end = min(hi, start + CB), sub = tid % LANES;
      for (int e0 = start; e0 < end; e0 += CB / LANES) {
        const int e = e0 + tid / LANES;
        float dot = 0.f, na = 0.f, nb = 0.f;
        if (e < end) {
          const float4 *p = reinterpret_cast<const float4 *>(cp.part) + (size_t)e * cp.H;
          for (int h0 = sub; h0 < cp.H; h0 += LANES * AHEAD) {
            float4 v[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) v[i] = h0 + LANES * i < cp.H ? p[h0 + LANES * i] : float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) { dot += v[i].x; na += v[i].y; nb += v[i].z; }
          }
        }
#pragma unroll
        for (int o = 1; o < LANES; o *= 2) {
          dot += __shfl_xor(dot, o, WAVE);
          na += __shfl_xor(na, o, WAVE);
          nb += __shfl_xor(nb, o, WAVE);
        }
        if (e < end && sub == 0) {
          const float c = dot / (fmaxf(sqrtf(na), 1e-8f) * fmaxf(sqrtf(nb), 1e-8f));
          const uint8_t low = c < cp.tau ? 1 : 0;
          if (cp.cos_out) cp.cos_out[e] = c;
          cp.flag_out[e] = low;  // (a chunk of several sweeps reads it back in the placement pass)
          mark[e - start] = low;
        }
      }
      __syncthreads();
      f = j < hi && mark[tid] != 0;
      __syncthreads();  // (before the next sweep's marks)
    } else if (j < hi) {
      f = flag[j] != 0;
    }
    mine += __popcll(__ballot(f));
  }
  if (lane == 0) wave_cnt[w] = mine;
  __syncthreads();
  int own = 0;
#pragma unroll
  for (int i = 0; i < CB / WAVE; ++i) own += wave_cnt[i];
  if (tid == 0) __hip_atomic_store(scan + 2 + bid, own + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int before = 0;
  if (lo < hi) {  // a chunk past the end places nothing and waits for nobody
    for (int i = tid; i < bid; i += CB) {
      int v;
      do {
        v = __hip_atomic_load(scan + 2 + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } while (v == 0);
      before += v - 1;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o, WAVE);
  __syncthreads();
  if (lane == 0) wave_cnt[w] = before;
  __syncthreads();
  before = 0;
#pragma unroll
  for (int i = 0; i < CB / WAVE; ++i) before += wave_cnt[i];
  __syncthreads();
  int total;
  if (one_sweep) {
    total = before + compact_sweep<CB>(f, row, sprev, lo + tid < hi, before, B, L, out_idx, out_off, out_cap, wave_cnt);
  } else {
    if constexpr (FROM != FROM_FLAGS) {  // every thread's flag stores have reached the L2
      wait_vmcnt<0>();
      __syncthreads();
    }
    total = compact_range<CB>(FROM != FROM_FLAGS ? own_flags : flag, rows, lo, hi, before, B, L, out_idx, out_off, out_cap,
                              FROM != FROM_FLAGS, wave_cnt);
  }
  // the workgroup that holds the end of the list (workgroup 0 of an empty one) writes the tail
  if ((lo < hi && hi == n) || (n == 0 && bid == 0))
    compact_tail<CB>(rows, n, total, B, L, out_off, out_cap, status, overflow_code);
  __syncthreads();
  if (tid == 0)
    s_last = __hip_atomic_fetch_add(scan + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == G - 1;
  __syncthreads();
  if (s_last) {
    for (int i = tid; i < G + 2; i += CB)
      __hip_atomic_store(scan + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Workgroups of a row kernel.  Where the count is on the device the capacity may be far above it, and
// workgroups without a row are not free (8192 of 1024 threads each for 330 rows: k_qkv_finalize 12.7 us, with
// 1024 of them 11.3 us).  Of the 1024-thread ones 512 are resident at once (two per CU; of k_qkv_finalize's forms with
// candidates, whose scalar registers allow seven waves a SIMD, 256); they take further rows in turn.  Full lists lose nothing by it:
// q/k/v stage at hidden 256 / 4096, 20480 listed rows, 96 -> 85 / 1937 -> 1820 us together with what the GEMMs gained.
constexpr int GRID_KNOWN = 8192, GRID_LISTED = 1024;
inline int row_grid(const Rows &rows, int cap) {
  const int most = rows.count ? GRID_LISTED : GRID_KNOWN;
  return cap < 1 ? 1 : (cap > most ? most : cap);
}
inline int row_grid(const Rows &rows) { return row_grid(rows, rows.cap); }

}  // namespace

void launch_gather_rmsnorm(DType t, const void *x, const void *gain, Rows rows, int d, float eps,
                           void *out, int by_token, const PlanMaker &job, hipStream_t s) {
  if (rows.cap <= 0 && !job.words) return;
  const int most = rows.count ? 4 * GRID_LISTED : 32768;  // (a quarter of the threads per workgroup)
  const int plans = job.words ? 1 : 0, grid = std::max(std::min(rows.cap, most), 1) + plans, wide_grid = row_grid(rows) + plans;
  auto go = [&](auto zero, auto job_c) {
    using T = decltype(zero);
    constexpr bool JOB = decltype(job_c)::value;
    const int nv = d / Vec16<T>::N;
#define DY_GATHER(NT, NV, G) k_gather_rmsnorm<T, NT, JOB, NV><<<G, NT, 0, s>>>((const T *)x, (const T *)gain, rows, d, eps, (T *)out, by_token, job)
    if (nv <= 2 * 256) DY_GATHER(256, 2, grid);
    else if (nv <= 256 * KEEP) DY_GATHER(256, KEEP, grid);
    else DY_GATHER(RB, KEEP, wide_grid);
#undef DY_GATHER
  };
  if (t == F32) go(float{}, std::false_type{});
  else if (plans) go(bf16_t{}, std::true_type{});
  else go(bf16_t{}, std::false_type{});
}

void launch_oproj_finalize(const float *part, Splits splits, const void *x,
                           const void *gain, Rows rows, int d, float eps, float *h, void *f,
                           const PlanMaker &job0, const PlanMaker &job1, hipStream_t s) {
  if (rows.cap <= 0) return;
  const int plans = (job0.words ? 1 : 0) + (job1.words ? 1 : 0);
  auto go = [&](auto jobs_c) {
    k_oproj_finalize<decltype(jobs_c)::value><<<row_grid(rows) + plans, RB, 0, s>>>(part, splits, (const bf16_t *)x, (const bf16_t *)gain, rows,
                                                                                      d, eps, h, (bf16_t *)f, job0, job1);
  };
  if (plans) go(std::true_type{});
  else go(std::false_type{});
}

void launch_down_finalize(const float *part, Splits splits, const float *h,
                          Rows rows, int d, void *out_cache, hipStream_t s) {
  const int done = splits.dev ? 0 : splits.done_to;
  if (rows.cap <= 0 || done >= rows.cap) return;
  k_down_finalize<<<row_grid(rows, rows.cap - done), RB, 0, s>>>(part, splits, h, rows, d, (bf16_t *)out_cache);
}

void launch_qkv_finalize(DType t, const float *part, Splits splits, Rows rows, const QkvOut &o, const CandidateOut *cand,
                         hipStream_t s) {
  const int done = splits.dev ? 0 : splits.done_to;
  if (rows.cap <= 0 || done >= rows.cap) return;
  const CandidateOut c = cand ? *cand : CandidateOut{};
#define DY_QKV_FIN(TT, C)                                                                               \
  k_qkv_finalize<TT, C><<<row_grid(rows, rows.cap - done), RB, 0, s>>>(                                 \
      part, splits, o.tab, rows, o.L, o.H, o.Hkv, o.dh, (const TT *)o.bq, (const TT *)o.bk, (const TT *)o.bv, \
      (TT *)o.q, (TT *)o.k, (TT *)o.v, o.q_by_token, (TT *)c.dv, (TT *)c.k, c.offsets, c.entry_of, c.entry_lo)
  if (t == F32) {
    if (c.layout == DV_BY_TOKEN) DY_QKV_FIN(float, DV_BY_TOKEN);  // (candidates alone: launch_qkv_f32 finishes all others)
    else DY_QKV_FIN(float, DV_BY_ENTRY);
  } else {
    if (c.layout == DV_NONE) DY_QKV_FIN(bf16_t, DV_NONE);
    else if (c.layout == DV_BY_TOKEN) DY_QKV_FIN(bf16_t, DV_BY_TOKEN);
    else if (c.layout == DV_BY_ENTRY) DY_QKV_FIN(bf16_t, DV_BY_ENTRY);
    else DY_QKV_FIN(bf16_t, DV_BY_SEQUENCE);
  }
#undef DY_QKV_FIN
}

inline int sal_grid(int cap) { return cap < 1 ? 1 : (cap > 65536 ? 65536 : cap); }

void launch_saliency(DType t, const void *c_new, void *c_cache, Rows rows, int D, float tau,
                     float *cos_out, uint8_t *flag_out, int commit, hipStream_t s) {
  if (rows.cap <= 0) return;
  if (t == F32)
    k_saliency<float><<<sal_grid(rows.cap), SAL_NT, 0, s>>>((const float *)c_new, (float *)c_cache, rows,
                                                        D, tau, cos_out, flag_out, commit);
  else
    k_saliency<bf16_t><<<sal_grid(rows.cap), SAL_NT, 0, s>>>((const bf16_t *)c_new, (bf16_t *)c_cache,
                                                         rows, D, tau, cos_out, flag_out, commit);
}

void launch_compact(const uint8_t *flag, Rows rows, int B, int L, int32_t *out_idx,
                    int32_t *out_offsets, int out_cap, int32_t *status, int32_t *scan, hipStream_t s) {
  const int cap = rows.cap < 0 ? 0 : rows.cap;
  int G = (cap + CB - 1) / CB;
  G = G < 1 ? 1 : (G > CMAXG ? CMAXG : G);
  int chunk = (cap + G - 1) / G;
  chunk = ((chunk + CB - 1) / CB) * CB;
  if (chunk < CB) chunk = CB;
  k_compact<FROM_FLAGS><<<G, CB, 0, s>>>(flag, rows, B, L, chunk, out_idx, out_offsets, out_cap, status, -6, scan, CosParts{}, ListPair{});
}

void launch_cos_compact(const float *cos_part, int H, float tau, float *cos_out, uint8_t *flag_out, Rows rows,
                        int B, int L, int32_t *out_idx, int32_t *out_offsets, int out_cap, int32_t *status,
                        int32_t *scan, hipStream_t s) {
  // 64 entries a workgroup: their sums are 32 KB at 32 heads
  constexpr int CC = 64;
  const int cap = rows.cap < 0 ? 0 : rows.cap;
  int G = (cap + CC - 1) / CC;
  G = G < 1 ? 1 : (G > CMAXG ? CMAXG : G);
  int chunk = (cap + G - 1) / G;
  chunk = ((chunk + CC - 1) / CC) * CC;
  if (chunk < CC) chunk = CC;
  k_compact<FROM_COS><<<G, CB, 0, s>>>(flag_out, rows, B, L, chunk, out_idx, out_offsets, out_cap, status, -6, scan,
                                       CosParts{cos_part, cos_out, flag_out, H, tau}, ListPair{});
}

void launch_merge_compact(Rows a, Rows b, int pos_lo, uint8_t *flag_out, int B, int L, int32_t *out_idx,
                          int32_t *out_offsets, int out_cap, int32_t *status, int32_t *scan, hipStream_t s) {
  const int T = B * L, G = (T + CB - 1) / CB;  // (T <= MERGE_TOKENS: a chunk is one sweep of the workgroup)
  k_compact<FROM_LISTS><<<G, CB, 0, s>>>(flag_out, Rows{nullptr, nullptr, T}, B, L, CB, out_idx, out_offsets, out_cap,
                                         status, -6, scan, CosParts{}, ListPair{a, b, flag_out, pos_lo});
}

// ---- approximate context update of the non-salient rows  [Sec. 3.3; Alg. 3 lines C <- ..., cosine] --
template <typename T>
__global__ __launch_bounds__(256) void k_clear_rows(Rows rows, T *dv, int dkv) {
  const int n = row_count(rows);
  constexpr int N = Vec16<T>::N;
  Vec16<T> zero;
#pragma unroll
  for (int e = 0; e < N; ++e) zero.set(e, 0.f);
  for (int j = blockIdx.x; j < n; j += gridDim.x) {
    const int r = rows.idx ? rows.idx[j] : j;
    for (int v = threadIdx.x; v < dkv / N; v += 256) st16(dv + (size_t)r * dkv + v * N, zero);
  }
}

// One workgroup per token of the step (entry j of `win`, token r).  Salient tokens (pos[r] != 0) take
// their exact row, all others the cached row plus the approximate residual; the cosine is taken over
// the stored (rounded) values against the cached row, which is read before it is overwritten.
// cos_out is indexed by token, flag_out by window entry.
// Residual: dc[j] (CACHED = false), or rebuilt from the partials of an attention pass over the compact
// candidate keys with the token's CACHED log-normaliser: sum over the key splits that hold keys of
// the token's sequence of part_o[s][j] * exp(m_s - lse[r, h])  (part_o is relative to the split's own
// running maximum m_s; nothing is renormalised).
struct CachedNorm {
  const float *part_o, *part_ml, *lse;
  const int32_t *key_offsets;
  int cap, H, dh, chunk, splits, L, key_cap;
};

template <typename T, bool CACHED>
__global__ __launch_bounds__(SAL_NT) void k_saliency_approx(Rows win, int D, const T *__restrict__ c_sal,
                                                             const T *__restrict__ dc,
                                                             int32_t *__restrict__ pos, T *c_cache,
                                                             float tau, float *__restrict__ cos_out,
                                                             uint8_t *__restrict__ flag_out, CachedNorm cn,
                                                             Residuals residuals) {
  __shared__ float red[3 * SAL_NT / WAVE];
  constexpr int N = Vec16<T>::N;
  const int nv = D / N;
  const int n = row_count(win);
  for (int j = blockIdx.x; j < n; j += gridDim.x) {
    const int r = win.idx ? win.idx[j] : j;
    const int p = pos[r];
    T *b = c_cache + (size_t)r * D;
    const T *src = p ? c_sal + (size_t)(p - 1) * D : dc + (size_t)j * D;
    int ns = 0;  // key splits that hold candidate keys of this token's sequence
    if (CACHED && !p) {
      const int sq = r / cn.L;
      const int lk = min(cn.key_offsets[sq + 1], cn.key_cap) - min(cn.key_offsets[sq], cn.key_cap);
      ns = (lk + cn.chunk - 1) / cn.chunk;
      ns = ns < cn.splits ? ns : cn.splits;
    }
    float dot = 0.f, na = 0.f, nb = 0.f;
    for (int v = threadIdx.x; v < nv; v += SAL_NT) {
      const Vec16<T> vb = ld16(b + v * N);
      Vec16<T> vn;
      if (CACHED && !p) {
        const int c = v * N, h = c / cn.dh;
        const float ref = cn.lse[(size_t)r * cn.H + h];
        float res[N];
#pragma unroll
        for (int i = 0; i < N; ++i) res[i] = 0.f;
        for (int sp = 0; sp < ns; ++sp) {
          const size_t row = (size_t)sp * cn.cap + j;
          const float wgt = __expf(cn.part_ml[(row * cn.H + h) * 2] - ref);
          const float4 *po = reinterpret_cast<const float4 *>(cn.part_o + row * D + c);
#pragma unroll
          for (int q4 = 0; q4 < N / 4; ++q4) {
            const float4 o = po[q4];
            res[4 * q4] += o.x * wgt; res[4 * q4 + 1] += o.y * wgt;
            res[4 * q4 + 2] += o.z * wgt; res[4 * q4 + 3] += o.w * wgt;
          }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) vn.set(i, vb.get(i) + res[i]);
      } else {
        const Vec16<T> vs = ld16(src + v * N);
#pragma unroll
        for (int i = 0; i < N; ++i) vn.set(i, p ? vs.get(i) : vb.get(i) + vs.get(i));
      }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const float fa = vn.get(i), fb = vb.get(i);
        dot += fa * fb;
        na += fa * fa;
        nb += fb * fb;
      }
      st16(b + v * N, vn);
    }
    block_sum3<SAL_NT>(dot, na, nb, red);
    if (threadIdx.x == 0) {
      const float s = dot / (fmaxf(sqrtf(na), 1e-8f) * fmaxf(sqrtf(nb), 1e-8f));
      if (cos_out) cos_out[r] = s;
      flag_out[j] = (s < tau) ? 1 : 0;
      // The map goes back to zero as it is consumed: every marked token is a token of the step, this
      // workgroup alone reads its entry, and all its threads did so before the barriers of the sum.
      if (p) pos[r] = 0;
    }
    if (!CACHED && p && residuals.dv) {
      Vec16<T> zero;
#pragma unroll
      for (int e = 0; e < N; ++e) zero.set(e, 0.f);
      T *dv = (T *)residuals.dv + (size_t)candidate_row(residuals.offsets, residuals.cap, residuals.L, r, p - 1).row * residuals.dkv;
      for (int v = threadIdx.x; v < residuals.dkv / N; v += SAL_NT) st16(dv + v * N, zero);
    }
  }
}

// The tokens at positions [lo, L) of every sequence as an index list (a response-only step's rows).
__global__ __launch_bounds__(256) void k_make_window(int B, int L, int lo, int32_t *idx, int32_t *off) {
  const int w = L - lo, n = B * w;
  for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256) idx[j] = (j / w) * L + lo + j % w;
  if (blockIdx.x == 0)
    for (int b = threadIdx.x; b <= B; b += 256) off[b] = b * w;
}

// flag[r] = 1 for the tokens r of a list at positions >= lo of their sequence (an id outside [0, T)
// is ignored rather than written through)
__global__ __launch_bounds__(256) void k_mark_flags(Rows rows, int T, int L, int lo, uint8_t *flag) {
  const int n = row_count(rows);
  for (int j = blockIdx.x * 256 + threadIdx.x; j < n; j += gridDim.x * 256) {
    const int r = rows.idx[j];
    if ((unsigned)r < (unsigned)T && r % L >= lo) flag[r] = 1;
  }
}

void launch_saliency_approx(DType t, Rows win, int D, const void *c_sal, const void *dc, int32_t *pos,
                            void *c_cache, float tau, float *cos_out, uint8_t *flag_out,
                            const AttnArgs *cached, const float *lse, int L, Residuals residuals, hipStream_t s) {
  if (win.cap <= 0) return;
  const int grid = win.cap > 65536 ? 65536 : win.cap;
  CachedNorm cn{};
  if (cached)
    cn = CachedNorm{cached->part_o, cached->part_ml, lse, cached->key_offsets, cached->rows.cap,
                    cached->H, cached->dh, cached->chunk, cached->splits, L, cached->key_cap};
#define DY_SAL_APPROX(TT, C)                                                                        \
  k_saliency_approx<TT, C><<<grid, SAL_NT, 0, s>>>(win, D, (const TT *)c_sal, (const TT *)dc, pos, \
                                                   (TT *)c_cache, tau, cos_out, flag_out, cn, residuals)
  if (t == F32) {
    if (cached) DY_SAL_APPROX(float, true);
    else DY_SAL_APPROX(float, false);
  } else {
    if (cached) DY_SAL_APPROX(bf16_t, true);
    else DY_SAL_APPROX(bf16_t, false);
  }
#undef DY_SAL_APPROX
}

void launch_make_window(int B, int L, int lo, int32_t *idx, int32_t *off, hipStream_t s) {
  const int n = B * (L - lo);
  k_make_window<<<n > 0 ? (n + 255) / 256 : 1, 256, 0, s>>>(B, L, lo, idx, off);
}

void launch_mark_flags(Rows rows, int T, int L, int lo, uint8_t *flag, hipStream_t s) {
  if (rows.cap <= 0) return;
  k_mark_flags<<<(rows.cap + 255) / 256, 256, 0, s>>>(rows, T, L, lo, flag);
}

void launch_clear_rows(DType t, Rows rows, void *dv, int dkv, hipStream_t s) {
  if (rows.cap <= 0) return;
  if (t == F32) k_clear_rows<float><<<row_grid(rows), 256, 0, s>>>(rows, (float *)dv, dkv);
  else k_clear_rows<bf16_t><<<row_grid(rows), 256, 0, s>>>(rows, (bf16_t *)dv, dkv);
}

// Row-major [n_out, n_in] matrix of 2-byte elements -> the panel layout the bf16 GEMMs read
// (panels of 32 rows, K-slice-major inside a panel): thread u moves the 16 bytes of destination unit u.
__global__ __launch_bounds__(256) void k_pack_weight(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                     int n_in, size_t units) {
  const int kslices = n_in / 64;
  for (size_t u = (size_t)blockIdx.x * 256 + threadIdx.x; u < units; u += (size_t)gridDim.x * 256) {
    const int c8 = (int)(u % 8), r = (int)((u / 8) % 32);
    const size_t pk = u / 256;  // panel * kslices + slice
    const int kt = (int)(pk % kslices);
    const size_t row = (pk / kslices) * 32 + r;
    dst[u] = src[(row * (size_t)n_in + (size_t)kt * 64) / 8 + c8];
  }
}

void launch_pack_weight(const void *src, int n_out, int n_in, void *dst, hipStream_t s) {
  const size_t units = (size_t)n_out * n_in / 8;
  if (units == 0) return;
  const size_t want = (units + 255) / 256;
  k_pack_weight<<<(unsigned)(want < 65536 ? want : 65536), 256, 0, s>>>((const uint4 *)src, (uint4 *)dst, n_in, units);
}

void launch_fill_i32(int32_t *p, int32_t v, int n, hipStream_t s) {
  if (n <= 0) return;
  k_fill_i32<<<(n + 255) / 256, 256, 0, s>>>(p, v, n);
}

}  // namespace dy
