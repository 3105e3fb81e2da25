// bf16 salient-row GEMM for the gfx950 matrix cores with asynchronous global -> LDS copies.
//   C[j,n] = sum_k A[row_j,k] * W[n,k]      (both operands K-contiguous)
//
// Weight layout.  W is stored in panels of 32 output rows, each panel K-slice-major:
//   W[n][k] lives at ((n/32) * (K/64) + k/64) * 2048 + (n%32) * 64 + k%64   (elements).
// The 128 bytes a tile row needs per K slice are then contiguous with those of the 31 other rows of
// its panel (4 KB), and a panel is read front to back while K advances: a workgroup that streams
// weights from HBM reads whole DRAM pages in order instead of one 128-byte piece per 8 KB row
// (measured at 106 rows on a 32-layer stack, whose weights always come from HBM: q/k/v GEMM 25.6 ->
// 23.7 us, gate|up 49.4 -> 46.2 us per layer against the row-major layout; a copy loop without
// products streams 6.0 TB/s from contiguous runs and 4.9-5.3 TB/s from 128-byte pieces).
//
// Data path.  K is cut into slices of 64 elements (128 bytes per tile row).  A slice of the
// (BM + BN) tile rows is copied straight from global memory into LDS by global_load_lds_dwordx4:
// every lane names its own 16-byte global source, the hardware writes lane i's data to
// LDS[M0 + 16*i].  One such instruction therefore fills 8 tile rows x 128 bytes.  No register is
// used for staging, so NS-1 slices can be in flight per workgroup while the MFMAs of the current
// slice run; the only synchronisation is one s_waitcnt vmcnt + one barrier per slice.  The row
// tiles of the ring loop (up to 256 rows) use the same copies through buffer descriptors and keep three to five
// whole slices or five halves of them in LDS (gemm_bf16_ring.h).
//
// LDS layout.  Rows are 128 bytes, unpadded (the copy engine writes lanes back to back), with an
// XOR swizzle instead: the 16-byte chunk c of tile row r lives at chunk position c ^ ((r/2) % 8).
// The copy applies it on the global side (the lane that fills position p of row r fetches chunk
// p ^ ((r/2) % 8)), the MFMA operand reads apply it on the LDS side.  The LDS of gfx950 has 64 banks
// (256 bytes per clock) and serves a 16-byte-per-lane read 16 lanes at a time: 16 neighbouring
// lanes (16 rows, same k) then touch 8 different positions in each of the two 128-byte bank halves
// (even rows / odd rows) = all 64 banks once.
//
// MFMA.  v_mfma_f32_32x32x16_bf16: lane l supplies 8 consecutive k of row (l%32) for A and of
// column (l%32) for B at k offset 8*(l/32); the accumulator block holds
//   row = 8*(r/4) + 4*(l/32) + (r%4),  col = l%32   in register r of lane l.
// The row tiles of the ring loop use v_mfma_f32_16x16x32_bf16 with a permuted order of the weight rows,
// so that neighbouring lanes hold neighbouring runs of columns of one row (gemm_bf16_ring.h).
//
// Tile walk.  The row count lives on the device; the grid is one workgroup per CU (k_gemm_planned) or sized
// from the list capacity (k_gemm_bf16), and each workgroup walks the existing tiles in a grouped order, remapped so
// that neighbouring tiles run on one XCD (workgroup i is dispatched to XCD i % 8) and share A / weight tiles in its L2.  gemm_tiles
// covers a window of list rows [row_lo, row_hi), so that a short last row tile can go to another tile
// shape.
//
// Epilogues.  A wave's loads and stores complete in order, and a wave of the ring loop is alone
// on its SIMD: a load issued behind stores (a residual, a register reloaded from scratch memory)
// returns only after all of them.  The epilogues therefore issue what they read ahead of the stores
// it could wait for, and the raw fp32 store of a K split is a compile-time form of the kernel (SPLIT)
// rather than a run-time branch beside the fused epilogue.
#pragma once
#include <type_traits>
#include "gemm_epilogues.h"
#include "gemm_plan.h"
#include "kernels.h"

namespace dy {
namespace mm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int BK = 64;    // K slice (elements)
constexpr int ROWB = 128; // bytes per tile row and slice
constexpr int N_XCD = 8;
constexpr int WPANEL = 32;  // output rows per weight panel

}  // namespace mm
}  // namespace dy
#include "gemm_bf16_ring.h"
namespace dy {
namespace mm {

// Tile shape: BM x BN output tile, WAVES_M x WAVES_N waves, DUAL = two weight matrices per tile (fused
// gate/up), NS LDS stages of one K slice each.  ONCE: weights that one workgroup alone reads go past the L2.
template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, bool DUAL_, int NS_, bool ONCE_ = false> struct Shape {
  static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_, NS = NS_;
  static constexpr bool DUAL = DUAL_, ONCE = ONCE_;
  static constexpr int NMAT = DUAL ? 2 : 1;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int MB = WM / 32, NB = WN / 32;
  static constexpr int NW = WAVES_M * WAVES_N;  // waves per workgroup (4 or 8)
  static constexpr int NT = NW * 64;
  static constexpr int A_LD = BM / (8 * NW);  // copy instructions per wave and slice (8 rows each)
  static constexpr int B_LD = BN / (8 * NW);
  static constexpr int LPS = A_LD + NMAT * B_LD;  // copies per wave and slice
  static constexpr int A_BYTES = BM * ROWB, W_BYTES = NMAT * BN * ROWB;
  // four waves on a tile of up to 256 rows with 256, 192 or 128 weight rows: the five-slot ring loop
  static constexpr bool RING = NW == 4 && BM == 256 && NS == 2;
  static constexpr int RING_ROWS = 16 * WAVES_M;  // a ring tile's rows are a multiple of this
  static constexpr size_t LDS_BYTES = RING ? (size_t)RING_SLOTS * RING_SLOT : (size_t)NS * (A_BYTES + W_BYTES);
  // shapes with three or more stages (weight streaming) run the loop pipelined over slices
  static constexpr bool PIPE = NS >= 3;
  static_assert(NW == 4 || NW == 8, "four or eight waves per workgroup");
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile is made of 32x32 blocks");
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile rows are copied in blocks of 8 per wave");
  static_assert(NS >= 2 && NS <= 8, "LDS stages");
  static_assert((NS - 1) * LPS < 64, "vmcnt immediate");
  static_assert(PIPE || MB * NB * NMAT > 2, "two-stage shapes interleave operand reads with enough products");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of one CU");
};

struct SplitStore {  // part != nullptr: raw fp32 tile part[z][j][n] instead of the fused epilogue
  float *part;
  size_t split_stride;
  int N;
};

// Operands of one GEMM, as the kernels take them.
struct GemmArgs {
  const bf16_t *A;
  const int32_t *gather;
  int lda;
  Rows rows;
  int N;
  WSeg seg;
  const bf16_t *W2;
  int K;
  float *part;  // raw result part[z][j][n], split stride = existing rows * N
};

// This lane's number, hidden from the optimiser and computed anew at every call.  What follows from it at the ends
// of a tile would otherwise be computed once per kernel, kept across the slice loops of every shape in it, which have
// no registers for that, and reloaded from scratch memory behind the copies in flight.
__device__ __forceinline__ int own_lane() {
  uint32_t all = ~0u;
  asm volatile("" : "+s"(all));
  return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
}

// How a workgroup walks the tiles: the first one's number and the distance to the next; the wave's number (scalar)
// and the LDS; whole: K is not split, and the epilogue finishes rows.  (Read off the thread's number once per kernel:
// a later shape's use of it would keep a register across
// the loop of an earlier one.)
struct Walk {
  int first, step, wave;
  unsigned char *smem;
  bool whole = false;
};
__device__ __forceinline__ Walk walk_of(unsigned char *smem) {
  return Walk{(int)blockIdx.x, (int)gridDim.x, (int)__builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), smem};
}

// Rows of a list that exist
__device__ __forceinline__ int rows_that_exist(const Rows &rows) { return rows.count ? min(*rows.count, rows.cap) : rows.cap; }

// f(MI) for the number of 16-row blocks per wave of a tile, of at most MAX: every count has a path of its own
template <int MAX, typename F> __device__ __forceinline__ bool with_blocks(int mi, F &&f) {
  if constexpr (MAX > 4) {
    if (mi == 8) return f(std::integral_constant<int, 8>{});
    if (mi == 7) return f(std::integral_constant<int, 7>{});
    if (mi == 6) return f(std::integral_constant<int, 6>{});
    if (mi == 5) return f(std::integral_constant<int, 5>{});
  }
  if (mi == 4) return f(std::integral_constant<int, 4>{});
  if (mi == 3) return f(std::integral_constant<int, 3>{});
  if (mi == 2) return f(std::integral_constant<int, 2>{});
  return f(std::integral_constant<int, 1>{});
}

// The tiles of rows [row_lo, min(M_all, row_hi)) of a list of M_all rows (row_lo is a multiple of BM) with `splitk` K splits,
// those that `walk` names.  Ring shapes: tiles of `ring_rows` rows (a multiple of RING_ROWS, at most BM), row_lo = 0.
// Splits are cut in whole K slices and may differ by one.
// SPLIT: the tile goes to the raw fp32 result part[z][j][n] instead of through the
// fused epilogue.  A compile-time switch: with both forms behind a run-time branch the compiler
// moves the accumulators out of the accumulation registers ahead of the branch, where they do not
// fit, and the epilogue's stores each wait for a reload from scratch memory.
template <typename SH, typename Epi, bool SPLIT>
__device__ __forceinline__ void gemm_tiles(const GemmArgs &ga, const Epi &epi, int M_all, int row_lo, int row_hi, int splitk,
                                           const Walk &walk, int ring_rows = SH::BM) {
  constexpr int BM = SH::BM, BN = SH::BN, MB = SH::MB, NB = SH::NB, NMAT = SH::NMAT, NS = SH::NS, NW = SH::NW;
  constexpr int group_m = 4;
  const bf16_t *const A = ga.A;
  const int32_t *const gather = Epi::GATHER ? ga.gather : nullptr;
  const bf16_t *const W2 = ga.W2;
  const int lda = ga.lda, N = ga.N, ldw = ga.K;
  const Rows rows = ga.rows;
  const WSeg &seg = ga.seg;

  const int M = min(M_all, row_hi);
  const SplitStore split{ga.part, (size_t)M_all * N, N};
  const int bm = SH::RING ? ring_rows : BM;
  const int tm_lo = SH::RING ? 0 : row_lo / BM;
  const int m_rel = max(M - tm_lo * BM, 0);
  // (ring tiles: list lengths are below 2^30 and a quotient's product with 1/bm may round either way)
  int tiles_m = (m_rel + BM - 1) / BM;
  if (SH::RING && bm != BM) {
    tiles_m = __builtin_amdgcn_readfirstlane((int)((float)m_rel * __builtin_amdgcn_rcpf((float)bm)));
    while (tiles_m * bm < m_rel) ++tiles_m;
    while (tiles_m > 0 && (tiles_m - 1) * bm >= m_rel) --tiles_m;
  }
  const int tiles_n = N / BN;
  const int first = walk.first, step = walk.step, wave = walk.wave;
  unsigned char *const smem_raw = walk.smem;
  const int lane = own_lane();
  const int wm0 = (wave / SH::WAVES_N) * SH::WM, wn0 = (wave % SH::WAVES_N) * SH::WN;
  const int l32 = lane % 32, lhi = lane / 32;
  const int KS = ldw / BK;  // K slices
  const uint32_t lds0 = lds_offset_of(smem_raw);

  // copy mapping of this lane inside an 8-row block: tile row r8, chunk position p, source chunk c
  const int r8 = lane / 8, cpos = lane % 8;
  // tile row of this lane in copy i is (i*NW + wave)*8 + r8, so (row/2) % 8 = ((wave & 1) * 4 + r8 / 2)
  const int csrc = cpos ^ (((wave & 1) << 2) | (r8 >> 1));
  // operand-read swizzle of this lane: chunk position of logical chunk (2*kk + lhi)
  int rd_off[BK / 16];
#pragma unroll
  for (int kk = 0; kk < BK / 16; ++kk) rd_off[kk] = (((2 * kk + lhi) ^ ((l32 >> 1) & 7)) * 16);

  // Tile order.  Workgroup p runs on XCD p % 8, and an XCD takes its workgroups in the order of p.
  // Each XCD gets a contiguous run of the FULL row tiles' tiles (walked in groups of group_m row tiles,
  // so that the tiles it runs at one time share operands in its L2) and, after those, its share of
  // the tiles of a last row tile that holds fewer than BM rows: those cost a fraction of a full tile
  // (see the partial loop below) and fill the end of every XCD's schedule instead of one XCD's.
  // With K splits the list of full tiles is the order above once per split, and so is that of the partial
  // ones: an XCD's run then mostly holds tiles of one split, which read the same part of K.
  const int has_tail = tiles_m * bm != m_rel ? 1 : 0;
  const int rows_full = tiles_m - has_tail;
  const int n_full = rows_full * tiles_n, n_part = has_tail * tiles_n;
  const int fx = (n_full * splitk + N_XCD - 1) / N_XCD, px = (n_part * splitk + N_XCD - 1) / N_XCD;
  const int total_all = (fx + px) * N_XCD;

  // Divisions are products with a reciprocal: for whole x below 2^21, (x + 1/2) / d lies at least 1 / (2 d)
  // from the next whole number, more than the product's rounding (an integer division is a chain of some
  // thirty instructions, eight of them in a row at the start of every tile).
  auto quot = [](int x, float inv) -> int { return __builtin_amdgcn_readfirstlane((int)(((float)x + 0.5f) * inv)); };
  auto inverse = [](int d) -> float {  // kept scalar
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, __builtin_amdgcn_rcpf((float)d))));
  };
  const int gsz = group_m * tiles_n;
  const float inv_full = inverse(n_full), inv_part = inverse(n_part), inv_gsz = inverse(gsz);
  // K slices of a split: the first k_rem splits have one more than the others
  const int k_base = splitk > 1 ? quot(KS, __builtin_amdgcn_rcpf((float)splitk)) : KS, k_rem = KS - k_base * splitk;
  auto k_first = [&](int z) -> int { return z * k_base + min(z, k_rem); };

  // tile (tm, tn) and K split z of position p in that order; false for the padding positions (uniform
  // for the workgroup)
  auto tile_at = [&](int p, int &tm, int &tn, int &z) -> bool {
    const int xcd = p % N_XCD, q = p / N_XCD;
    if (q < fx) {
      int logical = xcd * fx + q;
      if (logical >= n_full * splitk) return false;
      z = splitk > 1 ? quot(logical, inv_full) : 0;
      logical -= z * n_full;
      const int g = quot(logical, inv_gsz), r = logical - g * gsz;
      const int gm = min(group_m, rows_full - g * group_m);
      tn = quot(r, __builtin_amdgcn_rcpf((float)gm));
      tm = g * group_m + r - tn * gm;
    } else {
      const int lp = xcd * px + (q - fx);
      if (lp >= n_part * splitk) return false;
      z = splitk > 1 ? quot(lp, inv_part) : 0;
      tm = tiles_m - 1;
      tn = lp - z * n_part;
    }
    return true;
  };

  // Epilogue of one tile: the accumulators of this wave go through the fused epilogue (or, for a K
  // split, into the raw partial result).
  auto epilogue = [&](floatx16 (&acc)[NMAT][MB][NB], int m0, int n0, int tn, int z) {
    if constexpr (Epi::INTERLEAVE == 48) {
      // 32 x 96 wave tile = columns [0,48) of matrix 0 (gate) and [48,96) of matrix 1 (up): gate
      // column c pairs with tile column c + 48, which lane (c%32) ^ 16 holds one or two blocks on
      static_assert(NB == 3 && SH::WAVES_N == 1 && NMAT == 1, "half-interleaved tiles are 96 columns of one wave");
      const bool hi16 = (l32 & 16) != 0;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int j = m0 + wm0 + i * 32 + 8 * (e / 4) + 4 * lhi + (e % 4);
          const float a0 = acc[0][i][0][e], a1 = acc[0][i][1][e], a2 = acc[0][i][2][e];
          const float up0 = __shfl_xor(hi16 ? a1 : a2, 16, WAVE);  // up value of gate column l32
          const float up1 = __shfl_xor(a2, 16, WAVE);              // lanes 0..15: up value of gate column 32 + l32
          if (j < M) {
            epi.store(j, tn * 48 + l32, a0, up0);
            if (!hi16) epi.store(j, tn * 48 + 32 + l32, a1, up1);
          }
        }
    } else if constexpr (Epi::INTERLEAVE == 64) {
      // 32 x 128 wave tile = 64 gate + 64 up columns: the partner of a gate column is two blocks on
      // in the same lane
      static_assert(NB == 4 && SH::WAVES_N == 1 && NMAT == 1, "half-interleaved tiles are 128 columns of one wave");
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int j = m0 + wm0 + i * 32 + 8 * (e / 4) + 4 * lhi + (e % 4);
          if (j < M) {
            epi.store(j, tn * 64 + l32, acc[0][i][0][e], acc[0][i][2][e]);
            epi.store(j, tn * 64 + 32 + l32, acc[0][i][1][e], acc[0][i][3][e]);
          }
        }
    } else if (m0 + BM <= M) {
      // Full tile: no row checks, and every address is a wave-uniform base (scalar registers) plus a
      // byte offset per lane that is fixed for the tile.
      const int rbase = m0 + wm0, cbase = n0 + wn0;  // wave-uniform
      if constexpr (SPLIT) {
        float *pz = split.part + (size_t)z * split.split_stride;
        const uint32_t lb = ((uint32_t)(4 * lhi) * split.N + l32) * 4u;
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            float *r = pz + (size_t)(rbase + i * 32 + 8 * (e / 4) + (e % 4)) * split.N + cbase;
#pragma unroll
            for (int jn = 0; jn < NB; ++jn)
              *reinterpret_cast<float *>(reinterpret_cast<char *>(r + jn * 32) + lb) = acc[0][i][jn][e];
          }
      } else if constexpr (Epi::PRELOAD) {
        // A step of RS rows at a time: what the epilogue reads, then what it writes.  The reads of
        // step u + 1 are issued before the stores of step u: a wave's memory operations complete
        // in order, so a load behind stores would wait for all of them.
        constexpr int RS = NB >= 4 ? 8 : 16, STEPS = MB * 16 / RS;
        struct Pre {
          float v[RS][NB];
          int row[RS];
        };
        const uint32_t lbh = epi.lane_bytes_h(lhi, l32), lbo = epi.lane_bytes(lhi, l32);
        const int ld = epi.ld();
        auto row_of = [&](int u, int x) { return rbase + ((u * RS + x) / 16) * 32 + 8 * (((u * RS + x) % 16) / 4) + (x % 4); };
        auto load = [&](int u, Pre &p) {
#pragma unroll
          for (int x = 0; x < RS; ++x) {
            const int rr = row_of(u, x);
            p.row[x] = rows.idx ? *reinterpret_cast<const int *>(reinterpret_cast<const char *>(rows.idx + rr) + 16 * lhi) : 0;
#pragma unroll
            for (int jn = 0; jn < NB; ++jn) p.v[x][jn] = epi.get((size_t)rr * ld + cbase + jn * 32, lbh);
          }
        };
        Pre cur;
        load(0, cur);
#pragma unroll
        for (int u = 0; u < STEPS; ++u) {
          Pre nxt;
          if (u + 1 < STEPS) load(u + 1, nxt);
#pragma unroll
          for (int x = 0; x < RS; ++x) {
            const int i = (u * RS + x) / 16, e = (u * RS + x) % 16;
            if (rows.idx) {
              auto *o = epi.row_ptr(cur.row[x], cbase + l32);
#pragma unroll
              for (int jn = 0; jn < NB; ++jn) o[jn * 32] = from_f<std::remove_reference_t<decltype(o[0])>>(cur.v[x][jn] + acc[0][i][jn][e]);
            } else {
#pragma unroll
              for (int jn = 0; jn < NB; ++jn) epi.put((size_t)row_of(u, x) * ld + cbase + jn * 32, lbo, acc[0][i][jn][e], cur.v[x][jn]);
            }
          }
          if (u + 1 < STEPS) cur = nxt;
        }
      } else {
        const uint32_t lbo = epi.lane_bytes(lhi, l32);
        const int ld = epi.ld();
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const size_t u = (size_t)(rbase + i * 32 + 8 * (e / 4) + (e % 4)) * ld + cbase;
#pragma unroll
            for (int jn = 0; jn < NB; ++jn) epi.put(u + jn * 32, lbo, acc[0][i][jn][e], acc[NMAT - 1][i][jn][e]);
          }
      }
    } else if constexpr (Epi::PRELOAD) {
      if constexpr (!SPLIT) {
      // a 32-row block at a time: what the epilogue reads, then what it writes (two blocks in
      // flight cost more registers than the four-wave shapes have left: measured slower)
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        float pre[16][NB];
        int rowv[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int j = m0 + wm0 + i * 32 + 8 * (e / 4) + 4 * lhi + (e % 4);
          rowv[e] = (j < M && rows.idx) ? rows.idx[j] : j;
#pragma unroll
          for (int jn = 0; jn < NB; ++jn) pre[e][jn] = j < M ? epi.load(j, n0 + wn0 + jn * 32 + l32) : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int j = m0 + wm0 + i * 32 + 8 * (e / 4) + 4 * lhi + (e % 4);
          if (j < M) {
#pragma unroll
            for (int jn = 0; jn < NB; ++jn) epi.store(rowv[e], n0 + wn0 + jn * 32 + l32, acc[0][i][jn][e], pre[e][jn]);
          }
        }
      }
      } else {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int j = m0 + wm0 + i * 32 + 8 * (e / 4) + 4 * lhi + (e % 4);
            if (j < M) {
#pragma unroll
              for (int jn = 0; jn < NB; ++jn)
                split.part[(size_t)z * split.split_stride + (size_t)j * split.N + n0 + wn0 + jn * 32 + l32] =
                    acc[0][i][jn][e];
            }
          }
      }
    } else
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int j = m0 + wm0 + i * 32 + 8 * (e / 4) + 4 * lhi + (e % 4);
        if (j < M) {
          if constexpr (SPLIT) {
#pragma unroll
            for (int jn = 0; jn < NB; ++jn)
              split.part[(size_t)z * split.split_stride + (size_t)j * split.N + n0 + wn0 + jn * 32 + l32] =
                  acc[0][i][jn][e];
          } else {
            const int row = rows.idx ? rows.idx[j] : j;
#pragma unroll
            for (int jn = 0; jn < NB; ++jn)
              epi(j, row, n0 + wn0 + jn * 32 + l32, acc[0][i][jn][e], acc[NMAT - 1][i][jn][e]);
          }
        }
      }
  };

  if constexpr (SH::RING) {
    // Four-wave ring shapes.  The workgroup walks its tiles itself (the launcher starts one per CU),
    // and the ring is refilled for the next tile before the epilogue of the current one, so that
    // the first slices of a tile land while the previous tile's results are written.
    constexpr int WR = SH::WAVES_M, RR = SH::RING_ROWS, MAX_MI = BM / RR;
    using RingFull = Ring<NMAT, NB, BN, WR, MAX_MI>;
    constexpr int NWC = RingFull::NWC;
    static_assert(Epi::INTERLEAVE == 0 && SH::A_LD == 8 && NMAT * SH::B_LD == NWC, "ring shapes");
    const int wr = wave / SH::WAVES_N;  // wave row
    // Epilogue of one tile whose first row of this wave is rbase and first column cbase (both wave-uniform): this lane has
    // row rbase + RR i + 4 lq + e in element e of acc[t][i][..], column cbase + 16 G q + G l16 + h in block G q + h
    // (gemm_bf16_ring.h).  Row-ordered operands are addressed through buffer descriptors that end with the last
    // row: what lies past it is neither read nor written, without a branch per row (a branch around a load makes
    // the compiler wait for the load where the paths meet: 38000 instead of 14000 cycles for the down epilogue).
    constexpr int G = RingFull::G, NQ = 2 * NB / G;
    // Rows of q|k|v finished here: bias, rotation, rounding, and each value to where it belongs, where the raw result is
    // written, read and written again by a row kernel.  A head's column p turns with column p + HEAD / 2:
    //   SAME   a wave has whole heads of 128 columns: the partner is in the same lane, 64 columns on, and both use one table entry
    //   else   the weight rows of a run of 64 columns are those of 32 columns and of their partners (ring_sources): the
    //          partner is eight lanes on in the row of 16
    // What is read comes ahead of what it could wait for (a wave's memory operations complete in order): the list's entries
    // first, the table entries of row block i + AHEAD - 1 before block i is written.  Bound by the stores and the table's
    // loads, 16 cycles each of the CU's one path.  hidden 4096, GEMM and row kernel, us: dense 20480 rows 1466 + 211 -> 1469; lists of 2064
    // and 5160 rows 163 + 29 -> 170 + 5, 379 + 80 -> 392 + 5 (the row kernel is launched where the list's length may ask for a split).
    constexpr bool PAIRS = Epi::QKV == 128 && NQ != 2;  // the weight rows' order differs from the columns'
    constexpr bool SAME = Epi::QKV == 128 && NQ == 2;
    constexpr int NP = PAIRS && NQ > 1 ? 2 : 1;  // table entries of a row: one for all runs, or one for every second run
    constexpr int AHEAD = NP == 1 ? 3 : 2;       // row blocks whose table entries are in flight or in use
    auto qkv_rows = [&](auto &row, int rbase) {  // this lane's rows (tokens) of every row block
      constexpr int MI = sizeof(row) / sizeof(row[0]);
      const int lq = own_lane() / 16;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int n = __builtin_amdgcn_readfirstlane(min(max(M - rbase - RR * i, 0), 16));
        const auto list = make_srd(rows.idx + (rows.idx ? rbase + RR * i : 0), rows.idx ? n * 4u : 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) row[i][e] = rows.idx ? __builtin_amdgcn_raw_buffer_load_b32(list, lq * 16 + e * 4, 0, 0) : rbase + RR * i + 4 * lq + e;
      }
    };
    auto qkv_table = [&](auto &row, auto &tab, int cbase, int i) {  // the table entries of row block i
      if constexpr (Epi::QKV > 0) {
        const QkvOut &o = epi.o;
        const int l16 = own_lane() % 16;
        const bool any = (PAIRS ? cbase & ~127 : cbase) < (o.H + o.Hkv) * Epi::QKV;
        const auto table = make_srd(o.tab, any ? 0xfffffff0u : 0u);  // (values alone: nothing is read)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t pos = epi.position((uint32_t)row[i][e]);
#pragma unroll
          for (int u = 0; u < NP; ++u) {
            const int half = PAIRS ? ((cbase >> 6) + u) & 1 : 0;
            const uint32_t at = pos * (Epi::QKV * 4u) + (uint32_t)(32 * half + (SAME ? 4 * l16 : 4 * (l16 % 8))) * 8u;
            tab[i % AHEAD][e][u][0] = load_buf(table, at);
            tab[i % AHEAD][e][u][1] = load_buf(table, at + 16u);
          }
        }
      }
    };
    auto qkv_epilogue = [&](auto &acc, int rbase, int cbase) {
      if constexpr (Epi::QKV > 0) {
        constexpr int MI = sizeof(acc[0]) / sizeof(acc[0][0]), HEAD = Epi::QKV;
        const QkvOut &o = epi.o;
        const int ln = own_lane(), l16 = ln % 16, lq = ln / 16;
        const bool upper = (l16 & 8) != 0;  // !SAME: this lane has the second half's columns
        const int dq = o.H * HEAD, dkv = o.Hkv * HEAD;
        // (fetched together and selected from, as the weights' addresses in ring_sources)
        void *to_q = o.q, *to_k = o.k, *to_v = o.v;
        const void *bq = o.bq, *bk = o.bk, *bv = o.bv;
        asm volatile("" : "+s"(to_q), "+s"(to_k), "+s"(to_v), "+s"(bq), "+s"(bk), "+s"(bv));
        int row[MI][4];
        floatx4 tab[AHEAD][4][NP][2];
        qkv_rows(row, rbase);
#pragma unroll
        for (int i = 0; i < AHEAD - 1 && i < MI; ++i) qkv_table(row, tab, cbase, i);
        // where a run's columns go, wave-uniform but for the lane's own columns
        char *out[NQ];
        int row_bytes[NQ];
        bool turns[NQ], by_token[NQ];
        floatx4 bias[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int run = cbase + 64 * q, head = PAIRS ? run & ~127 : run, half = PAIRS ? (run >> 6) & 1 : 0;
          const bool in_q = head < dq, in_k = !in_q && head < dq + dkv;
          const int start = in_q ? 0 : in_k ? dq : dq + dkv;
          const int col = head - start + 32 * half + (PAIRS ? (upper ? 64 : 0) + 4 * (l16 % 8) : 4 * l16);
          out[q] = (char *)(in_q ? to_q : in_k ? to_k : to_v) + (size_t)col * 2;
          row_bytes[q] = (in_q ? dq : dkv) * 2;
          turns[q] = in_q || in_k;
          by_token[q] = !in_q || o.q_by_token;
          const void *b = in_q ? bq : in_k ? bk : bv;
          uint2 w = {0u, 0u};
          if (b) w = *reinterpret_cast<const uint2 *>((const bf16_t *)b + col);
          bias[q] = floatx4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                            __uint_as_float(w.y & 0xffff0000u)};
        }
        // TURN: the wave's columns are queries or keys (else values alone), wave-uniform.
        auto finish = [&](auto turn_c) {
          constexpr bool TURN = decltype(turn_c)::value;
#pragma unroll
          for (int i = 0; i < MI; ++i) {
            if (TURN && i + AHEAD - 1 < MI) qkv_table(row, tab, cbase, i + AHEAD - 1);
            const int n = __builtin_amdgcn_readfirstlane(min(max(M - rbase - RR * i, 0), 16));
            // (the accumulators are still where they were: without this the compiler moves them out of the second register
            // file ahead of the branch that led here, into scratch memory)
#pragma unroll
            for (int c = 0; c < 2 * NB; ++c) asm volatile("" : "+a"(acc[0][i][c]));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              floatx4 x[NQ], y[NQ];
#pragma unroll
              for (int q = 0; q < NQ; ++q) {
                x[q] = floatx4{acc[0][i][G * q][e], acc[0][i][G * q + 1][e], acc[0][i][G * q + 2][e], acc[0][i][G * q + 3][e]} + bias[q];
              }
#pragma unroll
              for (int q = 0; q < NQ; ++q) {
                const floatx4 *t = tab[i % AHEAD][e][q % NP];
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                  float turned = x[q][h];
                  if constexpr (TURN) {
                    const float co = t[h / 2][2 * (h % 2)], si = t[h / 2][2 * (h % 2) + 1];
                    if constexpr (SAME) {
                      const float ps = x[1 - q][h] * si;
                      turned = rotated(x[q][h], co, q == 0 ? -ps : ps);
                    } else {
                      const float partner = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x[q][h]), 0x128, 0xf, 0xf, false));
                      const float ps = partner * si;
                      turned = rotated(x[q][h], co, upper ? ps : -ps);
                    }
                  }
                  y[q][h] = !SAME && NQ > 1 && !turns[q] ? x[q][h] : turned;  // (a wave's runs may be on both sides of the last key column)
                }
              }
              if (4 * lq + e < n) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                  const size_t r = (size_t)(uint32_t)(by_token[q] ? row[i][e] : rbase + RR * i + 4 * lq + e);
                  *reinterpret_cast<uint2 *>(out[q] + r * (uint32_t)row_bytes[q]) = uint2{pack_bf16(y[q][0], y[q][1]), pack_bf16(y[q][2], y[q][3])};
                }
              }
            }
            __builtin_amdgcn_sched_barrier(0);  // (a row block at a time: more of them at once spill)
          }
        };
        bool any = false;
#pragma unroll
        for (int q = 0; q < NQ; ++q) any |= turns[q];
        if (any) {
          finish(std::true_type{});
        } else {
          finish(std::false_type{});
        }
      }
    };
    auto ring_epilogue = [&](auto &acc, int rbase, int cbase, int z) {
      constexpr int MI = sizeof(acc[0]) / sizeof(acc[0][0]);  // 16-row blocks
      const int ln = own_lane(), l16 = ln % 16, lq = ln / 16;
      // rows of block i that exist; descriptor of its rows of a [., N] operand of esz bytes per element
      auto left = [&](int i) -> int { return __builtin_amdgcn_readfirstlane(min(max(M - rbase - RR * i, 0), 16)); };
      auto block = [&](const void *p, int i, int esz) {
        return make_srd((const char *)p + ((size_t)(rbase + RR * i) * N + cbase) * esz, left(i) ? (uint32_t)(left(i) * N - cbase) * esz : 0);
      };
      uint32_t lane_row[4];  // element offsets of this lane's four rows in a block
#pragma unroll
      for (int e = 0; e < 4; ++e) lane_row[e] = (uint32_t)(4 * lq + e) * N + G * l16;
      if constexpr (SPLIT) {
        static_assert(!SPLIT || G == 4, "16-byte raw stores");
        if constexpr (Epi::QKV > 0) {
          if (walk.whole) {  // wave-uniform
            qkv_epilogue(acc, rbase, cbase);
            return;
          }
        }
        const float *pz = split.part + (size_t)z * split.split_stride;
        auto at = [&](int i, int q, int e) {
          return floatx4{acc[0][i][G * q][e], acc[0][i][G * q + 1][e], acc[0][i][G * q + 2][e], acc[0][i][G * q + 3][e]};
        };
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const auto part = block(pz, i, 4);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int q = 0; q < NQ; ++q) store_buf(at(i, q, e), part, lane_row[e] * 4u + 64 * G * q);
        }
      } else if constexpr (Epi::PRELOAD) {
        // what row block i + 1 reads is requested before block i is written: a wave's memory operations
        // complete in order, so a load behind stores would wait for all of them
        floatx4 pre[2][4][NQ];
        int row[2][4];
        auto load = [&](int i) {
          const auto res = block(epi.h, i, 4);
          const auto list = make_srd(rows.idx + (rows.idx ? rbase + RR * i : 0), rows.idx ? left(i) * 4u : 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            row[i & 1][e] = __builtin_amdgcn_raw_buffer_load_b32(list, lq * 16 + e * 4, 0, 0);
#pragma unroll
            for (int q = 0; q < NQ; ++q) pre[i & 1][e][q] = load_buf(res, lane_row[e] * 4u + 64 * G * q);
          }
        };
        load(0);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          if (i + 1 < MI) load(i + 1);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = 4 * lq + e;
            if (r < left(i)) {
#pragma unroll
              for (int q = 0; q < NQ; ++q) {
                const floatx4 a = {acc[0][i][G * q][e], acc[0][i][G * q + 1][e], acc[0][i][G * q + 2][e], acc[0][i][G * q + 3][e]};
                epi.store4(rows.idx ? row[i & 1][e] : rbase + RR * i + r, cbase + 16 * G * q + G * l16, a, pre[i & 1][e][q]);
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);  // (a row block at a time: more of them at once spill)
        }
      } else {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const auto act = block(epi.act, i, 2);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              float v[G];
#pragma unroll
              for (int h = 0; h < G; ++h) v[h] = epi.product(acc[0][i][G * q + h][e], acc[NMAT - 1][i][G * q + h][e]);
              store_buf(v, act, lane_row[e] * 2u + 32 * G * q);
            }
          __builtin_amdgcn_sched_barrier(0);  // (a row block at a time: more of them at once spill)
        }
      }
    };
    auto ring_sources = [&](int tm, int tn, int z, RingSrc &src) {
      const int kbeg = k_first(z) * BK;
      const int m0 = tm * bm, n0 = tn * BN;
      const int ln = own_lane(), r8 = ln / 8, csrc = (ln % 8) ^ (((wave & 1) << 2) | (r8 >> 1));  // as above
      // Lane offsets are 32 bits.  Without a gather list the descriptor starts at the tile's first
      // row, so the offsets stay below 256 rows; with one they are taken from the start of the
      // operand (the launcher checks that it spans less than 4 GiB).
      src.srd_a = make_srd(gather ? A : A + (size_t)m0 * lda, 0xfffffff0u);
      // (the eight list entries of a gathered operand are loaded back to back, then used)
      int srow[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int j = m0 + (i * NW + wave) * 8 + r8;
        srow[i] = j < M ? j : M - 1;  // rows past the end are clamped; their results are never stored
      }
      if (gather) {
#pragma unroll
        for (int i = 0; i < 8; ++i) srow[i] = gather[srow[i]];
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) srow[i] -= m0;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        uint32_t at = (uint32_t)srow[i] * (uint32_t)(lda * 2);
        asm volatile("" : "+v"(at));  // (a fused multiply-add has a 64-bit result: a second register per offset)
        src.va[i] = at + (uint32_t)(kbeg + csrc * 8) * 2u;
      }
      // The matrices' addresses and ends are fetched together and selected from: left to itself the compiler fetches
      // each descriptor's address from the kernel arguments when it knows which one it is, one wait after the other
      // (eight of them in the 256 x 256 tile).
      const void *w[4] = {seg.w[0], seg.w[1], seg.w[2], W2};
      int n_end[2] = {seg.n_end[0], seg.n_end[1]};
      asm volatile("" : "+s"(w[0]), "+s"(w[1]), "+s"(w[2]), "+s"(w[3]), "+s"(n_end[0]), "+s"(n_end[1]));
#pragma unroll
      for (int d = 0; d < RingFull::ND; ++d) {
        const int c = d * (NWC / RingFull::ND), t = c / SH::B_LD, i = c % SH::B_LD;
        // the copy's 8 tile rows hold every G-th weight row from nu on (wave-uniform): rows of one panel, and
        // so of one matrix, whose ends are multiples of 16 G (ring_groups_ok)
        int nu = n0 + RingFull::weight_row(i, wave);
        if constexpr (PAIRS) {
          // a run of 64 holds the 32 columns of half a head's half and their partners: panels 0 and 2, or 1 and 3, of the head
          if (walk.whole) nu += ((wave & 1) - ((n0 / 64 + i / 2) & 1)) * WPANEL;
        }
        const bool in1 = nu >= n_end[0], in2 = nu >= n_end[1];
        const void *base = t == 1 ? w[3] : in2 ? w[2] : in1 ? w[1] : w[0];
        const int nl = nu - (t == 1 ? 0 : in2 ? n_end[1] : in1 ? n_end[0] : 0);  // row in its matrix
        src.srd_w[d] = make_srd((const bf16_t *)base + ((size_t)(nl / WPANEL) * KS + kbeg / BK) * (WPANEL * BK) + (nl % WPANEL) * BK, 0xfffffff0u);
      }
      src.vw = (uint32_t)((G * r8 * BK + csrc * 8) * 2);
    };
    // 16-row blocks per wave of row tile t
    auto blocks_of = [&](int t) -> int { return (min(bm, M - t * bm) + RR - 1) / RR; };
    int tm = 0, tn = 0, z = 0, p = first;
    auto find = [&]() -> bool {  // the workgroup's tile at p or behind it
      while (p < total_all && !tile_at(p, tm, tn, z)) p += step;
      return p < total_all;
    };
    // Consecutive tiles with MI 16-row blocks of each wave, from the one at p on; returns whether there is another tile.
    // Everything about these tiles is in their own loop, epilogue included, and nothing but the tile's number passes
    // from one path to another (the first tile of a path fills the ring anew: only a last row tile changes the path).
    // Where the paths shared a loop, the sources of the copies, and where they met before the epilogue the
    // accumulators, went through other registers and scratch memory at the end of every tile.
    auto run_tiles_of = [&](auto mi_c, auto once_c) -> bool {
      constexpr int MI = decltype(mi_c)::value;
      using R = Ring<NMAT, NB, BN, WR, MI, decltype(once_c)::value>;
      uint32_t lds_at = lds0;
      asm volatile("" : "+s"(lds_at));  // (what follows from it is computed here, not once for all paths and kept)
      RingSrc src;
      ring_sources(tm, tn, z, src);
      R::fill(src, lds_at, wave, k_base + (z < k_rem ? 1 : 0));
      for (bool all_landed = false;; all_landed = true) {
        const int KT = k_base + (z < k_rem ? 1 : 0);
        const int rbase = tm * bm + 16 * wr, cbase = tn * BN + wn0, z_now = z;
        const int ln = own_lane(), l16 = ln % 16, lq = ln / 16;
        const unsigned char *rd_a = smem_raw + (16 * wr + l16) * ROWB, *rd_w = smem_raw + (wn0 + l16) * ROWB;
        int rd_off16[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) rd_off16[kk] = (((4 * kk + lq) ^ ((l16 >> 1) & 7)) * 16);
        floatx4 acc[NMAT][MI][2 * NB];
        R::tile(acc, lds_at, wave, src, rd_a, rd_w, rd_off16, KT, all_landed);
        p += step;
        const bool more = find(), same = more && blocks_of(tm) == MI;
        if (same) {
          ring_sources(tm, tn, z, src);
          R::fill(src, lds_at, wave, k_base + (z < k_rem ? 1 : 0));
        }
        ring_epilogue(acc, rbase, cbase, z_now);
        if (!same) return more;
      }
    };
    bool more = find();
    // All rows in one row tile of more than half the height, which is what 129 to 256 rows in one come to: the weights go past the L2,
    // where they would displace the activations that all workgroups share.  With more row tiles they are found there.  (hidden
    // 4096, 143 rows: step 184.5 -> 169.8 us; with 573 rows, past the L2 as well, 340 -> 362.)
    // The loops exist for the shapes that plans take for so few rows: 128 columns, K split where it may be, and 256 for gate|up (no
    // other for eight layer shapes of hidden 512 to 8192).  In the others they made the kernels longer for all rows: 330 rows, down
    // projection 35.9 -> 36.6 us; a loop of 8 x 1024 tokens 2013 -> 2035.
    constexpr bool ONCE_LOOPS = SH::ONCE && (BN * NMAT == 128 ? (NMAT == 2 || SPLIT) : BN * NMAT == 256 && NMAT == 2);
    if constexpr (ONCE_LOOPS) {
      static_assert(MAX_MI == 8, "row blocks of these shapes");
      if (M_all <= bm && blocks_of(0) > MAX_MI / 2) {
        const int mi = blocks_of(0);
        auto once = [&](auto mi_c) -> bool { return run_tiles_of(mi_c, std::true_type{}); };
        while (more) more = mi == 8 ? once(std::integral_constant<int, 8>{}) : mi == 7 ? once(std::integral_constant<int, 7>{})
                            : mi == 6 ? once(std::integral_constant<int, 6>{}) : once(std::integral_constant<int, 5>{});
        return;
      }
    }
    while (more) more = with_blocks<MAX_MI>(blocks_of(tm), [&](auto mi_c) -> bool { return run_tiles_of(mi_c, std::false_type{}); });
    return;
  }

  for (int p = first; p < total_all; p += step) {
    int tm, tn, z;
    if (!tile_at(p, tm, tn, z)) continue;
    const int m0 = (tm_lo + tm) * BM, n0 = tn * BN;
    const int kbeg = k_first(z) * BK, KT = k_base + (z < k_rem ? 1 : 0);

    // per-lane global sources of the copies it issues every slice
    const bf16_t *ap[SH::A_LD];
#pragma unroll
    for (int i = 0; i < SH::A_LD; ++i) {
      int j = m0 + (i * NW + wave) * 8 + r8;
      j = j < M ? j : M - 1;  // rows past the end are clamped; their results are never stored
      const int src = gather ? gather[j] : j;
      ap[i] = A + (size_t)src * lda + kbeg + csrc * 8;
    }
    // a column tile may span two of the stacked weight matrices: the matrix is looked up per row
    const bf16_t *wp[NMAT][SH::B_LD];
#pragma unroll
    for (int i = 0; i < SH::B_LD; ++i) {
      const int nrow = (i * NW + wave) * 8 + r8;
      const int n = n0 + nrow;
      const bf16_t *wbase;
      int nl;  // row inside its matrix
      if constexpr (Epi::INTERLEAVE > 0) {
        // tile tn = HALF rows of matrix 0 followed by the same HALF rows of matrix 1
        constexpr int HALF = Epi::INTERLEAVE;
        static_assert(BN == 2 * HALF, "one half tile per matrix");
        const bool second = nrow >= HALF;
        wbase = (const bf16_t *)(second ? seg.w[1] : seg.w[0]);
        nl = tn * HALF + (second ? nrow - HALF : nrow);
      } else {
        const bool in1 = n >= seg.n_end[0], in2 = n >= seg.n_end[1];
        wbase = (const bf16_t *)(in2 ? seg.w[2] : in1 ? seg.w[1] : seg.w[0]);
        nl = n - (in2 ? seg.n_end[1] : in1 ? seg.n_end[0] : 0);
      }
      // panel layout: slice kt of this row sits kt * (WPANEL * BK) elements further on
      const size_t woff = ((size_t)(nl / WPANEL) * (ldw / BK) + kbeg / BK) * (WPANEL * BK) + (nl % WPANEL) * BK + csrc * 8;
      wp[0][i] = wbase + woff;
      if (SH::DUAL)
        wp[NMAT - 1][i] = W2 + ((size_t)(n / WPANEL) * (ldw / BK) + kbeg / BK) * (WPANEL * BK) + (n % WPANEL) * BK + csrc * 8;
    }

    floatx16 acc[NMAT][MB][NB];
#pragma unroll
    for (int t = 0; t < NMAT; ++t)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) acc[t][i][j][e] = 0.f;

    // LDS: NS stages of the A tile, then NS stages of the weight tile(s)
    auto issue_a = [&](int kt) {  // A rows of slice kt -> A stage kt % NS
      const uint32_t sb = lds0 + (uint32_t)(kt % NS) * SH::A_BYTES + (uint32_t)wave * 1024u;
      const int ko = kt * BK;
#pragma unroll
      for (int i = 0; i < SH::A_LD; ++i) dma16(ap[i] + ko, sb + i * (NW * 1024u));
    };
    auto issue_w = [&](int kt) {  // weight rows of slice kt -> weight stage kt % NS
      const uint32_t sb = lds0 + (uint32_t)(NS * SH::A_BYTES) + (uint32_t)(kt % NS) * SH::W_BYTES +
                          (uint32_t)wave * 1024u;
      const int ko = kt * (WPANEL * BK);
#pragma unroll
      for (int t = 0; t < NMAT; ++t)
#pragma unroll
        for (int i = 0; i < SH::B_LD; ++i) {
          // (every weight is read by one workgroup; the row tiles that read them too where only a last row tile streams are long
          // done: dense 1300 rows of hidden 4096 589 -> 581 us, lists of as many equal)
          if constexpr (SH::ONCE) dma16_once(wp[t][i] + ko, sb + (uint32_t)(t * BN) * ROWB + i * (NW * 1024u));
          else dma16(wp[t][i] + ko, sb + (uint32_t)(t * BN) * ROWB + i * (NW * 1024u));
        }
    };

    __syncthreads();  // LDS free: the previous tile of this workgroup is fully consumed
    if constexpr (SH::PIPE) {
      // Weight-streaming shapes: one wave per SIMD and few products per slice, so nothing hides the
      // chain wait -> barrier -> operand reads -> products of a slice.  The loop is therefore
      // pipelined over slices: the operands of slice kt+1 are read (into a second register set)
      // while the products of slice kt run, and because a wave holds slice kt in registers when it
      // reaches the barrier of iteration kt, that stage is refilled at once: NS slices are in flight
      // instead of NS-1.
      // Few rows: only the first ALD of a wave's A_LD copies per slice hold rows below M (copy i of
      // wave w fills rows (i*NW + w)*8 ...), the others are left out -- with at most 64 (32) rows that
      // halves (quarters) the activation traffic from L2, which competes with the weight stream.
      // Tile rows that are never filled only feed results that are never stored.
      auto pipe_loop = [&](auto ald_c) {
      constexpr int ALD = decltype(ald_c)::value;
      constexpr int LPS = ALD + NMAT * SH::B_LD;  // copies per wave and slice
      auto issue_a_n = [&](int kt) {
        const uint32_t sb = lds0 + (uint32_t)(kt % NS) * SH::A_BYTES + (uint32_t)wave * 1024u;
        const int ko = kt * BK;
#pragma unroll
        for (int i = 0; i < ALD; ++i) dma16(ap[i] + ko, sb + i * (NW * 1024u));
      };
      constexpr int KS = BK / 16, RD = MB + NMAT * NB, MM = NMAT * MB * NB;
      bf16x8 af[2][KS][MB], bfr[2][KS][NMAT][NB];
      auto read_slice = [&](bf16x8 (&a)[KS][MB], bf16x8 (&b)[KS][NMAT][NB], int kt) {
        const unsigned char *sa = smem_raw + (size_t)(kt % NS) * SH::A_BYTES + (wm0 + l32) * ROWB;
        const unsigned char *sb = smem_raw + (size_t)NS * SH::A_BYTES + (size_t)(kt % NS) * SH::W_BYTES +
                                  (wn0 + l32) * ROWB;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
          for (int i = 0; i < MB; ++i) a[kk][i] = *reinterpret_cast<const bf16x8 *>(sa + i * 32 * ROWB + rd_off[kk]);
#pragma unroll
          for (int t = 0; t < NMAT; ++t)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              b[kk][t][j] = *reinterpret_cast<const bf16x8 *>(sb + (t * BN + j * 32) * ROWB + rd_off[kk]);
        }
      };
      auto slice = [&](int kt, auto cur_c) {
        constexpr int CUR = decltype(cur_c)::value;
        // slice kt+1 has landed: the copies issued after it may still be on their way
        if (kt + NS - 1 < KT) wait_vmcnt<(NS - 2) * LPS>();
        else wait_vmcnt<0>();
        wait_lgkmcnt0();  // the operands of slice kt are in registers: its stage is free
        __syncthreads();
        if (kt + NS < KT) { issue_a_n(kt + NS); issue_w(kt + NS); }
        read_slice(af[CUR ^ 1], bfr[CUR ^ 1], kt + 1 < KT ? kt + 1 : kt);  // (past the end: a harmless re-read)
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
          for (int t = 0; t < NMAT; ++t)
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
              for (int j = 0; j < NB; ++j)
                acc[t][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[CUR][kk][i], bfr[CUR][kk][t][j], acc[t][i][j], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, KS * RD, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, KS * MM, 0);
        __builtin_amdgcn_sched_barrier(0);
      };
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (s < KT) { issue_a_n(s); issue_w(s); }
      if (NS - 1 < KT) wait_vmcnt<(NS - 1) * LPS>();  // slice 0 has landed
      else wait_vmcnt<0>();
      __syncthreads();
      read_slice(af[0], bfr[0], 0);
      int kt = 0;
      for (; kt + 1 < KT; kt += 2) {
        slice(kt, std::integral_constant<int, 0>{});
        slice(kt + 1, std::integral_constant<int, 1>{});
      }
      if (kt < KT) slice(kt, std::integral_constant<int, 0>{});
      };
      const int a_need = (M - m0 + 8 * NW - 1) / (8 * NW);  // copies per wave that hold rows
      if (SH::A_LD >= 4 && a_need <= 1) pipe_loop(std::integral_constant<int, 1>{});
      else if (SH::A_LD >= 2 && a_need <= SH::A_LD / 2) pipe_loop(std::integral_constant<int, (SH::A_LD >= 2 ? SH::A_LD / 2 : 1)>{});
      else pipe_loop(std::integral_constant<int, SH::A_LD>{});
    } else if (NS == 2 && m0 + BM > M) {
      // A row tile that holds fewer than BM rows: copies of 8-row blocks past the end are left out,
      // and a wave multiplies only its 32-row blocks that hold rows (none at all for many waves), so
      // that the tile costs about what its weight copies cost.  Same barriers as the full loop.
      const int mbv_raw = (M - (m0 + wm0) + 31) / 32;
      const int mbv = mbv_raw < 0 ? 0 : (mbv_raw > MB ? MB : mbv_raw);  // wave-uniform
      auto issue_a_part = [&](int kt) {
        const uint32_t sb = lds0 + (uint32_t)(kt % NS) * SH::A_BYTES + (uint32_t)wave * 1024u;
        const int ko = kt * BK;
#pragma unroll
        for (int i = 0; i < SH::A_LD; ++i)
          if (m0 + (i * NW + wave) * 8 < M) dma16(ap[i] + ko, sb + i * (NW * 1024u));
      };
      issue_a_part(0);
      issue_w(0);
      for (int kt = 0; kt < KT; ++kt) {
        wait_vmcnt<0>();
        __syncthreads();
        if (kt + 1 < KT) {
          issue_a_part(kt + 1);
          issue_w(kt + 1);
        }
        if (mbv == 0) continue;  // wave-uniform; the barriers above are all this wave owes the tile
        const unsigned char *sa = smem_raw + (size_t)(kt % NS) * SH::A_BYTES + (wm0 + l32) * ROWB;
        const unsigned char *sb = smem_raw + (size_t)NS * SH::A_BYTES + (size_t)(kt % NS) * SH::W_BYTES +
                                  (wn0 + l32) * ROWB;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
          bf16x8 bfr[NMAT][NB];
#pragma unroll
          for (int t = 0; t < NMAT; ++t)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              bfr[t][j] = *reinterpret_cast<const bf16x8 *>(sb + (t * BN + j * 32) * ROWB + rd_off[kk]);
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            if (i < mbv) {
              const bf16x8 af = *reinterpret_cast<const bf16x8 *>(sa + i * 32 * ROWB + rd_off[kk]);
#pragma unroll
              for (int t = 0; t < NMAT; ++t)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                  acc[t][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr[t][j], acc[t][i][j], 0, 0, 0);
            }
          }
        }
      }
    } else {
    // slice by slice
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
      if (s < KT) { issue_a(s); issue_w(s); }

    for (int kt = 0; kt < KT; ++kt) {
      // slice kt has landed (this wave's part); a wave's copies complete in issue order
      if (kt + NS - 2 < KT) wait_vmcnt<(NS - 2) * SH::LPS>();
      else wait_vmcnt<0>();
      __syncthreads();  // ... all waves' parts; and everyone is done with slice kt-1
      if (kt + NS - 1 < KT) { issue_a(kt + NS - 1); issue_w(kt + NS - 1); }  // into the stage slice kt-1 left

      const unsigned char *sa = smem_raw + (size_t)(kt % NS) * SH::A_BYTES + (wm0 + l32) * ROWB;
      const unsigned char *sb = smem_raw + (size_t)NS * SH::A_BYTES + (size_t)(kt % NS) * SH::W_BYTES +
                                (wn0 + l32) * ROWB;
      // operand fragments of slice step kk+1 are fetched while the MFMAs of step kk run
      bf16x8 af[2][MB], bfr[2][NMAT][NB];
#pragma unroll
      for (int i = 0; i < MB; ++i) af[0][i] = *reinterpret_cast<const bf16x8 *>(sa + i * 32 * ROWB + rd_off[0]);
#pragma unroll
      for (int t = 0; t < NMAT; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          bfr[0][t][j] = *reinterpret_cast<const bf16x8 *>(sb + (t * BN + j * 32) * ROWB + rd_off[0]);
#pragma unroll
      for (int kk = 0; kk < BK / 16; ++kk) {
        const int c = kk & 1, n = c ^ 1;
        if (kk + 1 < BK / 16) {
#pragma unroll
          for (int i = 0; i < MB; ++i)
            af[n][i] = *reinterpret_cast<const bf16x8 *>(sa + i * 32 * ROWB + rd_off[kk + 1]);
#pragma unroll
          for (int t = 0; t < NMAT; ++t)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              bfr[n][t][j] = *reinterpret_cast<const bf16x8 *>(sb + (t * BN + j * 32) * ROWB + rd_off[kk + 1]);
        }
#pragma unroll
        for (int t = 0; t < NMAT; ++t)
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
              acc[t][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[c][i], bfr[c][t][j], acc[t][i][j], 0, 0, 0);
      }
      // Instruction order of the slice: the first step's operand reads, then the LDS reads of step
      // kk+1 spread one by one between the MFMAs of step kk (the scheduler alone fetches each
      // operand right before its use and leaves the matrix pipe waiting on the LDS).
      {
        constexpr int RD = MB + NMAT * NB, MM = NMAT * MB * NB;
        __builtin_amdgcn_sched_group_barrier(0x100, RD, 0);
#pragma unroll
        for (int kk = 0; kk + 1 < BK / 16; ++kk) {
#pragma unroll
          for (int q = 0; q < RD; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          }
          if (MM > RD) __builtin_amdgcn_sched_group_barrier(0x008, MM - RD, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, MM, 0);
      }
    }
    }

    epilogue(acc, m0, n0, tn, z);
  }
}

// One tile shape, chosen by the launcher.
template <typename SH, typename Epi, bool SPLIT>
__global__ __launch_bounds__(SH::NT) void k_gemm_bf16(GemmArgs ga, Epi epi, int splitk) {
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  gemm_tiles<SH, Epi, SPLIT>(ga, epi, rows_that_exist(ga.rows), 0, 0x7fffffff, splitk, walk_of(smem_raw));
}

// Row tiles of the ring loop (and the weight-streaming tiles of a short last row tile, or of a list with few
// rows), by the plan that fits the rows that exist (gemm_plan.h).  One workgroup per CU.
//   Kind::Epi      fused epilogue of the row tiles; Kind::FUSED / RAW: which of its forms exist
//   Kind::X, L, W  tile shapes (W: void where there is none); Kind::stream(...) runs the weight-streaming tiles
//   Kind::PLANS    the kernel may have to make its plan
// planned: PLAN_GIVEN: pl (the count is known on the host); PLAN_MADE: words, by the row kernel before; PLAN_HERE: made by every
// workgroup, the first of which leaves it in words for the row kernels (Splits::dev).
enum Planned { PLAN_GIVEN, PLAN_MADE, PLAN_HERE };
template <typename Kind>
__global__ __launch_bounds__(256) void k_gemm_planned(GemmArgs ga, typename Kind::Epi epi, PlanArgs pa, GemmPlan pl,
                                                      Planned planned, int32_t *words) {
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  Walk walk = walk_of(smem_raw);
  const int M = rows_that_exist(ga.rows);
  if (planned == PLAN_MADE) pl = load_plan(words);
  if constexpr (Kind::PLANS) {
    if (planned == PLAN_HERE) {
      pl = plan_on_device(pa, M, walk.wave, (uint32_t *)smem_raw);
      __syncthreads();  // (the words are read before anything is copied over them)
    }
  }
  if constexpr (Kind::Epi::QKV > 0) walk.whole = pl.sk == 1 && epi.o.tab;
  if constexpr (Kind::PLANS) {
    if (planned == PLAN_HERE && blockIdx.x == 0 && threadIdx.x == 0) store_plan(pl, walk.whole, words);
  }
  if (pl.row_hi > 0) {
    if (Kind::RAW && (!Kind::FUSED || pl.sk > 1)) {
      if constexpr (Kind::RAW) {
        if (pl.xl == PLAN_X) gemm_tiles<typename Kind::X, typename Kind::Epi, true>(ga, epi, M, 0, pl.row_hi, pl.sk, walk, pl.bm);
        else if (pl.xl == PLAN_L) gemm_tiles<typename Kind::L, typename Kind::Epi, true>(ga, epi, M, 0, pl.row_hi, pl.sk, walk, pl.bm);
        else if constexpr (!std::is_void<typename Kind::W>::value) gemm_tiles<typename Kind::W, typename Kind::Epi, true>(ga, epi, M, 0, pl.row_hi, pl.sk, walk, pl.bm);
      }
    } else {
      if constexpr (Kind::FUSED) {
        if (pl.xl == PLAN_X) gemm_tiles<typename Kind::X, typename Kind::Epi, false>(ga, epi, M, 0, pl.row_hi, 1, walk, pl.bm);
        else if (pl.xl == PLAN_L) gemm_tiles<typename Kind::L, typename Kind::Epi, false>(ga, epi, M, 0, pl.row_hi, 1, walk, pl.bm);
        else if constexpr (!std::is_void<typename Kind::W>::value) gemm_tiles<typename Kind::W, typename Kind::Epi, false>(ga, epi, M, 0, pl.row_hi, 1, walk, pl.bm);
      }
    }
  }
  if (pl.row_hi < M) Kind::stream(ga, epi, M, pl.row_hi, pl.sk_tail, walk);
}

template <typename Kind> void set_lds_once_planned() {
  static bool done = false;
  if (!done) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_planned<Kind>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, RING_SLOTS * (int)RING_SLOT);
    done = true;
  }
}

template <typename SH, typename Epi, bool SPLIT> void set_lds_once() {
  static bool done = false;
  if (!done) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gemm_bf16<SH, Epi, SPLIT>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)SH::LDS_BYTES);
    done = true;
  }
}

}  // namespace mm
}  // namespace dy
