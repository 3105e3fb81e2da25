// Pieces shared by the partial-attention kernels: the mapping from a workgroup's tile number to
// (sequence, first query row, row count) over ragged per-sequence row lists, and the key-range
// split arithmetic.
#pragma once
#include "common.h"
#include "kernels.h"

namespace dy {

// Upper bound (host) of the number of query tiles: sum_b ceil(n_b / BQ) <= cap/BQ + B.
inline int max_q_tiles(const AttnArgs &a, int BQ) {
  if (!a.offsets) return a.B * ((a.L + BQ - 1) / BQ);
  int t = (a.rows.cap + BQ - 1) / BQ + a.B;
  return t < 1 ? 1 : t;
}

// Keys per split, a multiple of the key tile BK.
__host__ __device__ inline int split_chunk(int L, int splits, int BK) {
  int c = (L + splits - 1) / splits;
  return ((c + BK - 1) / BK) * BK;
}

// Tile number -> info[0] = sequence (or -1 if the tile does not exist), info[1] = index of its
// first query row in the row list, info[2] = rows in the tile.  Called by one thread.
__device__ inline void find_tile(const AttnArgs &a, int BQ, int tile, int *info) {
  info[0] = -1;
  info[1] = 0;
  info[2] = 0;
  if (!a.offsets) {
    const int per = (a.L + BQ - 1) / BQ;
    const int b = tile / per, t = tile % per;
    if (b < a.B) {
      info[0] = b;
      info[1] = b * a.L + t * BQ;
      info[2] = min(BQ, a.L - t * BQ);
    }
    return;
  }
  const int total = min(a.offsets[a.B], a.rows.cap);
  int t = tile;
  for (int b = 0; b < a.B; ++b) {
    const int lo = min(a.offsets[b], total), hi = min(a.offsets[b + 1], total);
    const int nt = (hi - lo + BQ - 1) / BQ;
    if (t < nt) {
      info[0] = b;
      info[1] = lo + t * BQ;
      info[2] = min(BQ, hi - lo - t * BQ);
      return;
    }
    t -= nt;
  }
}

// Work item of a workgroup of a 1-D launch over (key split, KV head, query tile, query head of the
// group).  Workgroup p runs on XCD p % 8, and an XCD takes its workgroups in the order of p: every
// XCD gets one contiguous range of the items in the order above, so all query tiles and all query
// heads that read the keys and values of one (sequence, KV head) run on ONE XCD, next to each other
// in time, and that K/V stream crosses the fabric once instead of once per tile and head.
constexpr int ATTN_XCD = 8;
inline int attn_grid(const AttnArgs &a, int q_tiles) {
  const long items = (long)q_tiles * a.H * a.splits;
  return (int)((items + ATTN_XCD - 1) / ATTN_XCD) * ATTN_XCD;
}
// returns false when the workgroup has no item
__device__ __forceinline__ bool attn_work_item(const AttnArgs &a, int q_tiles, int *tile, int *h, int *split) {
  const int items = q_tiles * a.H * a.splits;
  const int per_xcd = (items + ATTN_XCD - 1) / ATTN_XCD;
  const int p = blockIdx.x;
  const int w = (p % ATTN_XCD) * per_xcd + p / ATTN_XCD;
  if (p / ATTN_XCD >= per_xcd || w >= items) return false;
  const int g = a.H / a.Hkv;
  const int gi = w % g;
  int rest = w / g;
  *tile = rest % q_tiles;
  rest /= q_tiles;
  *h = (rest % a.Hkv) * g + gi;
  *split = rest / a.Hkv;
  return true;
}

// ---- grouped form (head_dim 128 kernel): the g = H / Hkv query heads that share a KV head are
// folded into the query rows of a tile.  Per sequence and KV head the "packed rows" are the pairs
// (row of the list, head of the group), numbered p = row * g + head: a tile is BQ consecutive
// packed rows, so a workgroup streams the keys and values of its KV head once for up to BQ
// (row, head) pairs instead of once per head, and ragged row counts leave g times fewer idle waves.
// With g = 1 this is the plain form above.
inline int max_q_tiles_grouped(const AttnArgs &a, int BQ) {
  const int g = a.H / a.Hkv;
  if (!a.offsets) return a.B * ((a.L * g + BQ - 1) / BQ);
  const long t = ((long)a.rows.cap * g + BQ - 1) / BQ + a.B;
  return t < 1 ? 1 : (int)t;
}
inline int attn_grid_grouped(const AttnArgs &a, int q_tiles) {
  const long items = (long)q_tiles * a.Hkv * a.splits;
  return (int)((items + ATTN_XCD - 1) / ATTN_XCD) * ATTN_XCD;
}
// inclusive sum over the lanes of a wave (vector-register moves only)
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8: sums inside rows of 16
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // last lane of row 0 / 2 -> row 1 / 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // last lane of row 1 -> rows 2 and 3
  return x;
}
// Work item of a workgroup: sequence (or -1: no item), index of its first row in the row list, first packed row of the tile,
// packed rows in it, whether the tile is its sequence's only one.
struct AttnItem { int seq = -1, row = 0, packed = 0, n = 0, only = 0, kv_head = 0, split = 0; };
// The item of workgroup p of a 1-D launch over (key split, KV head, tile of packed rows), XCD-aware as above.  Called by every wave with
// all its lanes; the results are uniform.  The items are those of the tiles that exist, not of the q_tiles that the list's capacity allows: each XCD takes
// an equal share of them, and they come before all workgroups without work.  (Numbered by the capacity, a list of 330
// entries with room for 8192 had its 256 items in four groups per XCD behind 64 idle workgroups each: 43 us instead of 35
// for 8 sequences of 1024 tokens, 32 heads.)
// A lane counts the tiles of one sequence (64 at a time): one round of loads, where a walk over the sequences waits for each
// of them in turn.
__device__ __forceinline__ AttnItem attn_work_item_grouped(const AttnArgs &a, int BQ, int q_tiles, int p) {
  const int g = a.H / a.Hkv, lane = threadIdx.x % WAVE;
  AttnItem it;
  int total = 0, lo = 0, hi = 0, upto = 0, tiles = q_tiles;
  auto tiles_of = [&](int b0) {  // rows [lo, hi) of this lane's sequence, and the tiles up to and with it
    const int b = b0 + lane;
    lo = hi = 0;
    if (b < a.B) {
      lo = min(a.offsets[b], total);
      hi = min(a.offsets[b + 1], total);
    }
    upto = wave_scan(((hi - lo) * g + BQ - 1) / BQ);
    return __builtin_amdgcn_readlane(upto, WAVE - 1);
  };
  if (a.offsets) {
    total = min(a.offsets[a.B], a.rows.cap);
    tiles = 0;
    for (int b0 = 0; b0 < a.B; b0 += WAVE) tiles += tiles_of(b0);
  }
  const int items = tiles * a.Hkv * a.splits, per_xcd = (items + ATTN_XCD - 1) / ATTN_XCD;
  const int w = (p % ATTN_XCD) * per_xcd + p / ATTN_XCD;
  if (p / ATTN_XCD >= per_xcd || w >= items) return it;
  int t = w % tiles;
  const int rest = w / tiles;
  it.kv_head = rest % a.Hkv;
  it.split = rest / a.Hkv;
  if (!a.offsets) {
    const int per = (a.L * g + BQ - 1) / BQ, b = t / per;
    it.seq = b;
    it.row = b * a.L;
    it.packed = (t % per) * BQ;
    it.n = min(BQ, a.L * g - it.packed);
    it.only = per == 1;
    return it;
  }
  for (int b0 = 0; b0 < a.B; b0 += WAVE) {
    if (a.B > WAVE) tiles_of(b0);  // (else still in the registers)
    const uint64_t past = __ballot(upto > t);  // the sequences at or after the tile's
    if (past) {
      const int s = __ffsll((unsigned long long)past) - 1;
      const int n = __builtin_amdgcn_readlane((hi - lo) * g, s);
      const int first = t - (__builtin_amdgcn_readlane(upto, s) - (n + BQ - 1) / BQ);
      it.seq = b0 + s;
      it.row = __builtin_amdgcn_readlane(lo, s);
      it.packed = first * BQ;
      it.n = min(BQ, n - first * BQ);
      it.only = n <= BQ;
      return it;
    }
    t -= __builtin_amdgcn_readlane(upto, WAVE - 1);
  }
  return it;
}

void launch_attention_f32(const AttnArgs &a, hipStream_t s);
void launch_attention_bf16(const AttnArgs &a, hipStream_t s);
void launch_attn_combine(DType t, const AttnArgs &a, hipStream_t s);

}  // namespace dy
