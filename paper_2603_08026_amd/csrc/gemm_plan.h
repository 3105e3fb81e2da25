// Launch plans of the bf16 GEMMs in row tiles, made from the number of rows that EXIST.
//
// The row count of a list lives on the device, and a list's capacity says little about it: a generation
// loop carries lists of B*L entries of which a few percent are used.  A plan made from the capacity then
// takes the shapes of a dense step for a few hundred rows (one request batch of 8 x 1024 tokens, 330
// salient rows: 32 tiles of the down projection on 256 CUs, 201 us against 55 us with a K split; two layers and four
// steps of that loop 4080 -> 2424 us).
// So plans are made on the device once the count is there: every candidate is priced by one lane of
// a workgroup, the cheapest wins, and the row kernels that follow read the chosen split back from words
// of device memory.  A workgroup of the row kernel ahead of the GEMM does that beside its rows (PlanJob, kernels.h); where there is
// none that knows the count (the out-projection, behind the compaction) every workgroup of the GEMM does it for itself, which takes 1.7 us
// before its first copy.  Where the host knows the count (dense steps) it evaluates the same functions and
// passes the plan in.
//
// Two sets of candidates.  The first has tiles of 256 rows (plan_price).  The second has tiles of any height
// that is a multiple of 32 (64) rows, and tiles of 192 columns (tile_price): rows divided evenly over their tiles
// leave no thin last one, and 256 CUs are filled by what divides the matrix into about as many pieces -- 330 rows
// are 256 tiles of 192 x 192, not 192 tiles of 256 x 256 of which half hold 74 rows.
#pragma once
#include <type_traits>
#include "common.h"

namespace dy {
namespace mm {

// A plan: rows [0, row_hi) of the list in tiles of bm rows (xl: 1: 256 columns wide, 2: 192, 0: 128) with sk K splits;
// the rows from row_hi on in 128-row weight-streaming tiles with sk_tail K splits.
struct GemmPlan { int xl, sk, row_hi, sk_tail, bm; };
constexpr int PLAN_L = 0, PLAN_X = 1, PLAN_W = 2;  // GemmPlan::xl

// What plans are made from.  N output columns, K; and for the kind of GEMM:
//   tiles_l / _x / _w  column tiles of 128 / 256 / 192 columns; tiles_x, tiles_w = 0: they do not divide N
//   w_cols             weight rows per output column (2 for gate|up)
//   stream_cols        columns of the weight-streaming tiles; 0: not to be used
//   split_ok           K splits (and a streamed tail that is split) may be used: a row kernel sums them
//   split_free         a row kernel follows whatever the split (q|k|v, out-projection); otherwise a split or a streamed
//                      tail costs a sum kernel.  The prices charge an unsplit result's way through memory, also where
//                      q|k|v rows leave the GEMM finished (their fit and takes_over's shares are older than that)
//   part_elems         fp32 elements of the buffer of raw results
//   cus, inv_cus       CUs of an XCD
//   stream_us          price of a streamed last row tile
//   sum_us             what a sum kernel costs that would not be launched without a split (down projection with a plan
//                      made on the host)
struct PlanArgs {
  int N, K, tiles_l, tiles_x, w_cols, stream_cols, split_ok, split_free, tiles_w;
  long part_elems;
  float cus, inv_cus, stream_us, sum_us;
};

constexpr int PLAN_BK = 64, PLAN_XCD = 8;
constexpr int STREAM_ROWS = 128;     // rows that one weight-streaming tile holds
constexpr int PLAN_MIN_SLICES = 8;   // K slices every split keeps (the ring loop needs 3)
constexpr int PLAN_MAX_SPLIT = 16;
constexpr int PLAN_CANDIDATES = 4 * PLAN_MAX_SPLIT;  // {128, 256 columns} x {last row tile padded, streamed} x splits

// K splits of the weight-streaming tiles: about one workgroup per CU
__host__ __device__ inline int stream_split(const PlanArgs &a, int M) {
  const int tiles = a.N / a.stream_cols;
  int s = 1;
  while (tiles * s < 192 && s < 8 && (a.K / PLAN_BK) / (s * 2) >= 4) s *= 2;
  while (s > 1 && (long)s * M * a.N > a.part_elems) s /= 2;
  return a.split_ok ? s : 1;
}

// Whether sk K splits may be taken at all (fewer may then as well)
__host__ __device__ inline bool can_split(const PlanArgs &a, int M, int sk) {
  return sk == 1 || (a.split_ok && a.K / PLAN_BK >= PLAN_MIN_SLICES * sk && (long)sk * M * a.N <= a.part_elems);
}
__host__ __device__ inline bool can_stream(const PlanArgs &a, int M) {
  return a.stream_cols && M % 256 > 0 && M % 256 <= STREAM_ROWS && M >= 256;
}

// Price of candidate c in microseconds, or a huge value if it cannot be taken.  The constants are
// fitted to measured times of seven GEMMs of two layer shapes (hidden 4096 and 3584).  Every candidate was then timed
// for 23 GEMMs of six layer shapes (hidden 256 to 4096) at 14 row counts from 140 to 5000: the candidate with the least
// price is on average 0.25 % slower than the fastest one, at worst 11 % (322 points, weights of up to 16 copies in
// turn).  What they say:
//   - a CU takes 51 us for the K loop of a 256 x 128 tile over K = 4096 and 1.31 times that for a
//     256 x 256 one, and 6.9 or 13.8 us per tile for what surrounds the loop;
//   - an XCD's CUs take its positions of the tile order in turn (gemm_tiles): full tiles first, then the
//     tiles of a last row tile with fewer than 256 rows, which cost a fraction of a full one (they
//     still walk all of K with their copies) and first fill the slots the full tiles leave;
//   - weights arrive at 4 TB/s whatever the tiles do; in the streaming tiles as with_stream_price says;
//   - every K split moves its fp32 sums once more, written and read.
__host__ __device__ inline float plan_price(const PlanArgs &a, int M, int c) {
  const int sk = c % PLAN_MAX_SPLIT + 1, xl = (c / PLAN_MAX_SPLIT) & 1, streamed = c / (2 * PLAN_MAX_SPLIT);
  const int tail = M % 256;
  const bool ok = (!xl || a.tiles_x != 0) && can_split(a, M, sk) && (!streamed || can_stream(a, M));
  const int tiles = (xl ? a.tiles_x : a.tiles_l) * sk;
  const int full = (M / 256 * tiles + PLAN_XCD - 1) / PLAN_XCD, part = (tail && !streamed) ? (tiles + PLAN_XCD - 1) / PLAN_XCD : 0;
  // (counts are whole numbers far below 2^20: the products with the reciprocal round to the right side)
  const float rounds = ceilf((float)full * a.inv_cus - 1e-4f), slack = rounds * a.cus - (float)full;
  const float more = fmaxf(ceilf(((float)part - slack) * a.inv_cus - 1e-4f), 0.f);  // rounds of partial tiles alone
  const float f = fminf(fmaxf(0.31f + 0.125f * (float)((tail + 31) / 32), 0.385f), 1.0f);
  const float per_split = 1.0f / (float)sk;
  const float loop = 51.3f / 4096.0f * (float)a.K * (xl ? 1.31f : 1.0f) * per_split;
  const float w_bytes = (float)a.N * (float)a.w_cols * (float)a.K * 2.0f;
  float t = fmaxf((rounds + f * more) * loop + (rounds + more) * (xl ? 13.8f : 6.9f), w_bytes * (1.0f / 4.04e6f));
  const float sums = 1.29e-6f * (float)M * (float)a.N;
  if (a.split_free) t += sums * (float)(sk - 1);
  else if (a.split_ok && (sk > 1 || streamed)) t += sums * (float)sk + 4.0f;
  if (streamed) t += a.stream_us;
  return ok ? t : 3e30f;
}

__host__ __device__ inline GemmPlan plan_of(const PlanArgs &a, int M, int c) {
  const int streamed = c / (2 * PLAN_MAX_SPLIT);
  return GemmPlan{(c / PLAN_MAX_SPLIT) & 1, c % PLAN_MAX_SPLIT + 1, streamed ? M - M % 256 : M, streamed ? stream_split(a, M) : 1, 256};
}

// Tiles of one shape, `mi` units of 32 (192 columns: 64) rows high: whole row tiles, rows of the last one, and what a tile
// (a whole one, the last one) costs per K slice and beside its slices.  The same for every number of K splits.
struct TileHeight { int cols, full, tail; float slice, fixed, tail_slice, tail_fixed; };
__host__ __device__ inline TileHeight tile_height(const PlanArgs &a, int M, int shape, int mi) {
  const bool l = shape == PLAN_L, x = shape == PLAN_X;
  const int cols = l ? a.tiles_l : x ? a.tiles_x : a.tiles_w, unit = l || x ? 32 : 64, bm = mi * unit;
  const int full = M / bm, tail = M - full * bm;
  auto slice = [&](float m) -> float {
    return l ? 0.261f + 0.0488f * m : x ? fmaxf(0.532f + 0.0557f * m, 0.287f + 0.1124f * m) : fmaxf(0.429f + 0.104f * m, 0.196f + 0.195f * m);
  };
  auto fixed = [&](float m) -> float { return l ? 1.96f + 0.50f * m : x ? 1.48f + 0.80f * m : 2.45f + 0.94f * m; };
  const float m = (float)mi, t = (float)((tail + unit - 1) / unit);
  return TileHeight{bm <= 256 ? cols : 0, full, tail, slice(m), fixed(m), slice(t), fixed(t)};
}

// The weights' stream, and a price with what its raw results and sums add (M rows, sk splits)
__host__ __device__ inline float weights_us(const PlanArgs &a) {
  return (float)a.N * (float)a.w_cols * (float)a.K * 2.0f * (1.0f / 4.03e6f);
}
__host__ __device__ inline float with_sums(const PlanArgs &a, int M, int sk, float us) {
  const float mn = 1e-6f * (float)M * (float)a.N;
  if (a.split_free || sk > 1) us += 0.384f * mn * (float)sk;
  else if (a.w_cols == 1) us *= 1.08f;  // (the down projection's own epilogue: residual and scatter)
  if (a.split_free) us += 1.58f * mn * (float)(sk - 1);
  else if (sk > 1) us += 1.58f * mn * (float)sk + a.sum_us;
  return us;
}

// Price in microseconds of M rows in tiles of a height h with sk K splits, or a huge value.
// Fitted to 8287 times: 16 GEMMs of four layer shapes (hidden 512 to 4096) at 18 row counts from 140 to 5000, every
// shape, height and up to ten splits, weights of up to 16 copies in turn.  The candidate with the least price is on
// average 1.0 % slower than the fastest of all (worst 18 %); the least time itself is 2 to 34 % below that of the best
// 256-row tiles.
//   - a K slice costs a fixed part (waits, the weight copies) and one per unit of rows; from five (three) units on
//     256 (192) columns are bound by their products
//   - tiles at the same time slow each other down: a chip that is half empty is 11 % faster per tile
//   - the weights' stream and the tiles' own time overlap, not entirely; a raw result is written at 10 TB/s beside it
__host__ __device__ inline float tile_price(const PlanArgs &a, int M, const TileHeight &h, int sk) {
  const bool ok = h.cols != 0 && can_split(a, M, sk);
  const float fx = (float)((h.full * h.cols * sk + PLAN_XCD - 1) / PLAN_XCD), px = h.tail ? (float)((h.cols * sk + PLAN_XCD - 1) / PLAN_XCD) : 0.0f;
  const float rounds = ceilf(fx * a.inv_cus - 1e-4f), more = fmaxf(ceilf((px - (rounds * a.cus - fx)) * a.inv_cus - 1e-4f), 0.0f);
  const float slices = (float)a.K * (1.0f / PLAN_BK) / (float)sk;
  const float empty = 1.0f - fminf((fx + px) * a.inv_cus / fmaxf(rounds + more, 1.0f), 1.0f);
  const float t = (rounds * (slices * h.slice + h.fixed) + more * (slices * h.tail_slice + h.tail_fixed)) * (1.0f - 0.22f * empty);
  const float w = weights_us(a), hi = fmaxf(t, w), lo = fminf(t, w);
  const float us = 1.8f + hi + 0.26f * lo * (lo / hi) * (lo / hi);
  return ok ? with_sums(a, M, sk, us) : 3e30f;
}

// Candidate c of the second set for one shape: heights of 1 to 8 units x 8 splits
constexpr int TILE_CANDIDATES = 64;
__host__ __device__ inline int tile_split(int c) {  // 1 2 3 4 5 6 8 12
  const int i = c % 8;
  return i < 6 ? i + 1 : i == 6 ? 8 : 12;
}
__host__ __device__ inline int tile_units(int c) { return c / 8 + 1; }

// The first set's choice in tiles of the best height, height h (units - 1)
__host__ __device__ inline float first_price(const PlanArgs &a, const GemmPlan &p, int M, int h) {
  const float us = tile_price(a, p.row_hi, tile_height(a, p.row_hi, p.xl, h + 1), p.sk);
  return p.row_hi < M ? us + a.stream_us : us;
}
// Whether a candidate of the second set, with sk splits, takes the place of the first set's choice p: by how much it has
// to be cheaper.  The prices' error is 8 % (rms), most of it between different numbers of splits: the sums of many results
// are priced too high, those of few too low.  Both choices of every GEMM were timed in a step's projections and FFN half, the
// sum kernels included: 31 row counts from 140 to 2300, eight layer shapes of hidden 512 to 4096, 567 pairs that differ.
//   - equal splits, and gate|up, which has none: 0.97 up to 1024 rows, 0.95 beyond (0.85 against a streamed last row tile):
//     gains 301 us in all and loses at most 2 in one place
//   - the down projection, whose splits cost a sum kernel: 0.85 gains 278 us and loses 10; 0.90 would lose 132
//   - q|k|v, out-projection: below 2.5e6 results a split less is a gain nearly wherever the price says so; with more of
//     them 0.88 up to 1024 rows; beyond, 0.78 where a row has no more results than K (the out-projection, whose row kernel
//     adds the splits of a row at little cost) and there are at most 7e6, 0.85 for q|k|v, against a streamed last row tile
//     and for more results: gains 605 us, loses 45, at most 5 in one place.  0.97 up to 1024 rows and 0.85 beyond gained 501
//     and lost 141 (step of 256 rows at hidden 4096, q|k|v in one split against two, 186 against 181 us; 960 rows, the
//     out-projection likewise, 5 us).  Out-projection and FFN half with 0.85 / 0.78, us: hidden 4096, 1470 rows 436.2 / 433.0, 1610
//     475.1 / 470.2, 2000 541.7 / 542.1 (the whole step 846.8 / 849.7); hidden 5120, 3670 rows 1443 / 1460, 3940 1480 / 1509;
//     hidden 6144, 2770 rows 1535 / 1548, 4030 2031 / 2058: the results of two splits are more memory traffic there than
//     one split's idle CUs are time.
__host__ __device__ inline bool takes_over(const PlanArgs &a, int M, const GemmPlan &p, float first, int sk, float second) {
  const bool same = p.row_hi == M && sk == p.sk, down = a.split_ok && !a.split_free;
  float share = M <= 1024 && !down ? 0.97f : same ? 0.95f : 0.85f;
  const float results = (float)M * (float)a.N;
  if (a.split_free && !same) share = results < 2.5e6f ? 0.98f : M <= 1024 ? 0.88f : p.row_hi < M || a.N > a.K || results > 7e6f ? 0.85f : 0.78f;
  return second < share * first;
}

// The first set's choice on the host: candidate number
inline int first_on_host(const PlanArgs &a, int M) {
  int best = 0;
  float best_t = 1e30f;
  for (int shape = 0; shape < (can_stream(a, M) ? 4 : 2); ++shape)
    for (int sk = 1; sk <= PLAN_MAX_SPLIT && can_split(a, M, sk); ++sk) {
      const int c = shape * PLAN_MAX_SPLIT + sk - 1;
      const float t = plan_price(a, M, c);
      if (t < best_t) { best_t = t; best = c; }
    }
  return best;
}
inline GemmPlan plan_on_host(const PlanArgs &a, int M) {
  if (M <= STREAM_ROWS && a.stream_cols) return GemmPlan{0, 1, 0, stream_split(a, M), 256};
  GemmPlan p = plan_of(a, M, first_on_host(a, M));
  float first = 2e30f;
  for (int h = 0; h < 8; ++h) {
    const float t = first_price(a, p, M, h);
    if (t < first) { first = t; p.bm = 32 * (h + 1); }
  }
  // The second set's least price, of those below the first one's (only these can take over).  No price is below the weights'
  // stream with its sums: with that, heights priced once for all splits and nothing priced that cannot be taken, a step's four
  // plans take 4 (hidden 512) to 6 us (4096) of host time instead of 18.
  GemmPlan q = p;
  float best_t = first;
  const float least = 1.8f + weights_us(a);
  for (int shape = 0; shape < 3; ++shape) {
    if (shape == PLAN_X ? !a.tiles_x : shape == PLAN_W && !a.tiles_w) continue;
    const int unit = shape == PLAN_W ? 64 : 32;
    // (heights that no row needs cost what the lowest height with one row tile costs)
    for (int mi = 1; mi * unit <= 256 && (mi - 1) * unit < M; ++mi) {
      const TileHeight h = tile_height(a, M, shape, mi);
      for (int i = 0; i < 8 && can_split(a, M, tile_split(i)); ++i) {
        const int sk = tile_split(i);
        if (with_sums(a, M, sk, least) >= best_t) {
          if (sk > 1) break;  // (more splits have more sums)
          continue;
        }
        const float t = tile_price(a, M, h, sk);
        if (t < best_t) { best_t = t; q = GemmPlan{shape, sk, M, 1, mi * unit}; }
      }
    }
  }
  return takes_over(a, M, p, first, q.sk, best_t) ? q : p;
}

// What the launchers of the three kinds of GEMM make their plans from.  ring: the ring loop's shapes can be taken
// (ring_ok); part_elems: elements of the buffer of raw results; cus: CUs of an XCD
// w_ok: the kind has tiles of 192 columns
inline PlanArgs plan_args(int N, int K, int bn_l, bool wide_ok, int cus, bool w_ok) {
  const int bn_w = bn_l / 2 * 3;
  return PlanArgs{N, K, N / bn_l, wide_ok && N % (2 * bn_l) == 0 ? N / (2 * bn_l) : 0, 1, 0, 0, 0, wide_ok && w_ok && N % bn_w == 0 ? N / bn_w : 0, 0,
                  (float)cus, 1.0f / (float)cus, 0.0f, 0.0f};
}
// The streaming tiles read the weights once, at 5.3 TB/s together and at most 34.5 GB/s each (gate|up has no K
// split: with 88 tiles of 5632 columns over K = 2048 a streamed last row tile takes 18 us, not the 11 of the rate of
// all CUs)
inline PlanArgs with_stream_price(PlanArgs a) {
  if (!a.stream_cols) return a;
  const float w_bytes = (float)a.N * (float)a.w_cols * (float)a.K * 2.0f, tiles = (float)(a.N / a.stream_cols * stream_split(a, 1));
  a.stream_us = 2.3f + fmaxf(w_bytes * (1.0f / 5.26e6f), w_bytes / tiles * (1.0f / 34.5e3f));
  return a;
}
// q|k|v, out-projection: fp32 result, a row kernel follows
inline PlanArgs raw_plan_args(int N, int K, size_t part_elems, bool ring, int cus) {
  PlanArgs a = plan_args(N, K, 128, ring, cus, true);
  a.stream_cols = N % 96 == 0 ? 96 : 64;
  a.split_ok = a.split_free = 1;
  a.part_elems = (long)part_elems;
  return with_stream_price(a);
}
// gate|up: SwiGLU in the epilogue
inline PlanArgs swiglu_plan_args(int N, int K, int cus) {
  PlanArgs a = plan_args(N, K, 64, true, cus, true);
  a.w_cols = 2;
  a.stream_cols = N % 48 == 0 ? 48 : N % 64 == 0 ? 64 : 0;
  return with_stream_price(a);
}
// down projection: residual and scatter in the epilogue, or fp32 sums of a K split
inline PlanArgs down_plan_args(int N, int K, size_t part_elems, bool ring, int cus) {
  PlanArgs a = plan_args(N, K, 128, ring, cus, false);
  a.stream_cols = 64;
  a.split_ok = 1;
  a.part_elems = (long)part_elems;
  return with_stream_price(a);
}
// Is the plan made on the host?  When the count is known here; and for a list of up to 256 entries, one row
// tile whatever its count: the same shapes serve, and most steps lose by the device's plan.  Steps of one layer, lists of 256
// entries, full / half full / 20 rows, us, planned here | on the device (ahead, in row kernels): 28 over 4 heads 205 / 176 / 142 |
// 209 / 188 / 158; hidden 1024 68 / 62 / 54 | 73 / 72 / 64; hidden 4096 192 / 176 / 142 | 195 / 156 / 136, where few rows in much room gain;
// 140 entries 159 / 154 / 136 | 163 / 176 / 157, 60 / 57 / 53 | 67 / 69 / 64, 161 / 152 / 137 | 164 / 145 / 135.
inline bool plan_known(bool count_on_device, int cap) { return !count_on_device || cap <= 256; }
// What the rows of a GEMM go through: nothing, weight-streaming tiles alone (streams: up to 128 rows, where the shape has such tiles), row tiles
// of the ring loop by a plan, or the eight-wave shapes, which need neither
enum class Way { NONE, STREAM, TILES, EIGHT };
inline Way way_of(int cap, bool streams, bool ring) {
  return cap <= 0 ? Way::NONE : streams && cap <= STREAM_ROWS ? Way::STREAM : ring ? Way::TILES : Way::EIGHT;
}
// Is a plan to be made on the device?  The launcher of a GEMM and what has its plan made ahead both ask here.
inline bool wants_plan(Way way, bool count_on_device, int cap) { return way == Way::TILES && !plan_known(count_on_device, cap); }
// The way of a GEMM whose kernel cannot make its plan: without one (made) the rows take the shapes that need none
inline Way way_with(Way way, bool count_on_device, int cap, bool made) { return wants_plan(way, count_on_device, cap) && !made ? Way::EIGHT : way; }
// Does the down projection get a sum kernel behind it, and so a plan that may split K or stream a last row tile?
// Always where the plan for the full length wants it.  Where the device may find fewer rows, also if the list is long
// (SUM_CAP) or K is: a few rows without a split take the whole K loop of one row tile, against the sum kernel's
// launch of about 4 us where it then finds nothing to do.  The line is at ten such launches (K = 3200 and longer).
// FFN half at hidden 4096, FFN 12288, lists of 3000 without / with the sum kernel: 40 rows 215 / 92 us, 330 rows
// 274 / 172 us; a full list of 2600 777 / 783 us.  At hidden 1024, FFN 1664, 330 rows would gain 6 us and a full list
// lose 4 of 86.
constexpr int SUM_CAP = 4096;
constexpr float SUM_LOOP_US = 40.0f;
inline float loop_us(int K) { return 51.3f / 4096.0f * (float)K; }  // K loop of a 256 x 128 tile (plan_price)
inline bool down_has_sums(const PlanArgs &a, int cap, bool known) {
  const GemmPlan full = plan_of(a, cap, first_on_host(a, cap));
  return full.sk > 1 || full.row_hi < cap || (!known && (cap > SUM_CAP || loop_us(a.K) >= SUM_LOOP_US));
}

// Two kernels make raw results in row tiles: one that can finish q|k|v rows where K is not split, and one that knows nothing else and is
// a third as long.  Few rows pay for a long kernel with instructions that the caches no longer hold, so the first is taken only where
// it has rows to finish: where the plan of a full list (full) does not split K, and unless the list is a carried one.
//   - known rows whose K is split, us with the short kernel / the long one: response windows of 768 and 1024 rows in a loop of hidden
//     4096 1891 / 1914 and 2249 / 2273, dense 560 rows of 28 over 4 heads 317 / 321; from 1150 to 4000 rows equal
//   - lists whose K is split even when they are full: 307 rows of hidden 4096 240.6 / 243.2, 360 of 28 over 4 heads 273.9 / 274.7
//   - a list with room for more than half of the tokens (few_of_room) is a carried one, which holds a few percent of them: K is
//     then split on the device.  4 % of 8 x 1024 tokens: step 248 / 252, loop 1961 / 1993.  With more of them the long kernel
//     would finish rows: 10 and 25 % of 16 x 1280 tokens 802 / 782 and 1878 / 1805, which the host cannot know.
//   - few results of a list planned on the device: the row kernel is launched all the same and had little to do.  Steps, q|k|v columns x
//     rows: 768 x 310 / 740 / 990 / 1230 / 3080 77.4 / 81.0, 92.9 / 94.9, 99.2 / 100.6, 125.7 / 125.2, 191.8 / 189.8; 1536 x 490 / 990 /
//     1540 78.6 / 80.3, 102.3 / 101.0, 101.6 / 99.4; 3072 x 370 / 620 / 1080 / 1540 92.3 / 93.5, 104.4 / 104.8, 116.1 / 117.0, 137.9 /
//     137.2 (hidden 2048: 1080 rows 186.0 / 189.2); 4608 x 720 / 1030 / 1340 400.7 / 402.9, 521.7 / 527.0, 670.6 / 667.1; but 6144 x
//     310 / 650 / 1000 133.8 / 132.6, 169.0 / 167.2, 211.2 / 209.6; 12288 x 570 / 970 398 / 393, 513 / 504
// Known rows lose nothing there, since their row kernel is not launched (768 columns x 140 rows 55.3 / 54.5).
// The out-projection and other raw results of a layer take the same of the two kernels, which then follow each other closely enough for
// their instructions to be in the caches (16 x 1280 tokens, 2064 rows, out-projection in the short one: 837 -> 845) - with heads of
// 128 columns: the long kernel for heads of 64 is another one, and raw results beside it take the short kernel (hidden 512,
// short / long: 140 rows 54.5 / 55.9, 1230 rows 120.1 / 121.6, dense 3072 rows 95.1 / 96.8; hidden 1024 and 2048 equal to 0.8 % faster).
constexpr int FINISH_ROWS = 1100, FINISH_COLS = 6144;
inline bool few_of_room(bool count_on_device, int cap, size_t tokens) { return count_on_device && (size_t)cap * 2 > tokens; }
inline bool few_results(bool known, int cap, int qkv_cols) { return !known && cap < FINISH_ROWS && qkv_cols < FINISH_COLS; }
inline bool finishing_kernel(bool few, const GemmPlan &full) { return !few && full.sk == 1; }

// Matrices of 16 MiB and more go past the L2 where one workgroup alone reads a weight.  The caches keep a layer of smaller ones until the
// next step, and its kernels do without the loops for it, which make them longer for all rows.  Steps with three layers' weights in
// turn, us, past the L2 / through it: hidden 1024 (layer of 25 MB, largest matrix 11 MB) 100 rows 70.2 / 68.4, 112 rows 68.9 / 66.0, 232
// rows 69.2 / 67.5; hidden 2048 (100 MB, matrices of 22, 25 and 45 MB) 20 rows 76.8 / 80.7, 100 rows 93.0 / 96.9, 140 rows
// 94.0 / 96.4; 28 over 4 heads (466 MB) 100 rows 180.6 / 188.6.  (One layer of hidden 2048 called again and again, as no
// model does, finds its weights in the last-level cache: 100 rows 93.0 / 87.6.)
inline bool past_l2(int n_rows_w, int K) { return (size_t)n_rows_w * (size_t)K * 2 >= ((size_t)16 << 20); }

// The ring loop's weight copies have one lane offset for all of a tile: the rows they gather lie in one group of
// RING_GROUP weight rows, and so must lie in one matrix.  (Ends of the stacked matrices; every head size the library
// accepts is a multiple of 64.)
constexpr int RING_GROUP = 64;
inline bool ring_groups_ok(int end0, int end1) { return end0 % RING_GROUP == 0 && end1 % RING_GROUP == 0; }

// Least of a positive price over the 64 lanes of a wave, with its lane in the low six bits (positive floats order like
// their bits); the result is uniform
__device__ __forceinline__ uint32_t least_of_wave(float price, int lane) {
  uint32_t k = (__float_as_uint(price) & ~63u) | (uint32_t)lane;
  auto dpp = [](uint32_t v, auto ctrl) -> uint32_t {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, decltype(ctrl)::value, 0xf, 0xf, false);
  };
  k = min(k, dpp(k, std::integral_constant<int, 0xb1>{}));   // quad_perm 1,0,3,2
  k = min(k, dpp(k, std::integral_constant<int, 0x4e>{}));   // quad_perm 2,3,0,1
  k = min(k, dpp(k, std::integral_constant<int, 0x141>{}));  // row_half_mirror
  k = min(k, dpp(k, std::integral_constant<int, 0x140>{}));  // row_mirror: every lane has its row's least
  const uint32_t r0 = __builtin_amdgcn_readlane(k, 0), r1 = __builtin_amdgcn_readlane(k, 16),
                 r2 = __builtin_amdgcn_readlane(k, 32), r3 = __builtin_amdgcn_readlane(k, 48);
  return min(min(r0, r1), min(r2, r3));
}

// A workgroup of four waves (all lanes active): wave 0 prices the first set, waves 1 to 3 a shape of the second each.
// words: eight words of LDS that nothing else uses yet (the caller's barrier before their reuse).  The result is uniform.
__device__ __forceinline__ GemmPlan plan_on_device(const PlanArgs &a, int M, int wave, uint32_t *words) {
  static_assert(PLAN_CANDIDATES == WAVE && TILE_CANDIDATES == WAVE, "a candidate per lane");
  if (M <= STREAM_ROWS && a.stream_cols) return GemmPlan{0, 1, 0, stream_split(a, M), 256};
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
  if (wave == 0) {
    const int c = (int)(least_of_wave(plan_price(a, M, lane), lane) & 63u);
    const GemmPlan p = plan_of(a, M, c);
    const uint32_t k = least_of_wave(lane < 8 ? first_price(a, p, M, lane) : 3e30f, lane);
    if (lane == 0) { words[0] = k; words[4] = (uint32_t)c; }
  } else {
    const int shape = wave - 1;
    const uint32_t k = least_of_wave(tile_price(a, M, tile_height(a, M, shape, tile_units(lane)), tile_split(lane)), lane);
    if (lane == 0) words[wave] = k;
  }
  __syncthreads();
  uint32_t w[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) w[i] = __builtin_amdgcn_readfirstlane(words[i]);
  GemmPlan p = plan_of(a, M, (int)w[4]);
  p.bm = 32 * ((int)(w[0] & 63u) + 1);
  int shape = 0;
  if (w[2] < w[1]) shape = 1;
  if (w[3] < w[1 + shape]) shape = 2;
  const uint32_t k = w[1 + shape];
  const int c = (int)(k & 63u);
  if (takes_over(a, M, p, __uint_as_float(w[0] & ~63u), tile_split(c), __uint_as_float(k & ~63u)))
    p = GemmPlan{shape, tile_split(c), M, 1, tile_units(c) * (shape == PLAN_W ? 64 : 32)};
  return p;
}

// Words of a plan in device memory: the first four are those of Splits::dev
enum PlanWord { PW_SK, PW_ROW_HI, PW_SK_TAIL, PW_DONE_TO, PW_XL, PW_BM, PLAN_WORDS = 8 };
// done: the row tiles finish their rows where K is not split
__device__ __forceinline__ void store_plan(const GemmPlan &p, bool done, int32_t *words) {
  words[PW_SK] = p.sk;
  words[PW_ROW_HI] = p.row_hi;
  words[PW_SK_TAIL] = p.sk_tail;
  words[PW_DONE_TO] = done && p.sk == 1 ? p.row_hi : 0;
  words[PW_XL] = p.xl;
  words[PW_BM] = p.bm;
}
__device__ __forceinline__ GemmPlan load_plan(const int32_t *words) {
  auto w = [&](PlanWord i) -> int { return __builtin_amdgcn_readfirstlane(words[i]); };
  return GemmPlan{w(PW_XL), w(PW_SK), w(PW_ROW_HI), w(PW_SK_TAIL), w(PW_BM)};
}

}  // namespace mm
}  // namespace dy
