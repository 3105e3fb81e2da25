// Slice loop of the bf16 GEMM tiles with four waves (one per SIMD; the accumulators in the second register
// file) and 160 KB of LDS as a ring of slices: whole slices where three or more fit (tile_slices), else halves
// of slices in five 32 KB slots (tile_halves).
//
// Why a ring of halves in the 256 x 256 tile.  A K slice of the tile is 64 KB (A tile 32 KB + weight tile 32 KB), and two whole
// slices are all that fit beside nothing else in the 160 KB of LDS.  With two stages, the copies of
// slice kt+2 can only be issued once slice kt has been read out, and must have landed before slice
// kt+1 is read out: the copy path runs empty before every barrier and is asked for a whole slice in a
// burst after it (measured: 64 KB take about 3000 cycles to land that way, with or without matrix
// work, against 2048 cycles of matrix instructions per slice).  Here the halves of a slice take
// slots of their own, in the order A(0) W(0) A(1) W(1) A(2) ..., slot = position % 5.  There is one
// barrier per slice, in its middle: by then a wave has the operands of the whole slice in registers
// (128 of them), so the two slots of slice kt are free; W(kt+2) is copied into one during the second
// half of slice kt and A(kt+3) into the other during the first half of slice kt+1 -- one copy after
// every eighth matrix instruction, all the time -- and the eight newest copies stay in flight across the barrier (s_waitcnt vmcnt(8) and a raw
// s_barrier: __syncthreads would wait for all of them).
//
// The copies are buffer loads with LDS destination: a scalar descriptor per source matrix, a 32-bit
// byte offset per lane that is fixed for the tile, and the K walk as a scalar offset, so a copy costs
// no vector address arithmetic between the matrix instructions (measured against per-lane 64-bit
// addresses: 2150 against 2340 cycles per slice).  Lane offsets are 32 bits: the activation
// descriptor starts at the tile's first row, and the launcher takes these shapes only when a gathered
// activation operand and every weight matrix span less than 4 GiB.
#pragma once
#include <type_traits>
#include "common.h"

namespace dy {
namespace mm {

typedef __attribute__((address_space(3))) void lds_void_t;

// lane i's 16 bytes at (descriptor base + voff + soff) -> LDS[lds_addr + 16 i]; lds_addr and soff
// are wave-uniform.  Completion is tracked by vmcnt, in issue order.  ONCE: of data that is read once: non-temporal (bit 1 of
// the cache policy).
template <bool ONCE = false>
__device__ __forceinline__ void dma16_buf(__amdgpu_buffer_rsrc_t srd, uint32_t voff, uint32_t soff, uint32_t lds_addr) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(srd, (lds_void_t *)(uintptr_t)lds_addr, 16, voff, soff, 0, ONCE ? 2 : 0);
}

// descriptor of a raw byte buffer (no stride, no swizzle, 32-bit data format) that covers `bytes`
// from p; reads past the end return zero instead of faulting
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_srd(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)bytes, 0x00020000);
}

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t uintx4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t uintx2;

// four floats, or two / four floats as bf16, at byte offset `off` of a buffer
__device__ __forceinline__ floatx4 load_buf(__amdgpu_buffer_rsrc_t srd, uint32_t off) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(srd, off, 0, 0));
}
__device__ __forceinline__ void store_buf(floatx4 v, __amdgpu_buffer_rsrc_t srd, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, v), srd, off, 0, 0);
}
__device__ __forceinline__ void store_buf(const float (&v)[2], __amdgpu_buffer_rsrc_t srd, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b32(pack_bf16(v[0], v[1]), srd, off, 0, 0);
}
__device__ __forceinline__ void store_buf(const float (&v)[4], __amdgpu_buffer_rsrc_t srd, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b64(uintx2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])}, srd, off, 0, 0);
}

constexpr uint32_t RING_SLOT = 32768;
constexpr int RING_SLOTS = 5;
constexpr int RING_MIN_SLICES = 3;
constexpr int RING_MAX_WSRC = 6;

// Sources of a wave's copies for one tile:
//   srd_a / va[i]   descriptor and lane offsets of its A copies (8 tile rows each; as many as the tile's height needs)
//   srd_w[d] / vw   the same for its weight copies (8, 6 or 4 for 256, 192 or 128 weight rows): a
//                   copy's 8 rows lie in one weight panel; the descriptor starts at the first of them, so that
//                   one lane offset serves all copies, and with G = 4 also at the first of the next copy's,
//                   which lie two weight rows on
struct RingSrc {
  __amdgpu_buffer_rsrc_t srd_a, srd_w[RING_MAX_WSRC];
  uint32_t va[8], vw;
};

// Matrix instruction and column order.  v_mfma_f32_16x16x32_bf16: element e of lane l's four registers is
// activation row 4 * (l / 16) + e and column l % 16 of its 16 x 16 block.  The weight rows of G blocks (four,
// or two where a wave has two of a matrix) are permuted on their way into LDS so that lane l % 16 of the G
// blocks holds columns G * (l % 16) .. + G - 1 of the 16 G: its results of a row are one store (16 bytes of
// fp32; 8 or 4 of bf16), and those of the 16 lanes fill 256 (128, 64) bytes of the row.  The store path takes
// four lanes at a time, and they have to lie next to each other: with the weights as FIRST operand, where a lane
// holds eight columns but neighbouring lanes different rows, a 16-byte store of a wave took 64 cycles instead
// of 16, and the raw store of a 256 x 128 tile 7700 cycles instead of 3400.
// The 16x16 form does the same products with less power than the 32x32 one, and the matrix clock is power-bound:
// operands in registers, all CUs busy, random values: 1.85 against 1.75 PFLOP/s.
//
// Tile heights.  A tile holds any number of rows up to 16 MI WR (WR wave rows, MI 16-row blocks of each), and everything a
// slice costs follows MI: its A copies, operand reads and products.  The blocks of 16 rows are dealt to the wave rows in
// turn (block i of wave row w holds rows 16 (WR i + w) .. + 15 of the tile), so that every wave of a tile with few rows has
// its share of them.  MI is the same for all waves, chosen per tile (gemm_bf16_dma.h).
//
// The loop for one wave: NMAT x NB column groups of 32, group g = t * NB + j reads weight-tile rows (t * BN + wn0 + 32 j ...).
// Wave grid 2 x 2: four column groups of a wave (a 256-row weight tile: 256 x 256 or 256 x (128+128) outputs) or two (128
// weight rows); wave grid 4 x 1: six groups, all 192 weight rows of the tile.  The halves of a slice fill as much of
// their slots as they need.

// ONCE: all rows are in one row tile, so that every weight is read by one workgroup once (gemm_bf16_dma.h).
template <int NMAT, int NB, int BN, int WR, int MI, bool ONCE = false> struct Ring {
  static constexpr int NCB = NMAT * NB;  // column groups per wave
  static constexpr int NC = 2 * NCB;     // 16-column blocks per wave
  static constexpr int AC = WR * MI / 2;        // activation copies per wave and slice (32 tile rows each)
  static constexpr int NWC = NMAT * BN / 32;    // weight copies per wave and slice
  static constexpr int PS = MI * NC;     // products per K step of 32 = per half slice
  static constexpr int RD = MI + NC;     // operand reads per K step
  // products between two operand reads, and reads at a time where there are fewer products than reads
  static constexpr int RSP = PS / 2 >= 2 * RD ? 2 : 1, RPP = (RD + PS - 1) / PS;
  static_assert((WR == 2 && (NWC == 8 || NWC == 4) && MI <= 8) || (WR == 4 && NWC == 6 && MI <= 4), "tile shapes of the ring");
  static_assert(AC >= 1 && AC <= 8 && PS % AC == 0 && PS % NWC == 0, "copies are spread evenly over the products");
  // 16-column blocks whose columns alternate: row x of a group of 16 G LDS rows holds weight row
  // G (x % 16) + x / 16 of the group, so that lane l16 of the G blocks has columns G l16 .. + G - 1
  static constexpr int G = (2 * NB) % 4 == 0 ? 4 : 2;
  // weight row (from the tile's first column on) in LDS rows (4 i + wave) * 8 of a matrix; the row r8 after it
  // holds weight row weight_row + G r8
  static __device__ __forceinline__ int weight_row(int i, int wave) {
    return G == 4 ? (i / 2) * 64 + (wave & 1) * 32 + (i & 1) * 2 + (wave >> 1) : i * 32 + (wave & 1) * 16 + (wave >> 1);
  }
  static constexpr int ROW = 128, A_STEP = 128, W_STEP = 4096;  // bytes per tile row; K walk per slice

  static constexpr int ND = G == 4 ? NWC / 2 : NWC;  // descriptors
  static_assert(ND <= RING_MAX_WSRC, "descriptors of the weight copies");
  static __device__ __forceinline__ void copy_w(const RingSrc &src, int c, uint32_t kt, uint32_t lds_addr) {
    dma16_buf<ONCE>(src.srd_w[c * ND / NWC], src.vw, kt * W_STEP + (G == 4 && c % 2 ? 2 * ROW : 0), lds_addr);
  }

  static __device__ __forceinline__ int w_row(int c) { return (((c / 2) / NB) * BN + ((c / 2) % NB) * 32 + (c % 2) * 16) * ROW; }
  static __device__ __forceinline__ int nxt(int s, int d) { const int t = s + d; return t >= RING_SLOTS ? t - RING_SLOTS : t; }

  // Whole slices that fit beside each other where a slice is small enough for three of them (0: the ring of half
  // slices).  CPS copies of a wave fill CPS * 4 KB.
  static constexpr int CPS = AC + NWC;
  static __host__ __device__ constexpr int stages_of(int cps) {
    const int n = (int)(RING_SLOTS * RING_SLOT / 4096) / cps;
    return n < 3 ? 0 : n > 5 ? 5 : n;
  }
  static constexpr int STAGES = stages_of(CPS);

  // Fills the ring for a tile of KT slices.  The ring must be free (every wave past the middle barrier of the previous
  // tile's last slice).
  //   half slices: A(0) W(0) A(1) W(1) A(2) into slots 0..4;  whole slices: slice s into stage s, as many as there are
  static __device__ __forceinline__ void fill(const RingSrc &src, uint32_t lds0, int wave, int KT) {
    // (hidden from the optimiser: the copies' LDS addresses are sums of it and a constant, which are otherwise all
    // computed once per kernel and kept, forty of them, at the cost of vector registers for their spills)
    uint32_t lds_w = lds0 + (uint32_t)wave * 1024u;
    asm volatile("" : "+s"(lds_w));
    if constexpr (STAGES > 0) {
      const int n = min(STAGES, KT);
      for (int st = 0; st < n; ++st) {
        const uint32_t to = lds_w + (uint32_t)st * (CPS * 4096u);
#pragma unroll
        for (int i = 0; i < AC; ++i) dma16_buf(src.srd_a, src.va[i], (uint32_t)st * A_STEP, to + i * 4096u);
#pragma unroll
        for (int c = 0; c < NWC; ++c) copy_w(src, c, st, to + (AC + c) * 4096u);
      }
    } else {
#pragma unroll
      for (int h = 0; h < RING_SLOTS; ++h) {
        const int kt = h / 2;
        if (h % 2 == 0) {
#pragma unroll
          for (int i = 0; i < AC; ++i) dma16_buf(src.srd_a, src.va[i], (uint32_t)kt * A_STEP, lds_w + h * RING_SLOT + i * 4096u);
        } else {
#pragma unroll
          for (int c = 0; c < NWC; ++c) copy_w(src, c, kt, lds_w + h * RING_SLOT + c * 4096u);
        }
      }
    }
  }

  // One tile: acc[matrix][16-row block][16-column block] = A tile x W tile over KT >= 3 slices; the ring has been
  // filled (fill with AC copies).
  //   all_landed      wait for everything this wave has in flight (a fill issued before the previous
  //                   tile's epilogue, whose own loads and stores are counted with it) instead of for
  //                   the first slice alone; wave-uniform
  //   rd_a / rd_w     this lane's operand-read addresses inside a slot (slot 0), without the chunk swizzle
  //   rd_off[s]       swizzled chunk offset of K step s
  template <typename Acc>
  static __device__ __forceinline__ void tile(Acc &acc, uint32_t lds0, int wave, const RingSrc &src,
                                              const unsigned char *rd_a, const unsigned char *rd_w,
                                              const int (&rd_off)[2], int KT, bool all_landed) {
    if constexpr (STAGES > 0) tile_slices(acc, lds0, wave, src, rd_a, rd_w, rd_off, KT, all_landed);
    else tile_halves(acc, lds0, wave, src, rd_a, rd_w, rd_off, KT, all_landed);
  }

  // Reads of the other K step that go behind product q of a half slice: [first_read(q), first_read(q + 1))
  static __device__ __forceinline__ constexpr int first_read(int q) {
    const int r = RPP > 1 ? q * RPP : (q + RSP - 1) / RSP;
    return r < RD ? r : RD;
  }

  // Small tiles: STAGES whole slices, slice kt in stage kt % STAGES.  Where a few rows meet a whole weight matrix the
  // weights come from HBM, and the ring of half slices leaves a weight copy half a slice to one slice of time to
  // arrive, less than the memory's latency once a slice takes 0.6 us; here it has STAGES - 1.5 to STAGES - 1.  The
  // stage of slice kt is free past the barrier in the middle of slice kt: W(kt + STAGES) follows in its second half,
  // A(kt + STAGES) in the first half of slice kt + 1.  Against halves in the same tiles (16 GEMMs, 140 to 5000 rows):
  // 128 columns and 32 / 64 / 128 / 256 rows 0.56 / 0.66 / 0.79 / 0.92 of the time, 256 columns and 64 / 128 / 160 rows
  // 0.78 / 0.85 / 0.89, 192 columns and 64 / 128 / 192 rows 0.79 / 0.88 / 0.92.
  template <typename Acc>
  static __device__ __forceinline__ void tile_slices(Acc &acc, uint32_t lds0, int wave, const RingSrc &src,
                                                     const unsigned char *rd_a, const unsigned char *rd_w,
                                                     const int (&rd_off)[2], int KT, bool all_landed) {
    constexpr int S = STAGES > 0 ? STAGES : 1;
    constexpr uint32_t STAGE = CPS * 4096u, A_BYTES = AC * 4096u;
    static_assert((S - 1) * CPS < 64, "vmcnt immediate");
    const uint32_t lds_w = lds0 + (uint32_t)wave * 1024u;
    // wait for all but the newest n slices (n known to be at most S - 1)
    auto wait_but = [](int n) {
      if (S > 4 && n >= 4) wait_vmcnt<(S > 4 ? 4 : 0) * CPS>();
      else if (S > 3 && n >= 3) wait_vmcnt<(S > 3 ? 3 : 0) * CPS>();
      else if (n >= 2) wait_vmcnt<2 * CPS>();
      else if (n == 1) wait_vmcnt<CPS>();
      else wait_vmcnt<0>();
    };
    if (all_landed) wait_vmcnt<0>();
    else wait_but(min(S, KT) - 1);  // slice 0 has landed (this wave's part)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    bf16x8 af[2][MI], bfr[2][NC];  // [K step][16-row block], [K step][16-column block]
    auto read = [&](int st, int x, uint32_t stage) {
      if (x < MI) af[st][x] = *reinterpret_cast<const bf16x8 *>(rd_a + stage + x * (16 * WR) * ROW + rd_off[st]);
      else bfr[st][x - MI] = *reinterpret_cast<const bf16x8 *>(rd_w + stage + A_BYTES + w_row(x - MI) + rd_off[st]);
    };
    auto prod = [&](int st, int p, bool zero) {  // product p of a K step: row block p / NC, column block p % NC
      const int i = p / NC, c = p % NC;
      auto &a = acc[c / (2 * NB)][i][c % (2 * NB)];
      const floatx4 sum = zero ? floatx4{0.f, 0.f, 0.f, 0.f} : a;  // (the first products of a tile start from zero)
      a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[st][i], bfr[st][c], sum, 0, 0, 0);
    };
    uint32_t cur = 0;  // stage of slice kt (byte offset; hidden from the optimiser as in tile_halves)
    asm volatile("" : "+s"(cur));
#pragma unroll
    for (int x = 0; x < RD; ++x) read(0, x, cur);

    // CA: A(kt - 1 + S) is copied; CW: W(kt + S) is.  MORE: slice kt + 1 exists.
    auto slice = [&](int kt, auto first_c, auto ca_c, auto cw_c, bool more) {
      constexpr bool FIRST = decltype(first_c)::value, CA = decltype(ca_c)::value, CW = decltype(cw_c)::value;
      const uint32_t nxt = cur + STAGE >= S * STAGE ? 0 : cur + STAGE, prv = cur ? cur - STAGE : (S - 1) * STAGE;
      auto copy_a_due = [](int q) { return (q + 1) % (PS / AC) == 0; };
#pragma unroll
      for (int q = 0; q < PS; ++q) {
#pragma unroll
        for (int r = first_read(q); r < first_read(q + 1); ++r) read(1, r, cur);
        if (CA && copy_a_due(q)) {
          const int i = (q + 1) / (PS / AC) - 1;
          dma16_buf(src.srd_a, src.va[i], (uint32_t)(kt - 1 + S) * A_STEP, lds_w + prv + i * 4096u);
        }
        prod(0, q, FIRST);
      }
#pragma unroll
      for (int q = 0; q < PS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (first_read(q + 1) > first_read(q)) __builtin_amdgcn_sched_group_barrier(0x100, RPP, 0);
        if (CA && copy_a_due(q)) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
      // Middle: slice kt+1 has landed, and with the barrier everyone's part of it; everyone has read slice kt.
      if (CA || CW) wait_vmcnt<(S - 2) * CPS>();
      else wait_but(KT - 2 - kt);
      wait_lgkmcnt0();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      auto copy_w_due = [](int q) { return (q + 1) % (PS / NWC) == 0; };
#pragma unroll
      for (int q = 0; q < PS; ++q) {
        if (more) {
#pragma unroll
          for (int r = first_read(q); r < first_read(q + 1); ++r) read(0, r, nxt);
        }
        if (CW && copy_w_due(q)) copy_w(src, (q + 1) / (PS / NWC) - 1, kt + S, lds_w + cur + A_BYTES + ((q + 1) / (PS / NWC) - 1) * 4096u);
        prod(1, q, false);
      }
#pragma unroll
      for (int q = 0; q < PS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (more && first_read(q + 1) > first_read(q)) __builtin_amdgcn_sched_group_barrier(0x100, RPP, 0);
        if (CW && copy_w_due(q)) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
      cur = nxt;
    };
    constexpr auto yes = std::true_type{};
    constexpr auto no = std::false_type{};
    int kt = 1;
    if (KT > S) {
      slice(0, yes, no, yes, true);
      for (; kt + S < KT; ++kt) slice(kt, no, yes, yes, true);
      slice(kt, no, yes, no, true);
      ++kt;
    } else {
      slice(0, yes, no, no, true);
    }
    for (; kt + 1 < KT; ++kt) slice(kt, no, no, no, true);
    slice(kt, no, no, no, false);
  }

  // Large tiles: five slots of half slices (see the head of this file).
  template <typename Acc>
  static __device__ __forceinline__ void tile_halves(Acc &acc, uint32_t lds0, int wave, const RingSrc &src,
                                              const unsigned char *rd_a, const unsigned char *rd_w,
                                              const int (&rd_off)[2], int KT, bool all_landed) {
    const uint32_t lds_w = lds0 + (uint32_t)wave * 1024u;
    auto copy_a = [&](int i, int kt, int slot) {
      dma16_buf(src.srd_a, src.va[i], (uint32_t)kt * A_STEP, lds_w + (uint32_t)slot * RING_SLOT + i * 4096u);
    };
    if (all_landed) wait_vmcnt<0>();
    else wait_vmcnt<2 * AC + NWC>();  // slice 0 has landed (this wave's part); the rest of the fill is behind it
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    bf16x8 af[2][MI], bfr[2][NC];  // [K step][16-row block], [K step][16-column block]
    auto read = [&](int st, int x, const unsigned char *sa, const unsigned char *sb) {
      if (x < MI) af[st][x] = *reinterpret_cast<const bf16x8 *>(sa + x * (16 * WR) * ROW + rd_off[st]);
      else bfr[st][x - MI] = *reinterpret_cast<const bf16x8 *>(sb + w_row(x - MI) + rd_off[st]);
    };
    auto prod = [&](int st, int p, bool zero) {  // product p of a K step: row block p / NC, column block p % NC
      const int i = p / NC, c = p % NC;
      auto &a = acc[c / (2 * NB)][i][c % (2 * NB)];
      const floatx4 sum = zero ? floatx4{0.f, 0.f, 0.f, 0.f} : a;  // (the first products of a tile start from zero)
      a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[st][i], bfr[st][c], sum, 0, 0, 0);
    };
    // slot of A(kt); W(kt) is in the next one.  (Hidden from the optimiser: with a known start the first
    // slice's operand addresses lie past the reach of an LDS offset and are computed once per kernel, which
    // has no registers to keep them.)
    int slot_a = 0;
    asm volatile("" : "+s"(slot_a));
#pragma unroll
    for (int x = 0; x < RD; ++x) read(0, x, rd_a + (uint32_t)slot_a * RING_SLOT, rd_w + (uint32_t)(slot_a + 1) * RING_SLOT);

    auto slice = [&](int kt, auto first_c, auto m1_c, auto m2_c) {
      // FIRST: slice 0 (A(2) is already on its way); M1 / M2: slices kt+1 / kt+2 exist.  The last
      // slice keeps its barrier: past it every wave has read the tile's last operands out of the
      // ring, which the caller may then refill for its next tile.
      constexpr bool FIRST = decltype(first_c)::value, M1 = decltype(m1_c)::value, M2 = decltype(m2_c)::value;
      constexpr bool CA = !FIRST && M2;
      const int slot_w = nxt(slot_a, 1), slot_a1 = nxt(slot_a, 2), slot_w1 = nxt(slot_a, 3), slot_a2 = nxt(slot_a, 4);
      const unsigned char *sa = rd_a + (uint32_t)slot_a * RING_SLOT, *sb = rd_w + (uint32_t)slot_w * RING_SLOT;
      // First half: products of K step 0; the operand reads of step 1 between the first of them; the
      // copies of A(kt+2) into the slot W(kt-1) left, evenly.  In the instruction order
      // (sched_group_barrier: product, read, copy) the scheduler left alone would fetch each operand
      // right before its use and bunch the copies.
      auto copy_a_due = [](int q) { return (q + 1) % (PS / AC) == 0; };
#pragma unroll
      for (int q = 0; q < PS; ++q) {
#pragma unroll
        for (int r = first_read(q); r < first_read(q + 1); ++r) read(1, r, sa, sb);
        if (CA && copy_a_due(q)) copy_a((q + 1) / (PS / AC) - 1, kt + 2, slot_a2);
        prod(0, q, FIRST);
      }
#pragma unroll
      for (int q = 0; q < PS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (first_read(q + 1) > first_read(q)) __builtin_amdgcn_sched_group_barrier(0x100, RPP, 0);
        if (CA && copy_a_due(q)) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
      // Middle: slice kt+1 has landed (the copies of A(kt+2) behind it may still be in flight), and
      // with the barrier everyone's part of it; everyone has read slice kt out of its slots.
      if (M1) {
        if (M2) wait_vmcnt<AC>();
        else wait_vmcnt<0>();
      }
      wait_lgkmcnt0();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      // Second half: products of K step 1, the copies of W(kt+2) into the slot A(kt) left, the
      // operands of step 0 of slice kt+1.
      const unsigned char *sa1 = rd_a + (uint32_t)slot_a1 * RING_SLOT, *sb1 = rd_w + (uint32_t)slot_w1 * RING_SLOT;
      auto copy_w_due = [](int q) { return (q + 1) % (PS / NWC) == 0; };
#pragma unroll
      for (int q = 0; q < PS; ++q) {
        if (M1) {
#pragma unroll
          for (int r = first_read(q); r < first_read(q + 1); ++r) read(0, r, sa1, sb1);
        }
        if (M2 && copy_w_due(q)) copy_w(src, (q + 1) / (PS / NWC) - 1, kt + 2, lds_w + (uint32_t)slot_a * RING_SLOT + ((q + 1) / (PS / NWC) - 1) * 4096u);
        prod(1, q, false);
      }
#pragma unroll
      for (int q = 0; q < PS; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (M1 && first_read(q + 1) > first_read(q)) __builtin_amdgcn_sched_group_barrier(0x100, RPP, 0);
        if (M2 && copy_w_due(q)) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
      }
      slot_a = slot_a1;
    };
    slice(0, std::true_type{}, std::true_type{}, std::true_type{});
    int kt = 1;
    for (; kt + 2 < KT; ++kt) slice(kt, std::false_type{}, std::true_type{}, std::true_type{});
    slice(kt, std::false_type{}, std::true_type{}, std::false_type{});
    slice(kt + 1, std::false_type{}, std::false_type{}, std::false_type{});
  }
};

}  // namespace mm
}  // namespace dy
