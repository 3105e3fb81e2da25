// Partial (row-sparse) attention, fp32 arithmetic: exact attention rows for the salient queries
// against all keys/values of their sequence, no mask.  [Sec. 3.3 salient path; Alg. 3: C_sal]
//
// Flash-style: a workgroup owns BQ query rows of one (sequence, head) and streams the keys in
// tiles of BK through LDS with an online softmax.  The key range can be split over several
// workgroups (few query rows, small batch); partial (max, sum, un-normalised output) triples are
// merged by k_attn_combine.  This file serves the fp32 storage type; the bf16 type has MFMA
// kernels of its own and shares only the combine kernel and the tile-to-sequence mapping.
//
// Bound: latency (13 rows against 128 keys of four heads are 16 workgroups).  A workgroup's life is the way to its
// first tile and, per tile, a round of loads, the scores and the products, so a tile's keys and values are loaded together
// while the tile before is worked on, and everything is read from LDS four floats at a time: 13 rows, 128 keys
// 14.5 -> 7.2 us (element by element, each tile loaded when it was due), error against 64 bits 6.3e-7 -> 4.5e-7.
#include "attention_common.h"

namespace dy {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

// 16 rows x 16 lanes: lane `sub` of a row scores keys sub and sub + 16 of a tile and owns columns 64 i + 4 sub .. + 3
template <int DH> struct F32Tile {
  static constexpr int BQ = 16, BK = 32, NT = 256;
  static constexpr int CH = DH / 4;              // 16-byte chunks of a row
  static constexpr int LD = BK * CH / NT;        // chunks of K (and of V) per thread and tile
  static constexpr int OC = DH / 64;             // output chunks per thread
  static constexpr int STR = DH + 4;             // LDS row stride of Q and K: 16 rows' chunks fall on all 64 banks
  static_assert(LD * NT == BK * CH && OC * 64 == DH, "head_dim 64 or 128");
};

template <int DH>
__global__ __launch_bounds__(256) void k_attn_f32(AttnArgs a) {
  using TL = F32Tile<DH>;
  constexpr int BQ = TL::BQ, BK = TL::BK, NT = TL::NT, CH = TL::CH, LD = TL::LD, OC = TL::OC, STR = TL::STR;
  __shared__ __align__(16) float Qs[BQ][STR];
  __shared__ __align__(16) float Ks[BK][STR];
  __shared__ __align__(16) float Vs[BK][DH];
  __shared__ __align__(16) float Ps[BQ][BK + 4];
  __shared__ int tile_info[3];

  const int tid = threadIdx.x;
  if (tid == 0) find_tile(a, BQ, blockIdx.x, tile_info);
  __syncthreads();
  const int b = tile_info[0];
  if (b < 0) return;  // uniform: no such tile
  const int j0 = tile_info[1], nq = tile_info[2];
  const int h = blockIdx.y, kvh = h / (a.H / a.Hkv), split = blockIdx.z;
  const int kbase = a.key_offsets ? min(a.key_offsets[b], a.key_cap) : b * a.L;
  const int Lk = a.key_offsets ? min(a.key_offsets[b + 1], a.key_cap) - kbase : a.L;
  const int k_lo = split * a.chunk, k_hi = min(Lk, k_lo + a.chunk);
  if (k_lo >= k_hi) return;  // uniform

  const float *q = (const float *)a.q;
  const float *kc = (const float *)a.k + ((size_t)kbase * a.Hkv + kvh) * DH;
  const float *vc = (const float *)a.v + ((size_t)kbase * a.Hkv + kvh) * DH;
  const size_t kv_stride = (size_t)a.Hkv * DH;
  const float scale = 1.0f / sqrtf((float)DH);
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};

  // (keys past the end: zeros; four-byte alignment is all that these 16-byte loads ask for)
  floatx4 rk[LD], rv[LD];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int e = tid + NT * i, r = e / CH, c = (e % CH) * 4;
      const bool ok = k0 + r < k_hi;
      rk[i] = ok ? *reinterpret_cast<const floatx4 *>(kc + (size_t)(k0 + r) * kv_stride + c) : zero;
      rv[i] = ok ? *reinterpret_cast<const floatx4 *>(vc + (size_t)(k0 + r) * kv_stride + c) : zero;
    }
  };
  load(k_lo);
  for (int e = tid; e < BQ * CH; e += NT) {
    const int r = e / CH, c = (e % CH) * 4;
    const size_t qrow = (r < nq) ? (a.q_by_token ? (size_t)a.rows.idx[j0 + r] : (size_t)(j0 + r)) : 0;
    *reinterpret_cast<floatx4 *>(&Qs[r][c]) = (r < nq) ? *reinterpret_cast<const floatx4 *>(q + (qrow * a.H + h) * DH + c) * scale : zero;
  }

  const int row = tid / 16, sub = tid % 16;
  floatx4 o[OC];
#pragma unroll
  for (int i = 0; i < OC; ++i) o[i] = zero;
  float m_run = -INFINITY, l_run = 0.f;

  for (int k0 = k_lo; k0 < k_hi; k0 += BK) {
    __syncthreads();  // previous tile fully consumed (also orders the Qs fill)
#pragma unroll
    for (int i = 0; i < LD; ++i) {
      const int e = tid + NT * i, r = e / CH, c = (e % CH) * 4;
      *reinterpret_cast<floatx4 *>(&Ks[r][c]) = rk[i];
      *reinterpret_cast<floatx4 *>(&Vs[r][c]) = rv[i];
    }
    __syncthreads();
    if (k0 + BK < k_hi) load(k0 + BK);
    floatx4 a0 = zero, a1 = zero;
#pragma unroll
    for (int e = 0; e < DH; e += 4) {
      const floatx4 qv = *reinterpret_cast<const floatx4 *>(&Qs[row][e]);
      a0 += qv * *reinterpret_cast<const floatx4 *>(&Ks[sub][e]);
      a1 += qv * *reinterpret_cast<const floatx4 *>(&Ks[sub + 16][e]);
    }
    float s0 = (a0[0] + a0[1]) + (a0[2] + a0[3]), s1 = (a1[0] + a1[1]) + (a1[2] + a1[3]);
    if (k0 + sub >= k_hi) s0 = -INFINITY;
    if (k0 + sub + 16 >= k_hi) s1 = -INFINITY;
    float mt = fmaxf(s0, s1);
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) mt = fmaxf(mt, __shfl_xor(mt, off, 16));
    const float m_new = fmaxf(m_run, mt);  // finite: every tile holds at least one valid key
    const float corr = __expf(m_run - m_new);
    const float p0 = __expf(s0 - m_new), p1 = __expf(s1 - m_new);
    float ps = p0 + p1;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) ps += __shfl_xor(ps, off, 16);
    l_run = l_run * corr + ps;
    m_run = m_new;
    Ps[row][sub] = p0;
    Ps[row][sub + 16] = p1;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < OC; ++i) o[i] *= corr;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const floatx4 p = *reinterpret_cast<const floatx4 *>(&Ps[row][kk]);
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < OC; ++i) o[i] += p[x] * *reinterpret_cast<const floatx4 *>(&Vs[kk + x][64 * i + 4 * sub]);
    }
  }

  if (row < nq) {
    const int j = j0 + row;
    const bool whole = a.splits == 1 && !a.partial;
    float *out = whole ? (float *)a.out + ((size_t)j * a.H + h) * DH : a.part_o + (((size_t)split * a.rows.cap + j) * a.H + h) * DH;
    const float by = whole ? 1.0f / l_run : 1.0f;
#pragma unroll
    for (int i = 0; i < OC; ++i) *reinterpret_cast<floatx4 *>(out + 64 * i + 4 * sub) = o[i] * by;
    if (!whole && sub == 0) {
      float *ml = a.part_ml + (((size_t)split * a.rows.cap + j) * a.H + h) * 2;
      ml[0] = m_run;
      ml[1] = l_run;
    }
  }
}

}  // namespace

void launch_attention_f32(const AttnArgs &a, hipStream_t s) {
  dim3 grid(max_q_tiles(a, F32Tile<64>::BQ), a.H, a.splits);
  if (a.dh == 64) k_attn_f32<64><<<grid, 256, 0, s>>>(a);
  else k_attn_f32<128><<<grid, 256, 0, s>>>(a);
}

}  // namespace dy
