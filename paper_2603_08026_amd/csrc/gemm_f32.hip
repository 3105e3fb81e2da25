// Salient-row GEMMs for the fp32 storage type: C[j,n] = sum_k A[row_j,k] * W[n,k] with fused
// epilogues, on the fp32 matrix instructions (fp32 products and sums; the fp32 path is the accuracy
// reference of the library).  The row count lives on the device: the grid is sized for the list's
// capacity and each workgroup loops over the tiles that exist.
#include "gemm_epilogues.h"
#include "kernels.h"

namespace dy {

namespace {

constexpr int KSTEP = 64;  // K elements of a wave's step

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

// q|k|v finished in the epilogue (QkvOut): a tile's columns are pairs that turn together
struct EpiQkvF32 {
  static constexpr bool DUAL = false, PAIRS = true;
  QkvOut o;
};
// out-projection: h[j] = x[row_j] + result
struct EpiResidualF32 {
  static constexpr bool DUAL = false, PAIRS = false;
  const float *x;
  float *h;
  int N;
  __device__ __forceinline__ void operator()(int j, int row, int n, float acc, float) const {
    h[(size_t)j * N + n] = acc + x[(size_t)row * N + n];
  }
};
struct EpiRawF32 : EpiStoreF32 { static constexpr bool PAIRS = false; };
struct EpiSwiGLUF32 : EpiSwiGLU<float> { static constexpr bool PAIRS = false; };
struct EpiDownF32 : EpiDown<float> { static constexpr bool PAIRS = false; };

// The activations' RMSNorm: rows are multiplied by `gain` on their way into the products, the results by the rows'
// 1 / sqrt(mean square + eps)
struct NormIn {
  const float *gain = nullptr;
  float eps = 0.f;
};

// Tile of 16 MT rows x 16 NT columns per workgroup; its four waves take K steps of 64 in turn (wave w the
// steps w, w + 4, ...) and their sums are added through LDS in the order of the waves.  A lane loads four
// neighbouring k of row l % 16 of a block (k = 4 (l / 16) .. + 3 of every 16) straight into registers, 16
// bytes at a time and all of a step at once, and the four are the k of four v_mfma_f32_16x16x4_f32: the
// order in which k is summed does not matter as long as both operands agree.  Weights are the first
// operand, so that a lane's four results are neighbouring columns of one row (row l % 16, columns
// 4 (l / 16) .. + 3).  fp32 products and sums throughout.
// NORM: the activations are normalised on the way (NormIn).  A workgroup reads its rows whole, so it has their sums of squares,
// and what a row is divided by goes out of its products: no launch and no pass of its own.
// PAIRS (q|k|v): the columns of a tile are those of TN / 2 pairs (p, p + dh / 2) of heads: 16 columns hold eight pairs, partners
// 32 lanes apart; of two blocks of 16 the second holds the partners of the first.
// Waves per SIMD: left to itself the compiler orders the norm's loop for fewer registers as soon as anything is added behind it, with a
// wait for all loads every few products; for at most three waves it asks for half a step's operands at once.  With the rows that overflow
// (below) looked after, us: hidden 4096, 90 / 186 / 458 rows 792 -> 682, 1258 -> 1132, 2996 -> 2768; hidden 2048, 821 rows 1226 -> 1140; hidden
// 1024, 913 rows 465 -> 457; hidden 256 equal.
template <typename Epi, int MT, int NT, bool NORM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NORM ? 2 : 1, NORM ? 3 : 8))) void k_gemm_f32(const float *__restrict__ A, const int32_t *gather,
                                                   int lda, Rows rows, int K, int N, WSeg seg,
                                                   const float *__restrict__ W2, NormIn norm, Epi epi) {
  constexpr int TM = 16 * MT, TN = 16 * NT, NMAT = Epi::DUAL ? 2 : 1;
  __shared__ floatx4 part[3][NMAT * MT * NT][64];
  __shared__ float squares[4][TM];
  // column of tile tn's column x (a multiple of 16 in block x / 16)
  auto column = [&](int tn, int x) -> int {
    if constexpr (Epi::PAIRS) {
      const int half = epi.o.dh / 2, second = x >= TN / 2 ? 1 : 0, pair = tn * (TN / 2) + x - second * (TN / 2);
      const int head = half == 64 ? pair / 64 : pair / 32;
      return head * 2 * half + pair - head * half + second * half;
    } else {
      return tn * TN + x;
    }
  };

  const int M = rows.count ? min(*rows.count, rows.cap) : rows.cap;
  const int tiles_n = N / TN, tiles_m = (M + TM - 1) / TM;
  const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
  const int l16 = lane % 16, lq = lane / 16;

  for (int tile = blockIdx.x; tile < tiles_m * tiles_n; tile += gridDim.x) {
    const int tm = tile / tiles_n, tn = tile % tiles_n;
    const int m0 = tm * TM;
    const float *ap[MT], *wp[NMAT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int j = min(m0 + 16 * i + l16, M - 1);  // rows past the end are clamped; their results are never stored
      ap[i] = A + (size_t)(gather ? gather[j] : j) * lda + 4 * lq;
    }
#pragma unroll
    for (int c = 0; c < NT; ++c) {
      const int n = column(tn, 16 * c + l16);  // looked up in the stacked weight matrices
      const bool in1 = n >= seg.n_end[0], in2 = n >= seg.n_end[1];
      const int start = in2 ? seg.n_end[1] : in1 ? seg.n_end[0] : 0;
      wp[0][c] = (const float *)(in2 ? seg.w[2] : in1 ? seg.w[1] : seg.w[0]) + (size_t)(n - start) * K + 4 * lq;
      if (NMAT == 2) wp[NMAT - 1][c] = W2 + (size_t)n * K + 4 * lq;
    }
    floatx4 acc[NMAT][MT][NT];
#pragma unroll
    for (int t = 0; t < NMAT; ++t)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int c = 0; c < NT; ++c) acc[t][i][c] = floatx4{0.f, 0.f, 0.f, 0.f};

    float ss[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) ss[i] = 0.f;
    for (int k0 = wave * KSTEP; k0 < K; k0 += 4 * KSTEP) {  // K is a multiple of KSTEP
      floatx4 a[KSTEP / 16][MT], w[KSTEP / 16][NMAT][NT], g[KSTEP / 16];
#pragma unroll
      for (int s = 0; s < KSTEP / 16; ++s) {
#pragma unroll
        for (int i = 0; i < MT; ++i) a[s][i] = *reinterpret_cast<const floatx4 *>(ap[i] + k0 + 16 * s);
#pragma unroll
        for (int t = 0; t < NMAT; ++t)
#pragma unroll
          for (int c = 0; c < NT; ++c) w[s][t][c] = *reinterpret_cast<const floatx4 *>(wp[t][c] + k0 + 16 * s);
        if (NORM) g[s] = *reinterpret_cast<const floatx4 *>(norm.gain + 4 * lq + k0 + 16 * s);
      }
      if constexpr (NORM) {
#pragma unroll
        for (int s = 0; s < KSTEP / 16; ++s)
#pragma unroll
          for (int i = 0; i < MT; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) ss[i] += a[s][i][e] * a[s][i][e];
            a[s][i] *= g[s];
          }
      }
#pragma unroll
      for (int s = 0; s < KSTEP / 16; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int t = 0; t < NMAT; ++t)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
              for (int c = 0; c < NT; ++c)
                acc[t][i][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][t][c][e], a[s][i][e], acc[t][i][c], 0, 0, 0);
    }

    __syncthreads();  // the sums of the previous tile have been read
    if (wave > 0) {
#pragma unroll
      for (int t = 0; t < NMAT; ++t)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int c = 0; c < NT; ++c) part[wave - 1][(t * MT + i) * NT + c][lane] = acc[t][i][c];
    }
    if constexpr (NORM) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        ss[i] += __shfl_xor(ss[i], 16, WAVE);
        ss[i] += __shfl_xor(ss[i], 32, WAVE);
        if (lq == 0) squares[wave][16 * i + l16] = ss[i];
      }
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int j = m0 + 16 * i + l16, row = j < M && rows.idx ? rows.idx[j] : j;
        float scale = 1.0f;
        if constexpr (NORM) {
          const float sum = (squares[0][16 * i + l16] + squares[1][16 * i + l16]) + (squares[2][16 * i + l16] + squares[3][16 * i + l16]);
          scale = 1.0f / sqrtf(sum / (float)K + norm.eps);
        }
        floatx4 v[NMAT][NT];
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
          for (int t = 0; t < NMAT; ++t) {
            v[t][c] = acc[t][i][c];
#pragma unroll
            for (int q = 0; q < 3; ++q) v[t][c] += part[q][(t * MT + i) * NT + c][lane];
            if (NORM) v[t][c] *= scale;
          }
        if constexpr (NORM) {
          // Squares whose sum overflows make the factor 0, and their products may have overflowed as well: those of the
          // normalised elements, 0 or NaN, are taken instead.  (Addresses computed anew, not kept across the loop over K.)
          if (scale == 0.0f) {
            int jr = min(m0 + 16 * i + l16, M - 1), tile_n = tn;
            asm volatile("" : "+v"(jr), "+s"(tile_n));
            const float *xr = A + (size_t)(gather ? gather[jr] : jr) * lda;
            for (int c = 0; c < NT; ++c)
              for (int t = 0; t < NMAT; ++t)
                for (int e = 0; e < 4; ++e) {
                  const int n = column(tile_n, 16 * c + 4 * lq) + e;
                  const int in = n >= seg.n_end[1] ? 2 : n >= seg.n_end[0] ? 1 : 0;
                  const float *wr = t == 1 ? W2 + (size_t)n * K : (const float *)(in == 2 ? seg.w[2] : in == 1 ? seg.w[1] : seg.w[0]) + (size_t)(n - (in ? seg.n_end[in - 1] : 0)) * K;
                  float sum = 0.f;
                  for (int k = 0; k < K; ++k) sum += xr[k] * scale * norm.gain[k] * wr[k];
#pragma unroll
                  for (int cc = 0; cc < NT; ++cc)
#pragma unroll
                    for (int tt = 0; tt < NMAT; ++tt)
#pragma unroll
                      for (int ee = 0; ee < 4; ++ee)
                        if (cc == c && tt == t && ee == e) v[tt][cc][ee] = sum;
                }
          }
        }
        if constexpr (Epi::PAIRS) {
          // this lane's columns of each block, four in a row: first ones or (16 columns, lanes from 32 on; second block) partners
          const QkvOut &o = epi.o;
          const int half = o.dh / 2, dq = o.H * o.dh, dkv = o.Hkv * o.dh, pos = row % o.L;
          floatx4 mine[NT], other[NT];
          int at[NT];  // column of the stacked matrices
#pragma unroll
          for (int c = 0; c < NT; ++c) {
            at[c] = column(tn, 16 * c + 4 * lq);
            const bool in_q = at[c] < dq, in_k = !in_q && at[c] < dq + dkv;
            const float *b = (const float *)(in_q ? o.bq : in_k ? o.bk : o.bv);
            mine[c] = v[0][c];
            if (b) mine[c] += *reinterpret_cast<const floatx4 *>(b + at[c] - (in_q ? 0 : in_k ? dq : dq + dkv));
          }
#pragma unroll
          for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) other[c][e] = NT == 1 ? __shfl_xor(mine[c][e], 32, WAVE) : mine[NT - 1 - c][e];
          if (j < M) {
#pragma unroll
            for (int c = 0; c < NT; ++c) {
              const bool in_q = at[c] < dq, in_k = !in_q && at[c] < dq + dkv;
              const bool second = NT == 1 ? lq >= 2 : c == 1;
              floatx4 y = mine[c];
              if (in_q || in_k) {
                const int in_head = o.dh == 64 ? at[c] % 64 : at[c] % 128, p = second ? in_head - half : in_head;
                const floatx4 *t = reinterpret_cast<const floatx4 *>(o.tab + ((size_t)pos * half + p) * 2);
                const floatx4 t0 = t[0], t1 = t[1];
                const float co[4] = {t0[0], t0[2], t1[0], t1[2]}, si[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const float ps = other[c][e] * si[e];
                  y[e] = rotated(mine[c][e], co[e], second ? ps : -ps);
                }
              }
              const int to = in_q && !o.q_by_token ? j : row;
              float *out = in_q ? (float *)o.q + (size_t)to * dq + at[c] : in_k ? (float *)o.k + (size_t)to * dkv + at[c] - dq : (float *)o.v + (size_t)to * dkv + at[c] - dq - dkv;
              *reinterpret_cast<floatx4 *>(out) = y;
            }
          }
        } else if (j < M) {
#pragma unroll
          for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) epi(j, row, tn * TN + 16 * c + 4 * lq + e, v[0][c][e], v[NMAT - 1][c][e]);
        }
      }
    }
  }
}

template <bool NORM, typename Epi, int MT, int NT>
void launch(GemmA A, Rows rows, int K, int N, WSeg seg, const void *w2, NormIn norm, Epi epi, hipStream_t s) {
  const long t = (long)((rows.cap + 16 * MT - 1) / (16 * MT)) * (N / (16 * NT));
  k_gemm_f32<Epi, MT, NT, NORM><<<(int)(t > 4096 ? 4096 : t), 256, 0, s>>>((const float *)A.a, A.gather, A.lda, rows, K, N, seg,
                                                                     (const float *)w2, norm, epi);
}

// 16 x 16 tiles while those of a full list number at most two per CU: a few rows are bound by the latency
// of one round of loads, and small tiles put the whole of a short K in flight at once.  Beyond, 32 x 32
// (32 x 32 of each of gate and up): half the operand bytes per product.  Steps of a layer of hidden size
// 256 and FFN 768, against 64 x 64 tiles of plain FMAs that staged K in slices of 16 through LDS, a dozen
// workgroups each waiting for memory sixteen times in a row: 13 rows 193 -> 45 us (the four GEMMs 156 ->
// 18), 105 rows 247 -> 67 us, 2048 rows (dense) 369 -> 206 us; error against 64 bits 7.9e-7 -> 6.1e-7.  FFN half of
// wider layers (FFN three times as wide): hidden 1024, 13 / 400 / 2048 rows 544 / 718 / 1194 -> 33 / 150 / 617 us; hidden 4096
// 2277 / 4716 / 17540 -> 213 / 2054 / 9685 us.
template <bool NORM, typename Epi>
void run(GemmA A, Rows rows, int K, int N, WSeg seg, const void *w2, NormIn norm, Epi epi, hipStream_t s) {
  if (rows.cap <= 0) return;
  const long small = (long)((rows.cap + 15) / 16) * (N / 16);
  if (small <= 512) launch<NORM, Epi, 1, 1>(A, rows, K, N, seg, w2, norm, epi, s);
  else launch<NORM, Epi, 2, 2>(A, rows, K, N, seg, w2, norm, epi, s);
}

}  // namespace

void gemm_f32_raw(GemmA A, Rows rows, int K, WSeg seg, float *part, hipStream_t s) {
  run<false>(A, rows, K, seg.n_end[2], seg, nullptr, NormIn{}, EpiRawF32{{part, seg.n_end[2]}}, s);
}

void gemm_f32_down(GemmA A, Rows rows, int K, int N, const void *w_down, const float *h, void *out_cache, hipStream_t s) {
  run<false>(A, rows, K, N, wseg_one(w_down, N), nullptr, NormIn{}, EpiDownF32{{h, (float *)out_cache, N}}, s);
}

void launch_qkv_f32(const void *x, const void *gain, float eps, Rows rows, int K, WSeg seg, const QkvOut &out, hipStream_t s) {
  if (!gain) {
    run<false>(GemmA{x, nullptr, K}, rows, K, seg.n_end[2], seg, nullptr, NormIn{}, EpiQkvF32{out}, s);
    return;
  }
  run<true>(GemmA{x, rows.idx, K}, rows, K, seg.n_end[2], seg, nullptr, NormIn{(const float *)gain, eps}, EpiQkvF32{out}, s);
}

void launch_oproj_f32(GemmA A, Rows rows, int K, int N, const void *wo, const void *x, float *h, hipStream_t s) {
  run<false>(A, rows, K, N, wseg_one(wo, N), nullptr, NormIn{}, EpiResidualF32{(const float *)x, h, N}, s);
}

void launch_swiglu_f32(const float *h, const void *gain, float eps, Rows rows, int K, int N, const void *w_gate, const void *w_up,
                     void *act, hipStream_t s) {
  run<true>(GemmA{h, nullptr, K}, rows, K, N, wseg_one(w_gate, N), w_up, NormIn{(const float *)gain, eps}, EpiSwiGLUF32{{(float *)act, N}}, s);
}

}  // namespace dy
