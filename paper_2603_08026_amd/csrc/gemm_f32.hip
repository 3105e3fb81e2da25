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

// Tile of 16 MT rows x 16 NT columns per workgroup; its four waves take K steps of 64 in turn (wave w the
// steps w, w + 4, ...) and their sums are added through LDS in the order of the waves.  A lane loads four
// neighbouring k of row l % 16 of a block (k = 4 (l / 16) .. + 3 of every 16) straight into registers, 16
// bytes at a time and all of a step at once, and the four are the k of four v_mfma_f32_16x16x4_f32: the
// order in which k is summed does not matter as long as both operands agree.  Weights are the first
// operand, so that a lane's four results are neighbouring columns of one row (row l % 16, columns
// 4 (l / 16) .. + 3).  fp32 products and sums throughout.
template <typename Epi, int MT, int NT>
__global__ __launch_bounds__(256) void k_gemm_f32(const float *__restrict__ A, const int32_t *gather,
                                                   int lda, Rows rows, int K, int N, WSeg seg,
                                                   const float *__restrict__ W2, Epi epi) {
  constexpr int TM = 16 * MT, TN = 16 * NT, NMAT = Epi::DUAL ? 2 : 1;
  __shared__ floatx4 part[3][NMAT * MT * NT][64];

  const int M = rows.count ? min(*rows.count, rows.cap) : rows.cap;
  const int tiles_n = N / TN, tiles_m = (M + TM - 1) / TM;
  const int lane = threadIdx.x % WAVE, wave = threadIdx.x / WAVE;
  const int l16 = lane % 16, lq = lane / 16;

  for (int tile = blockIdx.x; tile < tiles_m * tiles_n; tile += gridDim.x) {
    const int tm = tile / tiles_n, tn = tile % tiles_n;
    const int m0 = tm * TM, n0 = tn * TN;
    const float *ap[MT], *wp[NMAT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int j = min(m0 + 16 * i + l16, M - 1);  // rows past the end are clamped; their results are never stored
      ap[i] = A + (size_t)(gather ? gather[j] : j) * lda + 4 * lq;
    }
#pragma unroll
    for (int c = 0; c < NT; ++c) {
      const int n = n0 + 16 * c + l16;  // looked up in the stacked weight matrices
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

    for (int k0 = wave * KSTEP; k0 < K; k0 += 4 * KSTEP) {  // K is a multiple of KSTEP
      floatx4 a[KSTEP / 16][MT], w[KSTEP / 16][NMAT][NT];
#pragma unroll
      for (int s = 0; s < KSTEP / 16; ++s) {
#pragma unroll
        for (int i = 0; i < MT; ++i) a[s][i] = *reinterpret_cast<const floatx4 *>(ap[i] + k0 + 16 * s);
#pragma unroll
        for (int t = 0; t < NMAT; ++t)
#pragma unroll
          for (int c = 0; c < NT; ++c) w[s][t][c] = *reinterpret_cast<const floatx4 *>(wp[t][c] + k0 + 16 * s);
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
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int j = m0 + 16 * i + l16;
#pragma unroll
        for (int c = 0; c < NT; ++c) {
          floatx4 v[NMAT];
#pragma unroll
          for (int t = 0; t < NMAT; ++t) {
            v[t] = acc[t][i][c];
#pragma unroll
            for (int q = 0; q < 3; ++q) v[t] += part[q][(t * MT + i) * NT + c][lane];
          }
          if (j < M) {
            const int row = rows.idx ? rows.idx[j] : j;
#pragma unroll
            for (int e = 0; e < 4; ++e) epi(j, row, n0 + 16 * c + 4 * lq + e, v[0][e], v[NMAT - 1][e]);
          }
        }
      }
    }
  }
}

template <typename Epi, int MT, int NT>
void launch(GemmA A, Rows rows, int K, int N, WSeg seg, const void *w2, Epi epi, hipStream_t s) {
  const long t = (long)((rows.cap + 16 * MT - 1) / (16 * MT)) * (N / (16 * NT));
  k_gemm_f32<Epi, MT, NT><<<(int)(t > 4096 ? 4096 : t), 256, 0, s>>>((const float *)A.a, A.gather, A.lda, rows, K, N, seg,
                                                                     (const float *)w2, epi);
}

// 16 x 16 tiles while those of a full list number at most two per CU: a few rows are bound by the latency
// of one round of loads, and small tiles put the whole of a short K in flight at once.  Beyond, 32 x 32
// (32 x 32 of each of gate and up): half the operand bytes per product.  Steps of a layer of hidden size
// 256 and FFN 768, against 64 x 64 tiles of plain FMAs that staged K in slices of 16 through LDS, a dozen
// workgroups each waiting for memory sixteen times in a row: 13 rows 193 -> 45 us (the four GEMMs 156 ->
// 18), 105 rows 247 -> 67 us, 2048 rows (dense) 369 -> 206 us; error against 64 bits 7.9e-7 -> 6.1e-7.  FFN half of
// wider layers (FFN three times as wide): hidden 1024, 13 / 400 / 2048 rows 544 / 718 / 1194 -> 33 / 150 / 617 us; hidden 4096
// 2277 / 4716 / 17540 -> 213 / 2054 / 9685 us.
template <typename Epi>
void run(GemmA A, Rows rows, int K, int N, WSeg seg, const void *w2, Epi epi, hipStream_t s) {
  if (rows.cap <= 0) return;
  const long small = (long)((rows.cap + 15) / 16) * (N / 16);
  if (small <= 512) launch<Epi, 1, 1>(A, rows, K, N, seg, w2, epi, s);
  else launch<Epi, 2, 2>(A, rows, K, N, seg, w2, epi, s);
}

}  // namespace

void gemm_f32_raw(GemmA A, Rows rows, int K, WSeg seg, float *part, hipStream_t s) {
  run(A, rows, K, seg.n_end[2], seg, nullptr, EpiStoreF32{part, seg.n_end[2]}, s);
}

void gemm_f32_swiglu(GemmA A, Rows rows, int K, int N, const void *w_gate, const void *w_up, void *act, hipStream_t s) {
  run(A, rows, K, N, wseg_one(w_gate, N), w_up, EpiSwiGLU<float>{(float *)act, N}, s);
}

void gemm_f32_down(GemmA A, Rows rows, int K, int N, const void *w_down, const float *h, void *out_cache, hipStream_t s) {
  run(A, rows, K, N, wseg_one(w_down, N), nullptr, EpiDown<float>{h, (float *)out_cache, N}, s);
}

}  // namespace dy
