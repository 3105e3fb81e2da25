// The launches of the library's calls, recorded on a machine without a GPU: a program that stands in for the few runtime functions that
// the host code calls, runs a case and prints a line per launch - the kernel, and the words of GEMM plans that it makes or reads.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <map>
#include <string>

#include "../paper_2603_08026_amd/csrc/api.hip"

namespace {

std::map<const void *, std::string> &kernels() {
  static std::map<const void *, std::string> k;
  return k;
}
enum { GIVEN, MADE, HERE };  // how a planned GEMM comes by its plan

void print_words(const char *what, const void *p) {
  if (p) printf(" %s=%zx", what, (size_t)p);
}

}  // namespace

extern "C" {

void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid, dim3 *block,
                           dim3 *grid, int *wsize) {
  kernels()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t) {
  const std::string &name = kernels()[f];
  auto is = [&](const char *part) { return name.find(part) != std::string::npos; };
  auto maker = [&](int i) { return ((const PlanMaker *)args[i])->words; };
  printf("%s", name.c_str());
  if (is("k_gemm_planned")) {
    const int how = *(const int *)args[4];
    const void *words = *(void **)args[5];
    if (how == MADE) printf(" reads=%zx", (size_t)words);
    if (how == HERE) printf(" makes=%zx", (size_t)words);
  } else if (is("k_gather_rmsnorm")) {
    print_words("makes", maker(7));
  } else if (is("k_oproj_finalize")) {
    print_words("splits", ((const Splits *)args[1])->dev);
    print_words("makes", maker(9));
    print_words("makes", maker(10));
  } else if (is("k_qkv_finalize") || is("k_down_finalize")) {
    print_words("splits", ((const Splits *)args[1])->dev);
  }
  printf("\n");
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { return (*p = calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }

}  // extern "C"

// launch_probe CASE cap hidden heads kv_heads head_dim ffn B L row_lo cached_norm
int main(int argc, char **argv) {
  if (argc != 12) return 2;
  int v[10];
  for (int i = 0; i < 10; ++i) v[i] = atoi(argv[2 + i]);
  const std::string what = argv[1];
  const int cap = v[0], B = v[6], L = v[7], lo = v[8], cached = v[9];
  dyllm_layer_cfg cfg{};
  cfg.hidden = v[1]; cfg.n_heads = v[2]; cfg.n_kv_heads = v[3]; cfg.head_dim = v[4]; cfg.ffn_dim = v[5];
  cfg.max_batch = B; cfg.max_seq = L; cfg.dtype = DYLLM_BF16; cfg.rms_eps = 1e-5f; cfg.rope_theta = 1e4f;
  dyllm_ctx *ctx = nullptr;
  if (dyllm_create(&cfg, &ctx) != DYLLM_OK) return 3;
  static char mem[32][64];  // addresses that nothing follows
  int n = 0;
  auto any = [&]() { return (void *)mem[n++]; };
  dyllm_layer_weights w{};
  w.wq = any(); w.wk = any(); w.wv = any(); w.wo = any(); w.w_gate = any(); w.w_up = any(); w.w_down = any(); w.g_attn = any(); w.g_ffn = any();
  dyllm_layer_cache cache{};
  cache.k = any(); cache.v = any(); cache.c = any(); cache.out = any();
  if (cached) cache.lse = (decltype(cache.lse))any();
  const dyllm_index_list in{(int32_t *)any(), (int32_t *)any(), cap};
  dyllm_index_list out{(int32_t *)any(), (int32_t *)any(), cap};
  const void *x = any();
  float *cos = (float *)any();
  int rc = 0;
  if (what == "step") {
    rc = dyllm_layer_step(ctx, &w, &cache, x, &in, B, L, 0.5f, &out, cos, nullptr);
  } else if (what == "approx") {
    rc = dyllm_layer_step_approx(ctx, &w, &cache, x, &in, B, L, lo, 0.5f, cached, &out, cos, nullptr);
  } else if (what == "counted window") {  // a window whose rows the device counts
    const Window win{Rows{ctx->win_idx, ctx->win_off + B, B * (L - lo)}, ctx->win_off, lo};
    rc = enqueue_approx_layer(ctx, &w, &cache, x, &in, B, L, win, true, 0.5f, cached, &out, cos, nullptr);
  } else if (what == "ffn") {
    rc = dyllm_salient_ffn(ctx, &w, x, cache.c, &in, B, L, cache.out, nullptr);
  } else if (what == "attention") {  // rows in a tile, key splits, keys of a split
    const AttnArgs a = attn_args(ctx, ctx->qs, cache.k, cache.v, rows_of(&in, B), in.offsets, B, L, nullptr, 0);
    printf("plan bq=%d splits=%d chunk=%d\n", a.bq, a.splits, a.chunk);
  } else if (what == "down alone") {  // a GEMM whose plan nobody has made
    launch_gemm_down(BF16, ctx->act, rows_of(&in, B), cfg.ffn_dim, cfg.hidden, w.w_down, ctx->hs, cache.out, ctx->part_o, ctx->part_elems,
                     PlanJob{}, nullptr);
  } else if (what == "up alone") {
    launch_gemm_swiglu(ctx->fs, rows_of(&in, B), cfg.hidden, cfg.ffn_dim, w.w_gate, w.w_up, ctx->act, PlanJob{}, nullptr);
  } else {
    rc = 4;
  }
  if (rc) fprintf(stderr, "%d %s\n", rc, dyllm_last_error(ctx));
  return rc ? 1 : 0;
}
