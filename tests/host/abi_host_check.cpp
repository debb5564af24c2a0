// Host-only exercise of the C ABI under AddressSanitizer / UBSan: argument validation and the planners.
// The runtime calls that the entry points make are defined here: a launch is written down and nothing runs, so that a call with
// placeholder pointers walks its whole host path.
#include <cstdio>
#include <cstdint>
#include <cstring>
#include <map>
#include <string>
#include <vector>
#include "qerl_nvfp4.h"

struct Dim3 { uint32_t x, y, z; };
static std::map<const void*, std::string>& kernel_names() { static std::map<const void*, std::string> m; return m; }
static std::vector<std::string> launched;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle = nullptr; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) { kernel_names()[host] = device; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3*, Dim3*, size_t*, void**) { return 0; }
int hipLaunchKernel(const void* f, Dim3, Dim3, void**, size_t, void*) { launched.push_back(kernel_names()[f]); return 0; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x100000; return 0; }
}
static int count_launches(const char* kernel) {   // since the last call; null: of any kernel
  int n = 0;
  for (const std::string& k : launched) n += !kernel || k.find(kernel) != std::string::npos;
  return n;
}
int main() {
  int bad = 0;
  void* fake = (void*)0x10000;
  // validation paths (never reach a launch)
  bad += nvfp4_quantize(nullptr, 4, 32, 32, (uint8_t*)fake, (uint8_t*)fake, nullptr, fake, 1 << 20, nullptr) != QERL_ERR_NULL;
  bad += nvfp4_lora_linear(fake, 2, 40, 40, (const uint8_t*)fake, (const uint8_t*)fake, (const float*)fake, 16, nullptr, nullptr, 0, 0.f, fake, 16, fake, 1 << 24, nullptr) != QERL_ERR_SHAPE;
  bad += qerl_workspace_status(nullptr, nullptr) != QERL_ERR_NULL;
  bad += qerl_status_from_error_word(5) != QERL_ERR_TIMEOUT;
  // planners over a grid of shapes
  long plans = 0;
  const int64_t Hs[] = {128, 512, 1040, 2048, 3584, 4096, 5120, 8192}, Is[] = {64, 640, 2368, 4096, 13824, 18944, 27648};
  for (int M = 1; M <= 16; ++M)
    for (int64_t H : Hs)
      for (int64_t I : Is)
        for (int64_t r : {0, 8, 16, 64}) {
          bad += aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(M, H, I, H, r, r, r) == 0;
          ++plans;
        }
  for (int M : {1, 8, 16, 17, 64, 128, 300, 4096})
    for (int64_t H : Hs) {
      const int64_t Ns[3] = {H, 1024, 1024}, rs[3] = {64, 64, 64};
      bad += aqn_rmsnorm_nvfp4_lora_linear_group_workspace_bytes(M, H, Ns, rs, 3) == 0;
      bad += nvfp4_lora_linear_workspace_bytes(M, 27648, H, 64) == 0;
      bad += nvfp4_lora_linear_swiglu_workspace_bytes(M, H, 27648, 64) == 0;
      bad += nvfp4_lora_linear_backward_workspace_bytes(M, 27648, H, 64) == 0;
      bad += mxfp4_lora_linear_native_workspace_bytes(M, 27648, H, 64) < mxfp4_linear_native_workspace_bytes(M, 27648, H);
      qerl_backward_desc bd[3] = {};
      for (int i = 0; i < 3; ++i) { bd[i].N = Ns[i]; bd[i].r = 64; }
      bad += nvfp4_lora_linear_backward_group_workspace_bytes(M, H, bd, 3) < nvfp4_lora_linear_backward_workspace_bytes(M, H, H, 64);
      plans += 6;
    }
  {
    // the new entry points' validation: descriptors on the host, nothing launched
    qerl_backward_desc bd[2] = {};
    for (auto& d : bd) { d.dy_bf16 = fake; d.lddy = 32; d.N = 32; d.packed_t = fake; d.tensor_scale = (const float*)fake; d.r = 0; }
    bad += nvfp4_lora_linear_backward_group(nullptr, 4, 64, 64, bd, 2, fake, 64, nullptr, 0, nullptr) != QERL_ERR_WORKSPACE;
    bd[1].N = 30;
    bad += nvfp4_lora_linear_backward_group(nullptr, 4, 64, 64, bd, 2, fake, 64, fake, 1 << 20, nullptr) != QERL_ERR_SHAPE;
    bad += nvfp4_lora_linear_backward_group(nullptr, 4, 64, 64, bd, 5, fake, 64, fake, 1 << 20, nullptr) != QERL_ERR_SHAPE;
    bad += mxfp4_lora_linear_native(fake, 4, 64, 64, fake, 8, fake, fake, 12, 1.f, nullptr, fake, 8, fake, 1 << 30, nullptr) != QERL_ERR_SHAPE;
    bad += mxfp4_lora_linear_native(fake, 4, 64, 64, fake, 8, nullptr, fake, 8, 1.f, nullptr, fake, 8, fake, 1 << 30, nullptr) != QERL_ERR_NULL;
    bad += mxfp4_lora_linear_native(fake, 4, 64, 64, fake, 8, nullptr, nullptr, 0, 0.f, nullptr, fake, 8, fake, 16, nullptr) != QERL_ERR_WORKSPACE;
  }
  bad += nvfp4_prepack_bytes(27648, 5120) != (size_t)864 * 40 * 2304;
  // 9..16 tokens, ranks whose sums of x A^T alone exceed the workspace's area: the decode kernels, as below 9 tokens
  {
    const int64_t shapes[][4] = {{16, 1024, 1024, 512}, {9, 256, 2048, 512}, {16, 64, 1024, 512}, {9, 32, 1024, 296}, {9, 256, 1024, 384}};
    for (auto& s : shapes) {
      const int64_t M = s[0], N = s[1], K = s[2], r = s[3];
      launched.clear();
      bad += nvfp4_lora_linear_packed(fake, M, K, K, fake, (const float*)fake, N, fake, fake, r, 1.f, fake, N, fake, nvfp4_lora_linear_workspace_bytes(M, N, K, r), nullptr) != QERL_OK;
      bad += count_launches("panel") != 0 || count_launches("decode") == 0;
    }
    long walks = 0;
    for (int64_t M = 1; M <= 20; ++M)
      for (int64_t K : {16, 896, 1024, 1536, 4096})
        for (int64_t N : {1, 32, 129, 256, 1024, 5000})
          for (int64_t r : {0, 64, 72, 256, 296, 512, 1096, 4096}) {
            qerl_linear_desc d[3] = {};
            const int64_t Ns[3] = {N, 256, 40}, rs[3] = {r, r, 8};
            int64_t n_sum = 0, r_sum = 0;
            for (int i = 0; i < 3; ++i) {
              d[i].packed = fake; d[i].tensor_scale = (const float*)fake; d[i].N = d[i].ldy = Ns[i]; d[i].y_bf16 = fake; d[i].A_bf16 = d[i].B_bf16 = fake;
              d[i].r = rs[i]; d[i].lora_scale = 1.f;
              n_sum += Ns[i]; r_sum += rs[i];
            }
            bad += nvfp4_lora_linear_packed_group(fake, M, K, K, d, 3, fake, nvfp4_lora_linear_workspace_bytes(M, n_sum, K, r_sum), nullptr) != QERL_OK;
            bad += nvfp4_lora_linear_packed(fake, M, K, K, fake, (const float*)fake, N, fake, fake, r, 1.f, fake, N, fake, nvfp4_lora_linear_workspace_bytes(M, N, K, r), nullptr) != QERL_OK;
            bad += nvfp4_lora_linear_packed_swiglu(fake, fake, M, K, K, K, fake, (const float*)fake, N, fake, fake, r, 1.f, fake, N, fake, nvfp4_lora_linear_swiglu_workspace_bytes(M, N, K, r), nullptr) != QERL_OK;
            walks += 3;
          }
    printf("host check: %ld calls walked to their launches\n", walks);
  }
  // The composed calls on a workspace of the size that is asked for, and on the smallest that is accepted: never the one persistent
  // launch on the first (but a group without a norm up to 8 tokens, and a feed-forward block whose down has a bias), always on the
  // second where it is the smaller; up to 8 tokens and H = 8192 the size of that launch is enough for the separate ones.
  {
    long one_launch = 0, separate = 0;
    for (int64_t H : {512, 1024, 2048, 3584, 5120, 9216})
      for (int64_t I : {1024, 5504, 18944, 27648})
        for (int64_t r : {0, 16, 64})
          for (int64_t M : {1, 5, 8, 9, 12, 16}) {
            qerl_linear_desc g{}, d{};
            g.packed = fake; g.tensor_scale = (const float*)fake; g.N = g.ldy = I; g.y_bf16 = fake; g.A_bf16 = g.B_bf16 = fake; g.r = r;
            d = g;
            d.N = d.ldy = H;
            qerl_linear_desc grp[2] = {g, d};
            const int64_t Ns[2] = {I, H}, rs[2] = {r, r};
            for (int what = 0; what < 2; ++what) {
              auto call = [&](size_t bytes) {
                launched.clear();
                return what == 0 ? aqn_rmsnorm_nvfp4_lora_mlp(fake, M, H, H, fake, nullptr, 1e-6f, &g, &g, &d, fake, bytes, nullptr)
                                 : aqn_rmsnorm_nvfp4_lora_linear_group(fake, M, H, H, fake, nullptr, 1e-6f, grp, 2, fake, bytes, nullptr);
              };
              const size_t need = what == 0 ? aqn_rmsnorm_nvfp4_lora_mlp_workspace_bytes(M, H, I, H, r, r, r)
                                            : aqn_rmsnorm_nvfp4_lora_linear_group_workspace_bytes(M, H, Ns, rs, 2);
              bad += call(need) != QERL_OK || count_launches("block_kernel") != 0;
              ++separate;
              size_t lo = 0, hi = need / 256;
              while (hi - lo > 1) {
                const size_t mid = (lo + hi) / 2;
                (call(mid * 256) == QERL_OK ? hi : lo) = mid;
              }
              bad += call(hi * 256) != QERL_OK || call(hi * 256 - 256) != QERL_ERR_WORKSPACE;
              call(hi * 256);
              const int n = count_launches("block_kernel");
              bad += n != 0 && (n != 1 || count_launches(nullptr) != 1 || (M <= 8 && H <= 8192));
              one_launch += n;
            }
          }
    printf("host check: %ld composed calls as separate launches, %ld smallest workspaces with the one launch\n", separate, one_launch);
    bad += one_launch == 0;
  }
  printf("host check: %ld sizing calls, %d unexpected results\n", plans, bad);
  return bad != 0;
}
