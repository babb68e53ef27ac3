// Walks the host side of the C ABI with the HIP runtime and the kernel launchers stubbed out (every stub returns
// success; only the allocators hand out memory): run under a sanitizer, see test_host_api.py.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime.h>
#ifndef __align__
#define __align__(n) __attribute__((aligned(n)))
#endif
#ifndef HIP_SYMBOL
#define HIP_SYMBOL(x) (&x)
#endif
#include "../paper_2401_05031_amd/csrc/api.hip"

// (the runtime's header gives each allocator's exact signature; the stubs below are the functions themselves)
extern "C" hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(1, n); return hipSuccess; }
extern "C" hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
extern "C" hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
extern "C" hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
extern "C" hipError_t hipGetSymbolAddress(void** p, const void*) { static int32_t cell[64]; *p = cell; return hipSuccess; }

#define CHECK(e) do { if (!(e)) { std::fprintf(stderr, "line %d: %s\n", __LINE__, #e); return 1; } } while (0)

int main() {
  static char dev[64];   // stands for device memory: no stub touches it
  void* p = dev;
  const int queries[] = {1, 3, 480, 481};   // 480 is the most whose plan the device expands
  for (int dtype : {(int)OTAS_F32, (int)OTAS_BF16})
    for (int lanes : {1, 3}) {
      const otas_model_desc d = {3, 64, 1, 128, dtype, 1e-6f, 1};
      std::vector<otas_layer_weights> w(d.L);
      for (auto& l : w) std::fill((const void**)&l, (const void**)(&l + 1), p);
      otas_ctx* c = nullptr;
      CHECK(otas_create(&c, &d, w.data(), nullptr) == OTAS_OK);
      CHECK(otas_set_lanes(c, lanes) == OTAS_OK);
      for (int B : queries)
        for (int r : {0, 3}) {
          std::vector<int32_t> off(B + 1), out(B + 1), take(B, r), prm(B + 1);
          for (int q = 0; q < B; ++q) { off[q + 1] = off[q] + 5 + q % 9; prm[q + 1] = prm[q] + q % 3; }
          void* ws = (void*)(uintptr_t)256;
          int32_t* sz = (int32_t*)p;
          for (uint32_t flags : {0u, (uint32_t)(OTAS_FLAG_SIZE_BIAS | OTAS_FLAG_TRACE)})
            CHECK(otas_encoder_forward(c, p, off.data(), take.data(), B, flags, ws, (size_t)1 << 40, dev + 8, sz,
                                       out.data(), sz, sz) == OTAS_OK);
          for (int q = 0; q < B; ++q) {
            int32_t len[4];
            CHECK(otas_schedule(5 + q % 9, 0, r, 1, d.L, len) == OTAS_OK && out[q + 1] - out[q] == len[d.L]);
          }
          CHECK(otas_encoder_layers(c, 1, 3, p, sz + 1, off.data(), take.data(), B, 0, ws, (size_t)1 << 40, dev + 8, sz,
                                    out.data(), nullptr, nullptr) == OTAS_OK);
          for (int mode : {(int)OTAS_PROMPT_REPLACE, (int)OTAS_PROMPT_GROW})
            CHECK(otas_encoder_forward_deep(c, p, off.data(), B, mode, p, prm.data(), ws, (size_t)1 << 40, dev + 8, sz,
                                            out.data()) == OTAS_OK);
          CHECK(otas_prompt_prepend(c, p, off.data(), p, prm.data(), B, dev + 8, out.data()) == OTAS_OK);
          CHECK(otas_token_merge(c, p, p, 64, nullptr, off.data(), take.data(), B, ws, (size_t)1 << 40, dev + 8, sz,
                                 out.data(), nullptr, nullptr) == OTAS_OK);
          std::vector<otas_task_head> heads(3, otas_task_head{p, p, 7});
          CHECK(otas_task_heads(c, (float*)p, off.data(), std::vector<int32_t>(B, 2).data(), B, heads.data(), 3, p, p,
                                (float*)p, 8) == OTAS_OK);
        }
      CHECK(otas_destroy(c) == OTAS_OK);
    }
  std::puts("host api ok");
  return 0;
}
