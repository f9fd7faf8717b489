// Walks the host dispatch of the fused Q, K, V GEMMs over row counts, query counts
// and widths, with the groups and split cap of a prefill layer.  On a machine
// without a GPU a launch that the dispatch accepts ends in hipErrorNoDevice, one
// that it refuses in hipErrorInvalidValue.  Prints one line per width:
//   d, fused sizes, sizes with two launches, refused launches
#include <algorithm>
#include <cstdio>

#include "kernels.h"

using namespace spider;

int main() {
  int devices = 0;
  if (hipGetDeviceCount(&devices) == hipSuccess && devices > 0) {
    printf("a GPU is present: nothing is launched\n");  // the pointers below are not memory
    return 2;
  }
  void* p = reinterpret_cast<void*>(1 << 20);
  for (int d : {256, 1024, 2048, 3072, 4096, 5120, 6656, 8192}) {
    int fused = 0, apart = 0, refused = 0;
    auto launch = [&](GemmArgs g, int cap) {
      const hipError_t e = launch_gemm_bf16(g, cap, nullptr);
      (void)hipGetLastError();
      if (e == hipErrorInvalidValue) ++refused;
    };
    for (int R = 257; R <= 9000; R += R < 2100 ? 1 : 13)
      for (int nA : {0, 1, 4, 5, 64, 129, 256, 257, R}) {
        if (nA > R) continue;
        GemmArgs a{};
        a.K = a.lda = d;
        a.epilogue = EPI_PARTIAL_F32;
        const int M[3] = {nA, R, R};
        for (int i = nA ? 0 : 1; i < 3; ++i)
          a.g[a.ngroups++] = GemmGroup{p, nullptr, M[i], p, nullptr, d, p, d, (int64_t)R * d, 0, 0, 0};
        const int cap = std::min(2, std::max(1, std::min(8, 4096 / R)));
        if (!gemm_qkv_fused(a, cap)) continue;
        ++fused;
        const bool two = gemm_qkv_q_apart(a, cap);
        a.epilogue = EPI_QKV_BF16;
        a.rope = reinterpret_cast<const float2*>(p);
        a.pos = reinterpret_cast<const int32_t*>(p);
        a.ldvt = (R + 31) / 32 * 32;
        for (int i = 0; i < a.ngroups; ++i) a.g[i].kind = i == a.ngroups - 1 ? 2 : 1;
        if (!two) {
          launch(a, cap);
          continue;
        }
        ++apart;
        GemmArgs q = a;
        q.ngroups = 1;
        launch(q, cap);
        a.ngroups = 2;
        a.g[0] = a.g[1];
        a.g[1] = a.g[2];
        launch(a, cap);
      }
    printf("%d %d %d %d\n", d, fused, apart, refused);
  }
  return 0;
}
