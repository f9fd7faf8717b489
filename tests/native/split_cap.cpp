// Walks the host dispatch of the decoder GEMMs over row counts, widths, depths and split
// caps, and reads the split-K factor each launch chose: a launch that takes more than its
// cap writes past the partial-sum buffer that the cap was worked out from.  Nothing is
// launched: without a GPU the call ends in hipErrorNoDevice, its choice already made.
// Prints one line per kernel path: path, launches, launches above one split, over the cap;
// then the refused shapes of widths and depths that are multiples of 64
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
  const char* names[] = {"few", "stream", "tile", "staged"};
  int n[4] = {}, split[4] = {}, over[4] = {}, refused = 0;
  for (int N : {64, 192, 256, 384, 512, 640, 1024, 2048, 4096, 5120, 8192})
    for (int K : {32, 64, 96, 512, 1024, 2048, 4096, 5120, 5504, 11008, 13824})
      for (int cap = 1; cap <= 8; ++cap)
        for (int M = 1; M <= 4200; M += M < 300 ? 1 : 37) {
          GemmArgs a{};
          a.K = a.lda = K;
          a.epilogue = EPI_PARTIAL_F32;
          a.ngroups = 1;
          a.g[0] = GemmGroup{p, nullptr, M, p, nullptr, N, p, N, (int64_t)M * N, 0, 0, 0};
          a.split = 0;
          const hipError_t e = launch_gemm_bf16(a, cap, nullptr);
          (void)hipGetLastError();
          if (e == hipErrorInvalidValue) {  // a shape no kernel takes
            refused += N % 64 == 0 && K % 64 == 0;
            continue;
          }
          const int path = M <= 4 ? 0 : (M <= 256 ? 1 : (N % 256 == 0 && K % 64 == 0 ? 2 : 3));
          ++n[path];
          split[path] += a.split > 1;
          over[path] += a.split > cap || a.split < 1;
        }
  for (int i = 0; i < 4; ++i) printf("%s %d %d %d\n", names[i], n[i], split[i], over[i]);
  printf("refused %d\n", refused);
  return 0;
}
