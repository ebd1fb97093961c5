// The launches of the one-workgroup subspace step, recorded on the host: the
// sweep limit that reaches the kernels against the rotation log's size.
// Prints n, mode, sweeps asked for, and the largest limit a kernel received.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <utility>

static int g_sweeps;
template <typename... A>
static void record_last(A... a) {
  const long long v[] = {(long long)a...};
  g_sweeps = (int)v[sizeof...(a) - 1];
}
struct Recorder {
  template <typename G, typename B, typename L, typename S, typename D>
  void operator()(G, B, L, S, D) {}  // kernels of the descriptors alone
  template <typename G, typename B, typename L, typename S, typename D, typename... A>
  void operator()(G, B, L, S, D, A... a) {
    record_last(a...);
  }
};
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, ...) Recorder()(__VA_ARGS__)
#include "../../paper_1603_02732_amd/csrc/kernels_sub.hip"

namespace sgo {
void check_launch(const char*) {}
void allow_lds(const void*) {}
void launch_sub_congruence(hipStream_t, const CandDesc*, int, int) {}
}  // namespace sgo

int main() {
  for (int n = 33; n <= sgo::kJacWideMax; ++n)  // up to 32 bands nothing is logged
    for (int asked : {1, 39, 40, 41, 66, 1000, 2000000000}) {
      g_sweeps = 0;
      sgo::launch_sub_block(nullptr, nullptr, 1, n, 3, asked);
      const int n2 = n + (n & 1), m = n2 - 1, np = n2 / 2;
      const long long rotations = (long long)g_sweeps * m * np;
      const long long room = ((long long)sgo::jac_log_doubles(n, sgo::kJacMaxSweeps) - sgo::kJacLog) / 2;
      std::printf("%d %d %d %lld %lld\n", n, asked, g_sweeps, rotations, room);
    }
  return 0;
}
