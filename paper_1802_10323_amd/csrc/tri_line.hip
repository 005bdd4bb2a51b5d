// tri_line.hip - the elimination kernels of any line length (tri_line.h).
#include <hip/hip_runtime.h>

#include "async_launch.h"
#include "tri_line.h"

namespace poisson_dev {

namespace {

template <typename T, int RPC, int P, int NL, int W>
hipError_t launch(const TriFastArgs<T>& a, hipStream_t st) {
  void (*k)(TriFastArgs<T>) =
      a.g.layout == 0 ? tri_line_kernel<T, RPC, P, NL, W, 0> : tri_line_kernel<T, RPC, P, NL, W, 1>;
  const int blocks =
      async_resident_blocks(reinterpret_cast<const void*>(k), a.g.ntiles, NL * P);
  hipLaunchKernelGGL(k, dim3(blocks), dim3(NL * P), 0, st, a);
  return hipGetLastError();
}

// The launch of n's chunking, among those of the lengths from N on (one for
// each number of virtual rows)
template <typename T, int N>
hipError_t launch_n(const TriFastArgs<T>& a, int n, hipStream_t st) {
  if constexpr (N > 512) {
    return hipErrorInvalidValue;
  } else {
    constexpr TriLineShape S = tri_line_shape(N);
    if (tri_line_shape(n).rpc == S.rpc && tri_line_shape(n).p == S.p)
      return launch<T, S.rpc, S.p, S.nl, S.waves>(a, st);
    return launch_n<T, S.rpc * S.p + 1>(a, n, st);
  }
}

}  // namespace

const void* tri_line_kernel_any() {
  constexpr TriLineShape S = tri_line_shape(17);
  return reinterpret_cast<const void*>(&tri_line_kernel<double, S.rpc, S.p, S.nl, S.waves, 0>);
}

hipError_t line_elimination_launch(const TriFastArgs<double>& a, int n, hipStream_t stream) {
  return launch_n<double, 17>(a, n, stream);
}

hipError_t line_elimination_launch(const TriFastArgs<float>& a, int n, hipStream_t stream) {
  return launch_n<float, 17>(a, n, stream);
}

}  // namespace poisson_dev
