// r2r_line_part.hip - the per-length transform kernels (r2r_line.h) of one
// part of the lengths (POISSON_LINE_PART_INDEX, line_launch.h).
#include <hip/hip_runtime.h>

#include "async_launch.h"
#include "line_launch.h"
#include "r2r_line.h"

namespace poisson_dev {

template <typename T, int M>
static hipError_t line_launch(const R2RFastArgs<T>& a, hipStream_t stream) {
  constexpr LineShape S = line_shape(sizeof(T), M);
  using C = LineCfg<M, S.nl, S.nt>;
  using L = LineLayout<T, C>;
  // waves per SIMD that the LDS allows
  constexpr int W = 80 * 1024 / L::lds_bytes(PIPE_IV) > 0 ? 4 : 2;
  void (*k)(R2RFastArgs<T>) = nullptr;
  const int pipe = a.kind >= K_ND ? PIPE_IV : a.inverse ? PIPE_INV : PIPE_FWD;
  switch (pipe * 2 + a.g.layout) {
    case 0: k = r2r_line_kernel<T, C, PIPE_FWD, 0, W>; break;
    case 1: k = r2r_line_kernel<T, C, PIPE_FWD, 1, W>; break;
    case 2: k = r2r_line_kernel<T, C, PIPE_INV, 0, W>; break;
    case 3: k = r2r_line_kernel<T, C, PIPE_INV, 1, W>; break;
    case 4: k = r2r_line_kernel<T, C, PIPE_IV, 0, W>; break;
    default: k = r2r_line_kernel<T, C, PIPE_IV, 1, W>; break;
  }
  const int blocks = async_resident_blocks(reinterpret_cast<const void*>(k), a.g.ntiles, S.nt);
  hipLaunchKernelGGL(k, dim3(blocks), dim3(S.nt), 0, stream, a);
  return hipGetLastError();
}

#define POISSON_LINE_DEFINE(M_)                                                    \
  hipError_t line_launch_##M_(const R2RFastArgs<double>& a, hipStream_t stream) {  \
    return line_launch<double, M_>(a, stream);                                     \
  }                                                                                \
  hipError_t line_launch_##M_(const R2RFastArgs<float>& a, hipStream_t stream) {   \
    return line_launch<float, M_>(a, stream);                                      \
  }

#define POISSON_CAT2(a, b) a##b
#define POISSON_CAT(a, b) POISSON_CAT2(a, b)
POISSON_CAT(POISSON_LINE_PART, POISSON_LINE_PART_INDEX)(POISSON_LINE_DEFINE)

}  // namespace poisson_dev
