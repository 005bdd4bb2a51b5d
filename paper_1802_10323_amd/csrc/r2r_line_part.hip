// r2r_line_part.hip - the per-length transform kernels (r2r_line.h) of one
// part of the lengths (POISSON_LINE_PART_INDEX, line_launch.h).
#include <hip/hip_runtime.h>

#include "async_launch.h"
#include "line_launch.h"
#include "r2r_line.h"

namespace poisson_dev {

// FP64 values of a radix-20 or radix-25 butterfly take more than 128 registers
template <typename T, int M, int LAYOUT>
using LineTile = LineCfg<M, line_shape(sizeof(T), M, LAYOUT).nl, line_shape(sizeof(T), M, LAYOUT).nt,
                         sizeof(T) == 8 && line_shape(sizeof(T), M, LAYOUT).waves == 4 ? 18 : 25>;

template <typename T, int M, int LAYOUT>
static hipError_t line_launch_layout(const R2RFastArgs<T>& a, hipStream_t stream) {
  constexpr LineShape S = line_shape(sizeof(T), M, LAYOUT);
  using C = LineTile<T, M, LAYOUT>;
  void (*k)(R2RFastArgs<T>) = a.kind >= K_ND ? r2r_line_kernel<T, C, PIPE_IV, LAYOUT, S.waves>
                              : a.inverse    ? r2r_line_kernel<T, C, PIPE_INV, LAYOUT, S.waves>
                                             : r2r_line_kernel<T, C, PIPE_FWD, LAYOUT, S.waves>;
  const int blocks = async_resident_blocks(reinterpret_cast<const void*>(k), a.g.ntiles, S.nt);
  hipLaunchKernelGGL(k, dim3(blocks), dim3(S.nt), 0, stream, a);
  return hipGetLastError();
}

template <typename T, int M>
static hipError_t line_launch(const R2RFastArgs<T>& a, hipStream_t stream) {
  return a.g.layout == 0 ? line_launch_layout<T, M, 0>(a, stream) : line_launch_layout<T, M, 1>(a, stream);
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

#define POISSON_LINE_M(M_) M_,
template <>
const void* line_part_kernel<POISSON_LINE_PART_INDEX>() {
  constexpr int m[] = {POISSON_CAT(POISSON_LINE_PART, POISSON_LINE_PART_INDEX)(POISSON_LINE_M)};
  constexpr int M = m[0];
  return reinterpret_cast<const void*>(
      &r2r_line_kernel<double, LineTile<double, M, 0>, PIPE_FWD, 0, line_shape(8, M, 0).waves>);
}

}  // namespace poisson_dev
