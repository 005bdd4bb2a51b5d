// line_launch.h - entry into the per-length transform kernels (r2r_line.h).
//
// 58 lengths x 2 types x 3 pipelines x 2 layouts are compiled as separate
// objects of one source (r2r_line_part.hip with POISSON_LINE_PART_INDEX = 0
// .. 7),
// so that the build uses every core.
#pragma once
#include <hip/hip_runtime.h>

#include "r2r_fast.h"

namespace poisson_dev {

// Complex lengths M = n/2 = 2^a 3^b 5^c in [12, 512], by part (dealt out by
// size so that the parts compile in about the same time).
#define POISSON_LINE_PART0(F) F(12) F(30) F(60) F(96) F(144) F(225) F(324) F(480)
#define POISSON_LINE_PART1(F) F(15) F(32) F(64) F(100) F(150) F(240) F(360) F(486)
#define POISSON_LINE_PART2(F) F(16) F(36) F(72) F(108) F(160) F(243) F(375) F(500)
#define POISSON_LINE_PART3(F) F(18) F(40) F(75) F(120) F(162) F(250) F(384) F(512)
#define POISSON_LINE_PART4(F) F(20) F(45) F(80) F(125) F(180) F(256) F(400)
#define POISSON_LINE_PART5(F) F(24) F(48) F(81) F(128) F(192) F(270) F(405)
#define POISSON_LINE_PART6(F) F(25) F(50) F(90) F(135) F(200) F(288) F(432)
#define POISSON_LINE_PART7(F) F(27) F(54) F(216) F(300) F(320) F(450)
#define POISSON_LINE_LENGTHS(F)                                                                   \
  POISSON_LINE_PART0(F) POISSON_LINE_PART1(F) POISSON_LINE_PART2(F) POISSON_LINE_PART3(F)         \
  POISSON_LINE_PART4(F) POISSON_LINE_PART5(F) POISSON_LINE_PART6(F) POISSON_LINE_PART7(F)

// Tile of length M for elements of `bytes` bytes: lines and threads.  On a
// strided axis a tile's rows are nl elements, so wide tiles use each DRAM page
// better; the tile and its twiddles have to leave room in the 160 KiB of LDS
// for a second block (its FFT runs while the other's loads and stores move)
// up to M = 256 in FP64.  Beyond, 16 lines (128-byte rows) fill the LDS and
// one block has a CU to itself.
struct LineShape {
  int nl, nt;
};
constexpr LineShape line_shape(int bytes, int m) {
  const int rows = m * bytes / 8;   // FP32 lines are half as long in bytes
  const int nt = rows <= 15 ? 256 : 512;
  const int nl = rows <= 72 ? 64 : rows <= 135 ? 32 : rows <= 256 ? 16 : 16;
  return LineShape{nl * (bytes == 4 && m > 256 ? 2 : 1), nt};
}

// Launch the transform of complex length M described by `a` (arguments as for
// r2r_fast_kernel, the geometry made for line_shape(sizeof(T), M).nl lines).
// hipErrorInvalidValue if the length has no kernel.
#define POISSON_LINE_DECLARE(M_)                                                  \
  hipError_t line_launch_##M_(const R2RFastArgs<double>& a, hipStream_t stream);  \
  hipError_t line_launch_##M_(const R2RFastArgs<float>& a, hipStream_t stream);
POISSON_LINE_LENGTHS(POISSON_LINE_DECLARE)
#undef POISSON_LINE_DECLARE

constexpr bool line_length(int m) {
  switch (m) {
#define POISSON_LINE_CASE(M_) case M_:
    POISSON_LINE_LENGTHS(POISSON_LINE_CASE)
#undef POISSON_LINE_CASE
    return true;
    default: return false;
  }
}

template <typename T>
inline hipError_t line_transform_launch(const R2RFastArgs<T>& a, int m, hipStream_t stream) {
  switch (m) {
#define POISSON_LINE_CASE(M_) case M_: return line_launch_##M_(a, stream);
    POISSON_LINE_LENGTHS(POISSON_LINE_CASE)
#undef POISSON_LINE_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace poisson_dev
