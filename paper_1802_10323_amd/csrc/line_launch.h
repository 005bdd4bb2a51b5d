// line_launch.h - entry into the per-length transform kernels (r2r_line.h).
//
// 56 lengths x 2 types x 3 pipelines x 2 layouts are compiled as separate
// objects of one source (r2r_line_part.hip with POISSON_LINE_PART_INDEX = 0
// .. 7), so that the build uses every core.
#pragma once
#include <hip/hip_runtime.h>

#include "r2r_fast.h"

namespace poisson_dev {

// Complex lengths M = n/2 = 2^a 3^b 5^c in [12, 512], by part (dealt out by
// size so that the parts compile in about the same time).  Not 256: the staging
// forms of length 512 (r2r_async_kernel, r2r_regstage_kernel) have the better
// tiles there (along x 5.6 against 5.1 TB/s, along y 5.8 against 5.1).
#define POISSON_LINE_PART0(F) F(12) F(30) F(60) F(96) F(144) F(225) F(324) F(480)
#define POISSON_LINE_PART1(F) F(15) F(32) F(64) F(100) F(150) F(240) F(360) F(486)
#define POISSON_LINE_PART2(F) F(16) F(36) F(72) F(108) F(160) F(243) F(375) F(500)
#define POISSON_LINE_PART3(F) F(18) F(40) F(75) F(120) F(162) F(250) F(384) F(512)
#define POISSON_LINE_PART4(F) F(20) F(45) F(80) F(125) F(180) F(400)
#define POISSON_LINE_PART5(F) F(24) F(48) F(81) F(128) F(192) F(270) F(405)
#define POISSON_LINE_PART6(F) F(25) F(50) F(90) F(135) F(200) F(288) F(432)
#define POISSON_LINE_PART7(F) F(27) F(54) F(216) F(300) F(320) F(450)
#define POISSON_LINE_LENGTHS(F)                                                                   \
  POISSON_LINE_PART0(F) POISSON_LINE_PART1(F) POISSON_LINE_PART2(F) POISSON_LINE_PART3(F)         \
  POISSON_LINE_PART4(F) POISSON_LINE_PART5(F) POISSON_LINE_PART6(F) POISSON_LINE_PART7(F)

// Tile of length M for elements of `bytes` bytes: lines, threads, and waves per
// SIMD (registers: 512 / waves).  Measured on fields of 2^25 points, both
// directions and the types averaged (TB/s along x / y; FP32: us of one solve):
//  * short lengths: blocks of 256 threads, several to a CU, so that one's
//    loads and stores run during another's FFT (n = 192 in FP64: 16 lines and
//    256 threads 6.4 / 6.1, 32 lines and 512 threads 5.9 / 5.6; n = 128 in
//    FP32: 32 lines and 256 threads 115, 64 lines and 512 threads 124); 16 lines
//    are 128-byte rows on a strided axis, 32 lines of the shortest lengths 256
//    (n = 128 along y 5.5 against 5.3);
//  * past M = 135 a line has work for 32 threads (n = 480: 16 lines and 512
//    threads 6.0 / 5.9, 8 lines and 256 threads 5.6 / 5.2, 32 lines, one block
//    to a CU, 4.9 / 4.6);
//  * past M = 256 in FP64 the 16-line tile fills the LDS: one block with 256
//    registers.  On the contiguous axis, where short rows cost nothing, 8
//    lines while two blocks fit (n = 800 along x 4.9 against 4.5; along y 4.4
//    against 4.3 the other way on n = 640, 3.6 against 4.4 on n = 1024).  FP32
//    keeps two blocks (n = 1024: 489 against 641 us with one).
struct LineShape {
  int nl, nt, waves;
};
constexpr LineShape line_shape(int bytes, int m, int layout) {
  if (bytes == 4)
    return m <= 64 ? LineShape{32, 256, 4} : m <= 270 ? LineShape{32, 512, 4} : LineShape{16, 512, 4};
  if (m <= 64) return LineShape{layout == 0 ? 32 : 16, 256, 4};
  if (m <= 135) return LineShape{16, 256, 4};
  if (m <= 256) return LineShape{16, 512, 4};
  return layout == 1 && m <= 405 ? LineShape{8, 512, 4} : LineShape{16, 512, 2};
}

// Launch the transform of complex length M described by `a` (arguments as for
// r2r_fast_kernel, the geometry made for line_shape(sizeof(T), M, layout).nl
// lines).
// hipErrorInvalidValue if the length has no kernel.
#define POISSON_LINE_DECLARE(M_)                                                  \
  hipError_t line_launch_##M_(const R2RFastArgs<double>& a, hipStream_t stream);  \
  hipError_t line_launch_##M_(const R2RFastArgs<float>& a, hipStream_t stream);
POISSON_LINE_LENGTHS(POISSON_LINE_DECLARE)
#undef POISSON_LINE_DECLARE

// A kernel of part I (see async_kernel).
template <int I>
const void* line_part_kernel();
#define POISSON_LINE_PART_DECLARE(I_) template <> const void* line_part_kernel<I_>();
POISSON_LINE_PART_DECLARE(0) POISSON_LINE_PART_DECLARE(1) POISSON_LINE_PART_DECLARE(2)
POISSON_LINE_PART_DECLARE(3) POISSON_LINE_PART_DECLARE(4) POISSON_LINE_PART_DECLARE(5)
POISSON_LINE_PART_DECLARE(6) POISSON_LINE_PART_DECLARE(7)
#undef POISSON_LINE_PART_DECLARE

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
