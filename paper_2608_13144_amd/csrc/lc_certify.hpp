// What the two certification paths share (gfx950 only).
#pragma once

#include "lc_common.hpp"

namespace lc {

constexpr double kSqrt2 = 1.4142135623730951;  // float64 nearest to sqrt(2)

// Label of a row the float16 filter could not settle; never a class.
constexpr int32_t kCertPending = -2147483647 - 1;

// (w1, j1, w2): top-1, its class and top-2 of another set of classes.
__device__ __forceinline__ void top2_merge(double w1, int j1, double w2, double& v1, int& i1, double& v2) {
  if (w1 > v1 || (w1 == v1 && j1 < i1)) {
    v2 = v1 > v2 ? v1 : v2;
    v1 = w1;
    i1 = j1;
  } else {
    v2 = w1 > v2 ? w1 : v2;
  }
  v2 = w2 > v2 ? w2 : v2;
}

// Certification of N rows through the float16 filter (certify_filter.hip):
// label, radius, margin and norm of every row, or kCertPending as the label
// (and nothing else but the norm) of a row it leaves to the float64 kernel.
bool certify_filter_takes(int64_t N, int32_t d, int32_t C);
hipError_t certify_filter_run(const float* z, int64_t N, int32_t d, const float* W, const float* b, int32_t C,
                              double sigma, bool bf16, bool tight, const double* row_dist, int32_t* label_out,
                              float* r_out, float* margin_out, float* norm2_out, void* head_ws, hipStream_t s);

}  // namespace lc
