// The layer products on the integer matrix cores: their launch (which calls take them: `digits_plan`).
#pragma once
#include "common.hpp"
#include "gemm_rules.hpp"

namespace csgs {

template <int MODE>
void launch_digits(const DigitsPlan &d, const float *A, int64_t lda, const float *B, int64_t ldb, float *C, int64_t ldc, int M, int N, int K,
                   const int32_t *M_dev, hipStream_t st, const CompInst &ci);

}  // namespace csgs
