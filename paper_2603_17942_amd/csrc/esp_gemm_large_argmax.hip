// Large-tile GEMM, epilogue 1: arg-max over the columns (LM head at many tree rows).  (A source file each, so that they compile side by side.)
#include "esp_gemm_large.h"

hipError_t launch_gemm_large_argmax(hipStream_t st, const LargeGemm& g) { return large_dispatch<1>(st, g); }
hipError_t gemm_large_argmax_prepare() { return large_prepare<1>(); }
