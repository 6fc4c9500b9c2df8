// Large-tile GEMM, epilogue 0: fp32 tiles (or split-K partials) out.  (A source file each, so that they compile side by side.)
#include "esp_gemm_large.h"

hipError_t launch_gemm_large_out(hipStream_t st, const LargeGemm& g) { return large_dispatch<0>(st, g); }
hipError_t gemm_large_out_prepare() { return large_prepare<0>(); }
