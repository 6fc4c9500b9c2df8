// Large-tile GEMM, epilogue 2: SwiGLU of the gate/up projection.  (A source file each, so that they compile side by side.)
#include "esp_gemm_large.h"

hipError_t launch_gemm_large_swiglu(hipStream_t st, const LargeGemm& g) { return large_dispatch<2>(st, g); }
hipError_t gemm_large_swiglu_prepare() { return large_prepare<2>(); }
