// GEMM on packed weights, epilogue 2: SwiGLU of the gate/up projection.  (A source file each, so that they compile side by side.)
#include "esp_gemm_tile.h"

hipError_t launch_gemm_tile_swiglu(hipStream_t st, const TileGemm& g) { return tile_dispatch<2>(st, g); }
hipError_t gemm_tile_swiglu_prepare() { return tile_prepare<2>(); }
