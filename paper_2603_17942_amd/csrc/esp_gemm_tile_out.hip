// GEMM on packed weights, epilogue 0: fp32 tiles (or split-K partials) out.  (A source file each, so that they compile side by side.)
#include "esp_gemm_tile.h"

hipError_t launch_gemm_tile_out(hipStream_t st, const TileGemm& g) { return tile_dispatch<0>(st, g); }
hipError_t gemm_tile_out_prepare() { return tile_prepare<0>(); }
