// GEMM on packed weights, epilogue 3: fp32 tiles out and arg-max over the columns (LM head, up to 128 rows).  (A source file each, so that they compile side by side.)
#include "esp_gemm_tile.h"

hipError_t launch_gemm_tile_both(hipStream_t st, const TileGemm& g) { return tile_dispatch<3>(st, g); }
hipError_t gemm_tile_both_prepare() { return tile_prepare<3>(); }
