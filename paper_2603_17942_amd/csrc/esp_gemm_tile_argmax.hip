// GEMM on packed weights, epilogue 1: arg-max over the columns (LM head).  (A source file each, so that they compile side by side.)
#include "esp_gemm_tile.h"

hipError_t launch_gemm_tile_argmax(hipStream_t st, const TileGemm& g) { return tile_dispatch<1>(st, g); }
hipError_t gemm_tile_argmax_prepare() { return tile_prepare<1>(); }
