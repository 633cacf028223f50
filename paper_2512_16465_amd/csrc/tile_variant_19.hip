// Tile variant 19 of tile_variants.def.
#define GEMM_TILE_VARIANT_INDEX 19
#include "tile_variant.inc"
