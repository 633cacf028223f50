// Tile variant 18 of tile_variants.def.
#define GEMM_TILE_VARIANT_INDEX 18
#include "tile_variant.inc"
