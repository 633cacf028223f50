// Tile variant 20 of tile_variants.def.
#define GEMM_TILE_VARIANT_INDEX 20
#include "tile_variant.inc"
