// Tile variant 21 of tile_variants.def.
#define GEMM_TILE_VARIANT_INDEX 21
#include "tile_variant.inc"
