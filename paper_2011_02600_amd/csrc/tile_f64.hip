// The tile stage kernel in double precision.
#define SBP_TILE_F64
#include "tile.hip"
