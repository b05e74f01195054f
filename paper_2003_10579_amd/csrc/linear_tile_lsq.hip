// The least-squares instances of the steady-state kernel, compiled beside those of softmax regression (half the build time).
#define SSGD_TILE_LSQ
#include "linear_tile.hip"
