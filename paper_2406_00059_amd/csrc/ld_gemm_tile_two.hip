// The big-tile kernel on two bf16 terms of the activations.
#include "ld_gemm_tile_kernel.h"

void ldt::launch_tile_two(int bm, int bn, const TileLaunch &l) {
#define LD_TILE(AT_, BT_, US_) \
    if (bm == AT_ * 32 && bn == BT_ * 32) return launch_tile_epilogue<2, 0, AT_, BT_>(l);
    LD_TILES_TWO(LD_TILE)
#undef LD_TILE
}
