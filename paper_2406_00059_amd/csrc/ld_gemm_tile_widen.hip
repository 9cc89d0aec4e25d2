// The big-tile kernel on one fp16 term of the activations, on the bf16 matrix, widened in the kernel.
#include "ld_gemm_tile_kernel.h"

void ldt::launch_tile_widen(int bm, int bn, const TileLaunch &l) {
#define LD_TILE(AT_, BT_, US_) \
    if (bm == AT_ * 32 && bn == BT_ * 32) return launch_tile_epilogue<1, 1, AT_, BT_>(l);
    LD_TILES_F16(LD_TILE)
#undef LD_TILE
}
