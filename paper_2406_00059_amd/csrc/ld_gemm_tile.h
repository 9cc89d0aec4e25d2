// The big-tile kernel (products of more than 64 rows): what its three translation units (two terms, one on the fp16 image, one on the
// bf16 matrix) share with the planner.
#pragma once
#include "ld_gemm.h"
#include "ld_device.h"
#include "ld_internal.h"
#include <utility>

namespace ldt {

using ldd::bf16_t;

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // native 16-byte vector (keeps arrays of it in registers)

// Tiles of the two forms, in units of 32 rows and 32 columns, and measured us per 64-wide chunk of K: of the two-term form with two
// stages in LDS (see plan_big), of the one-term form as it runs, whose smallest tile has one time for two and three stages (the
// latter, in launches of up to one workgroup a CU, 11 % faster).  (Odd column units have no SwiGLU form.)
#define LD_TILES_TWO(X) \
    X(3, 4, 0.73) X(3, 6, 1.03) X(3, 8, 1.23) X(4, 4, 0.96) X(4, 6, 1.21) X(4, 8, 1.50) X(5, 6, 1.42) X(5, 8, 1.77) X(6, 6, 1.61) X(6, 8, 2.04)
#define LD_TILES_F16(X) X(4, 6, 0.74) X(4, 8, 0.91) X(6, 6, 0.95) X(6, 8, 1.16) X(7, 8, 1.30) X(8, 5, 0.99) X(8, 6, 1.15) X(8, 8, 1.42)

constexpr int TILE_MAX_K = 1 << 23;      // the lane offsets of the copies reach over 256 rows in 32 bits
// Stages of K chunks in LDS: three where they fit, else two.  The smallest tiles, two workgroups of which fit a CU with two stages
// each, keep two where a launch has more than one workgroup a CU (12288 x 4096 at 480 rows in 96 x 128 tiles: 98 us so, 104 with three).
constexpr int tile_lds(int terms, int bm, int bn, int stages) { return stages * (terms * bm + bn) * 128; }
constexpr int LDS_BYTES = 160 * 1024;
constexpr int tile_stages(int terms, int bm, int bn) { return tile_lds(terms, bm, bn, 3) <= LDS_BYTES ? 3 : 2; }
constexpr bool tile_twice(int terms, int bm, int bn) { return 2 * tile_lds(terms, bm, bn, 2) <= LDS_BYTES; }

// One launch: grid workgroups for n_ttiles row tiles, all column blocks and ks slabs of K.
struct TileLaunch {
    const uint16_t *W;
    const bf16_t *hi, *lo;
    int T, N, K, epi;
    float *y;
    int n_ttiles, ks;
    float *partial;
    ld::OperandImage out;
    bool quads;
    int grid;
    hipStream_t s;
};
void launch_tile_two(int bm, int bn, const TileLaunch &l);
void launch_tile_image(int bm, int bn, const TileLaunch &l);      // l.W: the matrix's fp16 image
void launch_tile_widen(int bm, int bn, const TileLaunch &l);      // l.W: the bf16 matrix

// Eight bf16 numbers as fp16: exact where fp16 can hold the value (8 significant bits fit into 11; truncation
// only below 2^-14, where a bf16 weight is lost in the sums anyway).
__device__ __forceinline__ f16x8 bf16x8_to_f16x8(const __attribute__((ext_vector_type(4))) uint32_t &w) {
    uint32_t h[4];
#pragma unroll
    for (int i = 0; i < 4; i++)
        h[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w[i] << 16), __uint_as_float(w[i] & 0xffff0000u)));
    return __builtin_bit_cast(f16x8, (__attribute__((ext_vector_type(4))) uint32_t){h[0], h[1], h[2], h[3]});
}

// SwiGLU of one (gate, up) pair with the last product rounded to float, as a store to memory would: where the
// value goes straight into the bf16 split, a product fused into the split's subtraction would change the low part.
__device__ __forceinline__ float swiglu(float gate, float up) {
#pragma clang fp contract(off)
    return gate / (1.0f + __expf(-gate)) * up;
}

}  // namespace ldt
