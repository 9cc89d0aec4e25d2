// Linear layers on T >= 2 rows with the matrix cores: Y[T, N] = X[T, K] W[N, K]^T, W bf16.
//
// Precision: the float32 activations are split into two bf16 numbers, x = hi + lo (|lo| <= 2^-9 |hi|),
// and both parts are multiplied with the (exact) bf16 weights and accumulated in float32, so the
// product carries ~16 significant bits of the activation instead of 8.  In the decode regime the
// kernel is bound by the weight stream from HBM, where the second MFMA pass is free.
//
// Two kinds of kernel by row count, fed by images of the activations (two bf16 terms, or one fp16 term where the caller allows it),
// which k_norm_split writes in a pass of its own or a producer writes directly (k_reduce_add_norm_split and the SwiGLU
// epilogues, the attention kernels, the fused reducers of ld_batch.hip):
//  - k_gemm_skinny (2..64 rows): weight-stream bound, see its comment.  It also takes the float rows themselves.
//  - k_gemm_tile (> 64 rows, ld_gemm_tile_kernel.h): MFMA-bound; both operands through LDS, see its comment.
// Workgroups that share a W panel (same columns, different token tiles) are mapped to the same XCD so
// that the panel is fetched into one L2 only.  Split-K partial sums are added in fixed slab order.
#include "ld_gemm.h"
#include "ld_gemm_tile.h"
#include "ld_device.h"
#include "ld_rope.h"
#include "ld_internal.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>

using namespace ldd;
using namespace ldt;

namespace {

constexpr float F16_LIMIT = 65504.f;   // largest finite fp16

constexpr int KC = 128;          // K granularity the launcher requires (largest chunk any variant stages)

// Sum of squares in a fixed order of fused multiply-adds: the kernels that normalise a row must agree bit for bit.
__device__ __forceinline__ float add_squares(float ss, const float4 &v) {
    ss = fmaf(v.x, v.x, ss);
    ss = fmaf(v.y, v.y, ss);
    ss = fmaf(v.z, v.z, ss);
    return fmaf(v.w, v.w, ss);
}

// v * rstd * g with both products rounded: the split that follows subtracts the rounded value's high part, and a
// product fused into that subtraction would give a different low part in one kernel than in another.
__device__ __forceinline__ float4 scale4(const float4 &v, float rstd, const float4 &g) {
#pragma clang fp contract(off)
    return make_float4(v.x * rstd * g.x, v.y * rstd * g.y, v.z * rstd * g.z, v.w * rstd * g.w);
}

// One workgroup per row.  ROW_REGS > 0: the row (at most 1024 * ROW_REGS long) is read once and kept in registers, all
// loads in flight together.  OCT: the images are written as [K / 8][T][8] (see k_gemm_skinny), else row-major.  (The fp16
// rows of a long pass, 2111 x 5120, were split here and rounded in a pass of their own before: 30 + 18 us.)
template <int ROW_REGS, bool OCT>
__global__ __launch_bounds__(256) void k_norm_split(const float *__restrict__ x, const float *__restrict__ g,
                                                    float eps, int K, ld::OperandImage out) {
    __shared__ float red[4];
    const int t = blockIdx.x;
    const float *row = x + (int64_t)t * K;
    float4 keep[ROW_REGS > 0 ? ROW_REGS : 1];
    if constexpr (ROW_REGS > 0) {
#pragma unroll
        for (int u = 0; u < ROW_REGS; u++) {
            const int i = threadIdx.x * 4 + u * 1024;
            if (i < K) keep[u] = *reinterpret_cast<const float4 *>(row + i);
        }
    }
    float rstd = 1.f;
    if (g) {
        float ss = 0.f;
        if constexpr (ROW_REGS > 0) {
#pragma unroll
            for (int u = 0; u < ROW_REGS; u++)
                if (threadIdx.x * 4 + u * 1024 < K) ss = add_squares(ss, keep[u]);
        } else {
            for (int i = threadIdx.x * 4; i < K; i += 1024) ss = add_squares(ss, *reinterpret_cast<const float4 *>(row + i));
        }
        ss = wave_sum(ss);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
        __syncthreads();
        rstd = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / K + eps);
    }
    auto store = [&](int i, float4 v) {
        if (g) v = scale4(v, rstd, *reinterpret_cast<const float4 *>(g + i));
        store_operand4(out, t, OCT ? octet_index(t, i, gridDim.x) : (int64_t)t * K + i, v);
    };
    if constexpr (ROW_REGS > 0) {
#pragma unroll
        for (int u = 0; u < ROW_REGS; u++)
            if (threadIdx.x * 4 + u * 1024 < K) store(threadIdx.x * 4 + u * 1024, keep[u]);
    } else {
        for (int i = threadIdx.x * 4; i < K; i += 1024) store(i, *reinterpret_cast<const float4 *>(row + i));
    }
}

// *flag is set when a bf16 matrix holds a value that fp16 cannot (beyond +-65504, or not a number).
__global__ __launch_bounds__(256) void k_weight_range(const bf16_t *__restrict__ w, int64_t n8, int *__restrict__ flag) {
    bool big = false;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (int64_t)gridDim.x * 256) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(w + i * 8));
#pragma unroll
        for (int e = 0; e < 4; e++)
            big = big || !(fabsf(__uint_as_float(v[e] << 16)) <= F16_LIMIT) || !(fabsf(__uint_as_float(v[e] & 0xffff0000u)) <= F16_LIMIT);
    }
    if (big) *flag = 1;
}

// The same look at a matrix, and its fp16 image written beside it (exact wherever *flag stays clear, up to values
// below 2^-14 in magnitude).
__global__ __launch_bounds__(256) void k_weight_to_f16(const bf16_t *__restrict__ w, int64_t n8, uint16_t *__restrict__ out,
                                                       int *__restrict__ flag) {
    bool big = false;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (int64_t)gridDim.x * 256) {
        const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(w + i * 8));
#pragma unroll
        for (int e = 0; e < 4; e++)
            big = big || !(fabsf(__uint_as_float(v[e] << 16)) <= F16_LIMIT) || !(fabsf(__uint_as_float(v[e] & 0xffff0000u)) <= F16_LIMIT);
        *reinterpret_cast<f16x8 *>(out + i * 8) = bf16x8_to_f16x8(v);
    }
    if (big) *flag = 1;
}

// Up to 64 rows (decode batches, short chunks): the weight stream is everything, so the kernel is built around never
// interrupting it and around asking for it in long runs.  One workgroup of eight waves per CU stays for the whole
// launch and owns a set of W rows and a slab of K (2048 wide, 1024 for more than 32 rows); its waves split the slab
// and keep the (hi, lo) X fragments of their share in registers for good.  W arrives 16 rows at a time, each row's
// whole slab (4 KB in a row, 2 KB for more than 32 rows) by one wave, copied straight into LDS (global_load_lds,
// non-temporal): 128 KB (96 KB) per CU are in flight and no register waits for them.  The access shape is what the rate
// depends on: streaming the 7B gate/up (down) matrix alone takes 28.7 (17.4) us in runs of 4 KB per wave, 31.6 (20.7) us
// with 512 bytes of two rows per instruction and 32.7 (21.8) us with 128 bytes of eight.
// Per 16-row tile: wait for the own copies, barrier, read fragments (lane = row), barrier, request the tile that takes
// this one's place, add up the tile before, multiply.  The sum over the eight waves goes through LDS in wave order; one
// partial sum per K slab goes to scratch and a reduction kernel adds the slabs in order (for SwiGLU the gate and up rows
// are plain rows here and are paired by the reduce kernel).  What bounds small matrices instead is the X fragments, which
// come before the first tile (256 KB a workgroup at 32 rows): 4096x4096 at 17 - 32 rows is 1.5 us slower than a form that
// held 512 columns of X a workgroup.
// LDS: piece p (16 bytes) of a row's slab sits in slot p ^ row: the 16 rows that a fragment read touches at one p then
// lie in 16 different bank groups, and a lane of a copy may fetch any piece into its fixed slot.
constexpr int SK_WAVES = 8;
constexpr int sk_steps(int tt) { return tt > 2 ? 4 : 8; }                       // 32-wide k-steps of a wave, at most
constexpr int sk_slab(int tt) { return SK_WAVES * sk_steps(tt) * 32; }          // K slab of a workgroup, at most

// LDS accesses of this kernel are written in assembly (reads with their wait in the same block): the compiler cannot
// tell which copies in flight they have nothing to do with and would wait for all of them first.
__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
__device__ __forceinline__ void ds_read_b128xn(u32x4 (&w)[8], const uint32_t (&a)[8]) {
    asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                 "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7])
                 : "memory");
}
__device__ __forceinline__ void ds_read_b128xn(u32x4 (&w)[4], const uint32_t (&a)[4]) {
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
                 : "memory");
}

// TT: 16-row tiles of X.  SRC: X comes as [part][K / 8][T][8] (OCTETS, the layout the producers of a decode batch write: a
// fragment load is then four runs of 256 bytes instead of sixteen of 64, 2 us less per launch at 32 rows and 4 us at
// 64), as row-major images (ROWS), or as the float rows themselves (FLOATS), multiplied by the gain g and split here, with the
// sums of squares of each wave's share in ss_part[row][slab][wave] for the kernel that adds the slabs: as many bytes as two
// images, and no pass in front that writes them.  grid: ks * row groups, block b takes K slab b % ks of row group b / ks.
enum SkinnySource { SK_ROWS, SK_OCTETS, SK_FLOATS };
struct FloatRows { const float *x, *g; float *ss_part; };
template <int TT, SkinnySource SRC>
__global__ __launch_bounds__(64 * SK_WAVES, 2) void k_gemm_skinny(const bf16_t *__restrict__ W, const bf16_t *__restrict__ xhi,
                                                                  const bf16_t *__restrict__ xlo, int T, int n_rows, int K,
                                                                  int ks, float *__restrict__ partial, FloatRows fr) {
    constexpr int STEPS = sk_steps(TT), ROWB = sk_slab(TT) * 2;      // ROWB: bytes of LDS per row of a stage
    constexpr int STAGE = 16 * ROWB, S = TT > 2 ? 3 : 2;             // 2 stages of 64 KB, or 3 of 32 KB
    constexpr int IPR = ROWB / 1024, P = 2 * IPR;                    // copy instructions per row; per wave and stage
    __shared__ __attribute__((aligned(1024))) char ring[S * STAGE];
    __shared__ __attribute__((aligned(1024))) char red[2][SK_WAVES * TT * 1024];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int kz = blockIdx.x % ks, grp = blockIdx.x / ks, n_grp = gridDim.x / ks;
    // The group's tiles start at W rows row0, row0 + stride, ... below row1: a range of its own, cut in units of four, so that all
    // groups have the same share; or, where rows are a multiple of 16 KB apart, every n_grp-th tile, so that the groups read
    // next to each other: 8192x8192 at 2 / 32 rows 38.1 / 41.9 us in ranges, 30.0 / 34.8 so (at 4 KB apart and odd lengths level
    // to 3 % slower).  The slab [k0, k0 + 32 steps) is cut in units of 128; s0, ns: this wave's k-steps of it
    const bool dealt = K % 8192 == 0;
    const int64_t units = (n_rows + 3) / 4, n128 = K / 128;
    const int row0 = dealt ? grp * 16 : (int)(units * grp / n_grp) * 4, stride = dealt ? n_grp * 16 : 16;
    const int row1 = dealt ? n_rows : min((int)(units * (grp + 1) / n_grp) * 4, n_rows);
    const int k0 = (int)(n128 * kz / ks) * 128, steps = (int)((n128 * (kz + 1) / ks) * 128 - k0) / 32;
    const int s0 = steps * wave / SK_WAVES, ns = steps * (wave + 1) / SK_WAVES - s0;      // ns <= STEPS
    const int n_tiles = (row1 - row0 + stride - 1) / stride;
    const int last_piece = steps * 4 - 1;
    const uint32_t red_base = lds_address(red), ring_base = lds_address(ring);

    auto request = [&](int tile) {
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const int tr = 2 * wave + r;                                     // this wave's rows of the tile
            const int row = min(row0 + tile * stride + tr, row1 - 1);        // past the end: the last row again
            const bf16_t *src = W + (int64_t)row * K + k0;
#pragma unroll
            for (int j = 0; j < IPR; j++) {
                const int piece = min((j * 64 + lane) ^ tr, last_piece);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + piece * 8),
                                                 (__attribute__((address_space(3))) void *)(ring + (tile % S) * STAGE + tr * ROWB + j * 1024),
                                                 16, 0, 2);
            }
        }
    };
    // X fragments: lane (row l16, k group kg) holds 8 consecutive k of each 32-wide step; rows past T are never stored.
    // Requested ahead of W (loads return in order: behind it they cost 5 us more)
    u32x4 xf[TT][2][STEPS];      // FLOATS: the eight floats of a fragment until they are split
    float4 gain[SRC == SK_FLOATS ? STEPS : 1][2];
#pragma unroll
    for (int tt = 0; tt < TT; tt++)
#pragma unroll
        for (int part = 0; part < 2; part++)
#pragma unroll
            for (int s = 0; s < STEPS; s++) {
                const int t = min(tt * 16 + l16, T - 1), k = k0 + (s0 + min(s, max(ns - 1, 0))) * 32 + kg * 8;
                if constexpr (SRC == SK_FLOATS) {
                    xf[tt][part][s] = *reinterpret_cast<const u32x4 *>(fr.x + (int64_t)t * K + k + 4 * part);
                    if (tt == 0 && fr.g) gain[s][part] = *reinterpret_cast<const float4 *>(fr.g + k + 4 * part);
                } else {
                    const bf16_t *src = (part ? xlo : xhi) + (SRC == SK_OCTETS ? ((int64_t)(k >> 3) * T + t) * 8 : (int64_t)t * K + k);
                    xf[tt][part][s] = *reinterpret_cast<const u32x4 *>(src);
                }
            }

    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < S; i++)
        if (i < n_tiles) request(i);
    __builtin_amdgcn_sched_barrier(0);
    // waited for here, once: left to their first use, inside the loop, the wait would cover every copy in flight there
#pragma unroll
    for (int tt = 0; tt < TT; tt++)
#pragma unroll
        for (int part = 0; part < 2; part++)
#pragma unroll
            for (int s = 0; s < STEPS; s++) asm volatile("" : "+v"(xf[tt][part][s]));
    if constexpr (SRC == SK_FLOATS) {
#pragma unroll
        for (int tt = 0; tt < TT; tt++) {
            float ss = 0.f;
#pragma unroll
            for (int s = 0; s < STEPS; s++) {
                float4 a = __builtin_bit_cast(float4, xf[tt][0][s]), b = __builtin_bit_cast(float4, xf[tt][1][s]);
                if (fr.g) {
                    if (s < ns) ss = add_squares(add_squares(ss, a), b);
                    a = scale4(a, 1.f, gain[s][0]);
                    b = scale4(b, 1.f, gain[s][1]);
                }
                uint32_t l0, l1, l2, l3;
                const uint32_t h0 = split2_bf16(a.x, a.y, l0), h1 = split2_bf16(a.z, a.w, l1), h2 = split2_bf16(b.x, b.y, l2), h3 = split2_bf16(b.z, b.w, l3);
                xf[tt][0][s] = (u32x4){h0, h1, h2, h3};
                xf[tt][1][s] = (u32x4){l0, l1, l2, l3};
            }
            if (fr.g && grp == 0) {      // one group of each slab: the sums of squares of this wave's share
                ss += __shfl_xor(ss, 16, WAVE);
                ss += __shfl_xor(ss, 32, WAVE);
                const int t = tt * 16 + l16;
                if (kg == 0 && t < T) fr.ss_part[((int64_t)t * ks + kz) * SK_WAVES + wave] = ss;
            }
        }
    }

    // adds the eight waves' sums of a tile (in LDS since the barrier before) and stores them
    auto finish = [&](int tile) {
#pragma unroll
        for (int u = 0; u < (TT + 1) / 2; u++) {
            const int t = u * 32 + (threadIdx.x >> 4), r = threadIdx.x & 15, row = row0 + tile * stride + r;
            if (t < T && row < row1) {
                const uint32_t src = red_base + (tile & 1) * (SK_WAVES * TT * 1024) + t * 64 + r * 4;
                float v[SK_WAVES];
                static_assert(SK_WAVES == 8, "one read per wave below");
                constexpr int O = TT * 1024;
                asm volatile("ds_read_b32 %0, %8\n\tds_read_b32 %1, %8 offset:%9\n\tds_read_b32 %2, %8 offset:%10\n\t"
                             "ds_read_b32 %3, %8 offset:%11\n\tds_read_b32 %4, %8 offset:%12\n\tds_read_b32 %5, %8 offset:%13\n\t"
                             "ds_read_b32 %6, %8 offset:%14\n\tds_read_b32 %7, %8 offset:%15\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                             : "v"(src), "n"(O), "n"(2 * O), "n"(3 * O), "n"(4 * O), "n"(5 * O), "n"(6 * O), "n"(7 * O)
                             : "memory");
#pragma unroll
                for (int w = 1; w < SK_WAVES; w++) v[0] += v[w];
                partial[((int64_t)kz * T + t) * n_rows + row] = v[0];
            }
        }
    };

    for (int tile = 0; tile < n_tiles; tile++) {
        // the own copies of this tile have landed once no more than the younger tiles' are outstanding (copies return in
        // order; stores of partial sums among them only make the wait stricter)
        const int younger = min(n_tiles - 1 - tile, S - 1);
        if (younger == S - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * P) : "memory");
        else if (S > 2 && younger == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * P) : "memory");
        else if (S > 2 && younger == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(P) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        const uint32_t st = ring_base + (tile % S) * STAGE + l16 * ROWB;
        u32x4 wf[STEPS];
        uint32_t at[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; s++)      // a step past ns reads the last one's fragment again: not used
            at[s] = st + ((((s0 + min(s, max(ns - 1, 0))) * 4 + kg) ^ l16) * 16);
        ds_read_b128xn(wf, at);
        lds_barrier();
        if (tile + S < n_tiles) request(tile + S);
        if (tile) finish(tile - 1);      // the other half of red is written below
        f32x4 acc[TT][2];
#pragma unroll
        for (int tt = 0; tt < TT; tt++)
#pragma unroll
            for (int part = 0; part < 2; part++) acc[tt][part] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < STEPS; s++)
            if (s < ns)      // uniform over the wave
#pragma unroll
                for (int tt = 0; tt < TT; tt++)
#pragma unroll
                    for (int part = 0; part < 2; part++)
                        acc[tt][part] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[s]), __builtin_bit_cast(bf16x8, xf[tt][part][s]), acc[tt][part], 0, 0, 0);
        // lane (l16, kg) holds W rows 4 kg .. + 4 of the tile for X row l16
#pragma unroll
        for (int tt = 0; tt < TT; tt++) {
            const f32x4 v = acc[tt][0] + acc[tt][1];
            asm volatile("ds_write_b128 %0, %1" ::"v"(red_base + (tile & 1) * (SK_WAVES * TT * 1024) + wave * (TT * 1024) + (tt * 16 + l16) * 64 + kg * 16), "v"(v) : "memory");
        }
    }
    lds_barrier();
    finish(n_tiles - 1);
}

// Adds the ks K-slab partial sums in slab order and applies the epilogue.  norm.ss_part: the sums are scaled by the row's 1 / rms
// first, whose square sum comes in n parts.  One thread per V outputs of a row: four where rows are a multiple of four floats
// and 16-byte aligned, as long as that leaves two workgroups a CU (152 x 11008 SwiGLU pairs of two slabs 10.6 -> 7.2 us,
// 1056 x 4096 of four 23.7 -> 16.1; 20 x 11008 level, as one output a thread there).
struct RowNorm { const float *ss_part; int n, K; float eps; };
template <int EPI, int V>
__global__ __launch_bounds__(256) void k_splitk_reduce(const float *__restrict__ partial, int T, int N, int ks,
                                                       float *__restrict__ y, ld::OperandImage out, RowNorm norm) {
    typedef float vec __attribute__((ext_vector_type(V)));
    constexpr int WR = (EPI == ld::GEMM_SWIGLU) ? 2 : 1;
    const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (idx >= (int64_t)T * N) return;
    const int t = (int)(idx / N), n = (int)(idx % N);
    const float *p0 = partial + (int64_t)t * (WR * N) + n;
    const int64_t slab = (int64_t)T * (WR * N) / V;
    vec a = slab_sum(reinterpret_cast<const vec *>(p0), slab, ks, (vec)0.f);
    vec b = WR == 2 ? slab_sum(reinterpret_cast<const vec *>(p0 + N), slab, ks, (vec)0.f) : (vec)0.f;
    if (norm.ss_part) {
        const float4 *ss = reinterpret_cast<const float4 *>(norm.ss_part + (int64_t)t * norm.n);      // n is a multiple of 8
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int i = 0; i < norm.n / 4; i++) { const float4 v = ss[i]; sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w; }
        const float rstd = 1.0f / sqrtf((sum.x + sum.y + sum.z + sum.w) / norm.K + norm.eps);
#pragma unroll
        for (int e = 0; e < V; e++) {
            a[e] = mul_rounded(a[e], rstd);
            b[e] = mul_rounded(b[e], rstd);
        }
    }
    vec *dst = reinterpret_cast<vec *>(y + (int64_t)t * N + n);
    if constexpr (EPI == ld::GEMM_STORE) *dst = a;
    else if constexpr (EPI == ld::GEMM_ADD) *dst += a;
    else {
#pragma unroll
        for (int e = 0; e < V; e++) a[e] = swiglu(a[e], b[e]);
        if (!out.hi) *dst = a;
        else if constexpr (V == 4) store_operand4(out, t, (int64_t)t * N + n, make_float4(a[0], a[1], a[2], a[3]));
        else store_operand(out, t, (int64_t)t * N + n, a[0]);
    }
}

// Residual rows that feed the next normalised GEMM: finishes y (adds the ks K-slab partial sums in slab order, as
// k_splitk_reduce<GEMM_ADD> does; ks 0: the product kernel's epilogue has added them) and writes the next operand
// split(y * rsqrt(mean y^2 + eps) * g) in the same pass over the row, with k_norm_split's arithmetic in
// k_norm_split's order: the results are those of the two separate kernels, bit for bit.  One workgroup per row; N a
// multiple of 4.  ROW_REGS as there: the row stays in registers between the two halves.
template <int ROW_REGS>
__global__ __launch_bounds__(256) void k_reduce_add_norm_split(const float *__restrict__ partial, int T, int N, int ks,
                                                               float *__restrict__ y, const float *__restrict__ g, float eps,
                                                               ld::OperandImage out) {
    __shared__ float red[4];
    const int t = blockIdx.x;
    float *row = y + (int64_t)t * N;
    const float *prow = partial + (int64_t)t * N;
    const int64_t slab = (int64_t)T * N;
    float ss = 0.f;
    float4 keep[ROW_REGS > 0 ? ROW_REGS : 1];
    auto finish = [&](int i) {
        float4 v = *reinterpret_cast<const float4 *>(row + i);
        if (ks) {
            const float4 a = slab_sum(reinterpret_cast<const float4 *>(prow + i), slab / 4, ks, make_float4(0.f, 0.f, 0.f, 0.f));
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
            *reinterpret_cast<float4 *>(row + i) = v;
        }
        return v;
    };
    if constexpr (ROW_REGS > 0) {
#pragma unroll
        for (int u = 0; u < ROW_REGS; u++)
            if (threadIdx.x * 4 + u * 1024 < N) keep[u] = finish(threadIdx.x * 4 + u * 1024);
#pragma unroll
        for (int u = 0; u < ROW_REGS; u++)
            if (threadIdx.x * 4 + u * 1024 < N) ss = add_squares(ss, keep[u]);
    } else {
        for (int i = threadIdx.x * 4; i < N; i += 1024) ss = add_squares(ss, finish(i));
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float rstd = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / N + eps);
    auto store = [&](int i, const float4 &v) {
        store_operand4(out, t, (int64_t)t * N + i, scale4(v, rstd, *reinterpret_cast<const float4 *>(g + i)));
    };
    if constexpr (ROW_REGS > 0) {
#pragma unroll
        for (int u = 0; u < ROW_REGS; u++)
            if (threadIdx.x * 4 + u * 1024 < N) store(threadIdx.x * 4 + u * 1024, keep[u]);
    } else {
        for (int i = threadIdx.x * 4; i < N; i += 1024) store(i, *reinterpret_cast<const float4 *>(row + i));   // this thread's own stores
    }
}

int env_int(const char *name, int dflt) {
    const char *v = getenv(name);
    return v ? atoi(v) : dflt;
}
int cu_count() {
    hipDeviceProp_t p;
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess) n = p.multiProcessorCount;
    return n > 0 ? n : 256;
}
// Tile, workgroup count and split-K factor of the big-tile kernel for a row count: the candidate with the smallest
// estimated time.  Workgroups run in rounds of one per CU (256 of them); a round takes the tile's time per 64-wide chunk of K
// times its chunks, a last round that leaves CUs idle a little less (the others draw less power and run faster: 0.27 of the idle
// share in both forms); split-K adds the write and the ordered re-read of its partial sums.  The constants are fitted to the tiles
// and splits of the 7B, grouped-KV and 13B layer shapes.  One term, 512 - 3072 rows, on the image (widened): the choice is 0.6 % (1.1 %)
// slower than the best pair in the mean, 11 % (19 %) at worst, and nowhere slower than that of the times of two stages (0.9 % and 12 %, 2.0 %
// and 29 %).  192 x 192 at the 0.92 us that larger products show took 4096 x 4096 at 2048 rows from 128 x 256: 77.3 -> 81.6 us; at 1536 68.2
// -> 73.4. Two terms, 80 - 480 rows: 1.4 % and 9 %, with the times of tiles of two stages, though three take 5 - 13 % off the smaller ones.
// Fitted anew the choice was 0.8 % slower than the best, but K was cut in fewer slabs at 942 of 4917 sizes (65 .. 511 rows of these shapes)
// and in more at 222, and longer sums are less exact: rms error over rms of the result against float64 in one, two, four and eight slabs
// 2.520, 2.487, 2.470, 2.463e-6 (256 x 12288 x 4096), 3.636, 3.579, 3.554, 3.543e-6 (152 x 11008 x 4096 SwiGLU).  Nor is the plain product's
// time all there is: with the rotation that adds the slabs (ldk_qkv_rope) 256 x 12288 x 4096 takes 58.6 us in the two slabs of this model,
// 64.1 in the one of that, 256 x 15360 x 5120 80.2 and 85.3, while plain products gained up to 8 % (480 x 4096 x 11008 in five and four slabs
// 93.4 -> 87.3).  With six and four tiles instead of ten and eight the best pair would be some 3 % slower in the mean.
struct BigPlan { int bm, bn, n_ttiles, n_nblocks, ks; double est_us; };
struct Tile { int bm, bn; bool swiglu; double chunk_us; };
#define LD_TILE_ROW(AT_, BT_, US_) {32 * AT_, 32 * BT_, BT_ % 2 == 0, US_},
const Tile tiles_two[] = {LD_TILES_TWO(LD_TILE_ROW)};
const Tile tiles_f16[] = {LD_TILES_F16(LD_TILE_ROW)};
#undef LD_TILE_ROW
struct Costs { const Tile *first, *end; double idle, us_per_mb; };
const Costs costs_two{std::begin(tiles_two), std::end(tiles_two), 0.27, 0.44};
const Costs costs_f16{std::begin(tiles_f16), std::end(tiles_f16), 0.27, 0.46};
BigPlan plan_big(int T, int N, int K, int epi, const Costs &costs, bool *ignored = nullptr) {
    const bool swi = epi == ld::GEMM_SWIGLU;
    BigPlan best{};
    double best_t = 1e30;
    const Tile *first = costs.first, *end = costs.end;
    // tuning knob: "rows,columns,ks" of a tile (rows 2, 4: 128, 256); what is no plan of this form is ignored (see gemm_rows)
    const char *forced = getenv("LD_GEMM_BIG");
    int f_bm = 0, f_bn = 0, f_ks = 0;
    const bool parsed = forced && sscanf(forced, "%d,%d,%d", &f_bm, &f_bn, &f_ks) == 3 && f_ks >= 1;
    if (f_bm <= 4) f_bm *= 64;
    const bool known = parsed && std::any_of(first, end, [&](const Tile &t) { return t.bm == f_bm && t.bn == f_bn && (!swi || t.swiglu); });
    if (ignored) *ignored = forced && !known;
    for (const Tile *tl = first; tl != end; tl++) {
        if (known && (tl->bm != f_bm || tl->bn != f_bn)) continue;
        if (swi && !tl->swiglu) continue;
        const int nout = swi ? tl->bn / 2 : tl->bn;
        const int n_tt = (T + tl->bm - 1) / tl->bm, n_nb = (N + nout - 1) / nout;
        const int max_ks = std::max(1, std::min(8, K / 64 / 4));   // at least four chunks per slab
        for (int ks = 1; ks <= max_ks; ks++) {
            if (known && ks != std::min(f_ks, max_ks)) continue;
            const int64_t wgs = (int64_t)n_tt * n_nb * ks;
            const double rounds = (double)(wgs / 256) + (wgs % 256 ? 1.0 - costs.idle * (1.0 - (wgs % 256) / 256.0) : 0.0);
            double t = rounds * tl->chunk_us * ((K / 64 + ks - 1) / ks);
            if (ks > 1) t += 2.0 + costs.us_per_mb * 4e-6 * T * N * (swi ? 2 : 1) * ks;
            if (t < best_t) { best_t = t; best = {tl->bm, tl->bn, n_tt, n_nb, ks, t}; }
        }
    }
    return best;
}
BigPlan plan_big(int T, int N, int K, int epi, bool f16 = false, bool *ignored = nullptr) {
    return plan_big(T, N, K, epi, f16 ? costs_f16 : costs_two, ignored);
}

// Most rows the small-batch kernel takes: four 16-row tiles of X fit a wave's registers beside its fragments.  Feed-
// forward of the 7B shape at 33 / 48 / 49 / 64 rows against the kernels that took these rows before it (a 512-wide
// slab kernel in two groups of rows, then one with X staged chunk by chunk): 105 -> 79, 111 -> 84, 129 -> 88,
// 128 -> 91 us; at 2 / 16 / 32 rows 68 -> 64, 76 -> 68, 84 -> 74 us.
constexpr int SKINNY_MAX_ROWS = 64;
int skinny_tiles(int T) { return T <= 16 ? 1 : T <= 32 ? 2 : T <= 48 ? 3 : 4; }      // 16-row tiles of X
// K slabs: what the eight waves of a workgroup hold of X in registers, or a power of two of up to eight where that is up to a third more and
// saves work: the CUs divide into even groups, and a workgroup starts with less of X.  What it saves shows in the steps of the workgroup
// that has most of them, its 16-row tiles times its slab's columns; what it costs is the partial sums of the slabs added.  Hence: 3 to 4
// and 6 to 8 where the steps go down to 0.85 or less (0.925 for 3 to 4 of up to 32 rows and tiles enough, eight, to level out what is
// particular to the last one), 7 to 8 to 0.975.  us, fewest slabs -> power of two, by that ratio: 3 to 4, 0.71: 2048 x 5120 at 24 rows 15.1 ->
// 13.3; 0.86: 8192 x 6144 at 24 29.5 -> 27.0; 0.89: 15360 x 5120 at 20 39.4 -> 36.3, but 5120 x 5120 at 2 (five tiles) 13.1 -> 13.9; 0.95:
// 13824 x 3072 at 48 30.3 -> 31.8; 1.06: 13824 x 2304 at 48 27.8 -> 31.0.  6 to 8, 0.84: 4096 x 11008 at 8 20.9 -> 20.5; 0.88: 6144 x 11008
// at 24 34.0 -> 35.7.  7 to 8, 0.88: 3072 x 13824 at 16 23.3 -> 20.5; 0.98: 13824 x 13824 at 24 75.8 -> 77.2.  Over the 519 sizes that the
// limits were drawn from 3.6 % off, 1.5 % more at worst (with the power of two wherever it is up to a third more 3.6 % off, 11 % more); over
// 260 others 2.4 % off, 3 % more at worst.  Others are slower: 15360 x 5120 at 64 rows (5, 8) 52.1 -> 59.4, 12288 x 4096 at 20 (2, 4)
// 27.9 -> 30.8, 13824 x 13824 at 64 (14, 16) 99.9 -> 102.7.
int skinny_split(int T, int64_t n_rows, int K) {
    const int slab = sk_slab(skinny_tiles(T)), fewest = (K + slab - 1) / slab, p = fewest == 3 ? 4 : fewest == 6 || fewest == 7 ? 8 : fewest;
    if (p == fewest) return fewest;
    const int64_t units = (n_rows + 3) / 4;      // of the row groups, see the kernel
    auto tiles = [&](int ks) { const int64_t groups = std::min<int64_t>(256 / ks, (n_rows + 15) / 16); return ((units + groups - 1) / groups + 3) / 4; };
    auto steps = [&](int ks) { return tiles(ks) * ((K / 128 + ks - 1) / ks); };
    const int limit = fewest == 7 ? 975 : fewest == 3 && T <= 32 && tiles(p) >= 8 ? 925 : 850;      // thousandths
    return 1000 * steps(p) <= limit * steps(fewest) ? p : fewest;
}

int split_factor(int T, int N, int K, int epi, bool f16 = false) {
    if (T <= SKINNY_MAX_ROWS) return skinny_split(T, (int64_t)N * (epi == ld::GEMM_SWIGLU ? 2 : 1), K);
    return plan_big(T, N, K, epi, f16).ks;
}

}  // namespace

namespace ld {

bool gemm_supported(int T, int N, int K) { return T >= 2 && N > 0 && K > 0 && K % KC == 0; }

size_t gemm_split_bytes(int T, int K) { return (((size_t)2 * T * K * sizeof(bf16_t)) + 255) / 256 * 256; }

// Which rows past the last whole 256-row tile keep both bf16 terms in the one-term form.  The number of terms is part of a
// product's results, so it has a rule of its own that does not move when tiles or their measured times change: the rows
// keep both wherever a second stream of W (4 TB/s and 12 us) costs less than what they add to the time of 256 x 256 and
// 128 x 256 tiles at nominal rates (754 and 638 TFLOP/s; a last round that leaves CUs idle at least 0.74 of a whole one; K
// split in up to eight slabs at 9 TB/s for the partial sums, for the last column blocks alone at 3).
static double nominal_us(int T, int N, int K, int wr) {
    const int nout = 256 / wr, n_nb = (N + nout - 1) / nout, max_ks = std::max(1, std::min(8, K / 256));
    double best = 1e30;
    for (const int bm : {256, 128}) {
        const int64_t n_tt = (T + bm - 1) / bm, n_all = n_tt * n_nb;
        auto tile_us = [&](int k) { return 0.69 * 2.0 * bm * 256 * (double)k / ((bm == 256 ? 520.0 : 440.0) * 1e6 / 256.0); };
        for (int ks = 1; ks <= max_ks; ks++) {
            const int64_t wgs = n_all * ks;
            double t = ((double)(wgs / 256) + (wgs % 256 ? std::max((wgs % 256) / 256.0, 0.74) : 0.0)) * tile_us(K / ks);
            if (ks > 1) t += 3.0 + (double)T * N * wr * 4.0 * (2.0 * ks + 1.0) / 9.0e6;
            best = std::min(best, t);
        }
        const int64_t nb_a = n_all / 256 * 256 / n_tt, nb_b = n_nb - nb_a;
        if (bm != 256 || n_all <= 256 || n_all >= 512 || nb_a <= 0 || nb_b <= 0) continue;
        for (int ks = 2; ks <= max_ks; ks++) {
            const double cols_b = (double)std::min<int64_t>(N - nb_a * nout, nb_b * nout);
            best = std::min(best, (double)((nb_a * n_tt + 255) / 256) * tile_us(K) + (double)((nb_b * n_tt * ks + 255) / 256) * tile_us(K) / ks +
                                      6.0 + (double)T * cols_b * wr * 4.0 * (2.0 * ks + 1.0) / 3.0e6);
        }
    }
    return best;
}
// And by a second set of nominal rates, those of four tiles in rounds of 256 workgroups (0.89 of a round at least for the last
// one; K split in up to eight slabs at 0.48 us per MB of partial sums) against a stream at 5.2 TB/s and 10 us: between the two
// sets lie up to 128 row counts below 2200 per shape.
static double nominal_tiles_us(int T, int N, int K, int epi) {
    const struct { int bm, bn; bool swiglu; double us; } tiles[] = {{128, 256, true, 1.01}, {256, 160, false, 1.17}, {256, 192, true, 1.33}, {256, 256, true, 1.62}};
    const bool swi = epi == GEMM_SWIGLU;
    const int max_ks = std::max(1, std::min(8, K / 256));
    double best = 1e30;
    for (const auto &t : tiles) {
        if (swi && !t.swiglu) continue;
        const int nout = swi ? t.bn / 2 : t.bn;
        const int64_t items = (int64_t)((T + t.bm - 1) / t.bm) * ((N + nout - 1) / nout);
        for (int ks = 1; ks <= max_ks; ks++) {
            const int64_t wgs = items * ks;
            const double rounds = (double)(wgs / 256) + (wgs % 256 ? std::max((wgs % 256) / 256.0, 0.89) : 0.0);
            best = std::min(best, rounds * t.us * (K / 64) / ks + (ks > 1 ? 1.0 + 0.48 * 4e-6 * T * N * (swi ? 2 : 1) * ks : 0.0));
        }
    }
    return best;
}
// And by a third, eight tiles with two stages in LDS, chosen among as the planner does: it alone decides one of a thousand sizes (64 ..
// 60000 columns, K to 30000), none of the 7B, grouped-KV and 13B layer shapes below 4200 rows.  None of the three says what the tiles
// of today take, which would be left whole at a quarter of those shapes' tails: the second stream of W is there the price of the same results.
const Tile tiles_nominal[] = {{128, 192, true, 0.74}, {128, 256, true, 0.99}, {192, 192, true, 1.05}, {192, 256, true, 1.23},
                              {224, 256, true, 1.40}, {256, 160, false, 1.14}, {256, 192, true, 1.23}, {256, 256, true, 1.54}};
const Costs costs_nominal{std::begin(tiles_nominal), std::end(tiles_nominal), 0.31, 0.44};
static double stream_us(double bytes) { return bytes / 5.2e6 + 10.0; }      // ~5.2 TB/s + two launches
static bool tail_keeps_both_terms(int T, int r, int N, int K, int epi) {
    const int wr = epi == GEMM_SWIGLU ? 2 : 1;
    const double stream = (double)N * wr * K * 2.0;
    return nominal_us(T - r, N, K, wr) + stream / 4.0e6 + 12.0 < nominal_us(T, N, K, wr) ||
           nominal_tiles_us(T - r, N, K, epi) + stream_us(stream) < nominal_tiles_us(T, N, K, epi) ||
           plan_big(T - r, N, K, epi, costs_nominal).est_us + stream_us(stream) < plan_big(T, N, K, epi, costs_nominal).est_us;
}

// Rows that would only start one more, nearly empty 256-row tile (a mixed step's 4 x 257 + 28 rows, a 2048-row
// chunk beside 63 decode rows) are cut off and go through the small-batch kernels: in the two-term form where that costs less by the
// cost model that picks the tile (the weights are streamed once more), in the one-term form where the rule above wants both terms in
// them.  Returns the number of such tail rows (0: no cut).
int tail_rows(int T, int N, int K, int epi, bool f16) {
    const int r = T % 256;
    static const int enabled = env_int("LD_GEMM_TAIL", 1);   // tuning knob: 0 keeps every row in the tiled kernel
    if (!enabled || T <= 256 || r == 0 || r > 64 || getenv("LD_GEMM_BIG")) return 0;
    if (f16) return tail_keeps_both_terms(T, r, N, K, epi) ? r : 0;
    const double whole = plan_big(T, N, K, epi).est_us, main_part = plan_big(T - r, N, K, epi).est_us;
    return main_part + stream_us((double)N * (epi == GEMM_SWIGLU ? 2 : 1) * K * 2.0) < whole ? r : 0;
}

static size_t partial_bytes(int T, int N, int K, int epi, bool f16 = false) {
    const int ks = split_factor(T, N, K, epi, f16);
    return (ks > 1 || T <= SKINNY_MAX_ROWS) ? (size_t)ks * T * N * (epi == GEMM_SWIGLU ? 2 : 1) * sizeof(float) : 0;
}

size_t gemm_scratch_bytes(int T, int N, int K, int epi) {
    if (T > SKINNY_MAX_ROWS && K > TILE_MAX_K) return gemm_split_bytes(T, K) + partial_bytes(SKINNY_MAX_ROWS, N, K, epi);
    const int r = tail_rows(T, N, K, epi, false);
    size_t part = r ? std::max(partial_bytes(T - r, N, K, epi), partial_bytes(r, N, K, epi)) : partial_bytes(T, N, K, epi);
    if (T > 64) {      // the same pass in the fp16 form may split K differently
        const int rf = tail_rows(T, N, K, epi, true);
        part = std::max(part, partial_bytes(T - rf, N, K, epi, true));
        if (rf) part = std::max(part, partial_bytes(rf, N, K, epi));
    }
    return gemm_split_bytes(T, K) + part;
}

bool gemm_takes_octets(int T) { return T >= 2 && T <= SKINNY_MAX_ROWS; }

void launch_norm_split(const float *x, const float *g, float eps, int T, int K, uint16_t *xs, hipStream_t s, bool octets,
                       int f16_rows, int *f16_flag) {
    const OperandImage out{xs, xs + (size_t)T * K, f16_rows, f16_flag};
#define LD_NS(R_)                                                                                                      \
    do {                                                                                                               \
        if (octets) LD_LAUNCH((k_norm_split<R_, true>), dim3(T), dim3(256), 0, s, x, g, eps, K, out);                  \
        else LD_LAUNCH((k_norm_split<R_, false>), dim3(T), dim3(256), 0, s, x, g, eps, K, out);                        \
    } while (0)
    if (K <= 5 * 1024) LD_NS(5);
    else if (K <= 14 * 1024) LD_NS(14);
    else LD_NS(0);
#undef LD_NS
}

int skinny_slabs(int T, int64_t n_rows, int K) { return skinny_split(T, n_rows, K); }

static void launch_skinny(const uint16_t *W, const uint16_t *xhi, const uint16_t *xlo, int T, int n_rows, int K, float *partial, hipStream_t s,
                          SkinnySource src, const FloatRows &fr) {
    const int ks = skinny_split(T, n_rows, K);
    static const int n_cu = cu_count();
    // one workgroup per CU; fewer where a row group would get less than a tile
    const int n_grp = std::max(1, std::min(n_cu / ks, (n_rows + 15) / 16));
    const dim3 grid(n_grp * ks), block(64 * SK_WAVES);
#define LD_SKINNY(TT_)                                                                                                              \
    do {                                                                                                                            \
        if (src == SK_FLOATS) LD_LAUNCH((k_gemm_skinny<TT_, SK_FLOATS>), grid, block, 0, s, W, xhi, xlo, T, n_rows, K, ks, partial, fr);       \
        else if (src == SK_OCTETS) LD_LAUNCH((k_gemm_skinny<TT_, SK_OCTETS>), grid, block, 0, s, W, xhi, xlo, T, n_rows, K, ks, partial, fr);  \
        else LD_LAUNCH((k_gemm_skinny<TT_, SK_ROWS>), grid, block, 0, s, W, xhi, xlo, T, n_rows, K, ks, partial, fr);                \
    } while (0)
    switch (skinny_tiles(T)) {
        case 1: LD_SKINNY(1); break;
        case 2: LD_SKINNY(2); break;
        case 3: LD_SKINNY(3); break;
        default: LD_SKINNY(4);
    }
#undef LD_SKINNY
}
void launch_gemm_skinny(const uint16_t *W, const uint16_t *xhi, const uint16_t *xlo, int T, int n_rows, int K,
                        float *partial, hipStream_t s, bool octets) {
    launch_skinny(W, xhi, xlo, T, n_rows, K, partial, s, octets ? SK_OCTETS : SK_ROWS, FloatRows{});
}

static bool row_quads(int N, const float *y, const float *partial, const OperandImage &out) {
    return N % 4 == 0 && (((uintptr_t)y | (uintptr_t)partial | (uintptr_t)out.hi | (uintptr_t)out.lo) & 15) == 0;
}
static void launch_reduce(const float *partial, int T, int N, int ks, int epi, float *y, const OperandImage &out, const RowNorm &norm, hipStream_t s) {
    const int64_t n = (int64_t)T * N;
    const bool four = row_quads(N, y, partial, out) && n >= 4 * 256 * 512;
    const dim3 grid((unsigned)((four ? n / 4 + 255 : n + 255) / 256)), block(256);
#define LD_REDUCE(EPI_)                                                                                                \
    do {                                                                                                               \
        if (four) LD_LAUNCH((k_splitk_reduce<EPI_, 4>), grid, block, 0, s, partial, T, N, ks, y, out, norm);           \
        else LD_LAUNCH((k_splitk_reduce<EPI_, 1>), grid, block, 0, s, partial, T, N, ks, y, out, norm);                \
    } while (0)
    if (epi == GEMM_STORE) LD_REDUCE(GEMM_STORE);
    else if (epi == GEMM_ADD) LD_REDUCE(GEMM_ADD);
    else LD_REDUCE(GEMM_SWIGLU);
#undef LD_REDUCE
}

// The float rows take longer to arrive than octets do (rows a multiple of 4 KB apart come out of a few channels of the cache; with
// 64 bytes of a row in a run and an exchange between lanes they take as long), the more the more 16-row tiles of them a workgroup
// holds, and with a norm the kernel that adds the slabs has their squares to add.  Ahead of the pass they replace, therefore, where
// that pass is long or the rows are few.  GPU time at 2 .. 64 rows on 21 shapes with and without a norm, matrices out of HBM, images ->
// floats, us (the width of the output hardly matters):
//  one tile, no norm: 4096 x 4096 at 2 rows 13.9 -> 12.5, at 16 15.2 -> 15.0; 2048 x 2048 at 12 10.1 -> 10.0, at 16 10.4 -> 10.8;
//   768 x 768 at 10 8.8 -> 8.6, at 16 8.8 -> 9.6;
//  one tile, norm: 12288 x 4096 at 2 24.1 -> 22.9, at 16 25.8 -> 25.5; 8192 x 2048 at 8 level, at 16 15.2 -> 16.1; 9216 x 3072 at 12
//   level, at 16 19.8 -> 20.2; 4096 x 1024 at 6 level, at 16 10.1 -> 11.5;
//  two tiles: 12288 x 4096 with a norm at 17 27.3 -> 27.7, at 20 27.9 -> 28.4; without one 4096 x 4096 at 17 16.9 -> 17.2, 5120 x 5120 at
//   17 20.3 -> 20.1, at 20 level, at 24 21.2 -> 21.4;
//  three, no norm: 4096 x 4096 at 33 18.8 -> 17.8, at 40 18.9 -> 18.4, at 48 level; 2048 x 2048 at 40 11.4 -> 12.2; norm: 12288 x 4096 at
//   33 30.9 -> 31.8;
//  rows of more than 8192 columns everywhere: 4096 x 11008 at 2 25.1 -> 21.3, at 20 29.1 -> 26.7, at 33 33.5 -> 29.3, at 64
//   39.2 -> 36.6.
// A matrix of up to 8 MB takes the GPU less time than three launches take the caller: one launch fewer counts (3072 x 1024 at 16
// rows, calls one after the other 13.2 -> 11.4, on the GPU 9.7 -> 11.3).
bool gemm_takes_floats(int T, int N, int K, bool norm) {
    if (!gemm_takes_octets(T)) return false;
    const int forced = env_flag("LD_GEMM_FLOATS", -1);      // tuning knob: 1 float rows, 0 images
    if (forced >= 0) return forced != 0;
    if (K > 8192) return true;
    if (T <= 16) return (int64_t)N * K <= 1 << 22 || (norm ? T <= 6 || T * 256 <= K : T <= 10 || K >= 2048);
    return !norm && (T <= 32 ? T <= 20 && K >= 5120 : T <= 40 && K >= 3072);
}

void launch_gemm_floats(const uint16_t *W, const float *x, const float *g, float eps, int T, int N, int K, int epi, float *y, void *scratch,
                        hipStream_t s) {
    // the scratch of the image form: its images' place (K floats a row) holds the sums of squares, one of each wave of each slab: with
    // at most one slab per 128 columns at most K / 16 a row
    float *ss = (float *)scratch, *partial = (float *)((char *)scratch + gemm_split_bytes(T, K));
    const int n_rows = N * (epi == GEMM_SWIGLU ? 2 : 1), ks = skinny_split(T, n_rows, K);
    launch_skinny(W, nullptr, nullptr, T, n_rows, K, partial, s, SK_FLOATS, {x, g, ss});
    launch_reduce(partial, T, N, ks, epi, y, {}, {g ? ss : nullptr, ks * SK_WAVES, K, eps}, s);
}

// The big-tile kernel over all output columns (+ the split-K reduction).
static void launch_tiles(const uint16_t *W, const bf16_t *hi, const bf16_t *lo, int T, int N, int K, int epi, float *y,
                         float *partial, const BigPlan &p, hipStream_t s, bool reduce, const OperandImage &out, int f16) {
    const int grid = (p.n_nblocks * p.n_ttiles * p.ks + 7) / 8 * 8;
    const bool quads = row_quads(N, y, partial, out);
    const TileLaunch l{W, hi, lo, T, N, K, epi, y, p.n_ttiles, p.ks, partial, out, quads, grid, s};
    if (f16 == 2) launch_tile_image(p.bm, p.bn, l);
    else if (f16) launch_tile_widen(p.bm, p.bn, l);
    else launch_tile_two(p.bm, p.bn, l);
    if (p.ks <= 1 || !reduce) return;
    launch_reduce(partial, T, N, p.ks, epi, y, out, {}, s);
}

// Where the rows of a product go next.
struct RowsNext { const float *g; float eps; OperandImage out; const RopeKvArgs *rope; int row0; };

// Products with an operand of 4 GiB or more keep both terms in every row, wherever their tails are cut.
int gemm_f16_rows(int T, int N, int K, int epi) {
    if (T <= SKINNY_MAX_ROWS || K > TILE_MAX_K) return 0;
    const int64_t limit = (int64_t)1 << 31;      // elements
    if ((int64_t)T * K >= limit || (int64_t)N * (epi == GEMM_SWIGLU ? 2 : 1) * K >= limit) return 0;
    return T - tail_rows(T, N, K, epi, true);
}

// nx != nullptr with GEMM_ADD: y's rows are finished and turned into the next operand by one fused kernel in
// place of the split-K reduction.  With GEMM_SWIGLU: the epilogue (or the split-K reduction) writes its result
// as the next operand instead of floats.
// f16 (more than 64 rows): the rows are one fp16 image (hi), multiplied in the single-term form; W16: the matrix's fp16
// image where the caller keeps one (the kernel then reads it in W's place and converts nothing), else nullptr.
static void gemm_rows(const uint16_t *W, const bf16_t *hi, const bf16_t *lo, int T, int N, int K, int epi, float *y,
                      float *partial, hipStream_t s, const RowsNext *nx, bool f16, const uint16_t *W16, bool octets) {
    const bool chain_rope = nx && epi == GEMM_STORE && nx->rope;
    const bool chain_add = (nx && epi == GEMM_ADD) || chain_rope;      // a finishing kernel replaces the split-K reduction
    const OperandImage out = nx && epi == GEMM_SWIGLU ? nx->out : OperandImage{};
    auto finish = [&](int ks) {      // ks: slabs whose partial sums the finishing kernel still has to add
        if (chain_rope) {
            launch_rope(partial, T, ks, y, *nx->rope, nx->rope->pool, nx->row0, s);
        } else if (N <= 5 * 1024) {
            LD_LAUNCH((k_reduce_add_norm_split<5>), dim3(T), dim3(256), 0, s, partial, T, N, ks, y, nx->g, nx->eps, nx->out);
        } else {
            LD_LAUNCH((k_reduce_add_norm_split<0>), dim3(T), dim3(256), 0, s, partial, T, N, ks, y, nx->g, nx->eps, nx->out);
        }
    };
    if (T <= SKINNY_MAX_ROWS) {
        const int ks = split_factor(T, N, K, epi), n_rows = N * (epi == GEMM_SWIGLU ? 2 : 1);
        launch_gemm_skinny(W, hi, lo, T, n_rows, K, partial, s, octets);
        if (chain_add) finish(ks);     // the skinny kernel writes partial sums even for one slab
        else launch_reduce(partial, T, N, ks, epi, y, out, {}, s);
        return;
    }
    bool ignored = false;
    const BigPlan p = plan_big(T, N, K, epi, f16, &ignored);
    if (ignored) fprintf(stderr, "libld: LD_GEMM_BIG names no plan of the %s form: ignored\n", f16 ? "one-term" : "two-term");
    launch_tiles(f16 && W16 ? W16 : W, hi, lo, T, N, K, epi, y, partial, p, s, !chain_add, out, f16 ? (W16 ? 2 : 1) : 0);
    if (chain_add) finish(p.ks > 1 ? p.ks : 0);
}

void launch_gemm(const uint16_t *W, uint16_t *xs, int T, int N, int K, int epi, float *y, hipStream_t s,
                 const GemmNext *next, int *f16_flag, const uint16_t *W16, bool octets) {
    float *partial = (float *)((char *)xs + gemm_split_bytes(T, K));
    const bf16_t *hi = xs, *lo = xs + (size_t)T * K;
    const bool f16 = f16_flag && gemm_f16_rows(T, N, K, epi) > 0;
    // n rows from row0 on.  The next operand is a [2][T][N] image
    auto rows = [&](int row0, int n, bool one_term, const uint16_t *w16, bool oct) {
        RowsNext nx{};
        if (next) {
            uint16_t *nh = next->xs ? next->xs + (size_t)row0 * N : nullptr, *nl = nh ? nh + (size_t)T * N : nullptr;
            nx = {next->g, next->eps, {nh, nl, next->f16_rows - row0, f16_flag}, next->rope, row0};
        }
        gemm_rows(W, hi + (size_t)row0 * K, lo + (size_t)row0 * K, n, N, K, epi, y + (size_t)row0 * N, partial, s, next ? &nx : nullptr,
                  one_term, w16, oct);
    };
    // groups of rows share the partial-sum scratch: the stream orders each behind the reduction of the one before
    if (T > SKINNY_MAX_ROWS && K > TILE_MAX_K) {
        for (int row0 = 0; row0 < T; row0 += SKINNY_MAX_ROWS) rows(row0, std::min(SKINNY_MAX_ROWS, T - row0), false, nullptr, false);
        return;
    }
    // the rows beyond a multiple of 256 that go through the small-batch kernel keep both terms
    const int r = tail_rows(T, N, K, epi, f16);
    rows(0, T - r, f16, W16, octets);
    if (r) rows(T - r, r, false, nullptr, false);
}

void launch_weight_range_check(const uint16_t *W, int64_t n, int *flag, hipStream_t s) {
    LD_LAUNCH(k_weight_range, dim3(1024), dim3(256), 0, s, W, n / 8, flag);
}

void launch_weight_to_f16(const uint16_t *W, int64_t n, uint16_t *out, int *flag, hipStream_t s) {
    LD_LAUNCH(k_weight_to_f16, dim3(1024), dim3(256), 0, s, W, n / 8, out, flag);
}

}  // namespace ld
