// k_gemm_tile, included by the three translation units that instantiate it.
#pragma once
#include "ld_gemm_tile.h"

using namespace ldd;
using namespace ldt;

namespace {

// The big-tile kernel.  Four waves, one per SIMD (512 registers each), two by two, a wave owning AT x BT accumulator
// tiles of 16 x 16: the fewest operand bytes out of LDS per MFMA that the registers allow.  K advances in chunks of 64
// (rows of 128 bytes: whole cache lines), two or three stages, copied straight into LDS (buffer loads with the lds bit: a
// scalar base, a lane offset that never changes and a scalar step along K, so that a copy costs no vector
// arithmetic).
// What bounds it with real numbers in the operands is the power the matrix cores draw: on zeros 2048 x 8192 x 13824 takes
// 293 us, on normal ones 386 (32 x 32 x 16 MFMAs).  A loop of MFMAs alone reaches, on normal operands, 1688 TFLOP/s in fp16 and 1842
// in bf16 with 32 x 32 x 16, 1968 and 2105 with 16 x 16 x 32 (2440 - 2470 both on zeros): half as many accumulator bytes go in
// and out per product.  Hence the small MFMA: products with their operand passes 2048 x 8192 x 13824 430 -> 401 us,
// 2048 x 5120 x 13824 339 -> 281, 2111 x 27648 x 5120 568 -> 527, in two terms 152 x 4096 x 11008 54 -> 50.
// Beside that it is how the copies are issued and how long they have to arrive.  A copy whose turn comes while the CU's address
// unit is busy holds up the MFMAs behind it, and two stages leave a copy less than a chunk's time to arrive; so
//  - the operands of a chunk are all in registers before its second half (112 - 128 registers), its stage is free
//    from then on, and
//  - the copies of the chunk after next are spread over a whole chunk's MFMAs, a few per k-step, none in a row
//    (1118 -> 1245 TFLOP/s with the larger MFMA; 1454 without any copies).
// Where three stages fit (up to 53 KB each) a copy has two chunks' time and a chunk one barrier instead of two: with up to one
// workgroup a CU 5 - 13 % off the smaller tiles' launches (4096 x 4096 at 1028 rows in fp16, 128 x 192 tiles: 67 -> 58 us; at 300
// rows in two terms, 96 x 128: 40 -> 35), 0 - 7 % beyond.  Four stages are level with three; reading the operands eight MFMAs
// ahead of the barrier gives 0.3 % to the larger tiles.
// The matrix instructions are assembly, issued exactly in the order written here (see tile_mfma_bf16).
// One copy instruction covers 8 rows x 128 bytes; piece p (16 bytes) of row r sits in slot p ^ ((r >> 1) & 7) of its row:
// 16 consecutive rows at one p lie in 16 bank groups.
//
// TERMS 2: (hi, lo) bf16 images of the activations against the bf16 matrix, both into the same accumulators.
// TERMS 1 (rows that nobody reads at full precision, see launch_gemm): the activations as one fp16 image (xhi); WF 1: W
// is the bf16 matrix and a wave turns its fragments into fp16 on their way to the matrix cores (exact for 2^-14 <= |w| <
// 65520, which the launcher has checked on the whole matrix); WF 2: W is the matrix's fp16 image (k_weight_to_f16).
// Same values, same sums either way.
#if defined(__HIP_DEVICE_COMPILE__)
struct BufferCopy {      // 16 bytes per lane from base + lane offset + scalar offset into LDS, 1 KB in a row per wave
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ BufferCopy(const void *base)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, -1, 0x00020000)) {}
    __device__ __forceinline__ void operator()(char *dst, uint32_t lane_off, uint32_t off) const {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, lane_off, off, 0, 0);
    }
};
#else
struct BufferCopy {
    __device__ BufferCopy(const void *) {}
    __device__ void operator()(char *, uint32_t, uint32_t) const {}
};
#endif

// c += w x on the matrix cores, c in accumulation registers.  In assembly because the result has to land in the registers it
// came from: left to the compiler, which sees no need for that with MFMAs this short, a chunk carries some 400 copies.  The operands come from LDS reads
// (the compiler waits for those); an operand that vector arithmetic has just written needs two wait states.
__device__ __forceinline__ void tile_mfma_bf16(f32x4 &c, const u32x4 &w, const u32x4 &x) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
}
__device__ __forceinline__ void tile_mfma_f16(f32x4 &c, const u32x4 &w, const u32x4 &x) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
}
// Moved out of the accumulation registers here and not earlier: all at once they do not fit beside the rest.
__device__ __forceinline__ f32x4 tile_result(const f32x4 &c) {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; e++) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[e]) : "a"(c[e]));
    return v;
}
__device__ __forceinline__ void tile_mfma_f16_after_valu(f32x4 &c, const u32x4 &w, const u32x4 &x) {
    asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
}

// f(0), f(1), .. f(N - 1) with the number as a constant.
template <int... I, typename F>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F &&f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void each(F &&f) { each_of(std::make_integer_sequence<int, N>{}, f); }

template <int TERMS, int WF, int AT, int BT, int EPI, int S>
__global__ __launch_bounds__(256, 1) void k_gemm_tile(const bf16_t *__restrict__ W, const bf16_t *__restrict__ xhi,
                                                      const bf16_t *__restrict__ xlo, int T, int N, int K,
                                                      float *__restrict__ y, int n_ttiles, int ks,
                                                      float *__restrict__ partial, ld::OperandImage out, bool quads) {
    constexpr bool SWI = (EPI == ld::GEMM_SWIGLU);
    constexpr int BM = 32 * AT, BN = 32 * BT, NOUT = SWI ? BN / 2 : BN;
    constexpr int ROWS = TERMS * BM + BN, STAGE = ROWS * 128;
    static_assert(!SWI || BT % 2 == 0, "a wave holds as many gate as up tiles, and the four waves' copies j cover 32 rows of one matrix");
    constexpr int WOUT = SWI ? BT / 2 : BT;           // output column tiles per wave
    constexpr int P = ROWS / 32;                      // copies per wave and chunk: copy j of wave w covers rows (4 j + w) 8 .. + 8
    constexpr int NA = TERMS * AT, NM = NA * BT, NR = NA + BT;      // A tiles, MFMAs and operand reads of a k-step
    // two stages: copies (for the chunk after next) issued in the second half of a chunk; the rest in the first half of the chunk that
    // follows.  Three: all in the chunk that follows
    constexpr int PRE = S == 2 ? (P * 12 + 15) / 16 : 0, YOUNGER = (S - 2) * P + PRE;      // copies of the chunks behind the next
    // A tiles of the first k-step that are multiplied after its stage is given up, and of the last one that are multiplied
    // while the next chunk's operands are read
    constexpr int NL = NA >= 4 ? NA / 4 : 1, NF = NA >= 4 ? NA / 4 : 1;
    extern __shared__ __attribute__((aligned(1024))) char lds[];

    // Blocks b, b + 8, ... run on one XCD.  Each XCD takes an equal run of the work items (K slab fastest, then row tile,
    // then column block), so that its workgroups share W panels in its L2 and no XCD gets an item more than another
    const int xcd = blockIdx.x & 7, n_items = n_ttiles * ks * ((N + NOUT - 1) / NOUT);
    const int item = (int)((int64_t)n_items * xcd / 8) + (blockIdx.x >> 3);
    if (item >= (int)((int64_t)n_items * (xcd + 1) / 8)) return;
    const int kz = item % ks, tt_idx = item / ks % n_ttiles, nb = item / (ks * n_ttiles);
    const int t0 = tt_idx * BM, n0 = nb * NOUT;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;

    // lane offsets of the copies from the tile's first row of each matrix (rows clamped: clamped rows are never stored)
    uint32_t coff[P];
#pragma unroll
    for (int j = 0; j < P; j++) {
        const int vr = (4 * j + wave) * 8 + (lane >> 3);                       // row of the stage
        int row;
        if (32 * j < TERMS * BM) {
            row = min(vr % BM, T - 1 - t0);
        } else {
            row = min((vr - TERMS * BM) % NOUT, N - 1 - n0);      // SwiGLU: the gate rows, then the up rows of the same columns
        }
        coff[j] = ((uint32_t)row * (uint32_t)K + ((lane & 7) ^ ((vr >> 1) & 7)) * 8) * 2u;
    }
    const BufferCopy from_hi(xhi + (int64_t)t0 * K), from_lo((TERMS == 2 ? xlo : xhi) + (int64_t)t0 * K), from_w(W + (int64_t)n0 * K),
        from_up(W + (int64_t)(SWI ? N + n0 : n0) * K);
    const int c_begin = (int)((int64_t)kz * (K / 64) / ks), n = (int)((int64_t)(kz + 1) * (K / 64) / ks) - c_begin;      // >= 2 chunks
    auto copy = [&](int c, int st, int j) {      // copy j of chunk c into stage st
        char *dst = lds + st * STAGE + (4 * j + wave) * 1024;
        const uint32_t off = (uint32_t)(c_begin + min(c, n - 1)) * 128u;
        if (32 * j < BM) from_hi(dst, coff[j], off);
        else if (32 * j < TERMS * BM) from_lo(dst, coff[j], off);
        else if (32 * j >= TERMS * BM + NOUT) from_up(dst, coff[j], off);
        else from_w(dst, coff[j], off);
    };

    f32x4 acc[AT][BT];
#pragma unroll
    for (int i = 0; i < AT; i++)
#pragma unroll
        for (int j = 0; j < BT; j++) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    struct Frags { u32x4 a[NA], w[BT]; };
    const int sw = (l16 >> 1) & 7;
    auto read = [&](Frags &f, int st, int kstep, int r) {      // operand read r of a k-step, in the order of use
        const char *base = lds + st * STAGE + l16 * 128 + (((kstep * 4 + kg) ^ sw) * 16);
        const int i = r == 0 ? 0 : r - BT, j = r - 1;
        if (r == 0 || r > BT) f.a[i] = *reinterpret_cast<const u32x4 *>(base + ((i / AT) * BM + (wm * AT + i % AT) * 16) * 128);
        else f.w[j] = *reinterpret_cast<const u32x4 *>(base + (TERMS * BM + j / WOUT * NOUT + (wn * WOUT + j % WOUT) * 16) * 128);
    };
    // MFMA m of a k-step: A tile m / BT, W tile m % BT
    auto mfma = [&](Frags &f, int m) {
        const int i = m / BT, j = m % BT;
        if (WF == 1 && i == 0) f.w[j] = __builtin_bit_cast(u32x4, bf16x8_to_f16x8(f.w[j]));
        if constexpr (WF == 0) tile_mfma_bf16(acc[i % AT][j], f.w[j], f.a[i]);
        else if (WF == 1 && i == 0) tile_mfma_f16_after_valu(acc[i % AT][j], f.w[j], f.a[i]);
        else tile_mfma_f16(acc[i % AT][j], f.w[j], f.a[i]);
    };
    // nm MFMAs (from number m0 of f on, then from the first of g on) in this order, nr operand reads and nc copies spread
    // evenly between them
    auto mix = [&](Frags &f, Frags &g, int m0, int nm, int nr, auto &&rd, int nc, auto &&cp) {
#pragma unroll
        for (int k = 0; k < nm; k++) {
            if (m0 + k < NM) mfma(f, m0 + k);
            else mfma(g, m0 + k - NM);
#pragma unroll
            for (int r = (k * nr + nm - 1) / nm; r < ((k + 1) * nr + nm - 1) / nm; r++) rd(r);
#pragma unroll
            for (int c = (k * nc + nm - 1) / nm; c < ((k + 1) * nc + nm - 1) / nm; c++) cp(c);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

#pragma unroll
    for (int c = 0; c < S; c++) {
#pragma unroll
        for (int j = 0; j < (c < S - 1 ? P : PRE); j++) copy(c, c, j);
        // the count below lets all copies but chunk 0's be outstanding (arithmetic may cross)
        __builtin_amdgcn_sched_barrier(7);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(YOUNGER) : "memory");
    asm volatile("s_barrier" ::: "memory");
    Frags f0, f1;
#pragma unroll
    for (int r = 0; r < NR; r++) read(f0, 0, 0, r);
    auto none = [](int) {};
    // One loop for all chunks.  Past the last one the copies fetch it again, into the stage that nobody reads any more.  Two stages are told
    // apart by the parity of i, and their second barrier has no reads to wait for: with the general form's few scalar instructions more a chunk
    // the fp16 products of 14336 x 4096 pairs took 106.6 instead of 105.1 us at 512 rows, 213.6 instead of 209.3 at 1024 (96 products 0.2 %)
    int i = 0, at = 0;
    do {
        const int st = S == 2 ? i & 1 : at, next = S == 2 ? st ^ 1 : st + 1 == S ? 0 : st + 1, last = S == 2 ? st ^ 1 : st == 0 ? S - 1 : st - 1;
        asm volatile("s_nop 1" ::: "memory");      // before the first pass: the cleared accumulators
        if constexpr (S == 2) {
            mix(f0, f0, 0, NM - NL * BT, NR, [&](int r) { read(f1, st, 1, r); }, P - PRE, [&](int c) { copy(i + 1, last, PRE + c); });
            // every wave has this chunk's operands in registers: its stage is requested again, for chunk i + 2
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            mix(f0, f1, NM - NL * BT, (NL + NA - NF) * BT, 0, none, PRE, [&](int c) { copy(i + 2, st, c); });
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(YOUNGER) : "memory");
        } else {      // the stage of the chunk before is free: every wave has passed the barrier below with its operands in registers
            constexpr int M1 = NM, M2 = (NA - NF) * BT, P1 = (P * M1 + M1 + M2 - 1) / (M1 + M2);
            mix(f0, f0, 0, M1, NR, [&](int r) { read(f1, st, 1, r); }, P1, [&](int c) { copy(i + S - 1, last, c); });
            mix(f1, f1, 0, M2, 0, none, P - P1, [&](int c) { copy(i + S - 1, last, P1 + c); });
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(YOUNGER) : "memory");
        }
        // the own copies of chunk i + 1 have landed (only those of later chunks are younger), and after the barrier everyone's
        mix(f1, f1, NM - NF * BT, NF * BT, NR, [&](int r) { read(f0, next, 0, r); }, 0, none);
        at = next;
    } while (++i < n);
    // the copies have left, and the last results are in their registers before anything reads them (the compiler does not
    // see into the assembly)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // accumulator (a, j) of lane (l16, kg): row t0 + (wm AT + a) 16 + l16, four columns from n0 + (wn WOUT + j) 16 + 4 kg on
    const int ncols = SWI ? 2 * N : N;            // row length of the partial-sum buffer
    // Four columns at once at any float's address: one at a time, a store touches four bytes of each of 64 sectors, which rows that
    // are no multiple of four floats paid for
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    auto put = [&](float *dst, const f32x4 &v, int left) {
        if (left >= 4) {
            *reinterpret_cast<f32x4_any *>(dst) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++)
                if (e < left) dst[e] = v[e];
        }
    };
    each<WOUT>([&](auto j) __attribute__((always_inline)) {
        const int col = n0 + (wn * WOUT + j) * 16 + 4 * kg, left = N - col;
        if (left <= 0) return;
        each<AT>([&](auto a) __attribute__((always_inline)) {
            const int t = t0 + (wm * AT + a) * 16 + l16;
            if (t >= T) return;
            if (ks > 1) {
                float *dst = partial + ((int64_t)kz * T + t) * ncols + col;
                put(dst, tile_result(acc[a][j]), left);
                if constexpr (SWI) put(dst + N, tile_result(acc[a][j + WOUT]), left);
                return;
            }
            float *dst = y + (int64_t)t * N + col;
            f32x4 v = tile_result(acc[a][j]);
            if constexpr (EPI == ld::GEMM_ADD) {
                if (left >= 4) {
                    v += *reinterpret_cast<const f32x4_any *>(dst);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        if (e < left) v[e] += dst[e];
                }
            }
            if constexpr (SWI) {
                const f32x4 up = tile_result(acc[a][j + WOUT]);
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = swiglu(v[e], up[e]);
                if (out.hi) {
                    if (quads) {      // rows a multiple of four columns, 16-byte aligned
                        store_operand4(out, t, (int64_t)t * N + col, make_float4(v[0], v[1], v[2], v[3]));
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            if (e < left) store_operand(out, t, (int64_t)t * N + col + e, v[e]);
                    }
                    return;
                }
            }
            put(dst, v, left);
        });
    });
}

template <int TERMS, int WF, int AT, int BT, int EPI, int S>
void launch_tile_stages(const TileLaunch &l) {
    constexpr int lds_bytes = tile_lds(TERMS, AT * 32, BT * 32, S);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)k_gemm_tile<TERMS, WF, AT, BT, EPI, S>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        attr_set = true;
    }
    LD_LAUNCH((k_gemm_tile<TERMS, WF, AT, BT, EPI, S>), dim3(l.grid), dim3(256), lds_bytes, l.s, l.W, l.hi, l.lo, l.T, l.N, l.K, l.y,
              l.n_ttiles, l.ks, l.partial, l.out, l.quads);
}
template <int TERMS, int WF, int AT, int BT, int EPI>
void launch_tile(const TileLaunch &l) {
    if constexpr (tile_twice(TERMS, AT * 32, BT * 32)) {
        if (l.grid > 256) return launch_tile_stages<TERMS, WF, AT, BT, EPI, 2>(l);
    }
    launch_tile_stages<TERMS, WF, AT, BT, EPI, tile_stages(TERMS, AT * 32, BT * 32)>(l);
}
template <int TERMS, int WF, int AT, int BT>
void launch_tile_epilogue(const TileLaunch &l) {
    if (l.epi == ld::GEMM_STORE) launch_tile<TERMS, WF, AT, BT, ld::GEMM_STORE>(l);
    else if (l.epi == ld::GEMM_ADD) launch_tile<TERMS, WF, AT, BT, ld::GEMM_ADD>(l);
    else if constexpr (BT % 2 == 0) launch_tile<TERMS, WF, AT, BT, ld::GEMM_SWIGLU>(l);
}

}  // namespace
