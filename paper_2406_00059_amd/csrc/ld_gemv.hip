// Batch-1 matrix-vector product for bf16 matrices, organised by column slabs.
//
// HBM-bound: every matrix element is read exactly once, so the design goal is to keep as many
// 16-byte loads in flight per CU as possible, with as few vector-ALU instructions per loaded byte
// as possible, and with the same amount of work on every CU.
//
//  - Two workgroups of eight waves per CU; workgroup i owns the contiguous output range
//    [i N / G, (i+1) N / G), so all workgroups stream the same number of bytes (+-1 row).
//  - A workgroup's work is cut into items of two rows (the two of a pair, or neighbours) and one slab of columns, 2048 or 512
//    (CPS 4 or 1): a run of 4 KB or 1 KB of each row by one wave, 16 bytes a lane and load.  Its items, slab by slab, are
//    dealt to the waves in equal runs, and a wave keeps two items in flight.
//  - The input, multiplied by the RMSNorm gain, sits in LDS: it is requested before the first rows, and an item reads
//    its slab once for two rows, as many bytes as the rows have.
//  - An item ends in two sums across a wave (six shuffles), which wait in LDS: the only barriers are the one after
//    the input has arrived and the one before the epilogue.
//  What bounds it: HBM, and at both ends of the launch the latency of the input and of the last rows.  Long runs stream
//  faster (gate/up of the 7B shape, loads alone: 32.7 us in 128-byte runs, 28.7 in 4 KB), but where a wave would get two items
//  or fewer of 2048 columns it has nothing to overlap its sums with, and short slabs win (us, 2048 / 512 columns: 4096x4096
//  8.8 / 8.2, 2048x8192 8.9 / 8.1, 6144x4096 11.5 / 10.8; the other way about 4096x11008 17.4 / 18.5, 14336x4096 36.0 / 37.7).
//  - The RMSNorm scale 1 / rms(x) is a scalar, so it is applied to the finished dot products; its
//    sum of squares is accumulated when the input goes to LDS.
//  - Epilogues: store, residual add, SwiGLU (gate row r with up row N + r), and "RoPE + cache
//    append" for the fused q/k/v projection (row i of a head with row i + hd/2, then rotate by
//    the position's angle and write k, v straight into the paged pool).
#include "ld_gemv.h"
#include "ld_device.h"
#include "ld_internal.h"
#include <cstdlib>

using namespace ldd;

namespace {

constexpr int WAVES = 8;             // per workgroup, two workgroups per CU
constexpr int PIECE = WAVE * 8;      // columns that one load instruction of a wave covers
constexpr int LONG_SLAB = 4;         // pieces of a slab
constexpr int MAX_K = 16384;
constexpr int MAX_PARTS = 2048;      // partial sums of a workgroup: with the largest input 72 KB of LDS, two fit a CU

__device__ __forceinline__ float dot8(const u32x4_t &w, const float (&x)[8]) {
    float s = 0.f;
    s = fmaf(__uint_as_float(w.x << 16), x[0], s);
    s = fmaf(__uint_as_float(w.x & 0xffff0000u), x[1], s);
    s = fmaf(__uint_as_float(w.y << 16), x[2], s);
    s = fmaf(__uint_as_float(w.y & 0xffff0000u), x[3], s);
    s = fmaf(__uint_as_float(w.z << 16), x[4], s);
    s = fmaf(__uint_as_float(w.z & 0xffff0000u), x[5], s);
    s = fmaf(__uint_as_float(w.w << 16), x[6], s);
    s = fmaf(__uint_as_float(w.w & 0xffff0000u), x[7], s);
    return s;
}

// Matrix row of unit u, member m (m = 0: first row of the unit; m = 1: its partner row).
template <int EPI>
__device__ __forceinline__ int unit_row(int u, int m, int N, int half_hd) {
    if constexpr (EPI == ld::GEMV_SWIGLU) return u + m * N;
    else if constexpr (EPI == ld::GEMV_ROPE_KV) return (u / half_hd) * (2 * half_hd) + (u % half_hd) + m * half_hd;
    else return u;
}

// KMAX: columns the input's place in LDS is for.  CPS: pieces of a slab.
template <int KMAX, int CPS, int EPI, bool NORM>
__global__ __launch_bounds__(WAVES * WAVE, 4) void k_gemv1(const bf16_t *__restrict__ W, const float *__restrict__ x,
                                                        const float *__restrict__ g, float eps, int N, int K,
                                                        float *__restrict__ y, ld::RopeKvArgs rk) {
    constexpr int SLAB = CPS * PIECE;
    constexpr bool PAIRED = (EPI == ld::GEMV_SWIGLU || EPI == ld::GEMV_ROPE_KV);
    constexpr int UPI = PAIRED ? 1 : 2;        // output units of an item: it has two rows either way
    __shared__ __attribute__((aligned(16))) float xs[KMAX / 8][2][4];      // group g of eight columns: float4s (g / 64) 128 + g % 64 and 64 further
    __shared__ float part[MAX_PARTS];
    __shared__ float part_ss[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half_hd = (EPI == ld::GEMV_ROPE_KV) ? rk.hd / 2 : 1;
    const int n_units = (EPI == ld::GEMV_ROPE_KV) ? N / 2 : N;
    const int u_begin = (int)((int64_t)blockIdx.x * n_units / gridDim.x);
    const int units = (int)((int64_t)(blockIdx.x + 1) * n_units / gridDim.x) - u_begin;
    const int n_slabs = (K + SLAB - 1) / SLAB, per_slab = (units + UPI - 1) / UPI, n_items = per_slab * n_slabs;
    const int it_end = (wave + 1) * n_items / WAVES;

    // the input is requested before the first rows, so that waiting for it does not wait for them
    constexpr int XT = KMAX / 8 / (WAVES * WAVE);      // groups of eight columns a thread brings in
    float xv[XT][8], gv[NORM ? XT : 1][8];
#pragma unroll
    for (int i = 0; i < XT; i++) {
        const int col = (i * WAVES * WAVE + tid) * 8;
        if (col < K) {
            load8(x + col, xv[i]);
            if (NORM) load8(g + col, gv[i]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++) xv[i][e] = 0.f;
            if (NORM) {
#pragma unroll
                for (int e = 0; e < 8; e++) gv[i][e] = 0.f;
            }
        }
    }

    float before = 0.f;      // the old value for the residual add
    if (EPI == ld::GEMV_ADD && tid < units) before = y[u_begin + tid];

    u32x4_t bufA[2][CPS], bufB[2][CPS];
    auto issue = [&](u32x4_t (&buf)[2][CPS], int it) {
        const int slab = it / per_slab, u0 = u_begin + (it - slab * per_slab) * UPI;
#pragma unroll
        for (int r = 0; r < 2; r++) {
            if (!PAIRED && u0 + r >= u_begin + units) {      // an odd last row has no neighbour; the sum is not used
#pragma unroll
                for (int c = 0; c < CPS; c++) buf[r][c] = (u32x4_t){0u, 0u, 0u, 0u};
                continue;
            }
            const int u = PAIRED ? u0 : u0 + r;
            const bf16_t *p = W + (int64_t)unit_row<EPI>(u, PAIRED ? r : 0, N, half_hd) * K;
#pragma unroll
            for (int c = 0; c < CPS; c++) {
                const int col = slab * SLAB + c * PIECE + lane * 8;
                buf[r][c] = col < K ? load_stream16(p + col) : (u32x4_t){0u, 0u, 0u, 0u};
            }
        }
    };
    int it = wave * n_items / WAVES;
    if (it < it_end) issue(bufA, it);
    if (it + 1 < it_end) issue(bufB, it + 1);

    // cache append: position and physical block, looked up while the weights are on their way
    int kv_pos = 0;
    int64_t kv_phys = 0;
    if constexpr (EPI == ld::GEMV_ROPE_KV) {
        kv_pos = rk.pos[0];
        kv_phys = rk.table[(int64_t)rk.seq_slot[0] * rk.table_stride + (kv_pos >> 4)];
    }

    // the input (gain applied) goes to LDS, piece by piece in two planes, so that 64 lanes read 1 KB without conflicts
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < XT; i++) {
        const int o = i * WAVES * WAVE + tid;      // group of eight columns; piece o / 64, lane o % 64
        if (NORM) {
#pragma unroll
            for (int e = 0; e < 8; e++) {
                ss = fmaf(xv[i][e], xv[i][e], ss);
                xv[i][e] *= gv[i][e];
            }
        }
        float4 *at = reinterpret_cast<float4 *>(xs) + (o >> 6) * 128 + (o & 63);
        at[0] = make_float4(xv[i][0], xv[i][1], xv[i][2], xv[i][3]);
        at[64] = make_float4(xv[i][4], xv[i][5], xv[i][6], xv[i][7]);
    }
    if (NORM) {
        ss = wave_sum(ss);
        if (lane == 0) part_ss[wave] = ss;
    }
    lds_barrier();

    auto consume = [&](u32x4_t (&buf)[2][CPS], int item) {
        const int slab = item / per_slab;
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int c = 0; c < CPS; c++) {
            const float4 *at = reinterpret_cast<const float4 *>(xs) + (slab * CPS + c) * 128 + lane;
            const float4 lo = at[0], hi = at[64];
            const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            a0 += dot8(buf[0][c], v);
            a1 += dot8(buf[1][c], v);
        }
        // lanes below 32 end up with the first row's sum, the others with the second's
        const bool upper = lane >= 32;
        float s = (upper ? a1 : a0) + __shfl_xor(upper ? a0 : a1, 32, WAVE);
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) s += __shfl_xor(s, off, WAVE);
        if ((lane & 31) == 0) part[item * 2 + (lane >> 5)] = s;
    };
    for (; it < it_end; it += 2) {
        consume(bufA, it);
        if (it + 2 < it_end) issue(bufA, it + 2);
        if (it + 1 < it_end) {
            consume(bufB, it + 1);
            if (it + 3 < it_end) issue(bufB, it + 3);
        }
    }
    lds_barrier();

    float rstd = 1.f;
    if (NORM) {
        float s2 = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; w++) s2 += part_ss[w];
        rstd = 1.0f / sqrtf(s2 / K + eps);
    }
    for (int i = tid; i < units; i += WAVES * WAVE) {
        const int u = u_begin + i;
        float a = 0.f, b = 0.f;
        for (int sl = 0; sl < n_slabs; sl++) {
            const float *p = part + sl * per_slab * 2 + (PAIRED ? 2 * i : i);
            a += p[0];
            if (PAIRED) b += p[1];
        }
        a *= rstd;
        b *= rstd;
        if constexpr (EPI == ld::GEMV_STORE) {
            y[u] = a;
        } else if constexpr (EPI == ld::GEMV_ADD) {
            y[u] = (i == tid ? before : y[u]) + a;
        } else if constexpr (EPI == ld::GEMV_SWIGLU) {
            y[u] = a / (1.0f + __expf(-a)) * b;
        } else {
            const int hh = u / half_hd, i = u % half_hd, hd = 2 * half_hd;
            if (hh < rk.H + rk.Hkv) {   // q or k head: rotate the pair
                const float2 cs = rk.cos_sin[i];
                const float ra = a * cs.x - b * cs.y, rb = a * cs.y + b * cs.x;
                a = ra;
                b = rb;
            }
            if (hh < rk.H) {
                y[hh * hd + i] = a;
                y[hh * hd + i + half_hd] = b;
            } else {
                const int which = hh < rk.H + rk.Hkv ? 0 : 1;
                const int j = hh - rk.H - which * rk.Hkv;
                bf16_t *blk = rk.pool + kv_phys * kv_block_elems(rk.Hkv, hd);
                const int slot = kv_pos & 15;
                if (which == 0) {
                    blk[kv_k_offset(hd, j, slot, i)] = f32_to_bf16(a);
                    blk[kv_k_offset(hd, j, slot, i + half_hd)] = f32_to_bf16(b);
                } else {
                    blk[kv_v_offset(rk.Hkv, hd, j, slot, i)] = f32_to_bf16(a);
                    blk[kv_v_offset(rk.Hkv, hd, j, slot, i + half_hd)] = f32_to_bf16(b);
                }
            }
        }
    }
}

template <int KMAX, int CPS, bool NORM>
void launch_kmax(const bf16_t *W, const float *x, const float *g, float eps, int N, int K, int epi, float *y,
                 const ld::RopeKvArgs &rk, int grid, hipStream_t s) {
#define LD_GEMV1(EPI_) LD_LAUNCH((k_gemv1<KMAX, CPS, EPI_, NORM>), dim3(grid), dim3(WAVES * WAVE), 0, s, W, x, g, eps, N, K, y, rk)
    switch (epi) {
        case ld::GEMV_STORE: LD_GEMV1(ld::GEMV_STORE); break;
        case ld::GEMV_ADD: LD_GEMV1(ld::GEMV_ADD); break;
        case ld::GEMV_SWIGLU: LD_GEMV1(ld::GEMV_SWIGLU); break;
        default: LD_GEMV1(ld::GEMV_ROPE_KV); break;
    }
#undef LD_GEMV1
}

int env_int(const char *name, int dflt) {
    const char *v = getenv(name);
    return v ? atoi(v) : dflt;
}

}  // namespace

namespace ld {

bool gemv1_supported(int N, int K, int epi) {
    if (K % 8 || K <= 0 || N <= 0) return false;
    if (K > MAX_K) return false;
    if (epi == GEMV_ROPE_KV && N % 2) return false;
    return true;
}

void launch_gemv1(const uint16_t *W, const float *x, const float *g, float eps, int N, int K, int epi, float *y,
                  const RopeKvArgs *rk, hipStream_t s) {
    static int n_cu = 0;
    if (!n_cu) {
        hipDeviceProp_t p;
        int dev = 0;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&p, dev) == hipSuccess) n_cu = p.multiProcessorCount;
        if (n_cu <= 0) n_cu = 256;
    }
    const int n_units = epi == GEMV_ROPE_KV ? N / 2 : N;
    // Two workgroups per CU; more (which then follow one another) where a workgroup's partial sums would not fit.
    const int n_slabs = (K + LONG_SLAB * PIECE - 1) / (LONG_SLAB * PIECE);
    const bool paired = epi == GEMV_SWIGLU || epi == GEMV_ROPE_KV;
    const int max_units = MAX_PARTS / n_slabs / (paired ? 2 : 1) - 2;
    static const int forced = env_int("LD_GEMV_WGS_PER_CU", 0);   // tuning knob
    const int least = (n_units + max_units - 1) / max_units;
    int grid = n_cu * (forced > 0 ? forced : 2);
    while (grid < least) grid += n_cu;
    if (grid > n_units) grid = n_units;
    RopeKvArgs none{};
    const RopeKvArgs &r = rk ? *rk : none;
    // Slabs of one piece where a wave would get two items of long slabs or fewer (see the top of the file).  A workgroup with a
    // single row has half-empty items and stays with few of them (640x16384: 7.8 us, 8.5 in short slabs), and so do long
    // inputs, which every workgroup brings in for few rows (1024x16384: 8.9, 11.6).  At most 2 WAVES LONG_SLAB items of two
    // sums: well below MAX_PARTS.
    const int units = (n_units + grid - 1) / grid, items = (paired ? units : (units + 1) / 2) * n_slabs;
    const bool short_slabs = items <= 2 * WAVES && n_units >= 2 * grid && K <= 8192;
#define LD_KMAX(KMAX_, CPS_)                                                                 \
    do {                                                                                     \
        if (g) launch_kmax<KMAX_, CPS_, true>(W, x, g, eps, N, K, epi, y, r, grid, s);       \
        else launch_kmax<KMAX_, CPS_, false>(W, x, g, eps, N, K, epi, y, r, grid, s);        \
    } while (0)
    if (short_slabs) LD_KMAX(8192, 1);
    else if (K <= 8192) LD_KMAX(8192, LONG_SLAB);
    else LD_KMAX(MAX_K, LONG_SLAB);
#undef LD_KMAX
}

}  // namespace ld
