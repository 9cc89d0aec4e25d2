// Chunk-prefill attention over the paged KV pool on the matrix cores (bf16 pool, head_dim 128).
//
// A prefill segment is a run of consecutive rows of one sequence at consecutive positions; row r
// (position p_r) attends to every cached position j <= p_r: the earlier context plus, causally, the
// rows of its own chunk, whose keys/values were appended to the pool just before.  With an attention
// band of W positions it attends to max(0, p_r - W + 1) <= j <= p_r only: the walk over the KV positions
// starts at the first position the tile's first row sees, and a wave skips the steps that lie wholly
// before the band of its own first row.
//
// Work split: a workgroup (4 waves) takes 128 consecutive rows of a segment and one head; wave w owns rows
// [32w, 32w+32).  All four waves walk the same KV positions in steps of 32; the key rows and the (transposed) value
// tile of two steps (a unit) are copied into LDS in 16-byte pieces that were loaded into registers one unit earlier,
// behind block-table entries read another unit earlier, and shared by the four waves.  LDS is double buffered, with one
// barrier per unit.  Two workgroups fit a CU, so that one wave's softmax overlaps another's MFMAs.
//
// What bounds it: the work per step at two waves per SIMD, vector arithmetic and exponentials (which hold up the SIMD's MFMAs)
// as much as the MFMAs themselves.  Hence two steps a barrier; in F16 both steps' scores at once; and as little as possible around
// them: blocks are addressed in scalar registers, the range check of a widened pair is one instruction, a unit that lies below the
// last position is staged without a look at each piece, scores start at -m, and a maximum is looked for only where the
// exponentials against the last one have grown large.  The operands of the next MFMAs are read from LDS ahead of them, in an order that
// is pinned: left alone, the compiler reads each right before its use and waits for it.  Queries come in whole rows and shares go out in
// whole lanes: 16 bytes of each of 64 rows an instruction cost some 6000 and 2000 cycles a workgroup.
// 12 tiles x 32 heads (four segments of 257 rows) at contexts 2.2k .. 6.4k: 322 -> 214 -> 181 -> 171 us with these (one step at a time,
// two, no passes over the queries, the last three), 167 with the path for few rows; one 256-row chunk behind 1500, in two terms, 33 -> 31; one
// of 2048 behind 2048 151 -> 135; over 135 sets of tiles (4 .. 40 heads, 1 .. 24 tiles, walks of 4 .. 250 steps) the last three give 12 % in
// the mean, 9 % in two terms.
// Forming the next unit's scores between this one's exponentials, and staging between its value products, was level
// (209 and 79 us: its second set of scores fills the registers).  Two halves of a workgroup that take the matrix cores in turn, on
// pairs of tiles, reach 153 us in the first example but lose by up to three times where the work is small.
//
// Both products are computed transposed, so that the query index is the MFMA column (= lane % 32)
// everywhere and the online-softmax statistics of a query live in the lanes that hold its scores:
//   S^T[kv, q] = K[kv, :] . Q[q, :]      A = K rows   (LDS),
//                                        B = Q        (registers, split into bf16 hi + lo)
//   O^T[d, q] += V^T[d, kv] P^T[kv, q]   A = V^T      (LDS; the pool stores the values of a block
//                                                      transposed, [dim][16 positions]),
//                                        B = P^T      (the score registers themselves: in the 32x32
//                                                      accumulator layout a lane already holds, for
//                                                      its query, exactly the 8 kv slots of an operand)
// Row r of a score tile is NOT position kv0 + r: within each 16 rows, bits 2 and 3 of the row index are
// swapped (row r <-> position 16 (r/16) + tau(r%16), tau(r) = (r & 3) | (r & 4) << 1 | (r & 8) >> 1), so
// that the 8 accumulator registers a lane feeds into one value MFMA are 8 CONSECUTIVE positions, i.e. one
// 16-byte piece of the transposed value tile.
// Scores are kept in the log2 domain (q is pre-multiplied by log2(e)/sqrt(hd)); m, l and O are float32.
//
// Few tiles with long contexts (an observation appended to one long sequence) would leave most CUs idle and make every
// workgroup walk the whole context, and tiles of different length would leave them waiting for the longest, so the KV range
// of a tile is dealt out in shares of `per` steps to as many workgroups as it has shares; each writes its unnormalised
// output with its maximum and sum, and a merge kernel combines them in order.  Shares of one length, not one number of
// shares: four segments behind 0.5k .. 2.9k positions take 98 + 16 us per layer (walk + merge) in two shares each, 86 + 9 so.
#include "ld_attn_prefill.h"
#include "ld_device.h"
#include "ld_internal.h"
#include <type_traits>

using namespace ldd;

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;

constexpr int HD = 128;
constexpr int KVB = 32;          // kv positions per step
constexpr int KLD = HD + 8;      // LDS row stride of the key tile (elements): 272 bytes, conflict-free 16-byte reads
constexpr int MAX_SPLITS = 16;   // shares of a tile's KV steps, at most
constexpr int FEW_ROWS = 16;     // tiles of up to so many rows take few_rows()
constexpr int VLD = KVB + 8;     // LDS row stride of the transposed value tile (elements): 80 bytes

__device__ __forceinline__ int tau(int r) { return (r & 19) | ((r & 4) << 1) | ((r & 8) >> 1); }

// Two floats as packed fp16, rounded to nearest.
__device__ __forceinline__ uint32_t pack2_f16(float a, float b) {
    return __builtin_bit_cast(uint32_t, (f16x2){(_Float16)a, (_Float16)b});
}
// Eight bf16 numbers as fp16: exact where fp16 can hold the value (truncation below 2^-14, the largest finite
// fp16 beyond +-65504: the caller looks for such values with `mag`, the running maximum of the magnitudes, one instruction a
// pair.  It is NaN from the first NaN on).
__device__ __forceinline__ u32x4 bf16x8_to_f16x8(const u32x4 &w, float &mag) {
    u32x4 h;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float a = __uint_as_float(w[i] << 16), b = __uint_as_float(w[i] & 0xffff0000u);
        h[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
        mag = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mag, fabsf(a)), fabsf(b));
    }
    return h;
}

// 16 bytes from a lane's offset in a block that is the same for the whole wave: no address arithmetic in vector registers.
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ u32x4 load_in_block(const bf16_t *block, uint32_t off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(block), 0, -1, 0x00020000), off, 0, 0));
}
#else
__device__ u32x4 load_in_block(const bf16_t *, uint32_t) { return u32x4{}; }
#endif

// Partial results: [tile][head][share][128 rows][HD] and (m, l) likewise.  Place of dimensions 8 d8 + 4 hi .. + 4 of a row among the 128: as
// the lanes that have them store them, 1 KB in a row a wave.
__device__ __forceinline__ int part_place(int row, int d8, int hi) { return (((row >> 5) * (HD / 8) + d8) * 64 + hi * 32 + (row & 31)) * 4; }

// Steps of KVB positions that a tile walks: from the first position its first row sees (rounded down) to its last row's.
__device__ __forceinline__ int tile_start(const int4 &tile, int window) { return window > 0 ? (max(tile.z - window + 1, 0) & ~(KVB - 1)) : 0; }
__device__ __forceinline__ int tile_steps(const int4 &tile, int window) { return (tile.z + tile.y - 1 - tile_start(tile, window)) / KVB + 1; }

// The tile that comes rank-th when they are sorted by their steps (longest first, those of few rows, which take a fraction of the time, last;
// ties by index), and its index; more than a wave's lanes of them stay in their own order.
__device__ __forceinline__ int4 nth_longest(const int4 *__restrict__ tiles, int n_tiles, int window, int rank, int &index) {
    index = rank;
    if (n_tiles == 1 || n_tiles > WAVE) return tiles[rank];
    const int lane = threadIdx.x & 63;
    const int4 t = tiles[min(lane, n_tiles - 1)];
    const int own = t.y <= FEW_ROWS ? 0 : tile_steps(t, window);
    int before = 0;
    for (int i = 0; i < n_tiles; i++) {
        const int other = __builtin_amdgcn_readlane(own, i);
        before += other > own || (other == own && i < lane);
    }
    index = __ffsll(__ballot(lane < n_tiles && before == rank)) - 1;
    return make_int4(__builtin_amdgcn_readlane(t.x, index), __builtin_amdgcn_readlane(t.y, index), __builtin_amdgcn_readlane(t.z, index),
                     __builtin_amdgcn_readlane(t.w, index));
}

// Tiles of up to FEW_ROWS rows, which are not worth the staging (a 257-row segment ends in a tile of one row, whose walk took as long as
// half a full tile's): each wave walks every fourth step of the share by itself.  Four segments of 257 rows behind 2.2k .. 6.4k, GQA 4:1:
// 126 -> 119 us; four lone 5-row tiles of 32 heads over 8 50 -> 26 in two terms; 135 sets of tiles 4 % faster in the mean in two
// terms, 1 % in fp16 (33 rows upwards pay 0 - 3 % for the second path in the kernel).  Arithmetic and operands as in the decode kernel
// for grouped heads, a row of the tile in place of a head (two bf16 terms in both forms; in F16 the range is checked all the same).
union FewLds {
    char keys[4][4096];      // a block's keys on their way to operands, of each wave
    struct { float o[4][FEW_ROWS][HD + 4], ml[4][FEW_ROWS][2]; } waves;
};
template <bool F16>
__device__ __forceinline__ void few_rows(const float *__restrict__ q, int q_stride, const bf16_t *__restrict__ pool, int Hkv, const int32_t *__restrict__ trow,
                                         const int4 &tile, int h, int H, int kvh, int window, float scale_log2e, int kv_begin, int kv_end,
                                         FewLds &lds, float *__restrict__ part_o, float *__restrict__ part_ml, float *__restrict__ out,
                                         const ld::OperandImage &image, int *__restrict__ f16_flag) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, rg = lane >> 4;      // column of the 16 x 16 tiles: row of the tile
    const int last = tile.z + tile.y - 1, first_held = window > 0 ? (max(tile.z - window + 1, 0) & ~15) : 0;
    const int row = min(c, tile.y - 1), pos = tile.z + row, low = window > 0 ? max(pos - window + 1, 0) : 0;
    const int low_last = window > 0 ? max(last - window + 1, 0) : 0;      // all rows see [low_last, tile.z]
    const int64_t block_stride = kv_block_elems(Hkv, HD);
    float mag = 0.f;
    u16x2 most = {0, 0};      // F16: largest magnitudes of the keys and values
    bf16x8 qh[4], ql[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        float v[8];
        load8(q + (int64_t)(tile.x + row) * q_stride + h * HD + 32 * j + 8 * rg, v);
        u32x4 hw, lw;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const float a = v[2 * e] * scale_log2e, b = v[2 * e + 1] * scale_log2e;
            mag = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mag, fabsf(a)), fabsf(b));
            uint32_t lo;
            hw[e] = split2_bf16(a, b, lo);
            lw[e] = lo;
        }
        qh[j] = __builtin_bit_cast(bf16x8, hw);
        ql[j] = __builtin_bit_cast(bf16x8, lw);
    }
    f32x4 o[8];      // O^T: dims 16 nt + 4 rg + i of column c
#pragma unroll
    for (int nt = 0; nt < 8; nt++) o[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    // piece p (8 dims) of slot s sits in slot p ^ s of its 256-byte row
    char *tk = lds.keys[wave], *tk_st[4];
    const char *tk_ld[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int sl = 4 * j + rg;
        tk_st[j] = tk + sl * 256 + ((c ^ sl) & 15) * 16;
        tk_ld[j] = tk + c * 256 + ((sl ^ c) & 15) * 16;
    }
    const int steps = (kv_end - kv_begin + KVB - 1) / KVB, mine = (steps - wave + 3) / 4;      // of the share, of this wave
    u32x4 kf[2][4];
    u32x2 vf[8][2];
    for (int s0 = 0; s0 < mine; s0 += 32) {      // a lane has the table's entry of one of the next 64 blocks
        const int entry = trow[max(min((kv_begin >> 4) + 2 * (wave + 4 * (s0 + (lane >> 1))) + (lane & 1), last >> 4), first_held >> 4)];
        const int k = min(mine - s0, 32);
        auto block = [&](int t, int u) __attribute__((always_inline)) { return pool + (int64_t)__builtin_amdgcn_readlane(entry, 2 * t + u) * block_stride; };
        auto load_keys = [&](int t, int u) __attribute__((always_inline)) {
            const bf16_t *kp = block(t, u) + kv_k_offset(HD, kvh, 0, 0) + 8 * lane;
#pragma unroll
            for (int j = 0; j < 4; j++) kf[u][j] = *reinterpret_cast<const u32x4 *>(kp + 512 * j);
        };
        auto load_values = [&](int t, int u) __attribute__((always_inline)) {
            const bf16_t *vp = block(t, u) + kv_v_offset(Hkv, HD, kvh, 4 * rg, c);
#pragma unroll
            for (int nt = 0; nt < 8; nt++) vf[nt][u] = *reinterpret_cast<const u32x2 *>(vp + nt * 256);
        };
#pragma unroll
        for (int u = 0; u < 2; u++) { load_keys(0, u); load_values(0, u); }
        for (int t = 0; t < k; t++) {
            // the next step's keys are asked for when this one's are in LDS, its values when this one's are multiplied (the last step's
            // again behind it: without a condition)
            const int kv0 = kv_begin + KVB * (wave + 4 * (s0 + t)), next = min(t + 1, k - 1);
            if (kv0 + KVB - 1 > last || kv0 < first_held) {      // what was never written, or stands for a block that is not there
#pragma unroll
                for (int u = 0; u < 2; u++) {
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        const int p = kv0 + 16 * u + 4 * j + rg;
                        if (p > last || p < first_held) kf[u][j] = (u32x4){0u, 0u, 0u, 0u};
                    }
#pragma unroll
                    for (int nt = 0; nt < 8; nt++)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int p = kv0 + 16 * u + 4 * rg + e;
                            if (p > last || p < first_held) vf[nt][u][e / 2] &= e % 2 ? 0x0000ffffu : 0xffff0000u;
                        }
                }
            }
            if constexpr (F16) {      // as whole numbers: a NaN is the largest
                auto look = [&](uint32_t w) { most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, w & 0x7fff7fffu)); };
#pragma unroll
                for (int u = 0; u < 2; u++) {
#pragma unroll
                    for (int j = 0; j < 4; j++)
#pragma unroll
                        for (int e = 0; e < 4; e++) look(kf[u][j][e]);
#pragma unroll
                    for (int nt = 0; nt < 8; nt++) { look(vf[nt][u][0]); look(vf[nt][u][1]); }
                }
            }
            f32x4 sc[2];
#pragma unroll
            for (int u = 0; u < 2; u++) {
                sc[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 4; j++) *reinterpret_cast<u32x4 *>(tk_st[j]) = kf[u][j];
                load_keys(next, u);
                __builtin_amdgcn_wave_barrier();
                u32x4 kt[4];
#pragma unroll
                for (int j = 0; j < 4; j++) kt[j] = *reinterpret_cast<const u32x4 *>(tk_ld[j]);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const bf16x8 ka = __builtin_bit_cast(bf16x8, kt[j]);
                    sc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qh[j], sc[u], 0, 0, 0);
                    sc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, ql[j], sc[u], 0, 0, 0);
                }
            }
            if (kv0 + KVB - 1 > tile.z || kv0 < low_last) {      // element i of block u is position kv0 + 16 u + 4 rg + i
#pragma unroll
                for (int u = 0; u < 2; u++)
#pragma unroll
                    for (int i = 0; i < 4; i++) sc[u][i] = (uint32_t)(kv0 + 16 * u + 4 * rg + i - low) <= (uint32_t)(pos - low) ? sc[u][i] : -INFINITY;
            }
            float mb = -INFINITY;
#pragma unroll
            for (int u = 0; u < 2; u++)
#pragma unroll
                for (int i = 0; i < 4; i++) mb = fmaxf(mb, sc[u][i]);
            mb = fmaxf(mb, __shfl_xor(mb, 16, WAVE));
            mb = fmaxf(mb, __shfl_xor(mb, 32, WAVE));
            const float m_new = fmaxf(m, mb), ref = m_new > -INFINITY ? m_new : 0.f;
            const float scale = m > -INFINITY ? fast_exp2(m - ref) : 0.f;      // (o and l are zero with m)
            m = m_new;
            float p[8], psum = 0.f;
#pragma unroll
            for (int u = 0; u < 2; u++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    p[4 * u + i] = fast_exp2(sc[u][i] - ref);
                    psum += p[4 * u + i];
                }
            l = l * scale + psum;
            u32x4 ph, pl;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                uint32_t lo;
                ph[e] = split2_bf16(p[2 * e], p[2 * e + 1], lo);
                pl[e] = lo;
            }
            const bool rescale = __any(scale != 1.f);
#pragma unroll
            for (int nt = 0; nt < 8; nt++) {
                if (rescale) {
#pragma unroll
                    for (int i = 0; i < 4; i++) o[nt][i] *= scale;
                }
                const bf16x8 va = __builtin_bit_cast(bf16x8, (u32x4){vf[nt][0][0], vf[nt][0][1], vf[nt][1][0], vf[nt][1][1]});
                o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, __builtin_bit_cast(bf16x8, ph), o[nt], 0, 0, 0);
                o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, __builtin_bit_cast(bf16x8, pl), o[nt], 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < 2; u++) load_values(next, u);
        }
    }
    if constexpr (F16) {
        mag = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mag, bf16_to_f32(most[0])), bf16_to_f32(most[1]));
        if (!(mag <= 65504.f)) *f16_flag = 1;
    }
    l += __shfl_xor(l, 16, WAVE);
    l += __shfl_xor(l, 32, WAVE);
    lds_barrier();      // every wave is done with its keys
    if (c < tile.y) {
#pragma unroll
        for (int nt = 0; nt < 8; nt++) *reinterpret_cast<float4 *>(&lds.waves.o[wave][c][16 * nt + 4 * rg]) = make_float4(o[nt][0], o[nt][1], o[nt][2], o[nt][3]);
        if (rg == 0) *reinterpret_cast<float2 *>(lds.waves.ml[wave][c]) = make_float2(m, l);
    }
    lds_barrier();
    for (int idx = threadIdx.x; idx < tile.y * (HD / 4); idx += 256) {
        const int r = idx / (HD / 4), d = idx % (HD / 4) * 4;
        float M = -INFINITY, L = 0.f;
#pragma unroll
        for (int w = 0; w < 4; w++) M = fmaxf(M, lds.waves.ml[w][r][0]);
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < 4; w++) {      // a wave that saw no visible position has weight 0
            const float mw = lds.waves.ml[w][r][0], a = mw > -INFINITY ? fast_exp2(mw - M) : 0.f;
            const float4 x = *reinterpret_cast<const float4 *>(&lds.waves.o[w][r][d]);
            v.x += a * x.x; v.y += a * x.y; v.z += a * x.z; v.w += a * x.w;
            L += a * lds.waves.ml[w][r][1];
        }
        if (part_o) {
            *reinterpret_cast<float4 *>(part_o + part_place(r, d >> 3, (d >> 2) & 1)) = v;
            if (d == 0) *reinterpret_cast<float2 *>(part_ml + r * 2) = make_float2(M, L);
        } else {
            const float inv = 1.0f / L;
            v = make_float4(mul_rounded(v.x, inv), mul_rounded(v.y, inv), mul_rounded(v.z, inv), mul_rounded(v.w, inv));
            const int64_t e = ((int64_t)(tile.x + r) * H + h) * HD + d;
            if (image.hi) store_operand4(image, tile.x + r, e, v);
            else *reinterpret_cast<float4 *>(out + e) = v;
        }
    }
}

// F16 (the long passes whose rows the engine lets enter the products rounded to fp16): queries and probabilities as
// one fp16 term instead of two bf16 terms, keys and values widened from bf16 to fp16 when they are staged in LDS
// (once per workgroup, exact within the fp16 range): half the matrix-core work.  *f16_flag is set when a query, a
// key or a value lies beyond +-65504 (the pass is then repeated with two terms).
template <bool F16>
__global__ __launch_bounds__(256, 2) void k_attn_prefill(const float *__restrict__ q, int q_stride,
                                                         const bf16_t *__restrict__ pool, int Hkv,
                                                         const int32_t *__restrict__ table, int table_stride,
                                                         const int4 *__restrict__ tiles, int H, int window,
                                                         float scale_log2e, float *__restrict__ out,
                                                         int per, float *__restrict__ part_o, float *__restrict__ part_ml,
                                                         ld::OperandImage image, int *__restrict__ f16_flag) {
    struct Tiles { bf16_t ks[2][2][KVB][KLD], vt[2][2][HD][VLD]; };      // [buffer][step of the unit]
    struct Queries { bf16_t part[4][F16 ? 1 : 2][32][KLD]; };              // [wave][term]: ahead of them
    __shared__ __attribute__((aligned(16))) union Lds { Tiles tiles; Queries queries; FewLds few; } lds;
    auto &ks = lds.tiles.ks;
    auto &vt = lds.tiles.vt;
    // Work items longest first: shares in order, in each the tiles by their length, heads fastest.  Two workgroups share a
    // CU and run at each other's expense: in the tiles' own order long ones meet long ones.  Blocks b, b + 8, ... run on
    // one XCD: with the heads dealt out in eighths, the heads that read the same keys and values go through one L2.
    int tile_idx;
    const int4 tile = nth_longest(tiles, gridDim.y, window, blockIdx.y, tile_idx);      // x: first row, y: rows (<= 128), z: position of first row, w: seq slot
    const int h = H % 8 == 0 ? (blockIdx.x & 7) * (H / 8) + (blockIdx.x >> 3) : blockIdx.x;
    // this workgroup's share of the tile's KV steps: `per` of them, as many shares as the tile has (a short tile of an uneven
    // batch has fewer than the grid)
    const int n_steps = tile_steps(tile, window), split = blockIdx.z;
    if (split * per >= n_steps) return;
    const bool whole = n_steps <= per || gridDim.z == 1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int kvh = h / (H / Hkv);
    const int64_t block_stride = kv_block_elems(Hkv, HD);
    const int32_t *trow = table + (int64_t)tile.w * table_stride;

    const int wg_last_pos = tile.z + tile.y - 1;                       // last position any wave needs
    const int kv_start = tile_start(tile, window);
    const int kv_begin = kv_start + split * per * KVB;
    const int kv_end = split + 1 == gridDim.z ? wg_last_pos + 1 : min(kv_begin + per * KVB, wg_last_pos + 1);      // exclusive; the last share takes what is left
    if (tile.y <= FEW_ROWS) {
        const int64_t item = ((int64_t)tile_idx * H + h) * gridDim.z + split;
        few_rows<F16>(q, q_stride, pool, Hkv, trow, tile, h, H, kvh, window, scale_log2e, kv_begin, kv_end, lds.few, whole ? nullptr : part_o + item * 128 * HD,
                      part_ml + item * 256, out, image, f16_flag);
        return;
    }

    // this lane's query: row index inside the tile, validity, absolute position
    const int qi = wave * 32 + l32;
    const bool q_valid = qi < tile.y;
    const int q_pos = tile.z + min(qi, tile.y - 1);
    const int wave_last_pos = tile.z + min(wave * 32 + 31, tile.y - 1);
    const bool wave_active = wave * 32 < tile.y;
    // band: lowest position visible to this lane's query, to the wave's first query, to the tile's first query
    const int q_low = window > 0 ? max(q_pos - window + 1, 0) : 0;
    const int wave_low = window > 0 ? max(tile.z + wave * 32 - window + 1, 0) : 0;
    const int wave_first_pos = tile.z + wave * 32;                      // position of the wave's first query
    const int wave_low_hi = window > 0 ? max(wave_last_pos - window + 1, 0) : 0;   // lowest position its last query sees
    // first position of the lowest block any row of the tile sees: block-table entries below it may belong
    // to blocks the sequence has given up (ld_kv_trim) and are never dereferenced
    const int first_held_pos = window > 0 ? (max(tile.z - window + 1, 0) & ~15) : 0;

    // Q operand: for k-step j the lane supplies dims half*64 + j*8 .. +8 of its query (hi and lo parts; F16: one
    // fp16 term in qh).  The rows come as they lie in memory, two a load, and take the operand's form through LDS: a load of each
    // row's next 16 bytes touches 64 lines, sixteen times over
    u32x4 qh[8], ql[F16 ? 1 : 8];
    float mag = 0.f;                // F16: largest magnitude among the queries, keys and values that this lane rounded
    {
        auto &mine = lds.queries.part[wave];
        float4 raw[16];
#pragma unroll
        for (int i = 0; i < 16; i++)
            raw[i] = *reinterpret_cast<const float4 *>(q + (int64_t)(tile.x + min(wave * 32 + 2 * i + half, tile.y - 1)) * q_stride + h * HD + 4 * l32);
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const float4 v = make_float4(raw[i].x * scale_log2e, raw[i].y * scale_log2e, raw[i].z * scale_log2e, raw[i].w * scale_log2e);
            uint2 hi, lo;
            if constexpr (F16) {
                mag = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mag, fabsf(v.x)), fabsf(v.y));
                mag = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mag, fabsf(v.z)), fabsf(v.w));
                hi = make_uint2(pack2_f16(v.x, v.y), pack2_f16(v.z, v.w));
            } else {
                hi.x = split2_bf16(v.x, v.y, lo.x);
                hi.y = split2_bf16(v.z, v.w, lo.y);
                *reinterpret_cast<uint2 *>(&mine[F16 ? 0 : 1][2 * i + half][4 * l32]) = lo;
            }
            *reinterpret_cast<uint2 *>(&mine[0][2 * i + half][4 * l32]) = hi;
        }
        __builtin_amdgcn_wave_barrier();      // a lane reads what others of its wave wrote
#pragma unroll
        for (int j = 0; j < 8; j++) {
            qh[j] = *reinterpret_cast<const u32x4 *>(&mine[0][l32][half * 64 + j * 8]);
            if constexpr (!F16) ql[j] = *reinterpret_cast<const u32x4 *>(&mine[F16 ? 0 : 1][l32][half * 64 + j * 8]);
        }
    }

    f32x16 o[4];   // O^T: dims 32*nt + 8*(i/4) + 4*half + i%4 of this lane's query
#pragma unroll
    for (int nt = 0; nt < 4; nt++)
#pragma unroll
        for (int i = 0; i < 16; i++) o[nt][i] = 0.f;
    float m = -INFINITY, l = 0.f;

    // The pieces this thread copies per step: key rows (position kr, 16-byte piece kc of the row) and
    // value pieces (dimension vd, positions 8*vh .. +8 of block v of the step).
    const int kr = threadIdx.x >> 4, kc = (threadIdx.x & 15) * 8;       // + 16 rows for the second piece
    const int vd = threadIdx.x >> 1, vh = (threadIdx.x & 1) * 8;
    // lane offsets in bytes from a block's first element (a block has at most a few MB)
    const uint32_t k_off = (uint32_t)kv_k_offset(HD, kvh, kr, kc) * 2u, v_off = (uint32_t)kv_v_offset(Hkv, HD, kvh, vh, vd) * 2u;
    // Two steps of 32 positions make a unit, with one barrier each; the global loads run one unit ahead.
    u32x4 kreg[2][2], vreg[2][2];
    int entry[2][2];      // the table's entries of the unit to be loaded next, read one unit before
    auto look_up = [&](int kv0) {
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int v = 0; v < 2; v++)
                // a block past the last needed position is read again from the last needed block, one below
                // the first visible block from that block; never used
                entry[u][v] = trow[max(min(kv0 + KVB * u + 16 * v, wg_last_pos), first_held_pos) >> 4];
    };
    auto load_unit = [&] {
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int v = 0; v < 2; v++) {
                const bf16_t *blk = pool + (int64_t)entry[u][v] * block_stride;
                kreg[u][v] = load_in_block(blk, k_off);
                vreg[u][v] = load_in_block(blk, v_off);
            }
    };
    // Values of positions past the tile's last row were never written (the rest of the last block, or the
    // second block of a step that ends the walk): they may hold anything, also NaN, and a probability of zero
    // does not neutralise a NaN, so they are staged as zeros.  (Keys need nothing: their scores are replaced,
    // not multiplied.)
    auto stage_pieces = [&](int st, int kv_unit, auto whole_unit) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int v = 0; v < 2; v++) {
                const int kv0 = kv_unit + KVB * u;
                u32x4 kk = kreg[u][v], vv = vreg[u][v];
                if constexpr (F16) {
                    // a key row past the tile's last position was never written (its scores are masked): whatever it
                    // holds does not count as out of range
                    float seen = mag;
                    kk = bf16x8_to_f16x8(kk, seen);
                    if (whole_unit || kv0 + 16 * v + kr <= wg_last_pos) mag = seen;
                }
                *reinterpret_cast<u32x4 *>(&ks[st][u][16 * v + kr][kc]) = kk;
                const int p0 = kv0 + 16 * v + vh;      // position of this piece's first element
                if (!whole_unit && p0 + 7 > wg_last_pos) {
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        vv[e] = (p0 + 2 * e <= wg_last_pos ? vv[e] & 0x0000ffffu : 0u) |
                                (p0 + 2 * e + 1 <= wg_last_pos ? vv[e] & 0xffff0000u : 0u);
                }
                if constexpr (F16) vv = bf16x8_to_f16x8(vv, mag);
                *reinterpret_cast<u32x4 *>(&vt[st][u][vd][16 * v + vh]) = vv;
            }
    };
    auto stage = [&](int st, int kv_unit) {      // most units lie wholly below the last position: no look at each piece
        if (kv_unit + 2 * KVB - 1 <= wg_last_pos) stage_pieces(st, kv_unit, std::true_type{});
        else stage_pieces(st, kv_unit, std::false_type{});
    };
    // NT consecutive steps [u0, u0 + NT) of the unit at kv_unit: scores, softmax, output.  Two steps at a time (F16; the
    // two-term form has no registers left for that) give the matrix cores two independent chains of scores and the
    // softmax one maximum, one exchange and one look at the rescaling for 64 positions.
    constexpr int NT = F16 ? 2 : 1, RD = 4;      // RD: operands read ahead (3, 4 and 6 are level)
    f32x16 less_m;      // sixteen times minus the exponents' reference
#pragma unroll
    for (int i = 0; i < 16; i++) less_m[i] = 0.f;
    auto compute = [&](int kv_unit, int st, int u0) {
        const int kv0 = kv_unit + KVB * u0;
        // ---- S^T = K Q^T for 32 kv positions x 32 queries a step; tile row l32 is position kv0 + tau(l32).  The sums start
        // at -m, so that the scores come out relative to the exponents' reference
        f32x16 sc_t[NT];
        u32x4 f[RD];
        auto key = [&](int i) __attribute__((always_inline)) {      // operand i: k-step i / NT of step i % NT
            f[i % RD] = *reinterpret_cast<const u32x4 *>(&ks[st][u0 + i % NT][tau(l32)][half * 64 + i / NT * 8]);
        };
#pragma unroll
        for (int i = 0; i < RD; i++) key(i);
        __builtin_amdgcn_sched_barrier(0);
        // The matrix-core phases run at a raised wave priority: the other workgroup's wave on this SIMD then
        // fills the issue slots between the MFMAs with its softmax arithmetic instead of competing for them.
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 8 * NT; i++) {
            const int j = i / NT, n = i % NT;
            const u32x4 ka = f[i % RD];
            if constexpr (F16) {
                sc_t[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, ka), __builtin_bit_cast(f16x8, qh[j]), j ? sc_t[n] : less_m, 0, 0, 0);
            } else {
                sc_t[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka), __builtin_bit_cast(bf16x8, qh[j]), j ? sc_t[n] : less_m, 0, 0, 0);
                sc_t[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka), __builtin_bit_cast(bf16x8, ql[j]), sc_t[n], 0, 0, 0);
            }
            if (i + RD < 8 * NT) key(i + RD);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        // ---- online softmax; accumulator element i is row 8*(i/4) + 4*half + i%4 of the tile, which holds
        // position kv0 + 16*(i/8) + 8*half + i%8
        if (!(kv0 + NT * KVB - 1 <= wave_first_pos && kv0 >= wave_low_hi)) {
            // Not every position of the steps is visible to every query of the wave (at the diagonal and the band's edge): position
            // p is where p - q_low, unsigned, is at most q_pos - q_low.  Rows past the tile compute on a copy of the last row
            const uint32_t at0 = kv0 + 8 * half - q_low, most = q_pos - q_low;
#pragma unroll
            for (int n = 0; n < NT; n++)
#pragma unroll
                for (int i = 0; i < 16; i++) sc_t[n][i] = at0 + (uint32_t)(KVB * n + 16 * (i / 8) + i % 8) <= most ? sc_t[n][i] : -INFINITY;
        }
        uint32_t ph[NT][8], pl[NT][F16 ? 1 : 8];
        auto exponentials = [&]() __attribute__((always_inline)) {
            float sum = 0.f;
#pragma unroll
            for (int n = 0; n < NT; n++)
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float p0 = fast_exp2(sc_t[n][i]), p1 = fast_exp2(sc_t[n][i + 1]);      // masked: exp2(-inf) = 0
                    sum += p0 + p1;
                    if constexpr (F16) ph[n][i / 2] = pack2_f16(p0, p1);
                    else ph[n][i / 2] = split2_bf16(p0, p1, pl[n][i / 2]);
                }
            return sum;
        };
        float psum = exponentials();
        // m is the reference the exponents are taken against, not necessarily the running maximum: the maximum is looked for, and
        // m moved up to it, only where a lane's sum has grown past what fp16 surely holds (a sum of 256 over 32 positions has a term
        // of at least 2^3), or where a row has seen nothing yet.  o, l and m stay consistent, which is all the final division and
        // the split merge need.
        if (__any(!(psum <= 256.f) || !(m > -INFINITY))) {
            float mb = -INFINITY;      // relative to m
#pragma unroll
            for (int n = 0; n < NT; n++)
#pragma unroll
                for (int i = 0; i < 16; i++) mb = fmaxf(mb, sc_t[n][i]);
            // the other half of the wave holds the query's other scores
            const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(mb), __float_as_uint(mb), false, false);
            mb = fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1]));
            const bool first = !(m > -INFINITY), move = first ? mb > -INFINITY : mb > 3.f;
            const float up = move ? mb : 0.f, sc = first ? (move ? 0.f : 1.f) : fast_exp2(-up);
            if (move) m = (first ? 0.f : m) + up;
#pragma unroll
            for (int i = 0; i < 16; i++) less_m[i] = m > -INFINITY ? -m : 0.f;
#pragma unroll
            for (int n = 0; n < NT; n++)
#pragma unroll
                for (int i = 0; i < 16; i++) sc_t[n][i] -= up;
            l *= sc;
#pragma unroll
            for (int nt = 0; nt < 4; nt++)
#pragma unroll
                for (int i = 0; i < 16; i++) o[nt][i] *= sc;
            psum = exponentials();
        }
        l += psum;
        // ---- O^T += V^T P^T
        // slot e of this lane <-> position kv0 + 32*n + 16*mm + 8*half + e; operand i: step i / 8, half i / 4 % 2 of it, dimensions 32 (i % 4) + l32
        auto value = [&](int i) __attribute__((always_inline)) {
            f[i % RD] = *reinterpret_cast<const u32x4 *>(&vt[st][u0 + i / 8][i % 4 * 32 + l32][16 * (i / 4 % 2) + 8 * half]);
        };
#pragma unroll
        for (int i = 0; i < RD; i++) value(i);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 8 * NT; i++) {
            const int n = i / 8, mm = i / 4 % 2, nt = i % 4;
            const u32x4 va = f[i % RD];
            const u32x4 pbh = (u32x4){ph[n][4 * mm], ph[n][4 * mm + 1], ph[n][4 * mm + 2], ph[n][4 * mm + 3]};
            if constexpr (F16) {
                o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, va), __builtin_bit_cast(f16x8, pbh), o[nt], 0, 0, 0);
            } else {
                const u32x4 pbl = (u32x4){pl[n][4 * mm], pl[n][4 * mm + 1], pl[n][4 * mm + 2], pl[n][4 * mm + 3]};
                o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va), __builtin_bit_cast(bf16x8, pbh), o[nt], 0, 0, 0);
                o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va), __builtin_bit_cast(bf16x8, pbl), o[nt], 0, 0, 0);
            }
            if (i + RD < 8 * NT) value(i + RD);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };

    look_up(kv_begin);
    load_unit();
    // A walk that starts 16 positions before the first held block has read that block in their place.  Where it is also the
    // last, its unwritten slots pass for visible positions: neither as values nor for the range check.
    if (kv_begin < first_held_pos) kreg[0][0] = vreg[0][0] = (u32x4){0u, 0u, 0u, 0u};
    look_up(kv_begin + 2 * KVB);
    lds_barrier();      // the tiles take the queries' place
    int st = 0;
    for (int kv0 = kv_begin; kv0 < kv_end; kv0 += 2 * KVB) {
        // Stage this unit, then fetch the next.  One barrier per unit: a wave that writes buffer st for unit n has passed
        // the barrier of unit n-1, which every wave reaches only after it has finished reading buffer st for unit n-2.
        // (A unit that reaches past kv_end reads positions of the next share, which are skipped, or masked ones.)
        stage(st, kv0);
        lds_barrier();
        if (kv0 + 2 * KVB < kv_end) {
            load_unit();
            look_up(kv0 + 4 * KVB);
        }
        if (wave_active) {
#pragma unroll
            for (int u = 0; u < 2; u += NT) {
                const int at = kv0 + KVB * u;
                if (at < kv_end && at <= wave_last_pos && at + NT * KVB > wave_low) compute(kv0, st, u);   // else nothing visible to this wave
            }
        }
        st ^= 1;
    }
    // the two halves of a query's scores were summed separately
    l += __shfl_xor(l, 32, WAVE);
    if constexpr (F16) {
        if (!(mag <= 65504.f)) *f16_flag = 1;      // a magnitude that fp16 cannot hold, or a NaN
    }
    if (!whole) {      // unnormalised share
        if (q_valid) {
            const int64_t item = ((int64_t)tile_idx * H + h) * gridDim.z + split;
            float *op = part_o + item * 128 * HD;
#pragma unroll
            for (int nt = 0; nt < 4; nt++)
#pragma unroll
                for (int a = 0; a < 4; a++)
                    *reinterpret_cast<float4 *>(op + part_place(qi, 4 * nt + a, half)) =
                        make_float4(o[nt][4 * a], o[nt][4 * a + 1], o[nt][4 * a + 2], o[nt][4 * a + 3]);
            if (half == 0) *reinterpret_cast<float2 *>(part_ml + (item * 128 + qi) * 2) = make_float2(m, l);
        }
        return;
    }
    if (q_valid) {
        const float inv = 1.0f / l;
        const int64_t at = (int64_t)(tile.x + qi) * (H * HD) + h * HD;
#pragma unroll
        for (int nt = 0; nt < 4; nt++)
#pragma unroll
            for (int a = 0; a < 4; a++) {
                // products rounded to float: what a store would hold, also where they go straight into the split
                const float4 v = make_float4(mul_rounded(o[nt][4 * a], inv), mul_rounded(o[nt][4 * a + 1], inv),
                                             mul_rounded(o[nt][4 * a + 2], inv), mul_rounded(o[nt][4 * a + 3], inv));
                const int64_t e = at + nt * 32 + 8 * a + 4 * half;
                if (image.hi) {      // the output projection's operand instead of floats
                    store_operand4(image, tile.x + qi, e, v);
                } else {
                    *reinterpret_cast<float4 *>(out + e) = v;
                }
            }
    }
}

// Adds the shares of a tile's rows in order: half a wave per row (four dimensions a lane), eight rows of one head at a
// time.  A share that saw no visible position of the row has m = -inf and weight 0; some share always saw one.  Tiles
// that one workgroup walked whole are finished already.  What bounds it is the chain of its loads and, with many shares, their bytes:
// 8 full tiles of 32 heads 17.3 -> 16.0 us with four shares asked for at once, two of them 7.6 -> 7.0.
__global__ __launch_bounds__(256) void k_attn_prefill_merge(const int4 *__restrict__ tiles, int H, int window, int per, int ns,
                                                            const float *__restrict__ part_o,
                                                            const float *__restrict__ part_ml,
                                                            float *__restrict__ out, ld::OperandImage image) {
    const int4 tile = tiles[blockIdx.y];
    const int n = min((tile_steps(tile, window) + per - 1) / per, ns);
    const int r = blockIdx.z * 8 + (threadIdx.x >> 5), h = blockIdx.x, sub = threadIdx.x & 31;
    if (n <= 1 || r >= tile.y) return;
    const int64_t base = ((int64_t)blockIdx.y * H + h) * ns;
    const float2 ml = sub < n ? *reinterpret_cast<const float2 *>(part_ml + ((base + sub) * 128 + r) * 2) : make_float2(-INFINITY, 0.f);
    const float *po = part_o + base * 128 * HD + part_place(r, sub >> 1, sub & 1);
    // four shares at a time, the first of them asked for with the statistics: what is past the last one is read again and not used
    constexpr int AHEAD = 4;
    float4 v[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; u++) v[u] = *reinterpret_cast<const float4 *>(po + (int64_t)min(u, n - 1) * 128 * HD);
    float M = ml.x;
#pragma unroll
    for (int off = 1; off < MAX_SPLITS; off <<= 1) M = fmaxf(M, __shfl_xor(M, off, WAVE));
    const float weight = fast_exp2(ml.x - M);
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    float L = 0.f;
    for (int z0 = 0; z0 < n; z0 += AHEAD) {
        if (z0)
#pragma unroll
            for (int u = 0; u < AHEAD; u++) v[u] = *reinterpret_cast<const float4 *>(po + (int64_t)min(z0 + u, n - 1) * 128 * HD);
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            if (z0 + u >= n) break;
            const float a = __shfl(weight, z0 + u, 32);
            o.x += a * v[u].x; o.y += a * v[u].y; o.z += a * v[u].z; o.w += a * v[u].w;
            L += a * __shfl(ml.y, z0 + u, 32);
        }
    }
    const float4 r4 = make_float4(o.x / L, o.y / L, o.z / L, o.w / L);
    const int64_t e = ((int64_t)(tile.x + r) * H + h) * HD + sub * 4;
    if (image.hi) store_operand4(image, tile.x + r, e, r4);
    else *reinterpret_cast<float4 *>(out + e) = r4;
}

}  // namespace

namespace ld {

bool prefill_attention_supported(int dtype_is_bf16, int hd) { return dtype_is_bf16 && hd == HD; }

// Shares of the KV walk for the longest tile, and the steps of a share (shorter tiles have fewer shares).  Modelled in
// steps of a workgroup: a share costs its steps and ten more (launch, queries, first loads, result), a round of up to 256
// workgroups that, of up to 512 (two per CU) 1.15 times as much, and the merge two steps and 1 / 60 for each partial result of
// 64 KB.  At least 4 steps a share, and only as many shares as the scratch holds.  Fitted to every number of shares for 243 sets of
// tiles (4 .. 40 heads, 1 .. 16 tiles, walks of 4 .. 250 steps) and looked at again for 135 with the kernels as they are: the choice is
// 2.5 % (two terms 3.2 %) slower than the best in the mean, 29 % at worst, where tiles differ most in length.  A model that made the merge cheaper chose two shares for narrow bands over short
// segments: 22 -> 29 us for eight 64-row tiles of 32 heads with a band of 256, 22 so.
static int prefill_shares(int n_tiles, int H, int max_pos, int window, size_t scratch_bytes, int *per) {
    const int span = window > 0 ? std::min<int64_t>(max_pos + 1, (int64_t)window + 128 + KVB) : max_pos + 1;   // positions a tile walks
    const int steps = (span + KVB - 1) / KVB;
    const int64_t items = (int64_t)n_tiles * H;
    const size_t per_share = (size_t)items * 128 * (HD + 2) * sizeof(float);
    int best = 1;
    double best_t = 1e30;
    for (int n = 1; n <= MAX_SPLITS; n++) {
        const int p = ((steps + n - 1) / n + 1) & ~1;      // whole units of two steps
        if (n > 1 && (p < 4 || per_share * n > scratch_bytes)) break;
        const int64_t full = items * n / 512, rest = items * n % 512;
        const double rounds = full * 1.15 + (rest == 0 ? 0.0 : rest <= 256 ? 1.0 : 1.15);
        const double t = rounds * (p + 10) + (n > 1 ? 2.0 + items * n / 60.0 : 0.0);
        if (t < best_t) { best_t = t; best = n; }
    }
    *per = ((steps + best - 1) / best + 1) & ~1;
    return best;
}

size_t prefill_attention_scratch_bytes() { return (size_t)1536 * 128 * (HD + 2) * sizeof(float); }      // shares of 128 rows

void launch_prefill_attention(const float *q, int q_stride, const uint16_t *pool, int Hkv, const int32_t *table,
                              int table_stride, const int32_t *tiles, int n_tiles, int H, int window, int max_pos,
                              float *out, void *scratch, size_t scratch_bytes, hipStream_t s,
                              const OperandImage &image, int *f16_flag) {
    const float sl2 = 1.4426950408889634f / sqrtf((float)HD);
    // tiles are the second dimension of the grid, which ends at 65535: more of them go in several launches, one after the
    // other through the same scratch
    constexpr int MAX_TILES = 65535;
    for (int first = 0; first < n_tiles; first += MAX_TILES) {
        const int n = std::min(n_tiles - first, MAX_TILES);
        const int4 *t = (const int4 *)tiles + first;
        int per = 0;
        const int ns = prefill_shares(n, H, max_pos, window, scratch ? scratch_bytes : 0, &per);
        float *part_o = (float *)scratch;
        float *part_ml = part_o ? part_o + (size_t)n * 128 * H * ns * HD : nullptr;
        if (f16_flag)
            LD_LAUNCH(k_attn_prefill<true>, dim3(H, n, ns), dim3(256), 0, s, q, q_stride, pool, Hkv, table, table_stride, t, H, window,
                      sl2, out, per, part_o, part_ml, image, f16_flag);
        else
            LD_LAUNCH(k_attn_prefill<false>, dim3(H, n, ns), dim3(256), 0, s, q, q_stride, pool, Hkv, table, table_stride, t, H, window,
                      sl2, out, per, part_o, part_ml, image, f16_flag);
        if (ns > 1) LD_LAUNCH(k_attn_prefill_merge, dim3(H, n, 16), dim3(256), 0, s, t, H, window, per, ns, part_o, part_ml, out, image);
    }
}

}  // namespace ld
