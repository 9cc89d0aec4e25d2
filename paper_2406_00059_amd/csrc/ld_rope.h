// Rows of the q-k-v projection: rotary embedding and cache append, with the sum of the product's K slabs where it has them.
#pragma once
#include "ld_device.h"
#include "ld_gemv.h"
#include "ld_internal.h"

namespace ldd {

typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));      // four floats at any float's address

// Few rows, where only the latency of one row counts: one wave per row and head, a pair (i, i + HD / 2) a lane, nothing passed
// between lanes (one row 2.1 us, k_rope_rows 2.5).  Arguments and results as of k_rope_rows.
template <typename KVT>
__global__ __launch_bounds__(64) void k_rope_row(const float *__restrict__ partial, int T, int ks, float *__restrict__ y, ld::RopeKvArgs rk,
                                                 KVT *__restrict__ pool, int row0, bool store_kv) {
    const int t = blockIdx.y, hh = blockIdx.x, i = threadIdx.x, hd = rk.hd, half = hd / 2;
    if (i >= half) return;
    const int N = (rk.H + 2 * rk.Hkv) * hd;
    const float *prow = partial + (int64_t)t * N;
    float *row = y + (int64_t)t * N;
    auto value = [&](int col) { return ks ? slab_sum(prow + col, (int64_t)T * N, ks, 0.f) : row[col]; };
    const float2 c = reinterpret_cast<const float2 *>(rk.cos_sin)[(int64_t)(row0 + t) * half + i];
    const int c0 = hh * hd, j = hh - rk.H, vc = (rk.H + rk.Hkv + j) * hd;      // q heads, then k heads
    if (j < 0) {
        const float2 r = rope_rotate(value(c0 + i), value(c0 + i + half), c);
        row[c0 + i] = r.x;
        row[c0 + i + half] = r.y;
        return;
    }
    const int p = rk.pos[row0 + t], slot = p & 15;
    const int64_t phys = rk.table[(int64_t)rk.seq_slot[row0 + t] * rk.table_stride + (p >> 4)];
    KVT *blk = pool + phys * kv_block_elems(rk.Hkv, hd);
    const float a = value(c0 + i), b = value(c0 + i + half), va = value(vc + i), vb = value(vc + i + half);
    const float2 r = rope_rotate(a, b, c);
    store_elem(blk + kv_k_offset(hd, j, slot, i), r.x);
    store_elem(blk + kv_k_offset(hd, j, slot, i + half), r.y);
    store_elem(blk + kv_v_offset(rk.Hkv, hd, j, slot, i), va);
    store_elem(blk + kv_v_offset(rk.Hkv, hd, j, slot, i + half), vb);
    if (store_kv) {
        row[c0 + i] = a;
        row[c0 + i + half] = b;
        row[vc + i] = va;
        row[vc + i + half] = vb;
    }
}

// One workgroup: R consecutive rows of one head, HD / 8 threads a row, four pairs (i, i + HD / 2) a thread.  q heads are rotated in
// y; rotated k heads and v heads go into the paged pool (and, with store_kv, as they are into y).  ks > 0: the rows are the sums
// of ks slabs in `partial`, added in order; 0: they are in y.  Row t of the launch is row row0 + t of the pass.
// What bounds it is the rows' traffic, if the values are written well: a position's values lie 32 bytes apart (the pool keeps the
// 16 positions of a dimension together), so a kernel that takes one row at a time writes two bytes of every sector, sixteen
// times over.  Here they are turned around in LDS and neighbouring lanes write neighbouring positions.  Sixteen rows write the most of
// a sector at once; up to 128 rows, four to eight that fill one wave, which wait for nobody else.  1028 rows of 32 q, 32 k and 32 v
// heads 18.5 us one row at a time, 15.3 sixteen; 128 rows 4.9, 3.9, 3.5 four; 32 rows of as many sequences 3.4, 3.7, 3.3; but 256
// rows with the sum of two slabs, in a call of ldk_qkv_rope, 55.5 sixteen, 56.2 four.
template <int HD, typename KVT, int R>
__global__ __launch_bounds__(R * HD / 8) void k_rope_rows(const float *__restrict__ partial, int T, int ks, float *__restrict__ y, ld::RopeKvArgs rk,
                                                          KVT *__restrict__ pool, int row0, bool store_kv) {
    constexpr int HALF = HD / 2, TPR = HD / 8;
    __shared__ float vt[R][HD + 1];
    __shared__ int64_t at[R];      // first element of the row's block, -1 past the last row
    __shared__ int slots[R];
    const int r = threadIdx.x / TPR, i = threadIdx.x % TPR * 4, t = blockIdx.y * R + r, hh = blockIdx.x;
    const bool live = t < T;
    const int N = (rk.H + 2 * rk.Hkv) * HD;
    const float *prow = partial + (int64_t)t * N;
    float *row = y + (int64_t)t * N;
    auto value = [&](int col) -> float4_any {
        if (!ks) return *reinterpret_cast<const float4_any *>(row + col);
        float4_any acc = {0.f, 0.f, 0.f, 0.f};      // slab_sum's order and its grouping of the loads
        const int64_t stride = (int64_t)T * N;
        int z = 0;
        for (; z + 4 <= ks; z += 4) {
            float4_any v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) v[u] = *reinterpret_cast<const float4_any *>(prow + col + (z + u) * stride);
#pragma unroll
            for (int u = 0; u < 4; u++) acc += v[u];
        }
        for (; z < ks; z++) acc += *reinterpret_cast<const float4_any *>(prow + col + z * stride);
        return acc;
    };
    // The position is asked for first: behind the rotation, the chain from it over the block table to the block was one memory round
    // trip more.  So are the values, but not with sixteen rows (300 rows of 32 + 32 heads 6.3 -> 6.6 us: fewer workgroups a CU)
    const bool keep = hh >= rk.H;      // a k head and its v head
    const int c0 = hh * HD, j = hh - rk.H, vc = (rk.H + rk.Hkv + j) * HD;      // q heads, then k heads
    float4_any a, b, va, vb, ra, rb;
    int p = 0;
    int64_t phys = 0;
    if (live) {
        int seq = 0;
        if (keep) {
            p = rk.pos[row0 + t];
            seq = rk.seq_slot[row0 + t];
        }
        const float *cs = reinterpret_cast<const float *>(rk.cos_sin) + ((int64_t)(row0 + t) * HALF + i) * 2;
        const float4_any c01 = *reinterpret_cast<const float4_any *>(cs), c23 = *reinterpret_cast<const float4_any *>(cs + 4);
        a = value(c0 + i);
        b = value(c0 + i + HALF);
        if (keep) {
            if (R < 16) {
                va = value(vc + i);
                vb = value(vc + i + HALF);
            }
            phys = rk.table[(int64_t)seq * rk.table_stride + (p >> 4)];
        }
        const float2 c[4] = {make_float2(c01[0], c01[1]), make_float2(c01[2], c01[3]), make_float2(c23[0], c23[1]), make_float2(c23[2], c23[3])};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const float2 q = rope_rotate(a[e], b[e], c[e]);
            ra[e] = q.x;
            rb[e] = q.y;
        }
    }
    if (!keep) {
        if (live) {
            *reinterpret_cast<float4_any *>(row + c0 + i) = ra;
            *reinterpret_cast<float4_any *>(row + c0 + i + HALF) = rb;
        }
        return;
    }
    if (live) {
        if (R >= 16) {
            va = value(vc + i);
            vb = value(vc + i + HALF);
        }
        const int64_t first = phys * kv_block_elems(rk.Hkv, HD);
        const int slot = p & 15;
        KVT *k = pool + first + kv_k_offset(HD, j, slot, i);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            store_elem(k + e, ra[e]);
            store_elem(k + HALF + e, rb[e]);
            vt[r][i + e] = va[e];
            vt[r][i + HALF + e] = vb[e];
        }
        if (store_kv) {
            *reinterpret_cast<float4_any *>(row + c0 + i) = a;
            *reinterpret_cast<float4_any *>(row + c0 + i + HALF) = b;
            *reinterpret_cast<float4_any *>(row + vc + i) = va;
            *reinterpret_cast<float4_any *>(row + vc + i + HALF) = vb;
        }
        if (i == 0) { at[r] = first; slots[r] = slot; }
    } else if (i == 0) {
        at[r] = -1;
    }
    __syncthreads();
    const int vr = threadIdx.x % R;
    const int64_t first = at[vr];
    if (first < 0) return;
    for (int d = threadIdx.x / R; d < HD; d += TPR) store_elem(pool + first + kv_v_offset(rk.Hkv, HD, j, slots[vr], d), vt[vr][d]);
}

// The line between the two: they cross at 24 rows of 32 + 32 heads, 20 of 40 + 40, 70 of 32 + 8 and 110 of 4 + 4.
inline bool rope_few_rows(int T, int H, int Hkv) { return T <= 96 && (int64_t)T * (H + Hkv) <= 1536; }
template <typename KVT>
inline void launch_rope(const float *partial, int T, int ks, float *y, const ld::RopeKvArgs &rk, KVT *pool, int row0, hipStream_t s) {
    const bool store_kv = rk.store_kv && ks > 0;
    const int heads = rk.H + rk.Hkv;
#define LD_ROPE(KERNEL_, ROWS_, BLOCK_) LD_LAUNCH(KERNEL_, dim3(heads, (T + ROWS_ - 1) / ROWS_), dim3(BLOCK_), 0, s, partial, T, ks, y, rk, pool, row0, store_kv)
    if (rope_few_rows(T, rk.H, rk.Hkv)) LD_ROPE(k_rope_row<KVT>, 1, 64);
    else if (rk.hd == 128 && T <= 128) LD_ROPE((k_rope_rows<128, KVT, 4>), 4, 64);
    else if (rk.hd == 128) LD_ROPE((k_rope_rows<128, KVT, 16>), 16, 256);
    else if (T <= 128) LD_ROPE((k_rope_rows<64, KVT, 8>), 8, 64);
    else LD_ROPE((k_rope_rows<64, KVT, 16>), 16, 128);
#undef LD_ROPE
}

}  // namespace ldd
