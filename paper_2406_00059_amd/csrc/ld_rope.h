// Rows of the q-k-v projection: rotary embedding and cache append, with the sum of the product's K slabs where it has them.
#pragma once
#include "ld_device.h"
#include "ld_gemv.h"

namespace ldd {

typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));      // four floats at any float's address

// One workgroup: 16 consecutive rows of one head, HD / 8 threads a row, four pairs (i, i + HD / 2) a thread.  q heads are rotated in
// y; rotated k heads and v heads go into the paged pool (and, with store_kv, as they are into y).  ks > 0: the rows are the sums
// of ks slabs in `partial`, added in order; 0: they are in y.  Row t of the launch is row row0 + t of the pass.
// What bounds it is the rows' traffic, if the values are written well: a position's values lie 32 bytes apart (the pool keeps the
// 16 positions of a dimension together), so a kernel that takes one row at a time writes two bytes of every sector, sixteen
// times over.  Here they are turned around in LDS and neighbouring lanes write neighbouring positions.  1028 rows of 32 q, 32 k and 32 v
// heads 24.7 -> 19.3 us (one wave per row and head before); 256 rows, with the sum of two slabs, 10.6 + 8.1 -> 9.5.
template <int HD, typename KVT>
__global__ __launch_bounds__(2 * HD) void k_rope_rows(const float *__restrict__ partial, int T, int ks, float *__restrict__ y, ld::RopeKvArgs rk,
                                                      KVT *__restrict__ pool, int row0, bool store_kv) {
    constexpr int HALF = HD / 2, TPR = HD / 8;
    __shared__ float vt[16][HD + 1];
    __shared__ int64_t at[16];      // first element of the row's block, -1 past the last row
    __shared__ int slots[16];
    const int r = threadIdx.x / TPR, i = threadIdx.x % TPR * 4, t = blockIdx.y * 16 + r, hh = blockIdx.x;
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
    float4_any a, b, ra, rb;
    const int c0 = hh * HD;      // q heads, then k heads
    if (live) {
        const float *cs = reinterpret_cast<const float *>(rk.cos_sin) + ((int64_t)(row0 + t) * HALF + i) * 2;
        const float4_any c01 = *reinterpret_cast<const float4_any *>(cs), c23 = *reinterpret_cast<const float4_any *>(cs + 4);
        a = value(c0 + i);
        b = value(c0 + i + HALF);
        const float2 c[4] = {make_float2(c01[0], c01[1]), make_float2(c01[2], c01[3]), make_float2(c23[0], c23[1]), make_float2(c23[2], c23[3])};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const float2 p = rope_rotate(a[e], b[e], c[e]);
            ra[e] = p.x;
            rb[e] = p.y;
        }
    }
    if (hh < rk.H) {
        if (live) {
            *reinterpret_cast<float4_any *>(row + c0 + i) = ra;
            *reinterpret_cast<float4_any *>(row + c0 + i + HALF) = rb;
        }
        return;
    }
    const int j = hh - rk.H, vc = (rk.H + rk.Hkv + j) * HD;
    if (live) {
        const int p = rk.pos[row0 + t];
        const int64_t phys = rk.table[(int64_t)rk.seq_slot[row0 + t] * rk.table_stride + (p >> 4)];
        const float4_any va = value(vc + i), vb = value(vc + i + HALF);
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
    const int vr = threadIdx.x % 16;
    const int64_t first = at[vr];
    if (first < 0) return;
    for (int d = threadIdx.x / 16; d < HD; d += 2 * HD / 16) store_elem(pool + first + kv_v_offset(rk.Hkv, HD, j, slots[vr], d), vt[vr][d]);
}

}  // namespace ldd
