"""Per-kernel parity on the GPU: every kernel-level entry point against the oracle's step functions
on the same seeded inputs, element by element, at sizes spanning several tiles and ragged tails."""
import ctypes as C
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2406_00059_amd as ld
from paper_2406_00059_amd import binding
from workloads import gen
from helpers import MOVING_CTX, MOVING_HEADS, attention_and_bound, device_pool, logical_pool, moving_maximum_inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


_silu = np.vectorize(oracle.silu, otypes=[np.float64])      # the oracle's activation, element by element


def _mat(seed, stream, n, k, dtype):
    w = gen.normal(seed, stream, (n, k), std=0.05)
    return w.bfloat16() if dtype == "bf16" else w


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 7, 8, 19])
def test_linear_store_add_and_fused_norm(dtype, T):
    N, K = 301, 688           # ragged row count, K not a multiple of 512
    W = _mat(1, 1, N, K, dtype); x = gen.normal(1, 2, (T, K)); g = gen.normal(1, 3, (K,), std=0.1, mean=1.0)
    y0 = gen.normal(1, 4, (T, N))
    Wh = oracle.to_host_matrix(W)
    Wd, xd, gd = W.to(DEV), x.to(DEV), g.to(DEV)
    y = torch.empty(T, N, device=DEV)
    ld.ldk_linear(Wd, xd, y, ld.LDK_STORE)
    ref = np.stack([oracle.matvec(Wh, x[t].numpy()) for t in range(T)])
    np.testing.assert_allclose(y.cpu().numpy(), ref, rtol=0, atol=2e-6 * np.abs(ref).max())
    y = y0.to(DEV).clone()
    ld.ldk_linear(Wd, xd, y, ld.LDK_ADD, g=gd, eps=1e-5)
    refn = np.stack([oracle.matvec(Wh, oracle.rmsnorm(x[t].numpy(), g.numpy(), 1e-5)) for t in range(T)])
    np.testing.assert_allclose(y.cpu().numpy(), y0.numpy() + refn, rtol=0, atol=3e-6 * np.abs(refn).max())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5])
def test_linear_swiglu(dtype, T):
    F, K = 173, 256
    W = _mat(2, 1, 2 * F, K, dtype); x = gen.normal(2, 2, (T, K)); g = gen.normal(2, 3, (K,), std=0.1, mean=1.0)
    Wh = oracle.to_host_matrix(W)
    y = torch.empty(T, F, device=DEV)
    ld.ldk_linear(W.to(DEV), x.to(DEV), y, ld.LDK_SWIGLU, g=g.to(DEV), eps=1e-5)
    for t in range(T):
        gu = oracle.matvec(Wh, oracle.rmsnorm(x[t].numpy(), g.numpy(), 1e-5))
        ref = np.array([oracle.silu(gu[i]) * gu[F + i] for i in range(F)])
        np.testing.assert_allclose(y[t].cpu().numpy(), ref, rtol=0, atol=3e-6 * np.abs(ref).max())


def test_linear_full_7b_shapes_on_sampled_outputs():
    """The launch shapes of the 7B decode step (T = 1), checked on sampled output rows."""
    for N, K, epi in [(12288, 4096, ld.LDK_STORE), (4096, 11008, ld.LDK_ADD), (11008, 4096, ld.LDK_SWIGLU),
                      (32000, 4096, ld.LDK_STORE)]:
        rows = N * (2 if epi == ld.LDK_SWIGLU else 1)
        W = gen.normal(3, N, (rows, K), std=0.02, device=DEV).bfloat16()
        x = gen.normal(3, 7, (1, K), device=DEV)
        y = torch.zeros(1, N, device=DEV)
        ld.ldk_linear(W, x, y, epi)
        idx = gen.randint(3, 9, 0, N - 1, 48).tolist() + [0, N - 1]
        xh = x[0].cpu().numpy()
        for n in idx:
            a = oracle.matvec(oracle.to_host_matrix(W[n:n + 1]), xh)[0]
            if epi == ld.LDK_SWIGLU:
                a = oracle.silu(a) * oracle.matvec(oracle.to_host_matrix(W[N + n:N + n + 1]), xh)[0]
            assert abs(y[0, n].item() - a) <= 1e-5 * max(1.0, abs(a)) + 2e-6 * math.sqrt(K) * 0.02


@pytest.mark.parametrize("off", [0, 1], ids=["aligned", "4-bytes-off"])
@pytest.mark.parametrize("d", [1, 3, 4, 255, 260, 1024, 1028, 4096, 4100, 8188, 8192, 8196])
def test_rmsnorm_lengths_and_alignments(d, off):
    """Rows that are read four floats at a time and kept (a multiple of four, up to 8192, 16-byte aligned) and all others, gathered and in
    order, against float64.  Bound: at most 33 + 6 + 3 roundings of 2^-24 in the sum of squares, which count half, and a few behind it."""
    x = gen.normal(91, 1, (7 * d + off,), device=DEV)[off:].view(7, d); g = 1 + 0.1 * gen.normal(91, 2, (d,), device=DEV)
    out = torch.full((5 * d + off,), float("nan"), device=DEV)[off:].view(5, d)
    for idx in (None, [6, 0, 3, 3, 1]):
        ld.ldk_rmsnorm(x, g, out, 1e-5, row_idx=None if idx is None else torch.tensor(idx, dtype=torch.int32, device=DEV))
        v = x[:5].double() if idx is None else x[idx].double()
        ref = v / torch.sqrt((v * v).mean(1, keepdim=True) + 1e-5) * g.double()
        assert ((out.double() - ref).abs() <= 32 * 2.0 ** -24 * ref.abs()).all()


def test_embed_and_rmsnorm_gather():
    E = _mat(4, 1, 50, 256, "bf16"); tok = torch.tensor([3, 49, 0, 3], dtype=torch.int32)
    x = torch.empty(4, 256, device=DEV)
    ld.ldk_embed(E.to(DEV), tok.to(DEV), x)
    assert torch.equal(x.cpu(), E.float()[tok.long()])
    g = gen.normal(4, 2, (256,), std=0.1, mean=1.0)
    idx = torch.tensor([2, 0], dtype=torch.int32)
    out = torch.empty(2, 256, device=DEV)
    ld.ldk_rmsnorm(x, g.to(DEV), out, 1e-5, row_idx=idx.to(DEV))
    for r, src in enumerate([2, 0]):
        ref = oracle.rmsnorm(x[src].cpu().numpy(), g.numpy(), 1e-5)
        np.testing.assert_allclose(out[r].cpu().numpy(), ref, rtol=2e-6, atol=1e-7)


@pytest.mark.parametrize("dtype,hd", [("f32", 64), ("bf16", 128)])
def test_rope_and_cache_append_values_and_block_indexing(dtype, hd):
    H, Hkv, T, nblk = 4, 2, 5, 9
    nqkv = (H + 2 * Hkv) * hd
    qkv = gen.normal(5, 1, (T, nqkv))
    pos = torch.tensor([0, 15, 16, 17, 4000], dtype=torch.int32)
    slot = torch.tensor([0, 1, 1, 1, 2], dtype=torch.int32)
    table = torch.full((3, 256), -1, dtype=torch.int32)
    table[0, 0] = 4; table[1, 0] = 7; table[1, 1] = 2; table[2, 4000 // 16] = 5
    pdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    pool = torch.full((nblk, 2, Hkv, 16, hd), 512.0, dtype=pdt, device=DEV)
    cs = torch.empty(T, hd // 2, 2, device=DEV)
    q = qkv.to(DEV).clone()
    ld.ldk_rope_table(pos.to(DEV), hd, 10000.0, cs)
    ld.ldk_rope_kv_write(q, cs, pos.to(DEV), slot.to(DEV), table.to(DEV), pool, H, Hkv, hd)
    q, pool_h = q.cpu().numpy(), logical_pool(pool).float().cpu().numpy().astype(np.float64)
    touched = np.zeros(pool_h.shape[:4], bool)
    for t in range(T):
        p = int(pos[t]); blk = int(table[slot[t], p // 16]); s = p % 16
        for h in range(H):
            ref = oracle.rope_head(qkv[t, h * hd:(h + 1) * hd].numpy(), p)
            np.testing.assert_allclose(q[t, h * hd:(h + 1) * hd], ref, rtol=0, atol=4e-7 * np.abs(ref).max() + 1e-7)
        for j in range(Hkv):
            k = oracle.rope_head(qkv[t, (H + j) * hd:(H + j + 1) * hd].numpy(), p)
            v = qkv[t, (H + Hkv + j) * hd:(H + Hkv + j + 1) * hd].double().numpy()
            if dtype == "bf16":
                np.testing.assert_array_equal(pool_h[blk, 1, j, s], oracle.round_bf16(v))      # v: exact rounding
                # k is rotated in fp32 before rounding: equal to the oracle's rounding up to one bf16 step
                kr = oracle.round_bf16(k)
                assert np.all(np.abs(pool_h[blk, 0, j, s] - kr) <= np.abs(kr) * 2.0 ** -7 + 1e-30)
                assert np.mean(pool_h[blk, 0, j, s] == kr) > 0.9
            else:
                np.testing.assert_array_equal(pool_h[blk, 1, j, s], v)
                np.testing.assert_allclose(pool_h[blk, 0, j, s], k, rtol=0, atol=4e-7 * np.abs(k).max())
            touched[blk, :, j, s] = True
    assert np.all(pool_h[~touched] == 512.0), "a write landed outside the (block, slot) the table names"
    assert touched.sum() == T * 2 * Hkv


@pytest.mark.parametrize("dtype,hd", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("H,Hkv,T", [(3, 1, 95), (3, 1, 96), (3, 1, 97), (2, 2, 104), (20, 4, 64), (20, 4, 65), (32, 32, 24), (32, 32, 25), (16, 16, 67), (16, 4, 128), (16, 4, 129)])
def test_rope_rows_together_equal_rows_alone(dtype, hd, H, Hkv, T):
    """Many rows of one call (one wave a row up to 96 rows and 1536 rows times heads, four or eight rows a wave up to 128, sixteen a workgroup beyond) against a call
    for each row: the same bits in the rotated rows, and in the pool, which holds nothing else.  Rows of two sequences that start
    inside a block, and single rows of others."""
    N, n0 = (H + 2 * Hkv) * hd, T - T // 3
    qkv = gen.normal(71, hd, (T, N), device=DEV)
    pos = torch.tensor([13 + i for i in range(n0 // 2)] + [47 + i for i in range(n0 - n0 // 2)] + [(37 * i) % 200 for i in range(T - n0)], dtype=torch.int32, device=DEV)
    slot = torch.tensor([0] * (n0 // 2) + [1] * (n0 - n0 // 2) + [2 + i for i in range(T - n0)], dtype=torch.int32, device=DEV)
    n_seq, per = 2 + T - n0, 13
    table = torch.randperm(n_seq * per, generator=torch.Generator().manual_seed(T)).to(torch.int32).view(n_seq, per).to(DEV)
    cs = torch.empty(T, hd, device=DEV)
    ld.ldk_rope_table(pos, hd, 10000.0, cs)
    pools = [torch.full((n_seq * per, 2, Hkv, 16, hd), 3.0, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV) for _ in range(2)]
    a, b = qkv.clone(), qkv.clone()
    assert int(pos.max()) < per * 16
    ld.ldk_rope_kv_write(a, cs, pos, slot, table, pools[0], H, Hkv, hd)
    for t in range(T):
        ld.ldk_rope_kv_write(b[t:t + 1], cs[t:t + 1], pos[t:t + 1], slot[t:t + 1], table, pools[1], H, Hkv, hd)
    assert torch.equal(a, b) and torch.equal(*pools)
    assert not torch.equal(a[:, :H * hd], qkv[:, :H * hd]) and torch.equal(a[:, H * hd:], qkv[:, H * hd:])
    assert int((pools[0] != 3.0).any(-1).sum()) > 0


def _attention_case(seed, lens, H, Hkv, hd, dtype, spare=5):
    B = len(lens)
    nb = [(n + 15) // 16 for n in lens]
    total = sum(nb) + spare
    perm = gen.permutation(seed, 1, total).tolist()
    table = torch.full((B, max(nb)), 0, dtype=torch.int32)
    it = iter(perm)
    for b in range(B):
        for j in range(nb[b]):
            table[b, j] = next(it)
    pdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    pool = gen.normal(seed, 2, (total, 2, Hkv, 16, hd), device=DEV).to(pdt)
    # slots past a sequence's last position were never written: they may hold anything, so they hold NaN here
    # (a masked probability of zero times NaN would still poison the output), and so do the blocks no table
    # entry names
    used = torch.zeros(total, dtype=torch.bool)
    for b in range(B):
        used[table[b, :nb[b]].long()] = True
        if lens[b] % 16:
            pool[table[b, nb[b] - 1], :, :, lens[b] % 16:, :] = float("nan")
    pool[(~used).to(DEV)] = float("nan")
    q = gen.normal(seed, 3, (B, H, hd), device=DEV)
    return table, pool, q


def _attn_tol(dtype, hd, H, Hkv):
    """Relative tolerance of decode attention: the scalar kernel computes in float32 (2e-6); grouped heads
    on a bf16 pool with head_dim 128 run on the matrix cores with q and the probabilities split into two
    bf16 terms, which leaves 2^-17 = 7.6e-6 per operand element (3e-5 with the accumulation)."""
    return 3e-5 if (dtype == "bf16" and hd == 128 and 2 <= H // Hkv <= 16) else 2e-6


def _run_attention(table, pool, q, lens, H, Hkv, hd, window=0):
    B = len(lens)
    ctx = torch.tensor(lens, dtype=torch.int32, device=DEV)
    slot = torch.arange(B, dtype=torch.int32, device=DEV)
    out = torch.empty(B, H, hd, device=DEV)
    scratch = torch.empty(ld.ldk_attention_scratch_bytes(B, H, Hkv, hd, max(lens), window), dtype=torch.uint8,
                          device=DEV)
    ld.ldk_paged_attention(q, H * hd, device_pool(pool), table.to(DEV), slot, ctx, max(lens), H, Hkv, hd, out,
                           scratch, window=window)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _oracle_attention(table, pool, q, lens, Hkv, hd, rows=None, window=0):
    ph = oracle.to_host_matrix(pool.reshape(pool.shape[0], -1))
    kp = ph.reshape(-1)
    vp = kp[Hkv * 16 * hd:]                      # V half of each block starts Hkv*16*hd elements later
    strides = (2 * Hkv * 16 * hd, 16 * hd, hd)
    qh = q.cpu().numpy()
    if rows is None:
        return oracle.paged_attention(qh, kp, vp, strides, table.numpy(), lens, Hkv, window=window)
    sel = np.array(rows)
    return oracle.paged_attention(qh[sel], kp, vp, strides, table.numpy()[sel], [lens[r] for r in rows], Hkv,
                                  window=window)


@pytest.mark.parametrize("dtype,hd,H,Hkv", [("bf16", 128, 4, 4), ("f32", 64, 4, 4), ("bf16", 128, 8, 2), ("f32", 128, 2, 1),
                                            ("bf16", 128, 16, 2), ("bf16", 64, 6, 2), ("bf16", 128, 32, 8)])
def test_paged_attention_edge_lengths(dtype, hd, H, Hkv):
    lens = [1, 2, 15, 16, 17, 63, 255, 256, 257, 300, 1025]
    table, pool, q = _attention_case(21, lens, H, Hkv, hd, dtype)
    got = _run_attention(table, pool, q, lens, H, Hkv, hd)
    ref = _oracle_attention(table, pool, q, lens, Hkv, hd)
    assert np.max(np.abs(got - ref)) <= _attn_tol(dtype, hd, H, Hkv) * np.abs(ref).max() + 1e-6
    # ctx = 1 returns V of the single cached token
    v0 = pool[table[0, 0], 1, :, 0, :].float().cpu().numpy()
    for h in range(H):
        np.testing.assert_allclose(got[0, h], v0[h // (H // Hkv)], rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("window", [0, 20])
@pytest.mark.parametrize("dtype,hd,H,Hkv", [("bf16", 128, 2, 2), ("f32", 64, 4, 4), ("f32", 128, 2, 1), ("bf16", 64, 8, 2), ("f32", 64, 8, 1)])
def test_paged_attention_of_one_chunk(dtype, hd, H, Hkv, window):
    """Launches in which no row has more than one chunk (up to 64 positions; with many rows up to 512, several blocks a wave) finish
    their results without a merge: every group size of the scalar kernel, and a scratch of NaN that such a launch leaves as it is.  The
    same results as the operand of the output projection, in octets and in rows of a larger image: bit for bit their split."""
    groups = H // (H // Hkv if H // Hkv in (2, 4, 8) else 1)
    for lens in ([1, 2, 16, 17, 63, 64], [190, 449, 512, 500, 257] + [5] * (464 // groups)):
        T = len(lens)
        table, pool, q = _attention_case(27, lens, H, Hkv, hd, dtype)
        out = torch.full((T, H, hd), float("nan"), device=DEV)
        scratch = torch.full((ld.ldk_attention_scratch_bytes(T, H, Hkv, hd, max(lens), window) // 4,), float("nan"), device=DEV)
        args = (q, H * hd, device_pool(pool), table.to(DEV), torch.arange(T, dtype=torch.int32, device=DEV),
                torch.tensor(lens, dtype=torch.int32, device=DEV), max(lens), H, Hkv, hd)
        ld.ldk_paged_attention(*args, out, scratch, window=window)
        ref = _oracle_attention(table, pool, q, lens, Hkv, hd, window=window)
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= _attn_tol(dtype, hd, H, Hkv) * np.abs(ref).max() + 1e-6
        assert torch.isnan(scratch).all()
        rows = out.view(T, H * hd)
        hi = rows.bfloat16(); lo = (rows - hi.float()).bfloat16()
        images = _attention_images(args, scratch, window, T, octets=True).view(2, H * hd // 8, T, 8).transpose(1, 2).reshape(2, T, H * hd)
        assert torch.equal(images[0], hi) and torch.equal(images[1], lo)
        images = _attention_images(args, scratch, window, T + 3, octets=False).view(2, T + 3, H * hd)
        assert torch.equal(images[0, :T], hi) and torch.equal(images[1, :T], lo) and (images[:, T:] == 7.0).all()
        assert torch.isnan(scratch).all()


def _attention_images(args, scratch, window, image_rows, octets):
    """Decode attention that leaves (hi, lo) bf16 images, as the layers of the engine call it: args of ldk_paged_attention up to hd."""
    q, q_stride, pool, table, slot, ctx, max_ctx, H, Hkv, hd = args
    xs = torch.full((2 * image_rows * H * hd,), 7.0, dtype=torch.bfloat16, device=DEV)
    P, I = C.c_void_p, C.c_int
    f = C.CFUNCTYPE(I, P, I, P, I, P, I, P, P, I, I, I, I, I, I, P, P, C.c_size_t, P, I, C.c_bool, I, P)(
        ("_ZN2ld21paged_attention_splitEPKfiPKviPKiiS5_S5_iiiiiiPtPvmP12ihipStream_tibiPi", ld.lib()))
    rc = f(q.data_ptr(), q_stride, pool.data_ptr(), ld.LD_BF16 if pool.dtype == torch.bfloat16 else ld.LD_F32, table.data_ptr(), table.shape[1],
           slot.data_ptr(), ctx.data_ptr(), max_ctx, ctx.numel(), H, Hkv, hd, window, xs.data_ptr(), scratch.data_ptr(), scratch.numel() * 4,
           torch.cuda.current_stream().cuda_stream, image_rows, octets, 0, None)
    assert rc == ld.LD_OK
    return xs


@pytest.mark.parametrize("dtype,hd", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("chunks", [1, 2, 23, 24, 25, 47, 48, 49, 200, 257])
def test_paged_attention_chunk_counts(dtype, hd, chunks):
    """Decode attention merged from as many chunks of 64 positions, around the number the merge requests before it knows how
    many there are (12 per thread group: 24 and 48) and the 256 statistics its threads take at once; beside it, where the grid
    allows, a row of one position, whose other chunks are never written: the scratch is NaN before the call."""
    lens = [64 * chunks - 7] + [1] * (chunks < 250)
    table, pool, q = _attention_case(24, lens, 1, 1, hd, dtype)
    out = torch.empty(len(lens), 1, hd, device=DEV)
    scratch = torch.full((ld.ldk_attention_scratch_bytes(len(lens), 1, 1, hd, max(lens), 0) // 4,), float("nan"), device=DEV)
    ld.ldk_paged_attention(q, hd, device_pool(pool), table.to(DEV), torch.arange(len(lens), dtype=torch.int32, device=DEV),
                           torch.tensor(lens, dtype=torch.int32, device=DEV), max(lens), 1, 1, hd, out, scratch)
    ref = _oracle_attention(table, pool, q, lens, 1, hd)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= _attn_tol(dtype, hd, 1, 1) * np.abs(ref).max() + 1e-6


@pytest.mark.parametrize("window", [1, 5, 16, 17, 100, 256, 4096])
@pytest.mark.parametrize("dtype,hd,H,Hkv", [("bf16", 128, 8, 2), ("f32", 64, 4, 4)])
def test_paged_attention_band(dtype, hd, H, Hkv, window):
    """Attention band: the row sees its last `window` positions only; bands that start inside a block, at a
    block boundary, that are longer than the context, and of a single position."""
    lens = [1, 2, 15, 16, 17, 63, 255, 256, 257, 300, 1025]
    table, pool, q = _attention_case(22, lens, H, Hkv, hd, dtype)
    got = _run_attention(table, pool, q, lens, H, Hkv, hd, window=window)
    ref = _oracle_attention(table, pool, q, lens, Hkv, hd, window=window)
    assert np.max(np.abs(got - ref)) <= _attn_tol(dtype, hd, H, Hkv) * np.abs(ref).max() + 1e-6
    if window == 1:      # the own value
        for b, n in enumerate(lens):
            v = pool[table[b, (n - 1) // 16], 1, :, (n - 1) % 16, :].float().cpu().numpy()
            for h in range(H):
                np.testing.assert_allclose(got[b, h], v[h // (H // Hkv)], rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("H,Hkv", [(32, 32), (32, 8)])
def test_paged_attention_scratch_sized_for_the_cap_serves_every_shorter_context(H, Hkv):
    """The chunking follows the launch's longest context; scratch sized once for the cap must do for all
    shorter ones (the chunk count is not monotonic in the context length)."""
    hd, cap = 128, 16384
    lens_all = [1, 100, 1030, 2052, 3074, 4103, 5125, 7169, 9220, 13315, 16384]
    table, pool, q = _attention_case(23, [cap], H, Hkv, hd, "bf16")
    dpool = device_pool(pool)
    for T in (1, 3, 8):
        scratch = torch.empty(ld.ldk_attention_scratch_bytes(T, H, Hkv, hd, cap, 0), dtype=torch.uint8, device=DEV)
        qq = q.expand(T, H, hd).contiguous()
        slot = torch.zeros(T, dtype=torch.int32, device=DEV)
        out = torch.empty(T, H, hd, device=DEV)
        for n in lens_all:
            ctx = torch.full((T,), n, dtype=torch.int32, device=DEV)
            ld.ldk_paged_attention(qq, H * hd, dpool, table.to(DEV), slot, ctx, n, H, Hkv, hd, out, scratch)
        torch.cuda.synchronize()
        ref = _oracle_attention(table, pool, q, [lens_all[-1]], Hkv, hd)
        assert np.max(np.abs(out[0].cpu().numpy() - ref[0])) <= 3e-5 * np.abs(ref).max() + 1e-6


def test_paged_attention_grouped_band_serving_shape_sampled():
    """Batch 32, 32 query heads on 8 KV heads, contexts uniform in [512, 8192], band of 4096 positions:
    sampled rows (the longest, the shortest, one just over the band) against the oracle."""
    lens = gen.randint(20240602, 1, 512, 8192, 32).tolist()
    lens[3] = 4097
    table, pool, q = _attention_case(20240602, lens, 32, 8, 128, "bf16")
    got = _run_attention(table, pool, q, lens, 32, 8, 128, window=4096)
    assert np.isfinite(got).all()
    rows = [3, 9, int(np.argmax(lens)), int(np.argmin(lens))]
    ref = _oracle_attention(table, pool, q, lens, 8, 128, rows=rows, window=4096)
    err = np.max(np.abs(got[rows] - ref)) / np.abs(ref).max()
    assert err <= 2e-5, err


def test_paged_attention_microbench_shape():
    """Batch 16, 32 heads x 128, contexts uniform in [256, 4096] (the benchmark's draw), permuted block table:
    every (sequence, head) output against the oracle."""
    lens = gen.randint(20240601, 1, 256, 4096, 16).tolist()
    table, pool, q = _attention_case(20240601, lens, 32, 32, 128, "bf16")
    got = _run_attention(table, pool, q, lens, 32, 32, 128)
    assert np.isfinite(got).all()
    rows = list(range(16))
    ref = _oracle_attention(table, pool, q, lens, 32, 128, rows=rows)
    err = np.max(np.abs(got[rows] - ref)) / np.abs(ref).max()
    assert err <= 2e-5, err


def test_argmax_ties_and_brute_force():
    V = 32000
    lg = gen.normal(6, 1, (5, V))
    lg[1, [31999, 12, 700]] = 50.0
    lg[2, :] = 1.5
    lg[3, V - 1] = 60.0
    out = torch.empty(5, dtype=torch.int32, device=DEV)
    ld.ldk_argmax(lg.to(DEV), out)
    ref = [oracle.argmax(lg[r].numpy()) for r in range(5)]
    assert out.cpu().tolist() == ref and ref[1] == 12 and ref[2] == 0 and ref[3] == V - 1


def test_sampling_kernel_draws_the_oracles_tokens():
    """Gumbel-max token choice: for every row the kernel's draw equals the oracle's for the same (seed,
    position); rows with temperature 0 are the plain argmax; over many positions the draws of a small
    vocabulary follow softmax(logits / T)."""
    V, R = 32000, 12
    lg = gen.normal(7, 1, (R, V)) * 3.0
    temps = [0.0, 0.3, 0.7, 1.0, 1.5, 2.0] * 2
    seeds = [int(x) for x in gen.randint(7, 2, 0, 2 ** 40, R).tolist()]
    seeds[3] = 2 ** 64 - 5                                   # a seed above 2^63: unsigned arithmetic
    pos = [0, 1, 17, 4095, 8191, 100000, 5, 6, 7, 8, 9, 10]
    out = torch.empty(R, dtype=torch.int32, device=DEV)
    seed_t = torch.tensor([s - 2 ** 64 if s >= 2 ** 63 else s for s in seeds], dtype=torch.int64, device=DEV)
    ld.ldk_sample(lg.to(DEV), torch.tensor(temps, device=DEV), seed_t, torch.tensor(pos, dtype=torch.int32, device=DEV), out)
    got = out.cpu().tolist()
    for r in range(R):
        ref = oracle.sample_gumbel(lg[r].numpy(), temps[r], seeds[r], pos[r]) if temps[r] > 0 else oracle.argmax(lg[r].numpy())
        assert got[r] == ref, (r, got[r], ref)
    assert len(set(got[1:6])) > 1                            # the noise does move the choice
    # frequencies on a small vocabulary
    small = torch.tensor([1.2, -0.3, 0.0, 2.5, 2.4, -4.0, 0.7, 1.9])
    n = 20000
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    ld.ldk_sample(small.repeat(n, 1).to(DEV), torch.full((n,), 0.7, device=DEV), torch.full((n,), 777, dtype=torch.int64, device=DEV),
                  torch.arange(n, dtype=torch.int32, device=DEV), out)
    cnt = np.bincount(out.cpu().numpy(), minlength=8)
    p = np.exp(small.numpy() / 0.7); p /= p.sum()
    assert np.abs((cnt - n * p) / np.sqrt(n * p * (1 - p))).max() < 4.5
    ref = [oracle.sample_gumbel(small.numpy(), 0.7, 777, i) for i in range(2000)]
    assert out.cpu().tolist()[:2000] == ref


@pytest.mark.parametrize("dtype,hd,T", [("bf16", 128, 1), ("bf16", 128, 2), ("bf16", 128, 3), ("bf16", 128, 4), ("f32", 64, 1),
                                        ("bf16", 64, 1), ("bf16", 64, 4)])
def test_fused_qkv_projection_rope_cache_append(dtype, hd, T):
    """ldk_qkv_rope = RMSNorm + q/k/v projection + rotary embedding + cache append in one call
    (one fused kernel for a single bf16 row, a composition otherwise)."""
    H, Hkv, K, nblk = 6, 2, 1160, 7
    N = (H + 2 * Hkv) * hd
    W = _mat(8, 1, N, K, dtype); x = gen.normal(8, 2, (T, K)); g = gen.normal(8, 3, (K,), std=0.1, mean=1.0)
    pos = torch.tensor([37, 16, 95, 0][:T], dtype=torch.int32)
    slot = torch.tensor([1, 0, 1, 0][:T], dtype=torch.int32)
    table = torch.tensor([[3, 6, 0, 0, 0, 0], [5, 1, 4, 2, 0, 0]], dtype=torch.int32)   # logical -> physical
    pdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    pool = torch.full((nblk, 2, Hkv, 16, hd), 512.0, dtype=pdt, device=DEV)
    cs = torch.empty(T, hd // 2, 2, device=DEV)
    qkv = torch.zeros(T, N, device=DEV)
    ld.ldk_rope_table(pos.to(DEV), hd, 10000.0, cs)
    ld.ldk_qkv_rope(W.to(DEV), x.to(DEV), qkv, cs, pos.to(DEV), slot.to(DEV), table.to(DEV), pool, H, Hkv, hd,
                    g=g.to(DEV), eps=1e-5)
    qkv_h, pool_h = qkv.cpu().numpy(), logical_pool(pool).float().cpu().numpy().astype(np.float64)
    Wh = oracle.to_host_matrix(W)
    touched = np.zeros(pool_h.shape[:4], bool)
    for t in range(T):
        ref = oracle.matvec(Wh, oracle.rmsnorm(x[t].numpy(), g.numpy(), 1e-5))
        scale = np.abs(ref).max()
        p = int(pos[t]); blk = int(table[slot[t], p // 16]); s = p % 16
        for h in range(H):
            r = oracle.rope_head(ref[h * hd:(h + 1) * hd], p)
            np.testing.assert_allclose(qkv_h[t, h * hd:(h + 1) * hd], r, rtol=0, atol=4e-6 * scale)
        for j in range(Hkv):
            k = oracle.rope_head(ref[(H + j) * hd:(H + j + 1) * hd], p)
            v = ref[(H + Hkv + j) * hd:(H + Hkv + j + 1) * hd]
            tol = (2.0 ** -7 if dtype == "bf16" else 4e-6) * scale
            assert np.max(np.abs(pool_h[blk, 0, j, s] - k)) <= tol and np.max(np.abs(pool_h[blk, 1, j, s] - v)) <= tol
            if dtype == "bf16":
                assert np.mean(pool_h[blk, 0, j, s] == oracle.round_bf16(k)) > 0.9
                assert np.mean(pool_h[blk, 1, j, s] == oracle.round_bf16(v)) > 0.9
            touched[blk, :, j, s] = True
    assert np.all(pool_h[~touched] == 512.0) and touched.sum() == T * 2 * Hkv


@pytest.mark.parametrize("K", [4096, 5120, 8192, 11008, 13824])
@pytest.mark.parametrize("T", [2, 3, 4])
def test_linear_two_to_four_rows_every_row_length(T, K):
    """Decode batches of 2 .. 4 rows at the row lengths of the 7B and 13B shapes (model and FFN widths:
    8 to 27 K slabs of the small-batch matrix-core kernel), all three epilogues, ragged output counts."""
    N = 77
    W = _mat(12, K, 2 * N, K, "bf16"); x = gen.normal(12, 2, (T, K)); g = gen.normal(12, 3, (K,), std=0.1, mean=1.0)
    y0 = gen.normal(12, 4, (T, N))
    Wh = oracle.to_host_matrix(W)
    Wd, xd, gd = W.to(DEV), x.to(DEV), g.to(DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_SWIGLU), dtype=torch.uint8, device=DEV)
    gu = np.stack([oracle.matvec(Wh, oracle.rmsnorm(x[t].numpy(), g.numpy(), 1e-5)) for t in range(T)])
    y = torch.empty(T, N, device=DEV)
    ld.ldk_linear(Wd, xd, y, ld.LDK_SWIGLU, g=gd, eps=1e-5, scratch=scratch)
    ref = _silu(gu[:, :N]) * gu[:, N:]
    assert np.max(np.abs(y.cpu().numpy() - ref)) <= 2e-5 * np.abs(ref).max()
    y = y0.to(DEV).clone()
    ld.ldk_linear(Wd[:N], xd, y, ld.LDK_ADD, g=gd, eps=1e-5, scratch=scratch)
    assert np.max(np.abs(y.cpu().numpy() - (y0.numpy() + gu[:, :N]))) <= 2e-5 * np.abs(gu).max()
    plain = np.stack([oracle.matvec(Wh, x[t].numpy()) for t in range(T)])
    y = torch.empty(T, 2 * N, device=DEV)
    ld.ldk_linear(Wd, xd, y, ld.LDK_STORE, scratch=scratch)
    assert np.max(np.abs(y.cpu().numpy() - plain)) <= 2e-5 * np.abs(plain).max()


@pytest.mark.parametrize("T", [2, 5, 31, 32, 33, 41, 48, 49, 64, 100, 257, 300, 320, 321])
@pytest.mark.parametrize("epi", ["store", "add_norm", "swiglu_norm"])
def test_linear_matrix_core_path(T, epi):
    """bf16 matrices, several rows, K a multiple of 128, scratch given: the MFMA kernel with split
    (hi + lo) activations.  Ragged N (not a multiple of the 128-column tile) and ragged T (33, 41, 48: the
    small-batch kernel's second group of rows, full and ragged; 49: the first row count of the 64-row kernel)."""
    N, K = 333, 1152
    rows = 2 * N if epi == "swiglu_norm" else N
    W = _mat(9, 1, rows, K, "bf16"); x = gen.normal(9, 2, (T, K)); g = gen.normal(9, 3, (K,), std=0.1, mean=1.0)
    y0 = gen.normal(9, 4, (T, N))
    Wh = oracle.to_host_matrix(W)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_SWIGLU), dtype=torch.uint8, device=DEV)
    y = y0.to(DEV).clone()
    if epi == "store":
        ld.ldk_linear(W.to(DEV), x.to(DEV), y, ld.LDK_STORE, scratch=scratch)
        ref = np.stack([oracle.matvec(Wh, x[t].numpy()) for t in range(T)])
    elif epi == "add_norm":
        ld.ldk_linear(W.to(DEV), x.to(DEV), y, ld.LDK_ADD, g=g.to(DEV), eps=1e-5, scratch=scratch)
        ref = y0.numpy() + np.stack([oracle.matvec(Wh, oracle.rmsnorm(x[t].numpy(), g.numpy(), 1e-5)) for t in range(T)])
    else:
        ld.ldk_linear(W.to(DEV), x.to(DEV), y, ld.LDK_SWIGLU, g=g.to(DEV), eps=1e-5, scratch=scratch)
        gu = np.stack([oracle.matvec(Wh, oracle.rmsnorm(x[t].numpy(), g.numpy(), 1e-5)) for t in range(T)])
        ref = _silu(gu[:, :N]) * gu[:, N:]
    err = np.max(np.abs(y.cpu().numpy() - ref)) / np.abs(ref).max()
    assert err <= 2e-5, err


@pytest.mark.parametrize("floats", ["1", "0"], ids=["floats", "images"])
@pytest.mark.parametrize("T", [2, 15, 16, 17, 32, 33, 48, 49, 63, 64])
@pytest.mark.parametrize("N,K", [(5, 128), (301, 2048), (4099, 2176), (66, 11008), (7, 8192), (4105, 8192), (1023, 16384)])
def test_linear_small_batch_edges(T, N, K, floats, monkeypatch):
    """The small-batch kernel, fed by float rows and by bf16 images (the form of a decode batch's layers), at the edges of its tiles: one row below, at and above each count of 16-row tiles of X; fewer
    output rows than a tile, odd and ragged counts; K slabs where most waves have no share (128), of exactly the width a
    workgroup holds (2048), just beyond it (2176: two uneven slabs), a ragged FFN width, and rows a multiple of
    16 KB apart, whose tiles are dealt out in turn.  Against float64 on every
    output: the two bf16 terms leave 2^-18 of an activation, float32 sums about as much (2^-24 per addition, a random walk
    over K <= 16384 terms), so |error| <= 2^-16 sum_k |w x| holds with room, and a lost low term (2^-9) does not pass."""
    monkeypatch.setenv("LD_GEMM_FLOATS", floats)
    W = _mat(31, 1, N, K, "bf16").to(DEV); x = gen.normal(31, 2, (T, K), device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_STORE), dtype=torch.uint8, device=DEV)
    y = torch.full((T, N), float("nan"), device=DEV)
    ld.ldk_linear(W, x, y, ld.LDK_STORE, scratch=scratch)
    ref, mag = x.double() @ W.double().t(), x.double().abs() @ W.double().abs().t()
    assert ((y.double() - ref).abs() <= 2.0 ** -16 * mag).all()


@pytest.mark.parametrize("H,Hkv,hd", [(2, 1, 128), (3, 3, 64)])
@pytest.mark.parametrize("T", [64, 65, 79, 97, 128, 129, 257, 300])
def test_qkv_rope_equals_product_then_rotation(T, H, Hkv, hd):
    """ldk_qkv_rope on many rows (rotation, cache append and the sum of the product's slabs in one kernel from 65 rows on, in each of its
    forms: a row, four or eight, sixteen at a time) against ldk_linear followed by ldk_rope_kv_write: the same bits in the whole q-k-v buffer and in the whole pool.  Rows of
    two sequences at consecutive positions that start inside a block, single rows of a third, and a ragged last group of rows.
    The rows of the pool also against float64: one rounding to bf16 of a sum within 2^-16 of its terms."""
    K, N = 1152, (H + 2 * Hkv) * hd
    W = _mat(47, hd, N, K, "bf16").to(DEV); x = gen.normal(47, 2, (T, K), device=DEV)
    n0 = T // 2
    pos = torch.tensor([5 + i for i in range(n0)] + [16 + i for i in range(T - n0 - 1)] + [333], dtype=torch.int32, device=DEV)
    slot = torch.tensor([0] * n0 + [1] * (T - n0 - 1) + [2], dtype=torch.int32, device=DEV)
    table = torch.randperm(3 * 24, generator=torch.Generator().manual_seed(T)).to(torch.int32).view(3, 24).to(DEV)
    cs = torch.empty(T, hd, device=DEV)
    ld.ldk_rope_table(pos, hd, 10000.0, cs)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_STORE), dtype=torch.uint8, device=DEV)
    pools = [torch.full((72, 2, Hkv, 16, hd), 3.0, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    a, b = torch.full((T, N), float("nan"), device=DEV), torch.full((T, N), float("nan"), device=DEV)
    ld.ldk_qkv_rope(W, x, a, cs, pos, slot, table, pools[0], H, Hkv, hd, None, 1e-5, scratch)
    ld.ldk_linear(W, x, b, ld.LDK_STORE, scratch=scratch)
    ld.ldk_rope_kv_write(b, cs, pos, slot, table, pools[1], H, Hkv, hd)
    assert torch.equal(a, b) and torch.equal(pools[0], pools[1])
    ref, mag = x.double() @ W.double().t(), x.double().abs() @ W.double().abs().t()
    c = cs.view(T, hd // 2, 2).double()
    phys = table[slot.long(), pos.long() // 16].long()
    for j in range(Hkv):
        k0, v0 = (H + j) * hd, (H + Hkv + j) * hd
        u, v = ref[:, k0:k0 + hd // 2], ref[:, k0 + hd // 2:k0 + hd]
        rot = torch.cat([u * c[..., 0] - v * c[..., 1], u * c[..., 1] + v * c[..., 0]], 1)
        tol = 2.0 ** -16 * (mag[:, k0:k0 + hd // 2] + mag[:, k0 + hd // 2:k0 + hd]).repeat(1, 2)
        got = pools[0][phys, 0, j, pos.long() % 16].double()
        assert ((got - rot).abs() <= 2.0 ** -8 * rot.abs() + 2 * tol).all()
        got = pools[0].view(72, 2, Hkv, hd, 16)[phys, 1, j, :, pos.long() % 16].double()
        assert ((got - ref[:, v0:v0 + hd]).abs() <= 2.0 ** -8 * ref[:, v0:v0 + hd].abs() + 2 * 2.0 ** -16 * mag[:, v0:v0 + hd]).all()
    written = torch.zeros(72, 16, dtype=torch.bool, device=DEV); written[phys, pos.long() % 16] = True
    assert (pools[0].permute(0, 3, 1, 2, 4)[..., 0, :, :][~written] == 3.0).all()
    assert (pools[0].view(72, 2, Hkv, hd, 16)[:, 1].permute(0, 3, 1, 2)[~written] == 3.0).all()


@pytest.mark.parametrize("floats", ["1", "0"], ids=["floats", "images"])
@pytest.mark.parametrize("T", [2, 16, 17, 20, 21, 32, 33, 40, 41, 64])
@pytest.mark.parametrize("N,K,epi", [(5, 128, "store"), (301, 4096, "swiglu"), (66, 5120, "add"), (302, 11008, "add"), (7, 8320, "swiglu")])
def test_linear_small_batch_normalises_float_rows(T, N, K, epi, floats, monkeypatch):
    """The small-batch product with a norm, from float rows (split and squared in the product, the
    scale applied to the finished sums) and from images (a pass in front): rows of very different size, so that a scale or a sum of
    squares of another row shows.  Against float64: the bound of test_linear_small_batch_edges on the normalised row, and
    2^-20 for the sum of squares and its root."""
    monkeypatch.setenv("LD_GEMM_FLOATS", floats)
    code = {"store": ld.LDK_STORE, "add": ld.LDK_ADD, "swiglu": ld.LDK_SWIGLU}[epi]
    rows = 2 * N if epi == "swiglu" else N
    W = _mat(37, K, rows, K, "bf16").to(DEV); g = gen.normal(37, 3, (K,), std=0.1, mean=1.0).to(DEV)
    x = gen.normal(37, 2, (T, K), device=DEV) * (10.0 ** (torch.arange(T, device=DEV) % 5 - 2))[:, None]
    y0 = gen.normal(37, 4, (T, N), device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, code), dtype=torch.uint8, device=DEV)
    y = y0.clone()
    ld.ldk_linear(W, x, y, code, g=g, eps=1e-5, scratch=scratch)
    xn = x.double() / torch.sqrt((x.double() ** 2).mean(1, keepdim=True) + 1e-5) * g.double()
    full, mag = xn @ W.double().t(), xn.abs() @ W.double().abs().t()
    a, tol = full[:, :N], 2.0 ** -16 + 2.0 ** -20
    if epi == "swiglu":      # |d(silu(a) b)| <= 1.1 |b| |da| + |silu(a)| |db|
        ref = torch.nn.functional.silu(a) * full[:, N:]
        bound = tol * (1.1 * full[:, N:].abs() * mag[:, :N] + torch.nn.functional.silu(a).abs() * mag[:, N:]) + 1e-6 * ref.abs() + 1e-7
    else:
        ref, bound = a + (y0.double() if epi == "add" else 0), tol * mag[:, :N] + 1e-6
    assert ((y.double() - ref).abs() <= bound).all()


@pytest.mark.parametrize("plan", ["2,128,1", "2,128,3", "2,256,1", "2,256,2", "192,256,1", "192,256,4"])
@pytest.mark.parametrize("epi", ["store", "add", "swiglu"])
def test_linear_big_tile_every_plan(plan, epi, monkeypatch, capfd):
    """The big-tile kernel picks its tile and split-K factor from a cost estimate; here three of its tiles
    (128 x 128, 128 x 256, 192 x 256) are forced in turn, with and without split-K, on a shape that is ragged
    in tokens and in output columns, against the oracle on every output.  (A plan that was not taken is reported.)"""
    monkeypatch.setenv("LD_GEMM_BIG", plan)
    T, N, K = 333, 301, 1152
    rows = 2 * N if epi == "swiglu" else N
    W = _mat(11, 1, rows, K, "bf16"); x = gen.normal(11, 2, (T, K)); y0 = gen.normal(11, 4, (T, N))
    Wh = oracle.to_host_matrix(W)
    code = {"store": ld.LDK_STORE, "add": ld.LDK_ADD, "swiglu": ld.LDK_SWIGLU}[epi]
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, code), dtype=torch.uint8, device=DEV)
    y = y0.to(DEV).clone()
    ld.ldk_linear(W.to(DEV), x.to(DEV), y, code, scratch=scratch)
    ref = np.stack([oracle.matvec(Wh, x[t].numpy()) for t in range(T)])
    if epi == "add":
        ref = y0.numpy() + ref
    elif epi == "swiglu":
        ref = _silu(ref[:, :N]) * ref[:, N:]
    err = np.max(np.abs(y.cpu().numpy() - ref)) / np.abs(ref).max()
    assert err <= 2e-5, err
    assert "LD_GEMM_BIG" not in capfd.readouterr().err


@pytest.mark.parametrize("plan", ["256,256,1", "100,100,1", "128,256,0", "nonsense"])
def test_linear_unknown_forced_plan_is_reported(plan, monkeypatch, capfd):
    """A forced plan that the form does not have (256 x 256 exists for one term only) leaves the planner's choice and says so."""
    T, N, K = 333, 301, 1152
    W = _mat(11, 1, N, K, "bf16").to(DEV); x = gen.normal(11, 2, (T, K), device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_STORE), dtype=torch.uint8, device=DEV)
    ys = []
    for env in (None, plan):
        if env:
            monkeypatch.setenv("LD_GEMM_BIG", env)
        ys.append(torch.full((T, N), float("nan"), device=DEV))
        ld.ldk_linear(W, x, ys[-1], ld.LDK_STORE, scratch=scratch)
        assert ("LD_GEMM_BIG" in capfd.readouterr().err) == bool(env)
    assert torch.isfinite(ys[0]).all() and torch.equal(*ys)


@pytest.mark.parametrize("form,rows,cols", [("two", r, c) for r, c in ((96, 128), (96, 192), (96, 256), (128, 128), (128, 192), (128, 256), (160, 192), (160, 256), (192, 192), (192, 256))]
                         + [("f16", r, c) for r, c in ((128, 192), (128, 256), (192, 192), (192, 256), (224, 256), (256, 160), (256, 192), (256, 256))])
@pytest.mark.parametrize("K,ks", [(128, 1), (1152, 1), (1152, 4)])
def test_linear_every_tile(form, rows, cols, K, ks, monkeypatch, capfd):
    """Every tile of the big-tile kernel, in both forms (two bf16 terms; one fp16 term on the fp16 image and on the bf16
    matrix), forced in turn on a shape that is ragged in rows and columns: the fewest chunks of K the pipeline has to
    cope with (2), an ordinary run, and split K with uneven slabs (18 chunks over 4).  Against float64 on the inputs
    as the form rounds them: |error| <= 2^-16 sum_k |w x| (float32 sums of up to 1152 terms stay well below; for two
    terms 2^-18 per activation adds to it).  The 160-column tile has no SwiGLU form."""
    monkeypatch.setenv("LD_GEMM_BIG", "%d,%d,%d" % (rows, cols, ks))
    T, N = 333, 301
    W = _mat(41, K, 2 * N, K, "bf16").to(DEV); x = gen.normal(41, 2, (T, K), device=DEV)
    y0 = gen.normal(41, 4, (T, N), device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_SWIGLU), dtype=torch.uint8, device=DEV)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    Wh = torch.empty_like(W, dtype=torch.float16); ld.ldk_weights_to_f16(W, Wh, flag)
    hi = x.bfloat16().float()
    xr = ((hi + (x - hi).bfloat16().float()).half() if form == "f16" else x).double()
    full, mag = xr @ W.double().t(), xr.abs() @ W.double().abs().t()
    for epi, n in ((ld.LDK_STORE, N), (ld.LDK_ADD, N)) + (((ld.LDK_SWIGLU, 2 * N),) if cols != 160 else ()):
        outs = []
        for image in ((None, Wh) if form == "f16" else (None,)):
            y = y0.clone() if epi == ld.LDK_ADD else torch.full((T, N), float("nan"), device=DEV)
            if form == "f16":
                ld.ldk_linear_f16(W[:n], x, y, flag, epi, scratch=scratch, W_f16=None if image is None else image[:n])
            else:
                ld.ldk_linear(W[:n], x, y, epi, scratch=scratch)
            outs.append(y)
        if form == "f16":
            assert torch.equal(outs[0], outs[1]) and int(flag.item()) == 0
        a = full[:, :N]
        if epi == ld.LDK_SWIGLU:      # |d(silu(a) b)| <= 1.1 |b| |da| + |silu(a)| |db|
            ref = torch.nn.functional.silu(a) * full[:, N:]
            bound = 2.0 ** -16 * (1.1 * full[:, N:].abs() * mag[:, :N] + torch.nn.functional.silu(a).abs() * mag[:, N:]) + 1e-6 * ref.abs()
        else:
            ref, bound = a + (y0.double() if epi == ld.LDK_ADD else 0), 2.0 ** -16 * mag[:, :N] + 1e-6
        assert ((outs[-1].double() - ref).abs() <= bound + 1e-7).all(), epi
    assert "LD_GEMM_BIG" not in capfd.readouterr().err


@pytest.mark.parametrize("N,K", [(301, 4224), (640, 5120), (96, 6144), (130, 10368), (513, 11008), (37, 14336), (77, 2816), (77, 11392), (12, 24704),
                                 (5120, 4224), (8200, 5120), (8200, 2304)])
@pytest.mark.parametrize("T", [2, 20, 33, 64])
def test_linear_small_batch_slabs(T, N, K):
    """The small-batch product where its K slabs (2048 columns at most, 1024 beyond 32 rows) go up to a power of two (3 to 4, 6 and 7 to
    8) and where they stay (2, 3, 5, 11, 12, 13, 14, 25): uneven slabs, fewer columns than workgroups.  Against float64: two terms are off by
    at most 2^-16 of a product, the float32 sums by 2^-20 of the sum of magnitudes."""
    W = _mat(71, K, N, K, "bf16").to(DEV); x = gen.normal(71, 2, (T, K), device=DEV); g = 1 + 0.1 * gen.normal(71, 3, (K,), device=DEV)
    y = torch.full((T, N), float("nan"), device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_STORE), dtype=torch.uint8, device=DEV)
    for norm in (False, True):
        ld.ldk_linear(W, x, y, ld.LDK_STORE, g if norm else None, 1e-5, scratch)
        xd = x.double()
        if norm:
            xd = xd * g.double() / torch.sqrt((xd * xd).mean(1, keepdim=True) + 1e-5)
        ref, mag = xd @ W.double().t(), xd.abs() @ W.double().abs().t()
        assert ((y.double() - ref).abs() <= (2.0 ** -16 + 2.0 ** -20) * mag).all()


@pytest.mark.parametrize("T,N,K,epi,slabs", [(256, 12288, 4096, "STORE", 2), (152, 12288, 4096, "STORE", 4), (300, 12288, 4096, "STORE", 2),
                                             (152, 11008, 4096, "SWIGLU", 2), (200, 4096, 11008, "ADD", 8), (256, 15360, 5120, "STORE", 2)])
def test_linear_two_term_slabs(T, N, K, epi, slabs):
    """K is cut in as many slabs as ever where tiles take a two-term product (longer sums are less exact): the slabs whose partial sums the call
    leaves in its scratch.  The sums are finite, so what is still NaN was not written."""
    code = getattr(ld, "LDK_" + epi); R = N * (2 if epi == "SWIGLU" else 1)
    W = torch.full((R, K), 0.01, dtype=torch.bfloat16, device=DEV); x = torch.ones(T, K, device=DEV); y = torch.zeros(T, N, device=DEV)
    scratch = torch.full((T * K + 8 * T * R,), float("nan"), device=DEV)
    assert scratch.numel() * 4 >= ld.ldk_linear_scratch_bytes(T, N, K, code)
    ld.ldk_linear(W, x, y, code, scratch=scratch)
    written = scratch[T * K:].isfinite()
    assert int(written.sum()) == slabs * T * R and written[:slabs * T * R].all()


@pytest.mark.parametrize("form,rows,cols", [("two", 96, 128), ("f16", 128, 192), ("two", 128, 128), ("f16", 256, 160)])
@pytest.mark.parametrize("K,ks", [(128, 1), (256, 1), (384, 1), (896, 3), (1408, 3)])
def test_linear_tile_stages(form, rows, cols, K, ks, monkeypatch):
    """The smallest tile of each form keeps two stages in a launch of more than 256 workgroups (here 3 x 100 x ks of them) and has three in
    a smaller one (the first columns alone), as the tiles beside them have in both: 2, 4 and 6 chunks of K, and split K with
    uneven slabs (14 and 22 chunks over 3).  The same bits for the columns that both compute, and within
    2^-16 sum_k |w x| of float64 on the inputs as the form rounds them (see test_linear_every_tile)."""
    monkeypatch.setenv("LD_GEMM_BIG", "%d,%d,%d" % (rows, cols, ks))
    T, N, part = 2 * rows + 5, 99 * cols + 7, 20 * cols + 40
    W = _mat(47, K, N, K, "bf16").to(DEV); x = gen.normal(47, 2, (T, K), device=DEV)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    Wh = torch.empty_like(W, dtype=torch.float16); ld.ldk_weights_to_f16(W, Wh, flag)
    scratch = torch.empty(2 * T * K * 2 + 256 + ks * T * N * 4, dtype=torch.uint8, device=DEV)
    hi = x.bfloat16().float()
    xr = ((hi + (x - hi).bfloat16().float()).half() if form == "f16" else x).double()
    ref, mag = xr @ W.double().t(), xr.abs() @ W.double().abs().t()
    for image in ((None, Wh) if form == "f16" else (None,)):
        ys = []
        for n in (N, part):
            ys.append(torch.full((T, n), float("nan"), device=DEV))
            if form == "f16":
                ld.ldk_linear_f16(W[:n], x, ys[-1], flag, ld.LDK_STORE, scratch=scratch, W_f16=None if image is None else image[:n])
            else:
                ld.ldk_linear(W[:n], x, ys[-1], ld.LDK_STORE, scratch=scratch)
        assert torch.equal(ys[0][:, :part], ys[1])
        assert ((ys[0].double() - ref).abs() <= 2.0 ** -16 * mag + 1e-6).all()


@pytest.mark.parametrize("form", ["two", "f16"])
@pytest.mark.parametrize("T,N,ks", [(65, 4, 1), (333, 300, 1), (333, 300, 3), (257, 1028, 2), (300, 302, 1)])
def test_linear_tile_stores_of_four_columns(form, T, N, ks, monkeypatch):
    """The big-tile kernel stores four columns at a time at any float's address, and one at a time what is left of a row (302 columns;
    an output that starts 4 bytes past an aligned address): the same bits, nothing written beside the output, and within
    2^-16 sum_k |w x| of float64 on the inputs as the form rounds them (see test_linear_every_tile)."""
    monkeypatch.setenv("LD_GEMM_BIG", "128,256,%d" % ks)
    K = 1152
    W = _mat(43, N, 2 * N, K, "bf16").to(DEV); x = gen.normal(43, 2, (T, K), device=DEV); y0 = gen.normal(43, 4, (T, N), device=DEV)
    scratch = torch.empty(2 * T * K * 2 + 256 + ks * T * 2 * N * 4, dtype=torch.uint8, device=DEV)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    hi = x.bfloat16().float()
    xr = ((hi + (x - hi).bfloat16().float()).half() if form == "f16" else x).double()
    full, mag = xr @ W.double().t(), xr.abs() @ W.double().abs().t()
    for epi, n in ((ld.LDK_STORE, N), (ld.LDK_ADD, N), (ld.LDK_SWIGLU, 2 * N)):
        outs = []
        for shift in (0, 1):
            buf = torch.full((T * N + 8,), 7.0, device=DEV)
            y = buf[4 + shift:4 + shift + T * N].view(T, N)
            y.copy_(y0)
            if form == "f16":
                ld.ldk_linear_f16(W[:n], x, y, flag, epi, scratch=scratch)
            else:
                ld.ldk_linear(W[:n], x, y, epi, scratch=scratch)
            assert (buf[:4 + shift] == 7.0).all() and (buf[4 + shift + T * N:] == 7.0).all()
            outs.append(y)
        assert torch.equal(*outs)
        a = full[:, :N]
        if epi == ld.LDK_SWIGLU:
            ref = torch.nn.functional.silu(a) * full[:, N:]
            bound = 2.0 ** -16 * (1.1 * full[:, N:].abs() * mag[:, :N] + torch.nn.functional.silu(a).abs() * mag[:, N:]) + 1e-6 * ref.abs()
        else:
            ref, bound = a + (y0.double() if epi == ld.LDK_ADD else 0), 2.0 ** -16 * mag[:, :N] + 1e-6
        assert ((outs[0].double() - ref).abs() <= bound + 1e-7).all(), epi


@pytest.mark.parametrize("form,T,N,K", [("tiles", 257, 2044, 1152), ("tiles", 300, 1752, 1152)]
                         + [(form, T, N, K) for form in ("floats", "images") for T, N, K in ((40, 13824, 1152), (64, 8196, 2176))])
@pytest.mark.parametrize("epi", ["store", "add", "swiglu"])
def test_linear_reduction_of_four_outputs(form, T, N, K, epi, monkeypatch):
    """Slab sums of 524288 outputs and more are added four outputs a thread where the output is 16-byte aligned, one at a time where
    it starts 4 bytes past that: the same bits, behind the big tiles (two slabs) and behind the small-batch product with a norm, from
    float rows (whose scale the reduction applies) and from images.  Against float64 on every output: the bound of
    test_linear_small_batch_normalises_float_rows."""
    assert T * N >= 1 << 19 and N % 4 == 0
    monkeypatch.setenv("LD_GEMM_BIG", "128,256,2")
    monkeypatch.setenv("LD_GEMM_FLOATS", "1" if form == "floats" else "0")
    code = {"store": ld.LDK_STORE, "add": ld.LDK_ADD, "swiglu": ld.LDK_SWIGLU}[epi]
    W = _mat(59, N, N * (2 if epi == "swiglu" else 1), K, "bf16").to(DEV); g = gen.normal(59, 3, (K,), std=0.1, mean=1.0).to(DEV)
    x = gen.normal(59, 2, (T, K), device=DEV) * (10.0 ** (torch.arange(T, device=DEV) % 5 - 2))[:, None]
    y0 = gen.normal(59, 4, (T, N), device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, code), dtype=torch.uint8, device=DEV)
    outs = []
    for shift in (0, 1):
        buf = torch.full((T * N + 8,), 7.0, device=DEV)
        y = buf[4 + shift:4 + shift + T * N].view(T, N)
        y.copy_(y0)
        ld.ldk_linear(W, x, y, code, g=g, eps=1e-5, scratch=scratch)
        assert (buf[:4 + shift] == 7.0).all() and (buf[4 + shift + T * N:] == 7.0).all()
        outs.append(y)
    assert torch.equal(*outs)
    xn = x.double() / torch.sqrt((x.double() ** 2).mean(1, keepdim=True) + 1e-5) * g.double()
    full, mag = xn @ W.double().t(), xn.abs() @ W.double().abs().t()
    a, tol = full[:, :N], 2.0 ** -16 + 2.0 ** -20
    if epi == "swiglu":
        ref = torch.nn.functional.silu(a) * full[:, N:]
        bound = tol * (1.1 * full[:, N:].abs() * mag[:, :N] + torch.nn.functional.silu(a).abs() * mag[:, N:]) + 1e-6 * ref.abs() + 1e-7
    else:
        ref, bound = a + (y0.double() if epi == "add" else 0), tol * mag[:, :N] + 1e-6
    assert ((outs[0].double() - ref).abs() <= bound).all()


def test_linear_matrix_core_7b_shapes_sampled():
    """Launch shapes of the batch-32 decode step, of a 256-row prefill chunk, of a mixed step (32 decode rows
    + four 256-row chunks) and of a 2048-row chunk beside 63 decode rows, sampled outputs.  The last two have
    a tail of 32 / 63 rows past the last full 256-row tile, which is cut off and computed by the small-batch
    kernels: the rows on both sides of the cut are among the samples.  768 rows: three row tiles, a grid of
    less than one round."""
    _sampled_linear_cases((32, 256, 768, 1056, 2111),
                          [(12288, 4096, ld.LDK_STORE), (4096, 11008, ld.LDK_ADD), (11008, 4096, ld.LDK_SWIGLU)])


def test_linear_matrix_core_13b_shapes_sampled():
    """The four layer matrices of the 13B shape (row lengths 5120 and 13824) at the row counts of its batch-64
    step: 63 decode rows beside a 2048-row chunk (2111), and 2112 (one more decode row, or a chunk behind a
    pending token); sampled outputs, the rows on both sides of the 256-row tile cut among them."""
    _sampled_linear_cases((2111, 2112), [(15360, 5120, ld.LDK_STORE), (5120, 5120, ld.LDK_ADD),
                                         (5120, 13824, ld.LDK_ADD), (13824, 5120, ld.LDK_SWIGLU)])


def _sampled_linear_cases(row_counts, matrices):
    for T in row_counts:
        for N, K, epi in matrices:
            rows = N * (2 if epi == ld.LDK_SWIGLU else 1)
            W = gen.normal(3, N, (rows, K), std=0.02, device=DEV).bfloat16()
            x = gen.normal(3, 7 + T, (T, K), device=DEV)
            y = torch.zeros(T, N, device=DEV)
            scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, epi), dtype=torch.uint8, device=DEV)
            ld.ldk_linear(W, x, y, epi, scratch=scratch)
            ns = gen.randint(3, 9, 0, N - 1, 6).tolist() + [0, N - 1]
            ts = sorted(set(gen.randint(3, 10, 0, T - 1, 5).tolist() + [0, T - 1, max(T - T % 256 - 1, 0), min(T - T % 256, T - 1)]))
            xh = x.cpu().numpy(); yh = y.cpu().numpy()
            for n in ns:
                wr = oracle.to_host_matrix(W[n:n + 1]); wu = oracle.to_host_matrix(W[N + n:N + n + 1]) if epi == ld.LDK_SWIGLU else None
                for t in ts:
                    a = oracle.matvec(wr, xh[t])[0]
                    if wu is not None:
                        a = oracle.silu(a) * oracle.matvec(wu, xh[t])[0]
                    # two-term bf16 split of the activations: ~2^-17 per element, random-walk over K terms
                    assert abs(yh[t, n] - a) <= 1e-4 * max(1.0, abs(a)), (T, N, t, n, yh[t, n], a)


def test_linear_fp16_rows_sampled():
    """The form of the multi-row product that long prefill chunks take in the engine (ldk_linear_f16: activations
    rounded to fp16 in one term, bf16 matrix entries widened to fp16 exactly): sampled outputs against the oracle's
    dot product on the inputs rounded as the kernel rounds them (the 16-bit sum of the split image, then fp16; what
    remains is float32 accumulation: the two-term test's bound) and
    against the oracle on the exact inputs (the rounding itself: 2^-12 per term, random walk over K terms).  Row
    counts with a remainder of up to 64 rows (1056, 2111), which keeps both terms in some products and is not compared with the
    one-term result, with three and one row tiles, and one that stays on the
    small-batch kernel (32: bit-equal to ldk_linear).  With the matrix's fp16 image (ldk_weights_to_f16: equal to the
    bf16 values entry by entry, truncated toward zero below 2^-17 where fp16 has no bits left) the same call gives
    bit-equal results.  A value beyond the fp16 range in the input or in the matrix raises the flag."""
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    for T in (32, 256, 768, 1056, 2111):
        for N, K, epi in [(12288, 4096, ld.LDK_STORE), (4096, 11008, ld.LDK_ADD), (11008, 4096, ld.LDK_SWIGLU)]:
            rows = N * (2 if epi == ld.LDK_SWIGLU else 1)
            W = gen.normal(3, N, (rows, K), std=0.02, device=DEV).bfloat16()
            x = gen.normal(3, 7 + T, (T, K), device=DEV)
            y = torch.zeros(T, N, device=DEV); y2 = torch.zeros(T, N, device=DEV)
            scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, epi), dtype=torch.uint8, device=DEV)
            flag.zero_()
            ld.ldk_linear_f16(W, x, y, flag, epi, scratch=scratch)
            assert int(flag.item()) == 0
            ld.ldk_linear(W, x, y2, epi, scratch=scratch)
            r = T % 256 if T > 256 and T % 256 <= 64 else 0       # rows that may keep both terms
            if T <= 64:
                assert torch.equal(y, y2)
            else:
                assert not torch.equal(y[:T - r], y2[:T - r])     # the single-term form did run
            Wh = torch.zeros(rows, K, dtype=torch.float16, device=DEV); y3 = torch.zeros(T, N, device=DEV)
            ld.ldk_weights_to_f16(W, Wh, flag)
            assert int(flag.item()) == 0
            wf, whf = W.float(), Wh.float()
            fits = wf.abs() >= 2.0 ** -17
            assert torch.equal(whf[fits], wf[fits])
            assert bool(((whf.abs() <= wf.abs()) & ((wf - whf).abs() < 2.0 ** -24) & (whf * wf >= 0))[~fits].all())
            ld.ldk_linear_f16(W, x, y3, flag, epi, scratch=scratch, W_f16=Wh)
            assert int(flag.item()) == 0 and torch.equal(y3, y)
            del Wh, wf, whf, fits, y3
            ns = gen.randint(3, 9, 0, N - 1, 6).tolist() + [0, N - 1]
            ts = sorted(set(gen.randint(3, 10, 0, T - 1, 5).tolist() + [0, T - 1, max(T - T % 256 - 1, 0), min(T - T % 256, T - 1)]))
            xh = x.cpu().numpy(); yh = y.cpu().numpy()
            # what the kernel rounds: the sum of the two bf16 terms of the split image (16 bits), not x itself
            xc = x.cpu(); hi = xc.bfloat16().float(); lo = (xc - hi).bfloat16().float()
            xr = (hi + lo).half().float().numpy()
            for n in ns:
                wr = oracle.to_host_matrix(W[n:n + 1]); wu = oracle.to_host_matrix(W[N + n:N + n + 1]) if epi == ld.LDK_SWIGLU else None
                for t in ts:
                    vals = []
                    for xin in (xh, xr):
                        a = oracle.matvec(wr, xin[t])[0]
                        if wu is not None:
                            a = oracle.silu(a) * oracle.matvec(wu, xin[t])[0]
                        vals.append(a)
                    exact, rounded = vals
                    assert abs(yh[t, n] - exact) <= 2e-3 * max(1.0, abs(exact)), (T, N, t, n, yh[t, n], exact)
                    if T > 64 and t < T - r:
                        assert abs(yh[t, n] - rounded) <= 1e-4 * max(1.0, abs(rounded)), (T, N, t, n, yh[t, n], rounded)
    # values beyond the fp16 range
    T, N, K = 300, 4096, 4096
    W = gen.normal(3, 1, (N, K), std=0.02, device=DEV).bfloat16()
    x = gen.normal(3, 2, (T, K), device=DEV)
    y = torch.zeros(T, N, device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_STORE), dtype=torch.uint8, device=DEV)
    xb = x.clone(); xb[17, 1234] = 7.0e4
    flag.zero_(); ld.ldk_linear_f16(W, xb, y, flag, scratch=scratch); assert int(flag.item()) == 1
    xb[17, 1234] = -6.5e4           # the largest fp16 magnitude is 65504
    flag.zero_(); ld.ldk_linear_f16(W, xb, y, flag, scratch=scratch); assert int(flag.item()) == 0
    Wb = W.clone(); Wb[4000, 4095] = 1.0e5
    flag.zero_(); ld.ldk_linear_f16(Wb, x, y, flag, scratch=scratch); assert int(flag.item()) == 1
    Wh = torch.zeros(N, K, dtype=torch.float16, device=DEV)
    flag.zero_(); ld.ldk_weights_to_f16(Wb, Wh, flag); assert int(flag.item()) == 1
    Wb[4000, 4095] = float("nan")
    flag.zero_(); ld.ldk_linear_f16(Wb, x, y, flag, scratch=scratch); assert int(flag.item()) == 1
    flag.zero_(); ld.ldk_weights_to_f16(Wb, Wh, flag); assert int(flag.item()) == 1
    Wb[4000, 4095] = -65504.0 * 0.75   # bf16 has no 65504; -49128 rounds to a bf16 within range
    flag.zero_(); ld.ldk_weights_to_f16(Wb, Wh, flag); assert int(flag.item()) == 0 and float(Wh[4000, 4095]) == float(Wb[4000, 4095])


def test_linear_fp16_image_13b_shapes_bit_equal():
    """The four layer matrices of the 13B shape at the row count of its batch-64 step (63 decode rows beside a
    2048-row chunk): the fp16 form gives the same bits whether the kernel widens the bf16 weights itself or reads
    the matrix's fp16 image, and differs from the two-term form (so it did run)."""
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    T = 2111
    for N, K, epi in [(15360, 5120, ld.LDK_STORE), (5120, 5120, ld.LDK_ADD), (5120, 13824, ld.LDK_ADD), (13824, 5120, ld.LDK_SWIGLU)]:
        rows = N * (2 if epi == ld.LDK_SWIGLU else 1)
        W = gen.normal(5, N, (rows, K), std=0.02, device=DEV).bfloat16()
        x = gen.normal(5, 7 + K, (T, K), device=DEV)
        y0 = gen.normal(5, 8, (T, N), device=DEV)                 # the residual that LDK_ADD adds to
        scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, epi), dtype=torch.uint8, device=DEV)
        Wh = torch.zeros(rows, K, dtype=torch.float16, device=DEV)
        ld.ldk_weights_to_f16(W, Wh, flag)
        outs = []
        for img in (None, Wh):
            y = y0.clone()
            ld.ldk_linear_f16(W, x, y, flag, epi, scratch=scratch, W_f16=img)
            outs.append(y)
        y2 = y0.clone()
        ld.ldk_linear(W, x, y2, epi, scratch=scratch)
        assert int(flag.item()) == 0
        assert torch.equal(outs[0], outs[1]) and not torch.equal(outs[0], y2), (N, K, epi)
        assert float((outs[0] - y2).abs().max()) <= 2e-3 * max(1.0, float(y2.abs().max()))


@pytest.mark.parametrize("split", [False, True], ids=["whole", "kv-split"])
@pytest.mark.parametrize("window", [0, 40, 200])
@pytest.mark.parametrize("H,Hkv", [(4, 4), (8, 2)])
def test_prefill_attention_fp16_form(H, Hkv, window, split):
    """The form of chunk-prefill attention that the engine's long passes take (ldk_prefill_attention_f16: queries and
    probabilities as one fp16 term, keys and values widened to fp16 exactly): the segments of
    test_prefill_attention_segments, every row against the oracle's single-query attention.  What the form rounds
    is q (2^-12 per element of a 128-term score of a few units: ~1e-3 in the exponent's argument) and p (2^-12):
    bound 1e-3 of the largest output, thirty times the two-term bound and a third of what the cache's own bf16
    rounding of a key moves a score by.  A key or value beyond the fp16 range at a position the walk reads, or a
    query that is, raises the flag; the same values at positions no row sees do not."""
    hd = 128
    segs = [(37, 100), (0, 5), (1000, 300), (255, 1), (16, 32)]
    lens = [p + n for p, n in segs]
    table, pool, _ = _attention_case(31, lens, H, Hkv, hd, "bf16")
    T = sum(n for _, n in segs)
    q = gen.normal(31, 9, (T, H, hd), device=DEV)
    tiles, row_seq, row_pos, r = [], [], [], 0
    for s, (p0, n) in enumerate(segs):
        for off in range(0, n, 128):
            tiles.append([r + off, min(128, n - off), p0 + off, s])
        row_seq += [s] * n; row_pos += list(range(p0, p0 + n)); r += n
    tiles_d = torch.tensor(tiles, dtype=torch.int32, device=DEV)
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    scratch = torch.empty(ld.ldk_prefill_attention_scratch_bytes(), dtype=torch.uint8, device=DEV) if split else None

    def run(qq, pp):
        out = torch.zeros(T, H, hd, device=DEV)
        flag.zero_()
        ld.ldk_prefill_attention_f16(qq, H * hd, device_pool(pp), table.to(DEV), tiles_d, H, Hkv, hd, out, max(row_pos), flag,
                                     window=window, scratch=scratch)
        torch.cuda.synchronize()
        return out.cpu().numpy(), int(flag.item())

    got, f = run(q, pool)
    assert f == 0
    out2 = torch.zeros(T, H, hd, device=DEV)
    ld.ldk_prefill_attention(q, H * hd, device_pool(pool), table.to(DEV), tiles_d, H, Hkv, hd, out2, max(row_pos),
                             window=window, scratch=scratch)
    assert not np.array_equal(got, out2.cpu().numpy())      # the single-term form did run
    ph = oracle.to_host_matrix(pool.reshape(pool.shape[0], -1)).reshape(-1)
    ref = oracle.paged_attention(q.cpu().numpy(), ph, ph[Hkv * 16 * hd:], (2 * Hkv * 16 * hd, 16 * hd, hd),
                                 table.numpy()[row_seq], [p + 1 for p in row_pos], Hkv, window=window)
    err = np.max(np.abs(got - ref), axis=(1, 2)) / np.abs(ref).max()
    assert 3e-5 < err.max() <= 1e-3, (err.max(), int(err.argmax()), row_pos[int(err.argmax())])
    # out of range: the key of position 1100 of the third sequence (seen by its rows from 1100 on, inside every band)
    blk, slot = int(table[2, 1100 // 16]), 1100 % 16
    big = pool.clone(); big[blk, 0, Hkv - 1, slot, 5] = 7.0e4
    assert run(q, big)[1] == 1
    big = pool.clone(); big[blk, 1, 0, slot, 77] = -1.0e5
    assert run(q, big)[1] == 1
    # the last block of the second sequence (5 positions): slots 5..15 were never written and no row reads them as values;
    # its keys there are read and masked, so a key counts, a value slot beyond the tile is zeroed before it is looked at
    qb = q.clone(); qb[3, 1, 9] = 1.0e6
    assert run(qb, pool)[1] == 1


@pytest.mark.parametrize("what", [float("nan"), float("inf"), -float("inf"), 65536.0, 65280.0])
@pytest.mark.parametrize("part", [0, 1], ids=["key", "value"])
@pytest.mark.parametrize("pos", [0, 63, 64, 127, 190])
def test_prefill_attention_fp16_range_check(what, part, pos):
    """What raises the flag of the fp16 form: a NaN, an infinity or 65536 (the first magnitude fp16 cannot hold) in a key or a value
    that a row sees, in units that lie below the last position and in the last one, also beside the first and last position of a
    unit of 64; 65280, the largest bf16 number that fp16 holds, does not."""
    H, hd, lens = 2, 128, [191]
    table, pool, _ = _attention_case(53, lens, H, H, hd, "bf16")
    q = gen.normal(53, 9, (40, H, hd), device=DEV)
    tiles = torch.tensor([[0, 40, 151, 0]], dtype=torch.int32, device=DEV)
    pool = pool.clone()
    pool[int(table[0, pos // 16]), part, 1, pos % 16, 17] = what
    flag, out = torch.zeros(1, dtype=torch.int32, device=DEV), torch.zeros(40, H, hd, device=DEV)
    ld.ldk_prefill_attention_f16(q, H * hd, device_pool(pool), table.to(DEV), tiles, H, H, hd, out, 190, flag)
    assert int(flag.item()) == (what != 65280.0)


@pytest.mark.parametrize("what", [float("nan"), float("inf"), -65536.0])
@pytest.mark.parametrize("part", [0, 1], ids=["key", "value"])
@pytest.mark.parametrize("window,touched", [(61, range(96, 111)), (55, range(112, 117)), (33, range(128, 139))])
def test_prefill_attention_fp16_range_check_below_the_band(what, part, window, touched):
    """The flag of the fp16 form counts every position that the walk touches, also those below the band of every row: the walk
    starts at a multiple of 32, or at the first block the band still holds.  A value that the flag names raises it at each
    of them, one in the position before them does not."""
    H, hd, lens = 2, 128, [191]
    table, clean, _ = _attention_case(53, lens, H, H, hd, "bf16")
    q = gen.normal(53, 9, (20, H, hd), device=DEV)
    tiles = torch.tensor([[0, 20, 171, 0]], dtype=torch.int32, device=DEV)
    assert 171 - window + 1 == touched.stop
    for pos in (touched.start - 1, *touched):
        pool = clean.clone()
        pool[int(table[0, pos // 16]), part, 1, pos % 16, 17] = what
        flag, out = torch.zeros(1, dtype=torch.int32, device=DEV), torch.zeros(20, H, hd, device=DEV)
        ld.ldk_prefill_attention_f16(q, H * hd, device_pool(pool), table.to(DEV), tiles, H, H, hd, out, 190, flag, window=window)
        assert int(flag.item()) == (pos in touched), pos


@pytest.mark.parametrize("N,K,epi,norm", [(N, K, epi, norm) for epi in ("store", "add", "swiglu") for norm in (False, True) for N, K in [
    (1, 8), (2, 2040), (3, 2048), (513, 2056), (1025, 6152), (1537, 8192), (770, 8200), (1026, 16384), (4099, 2056), (4099, 8200), (2050, 16384), (16391, 1032)]] + [(140000, 16384, "store", False)])
def test_gemv_slab_edges(N, K, epi, norm):
    """The one-row product at the edges of its slabs of 2048 and 512 columns (the latter where a wave gets few items), of the two sizes its input has in LDS (8192 columns and
    16384), of the two-row items (odd and single rows, fewer outputs than workgroups, one more than two each) and beyond the
    partial sums that one workgroup per slot can hold, against float64.  Bound: a sum passes through at most 4 x 8 additions in a lane,
    6 across the wave and 8 over the slabs, so 64 roundings of 2^-24 of the sum of magnitudes cover it with the norm's."""
    e = {"store": ld.LDK_STORE, "add": ld.LDK_ADD, "swiglu": ld.LDK_SWIGLU}[epi]
    rows = N * (2 if epi == "swiglu" else 1)
    torch.manual_seed(N * 31 + K)
    W = torch.empty(rows, K, dtype=torch.bfloat16, device=DEV).normal_(0, 0.05)
    x, g = torch.randn(1, K, device=DEV), 1 + 0.1 * torch.randn(K, device=DEV)
    y0 = torch.randn(1, N, device=DEV)
    y = y0.clone()
    scratch = torch.empty(max(1, ld.ldk_linear_scratch_bytes(1, N, K, e)), dtype=torch.uint8, device=DEV)
    ld.ldk_linear(W, x, y, e, g if norm else None, 1e-5, scratch)
    xd = x[0].double()
    if norm:
        xd = xd * g.double() / torch.sqrt((xd * xd).mean() + 1e-5)
    s, mag = torch.empty(rows, dtype=torch.float64, device=DEV), torch.empty(rows, dtype=torch.float64, device=DEV)
    for r in range(0, rows, 20000):
        w = W[r:r + 20000].double()
        s[r:r + 20000], mag[r:r + 20000] = (w * xd).sum(1), (w * xd).abs().sum(1)
    tol = 64 * 2.0 ** -24 * mag
    if epi == "store":
        ref = s
    elif epi == "add":
        ref, tol = y0[0].double() + s, tol + 2.0 ** -23 * (y0[0].double().abs() + s.abs())
    else:      # |silu'| <= 1.1, |silu(a)| <= |a|; the exponential is good to some 2^-20 of the result
        a, b = s[:N], s[N:]
        ref = a * torch.sigmoid(a) * b
        tol = 1.1 * tol[:N] * (b.abs() + tol[N:]) + a.abs() * tol[N:] + 2.0 ** -20 * (a * b).abs()
    assert bool(((y[0].double() - ref).abs() <= tol).all()), float(((y[0].double() - ref).abs() / tol).max())


@pytest.mark.parametrize("shares", [1, 2, 16])
@pytest.mark.parametrize("window", [0, 333])
@pytest.mark.parametrize("H,Hkv,many", [(3, 3, False), (16, 4, False), (2, 1, True)])
def test_prefill_attention_uneven_tiles(H, Hkv, many, window, shares):
    """Tiles of 1, 32, 33, 64, 65 and 128 rows behind contexts of very different length (walks of 1 to 99 steps, even and odd), so that a
    short tile has fewer shares than a long one and the last share of each is cut; head counts that do and don't divide into
    the eight chip dies; more tiles than a wave has lanes (which then keep their own order); scratch for one, two and all shares,
    and a max_pos beyond every row.  Both forms against the oracle, with the bounds of the two tests around this one."""
    hd = 128
    segs = [(31 * i % 97, 1 + 5 * i % 40) for i in range(70)] if many else [(3000, 129), (17, 64), (700, 33), (0, 1), (1503, 32), (1000, 65)]
    table, pool, _ = _attention_case(35, [p + n for p, n in segs], H, Hkv, hd, "bf16")
    T = sum(n for _, n in segs)
    q = gen.normal(35, 9, (T, H, hd), device=DEV)
    tiles, row_seq, row_pos, r = [], [], [], 0
    for s, (p0, n) in enumerate(segs):
        for off in range(0, n, 128):
            tiles.append([r + off, min(128, n - off), p0 + off, s])
        row_seq += [s] * n; row_pos += list(range(p0, p0 + n)); r += n
    tiles_d, flag = torch.tensor(tiles, dtype=torch.int32, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    size = min(shares * len(tiles) * H * 128 * (hd + 2) * 4, ld.ldk_prefill_attention_scratch_bytes())
    scratch = torch.empty(size, dtype=torch.uint8, device=DEV) if shares > 1 else None
    out, out16 = torch.zeros(T, H, hd, device=DEV), torch.zeros(T, H, hd, device=DEV)
    args = (H * hd, device_pool(pool), table.to(DEV), tiles_d, H, Hkv, hd)
    ld.ldk_prefill_attention(q, *args, out, max(row_pos) + 500 * (shares - 1), window=window, scratch=scratch)
    ld.ldk_prefill_attention_f16(q, *args, out16, max(row_pos), flag, window=window, scratch=scratch)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    ph = oracle.to_host_matrix(pool.reshape(pool.shape[0], -1)).reshape(-1)
    ref = oracle.paged_attention(q.cpu().numpy(), ph, ph[Hkv * 16 * hd:], (2 * Hkv * 16 * hd, 16 * hd, hd),
                                 table.numpy()[row_seq], [p + 1 for p in row_pos], Hkv, window=window)
    for got, bound in ((out, 3e-5), (out16, 1e-3)):
        err = np.max(np.abs(got.cpu().numpy() - ref), axis=(1, 2)) / np.abs(ref).max()
        assert err.max() <= bound, (err.max(), int(err.argmax()), row_pos[int(err.argmax())])


@pytest.mark.parametrize("window", [0, 300])
@pytest.mark.parametrize("rows", [7, 200])
@pytest.mark.parametrize("growth", [-0.03, 0.01, 0.03])
def test_prefill_attention_moving_maximum(growth, rows, window):
    """Scores that fall or rise along the walk, by up to 50 in the exponent, so that the reference of the exponentials stays where the first
    positions put it, is moved now and then, differently in each row and half of a wave.  Both forms against float64 on the operands as
    they round them (tiles of up to 16 rows take two terms in both), bound beside it; a wrong rescaling lies far
    outside (test_moving_maximum_bound_sees_wrong_rescaling)."""
    hd, H, ctx = 128, MOVING_HEADS, MOVING_CTX
    table, pool, _ = _attention_case(67, [ctx + rows], H, H, hd, "bf16")
    q, k, v = moving_maximum_inputs(growth, rows, DEV)
    pos = torch.arange(ctx + rows)
    for part, x in ((0, k), (1, v)):
        pool[table[0, pos // 16].long().to(DEV), part, :, (pos % 16).to(DEV), :] = x
    tiles = [[off, min(128, rows - off), ctx + off, 0] for off in range(0, rows, 128)]
    tiles_d, flag = torch.tensor(tiles, dtype=torch.int32, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    out, out16 = torch.zeros(rows, H, hd, device=DEV), torch.zeros(rows, H, hd, device=DEV)
    args = (H * hd, device_pool(pool), table.to(DEV), tiles_d, H, H, hd)
    ld.ldk_prefill_attention(q, *args, out, ctx + rows - 1, window=window)
    ld.ldk_prefill_attention_f16(q, *args, out16, ctx + rows - 1, flag, window=window)
    assert int(flag.item()) == 0
    for got, form in ((out, "two"), (out16, "f16" if rows > 16 else "two")):
        ref, bound = attention_and_bound(q, k, v, ctx, window, form)
        assert ((got.double() - ref).abs() <= bound).all(), (form, float(((got.double() - ref).abs() / bound).max()))


@pytest.mark.parametrize("split", [False, True], ids=["whole", "kv-split"])
@pytest.mark.parametrize("window", [0, 1, 50, 4500])
@pytest.mark.parametrize("H,Hkv", [(3, 3), (8, 1)])
def test_prefill_attention_few_rows(H, Hkv, window, split):
    """Tiles of up to 16 rows, whose waves walk every fourth step of a share by themselves, and the first beyond them: 1, 2, 15, 16 and 17
    rows alone and behind a full tile; last positions just before, at and behind a block's and a step's end; walks of fewer steps
    than waves and, at 4200 and 8300 positions, of more than the 32 that a wave looks up at a time.  What was never written
    is NaN.  Both forms against the oracle: the tiles of up to 16 rows take two terms in both, so the bound of the two-term form holds for them."""
    hd = 128
    segs = [(0, 1), (14, 1), (15, 2), (30, 1), (31, 15), (97, 15), (112, 16), (113, 16), (90, 17), (0, 16), (200, 129), (75, 144), (60, 145), (4200, 16), (8300, 3)]
    lens = [p + n for p, n in segs]
    table, pool, _ = _attention_case(61, lens, H, Hkv, hd, "bf16")
    T = sum(n for _, n in segs)
    q = gen.normal(61, 9, (T, H, hd), device=DEV)
    tiles, row_seq, row_pos, few, r = [], [], [], [], 0
    for s, (p0, n) in enumerate(segs):
        for off in range(0, n, 128):
            tiles.append([r + off, min(128, n - off), p0 + off, s])
            few += [tiles[-1][1] <= 16] * tiles[-1][1]
        row_seq += [s] * n; row_pos += list(range(p0, p0 + n)); r += n
    tiles_d, flag = torch.tensor(tiles, dtype=torch.int32, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)
    scratch = torch.empty(ld.ldk_prefill_attention_scratch_bytes(), dtype=torch.uint8, device=DEV) if split else None
    out, out16 = torch.zeros(T, H, hd, device=DEV), torch.zeros(T, H, hd, device=DEV)
    args = (H * hd, device_pool(pool), table.to(DEV), tiles_d, H, Hkv, hd)
    ld.ldk_prefill_attention(q, *args, out, max(row_pos), window=window, scratch=scratch)
    ld.ldk_prefill_attention_f16(q, *args, out16, max(row_pos), flag, window=window, scratch=scratch)
    assert int(flag.item()) == 0
    ph = oracle.to_host_matrix(pool.reshape(pool.shape[0], -1)).reshape(-1)
    ref = oracle.paged_attention(q.cpu().numpy(), ph, ph[Hkv * 16 * hd:], (2 * Hkv * 16 * hd, 16 * hd, hd),
                                 table.numpy()[row_seq], [p + 1 for p in row_pos], Hkv, window=window)
    for got, bound in ((out, 3e-5), (out16, np.where(few, 3e-5, 1e-3))):
        err = np.max(np.abs(got.cpu().numpy() - ref), axis=(1, 2)) / np.abs(ref).max()
        assert np.all(err <= bound), (err.max(), int(err.argmax()), row_pos[int(err.argmax())])


@pytest.mark.parametrize("what", [float("nan"), -float("inf"), 65536.0, 65280.0])
@pytest.mark.parametrize("part", [0, 1], ids=["key", "value"])
@pytest.mark.parametrize("pos", [95, 96, 111, 127, 128, 157, 171, 172, 175])
def test_prefill_attention_few_rows_fp16_range_check(what, part, pos):
    """The flag of the fp16 form in a tile of 11 rows at 161 .. 171 with a band of 61: raised by what the walk touches, from the first
    block that the band holds (position 96) to the last row's position, as in the larger tiles; not by the rest of the last block."""
    H, hd, lens = 2, 128, [172]
    table, pool, _ = _attention_case(53, lens, H, H, hd, "bf16")
    q = gen.normal(53, 9, (11, H, hd), device=DEV)
    tiles = torch.tensor([[0, 11, 161, 0]], dtype=torch.int32, device=DEV)
    pool = pool.clone()
    pool[int(table[0, pos // 16]), part, 1, pos % 16, 17] = what
    flag, out = torch.zeros(1, dtype=torch.int32, device=DEV), torch.zeros(11, H, hd, device=DEV)
    ld.ldk_prefill_attention_f16(q, H * hd, device_pool(pool), table.to(DEV), tiles, H, H, hd, out, 171, flag, window=61)
    assert int(flag.item()) == (what != 65280.0 and 96 <= pos <= 171)


def test_calls_without_a_stream_run_on_the_current_one():
    """The stream of a call that names none: torch's current stream of the calling thread, also inside a stream context and a capture."""
    import threading
    same = lambda: binding._stream(None) == torch.cuda.current_stream().cuda_stream
    assert same()
    s = torch.cuda.Stream()
    seen = []
    with torch.cuda.stream(s):
        assert same() and binding._stream(None) == s.cuda_stream
        t = threading.Thread(target=lambda: seen.append(same() and binding._stream(None) != s.cuda_stream)); t.start(); t.join()
    assert same() and seen == [True]
    x, y = torch.ones(64, device=DEV), torch.zeros(64, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=s):
        y.copy_(x)
        assert same() and binding._stream(None) == s.cuda_stream


@pytest.mark.parametrize("split", [False, True], ids=["whole", "kv-split"])
@pytest.mark.parametrize("window", [0, 1, 40, 128, 200, 5000])
@pytest.mark.parametrize("H,Hkv", [(4, 4), (8, 2)])
def test_prefill_attention_segments(H, Hkv, window, split):
    """Chunk-prefill attention (matrix cores): segments of different sequences, a fresh prompt (position 0),
    an observation appended to a long context, a segment longer than one 128-row tile; causal inside
    the chunk; permuted block table; with and without an attention band (shorter than a wave's 32 rows,
    shorter and longer than a tile, longer than every context).  Every row against the oracle's
    single-query attention.  With scratch the KV range of a tile is split over several workgroups and merged
    (some shares are empty or wholly masked for some rows); without it every tile walks its whole range."""
    hd = 128
    segs = [(37, 100), (0, 5), (1000, 300), (255, 1), (16, 32)]          # (first position, rows) per sequence
    lens = [p + n for p, n in segs]
    table, pool, _ = _attention_case(31, lens, H, Hkv, hd, "bf16")
    T = sum(n for _, n in segs)
    q = gen.normal(31, 9, (T, H, hd), device=DEV)
    tiles, row_seq, row_pos, r = [], [], [], 0
    for s, (p0, n) in enumerate(segs):
        for off in range(0, n, 128):
            tiles.append([r + off, min(128, n - off), p0 + off, s])
        row_seq += [s] * n; row_pos += list(range(p0, p0 + n)); r += n
    out = torch.zeros(T, H, hd, device=DEV)
    scratch = torch.empty(ld.ldk_prefill_attention_scratch_bytes(), dtype=torch.uint8, device=DEV) if split else None
    ld.ldk_prefill_attention(q, H * hd, device_pool(pool), table.to(DEV), torch.tensor(tiles, dtype=torch.int32, device=DEV),
                             H, Hkv, hd, out, max(row_pos), window=window, scratch=scratch)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    ph = oracle.to_host_matrix(pool.reshape(pool.shape[0], -1)).reshape(-1)
    ref = oracle.paged_attention(q.cpu().numpy(), ph, ph[Hkv * 16 * hd:], (2 * Hkv * 16 * hd, 16 * hd, hd),
                                 table.numpy()[row_seq], [p + 1 for p in row_pos], Hkv, window=window)
    err = np.max(np.abs(got - ref), axis=(1, 2)) / np.abs(ref).max()
    assert err.max() <= 3e-5, (err.max(), int(err.argmax()), row_pos[int(err.argmax())])


@pytest.mark.parametrize("f16", [False, True], ids=["two-term", "fp16"])
@pytest.mark.parametrize("window", [1, 5, 13])
def test_prefill_attention_band_inside_the_last_block(window, f16):
    """Bands of fewer than 16 positions over tiles whose first visible block is also the last, partly written one and lies in the
    upper half of a 32-position step: the lower half of the step then has no block of its own and reads that one, whose
    unwritten slots hold NaN.  They neither reach an output nor count as beyond the fp16 range.  Bounds as in the tests above
    (two terms 3e-5, one fp16 term 1e-3 of the largest output)."""
    hd, H, Hkv = 128, 4, 2
    segs = [(1300, 1), (1300, 3), (16, 1), (20, 2), (1317, 1), (1310, 2), (55, 9)]
    table, pool, _ = _attention_case(37, [p + n for p, n in segs], H, Hkv, hd, "bf16")
    tiles, row_seq, row_pos = [], [], []
    for s, (p0, n) in enumerate(segs):
        tiles.append([len(row_pos), n, p0, s])
        row_seq += [s] * n; row_pos += list(range(p0, p0 + n))
    q = gen.normal(37, 9, (len(row_pos), H, hd), device=DEV)
    out, flag = torch.zeros_like(q), torch.zeros(1, dtype=torch.int32, device=DEV)
    args = (q, H * hd, device_pool(pool), table.to(DEV), torch.tensor(tiles, dtype=torch.int32, device=DEV), H, Hkv, hd, out, max(row_pos))
    if f16:
        ld.ldk_prefill_attention_f16(*args, flag, window=window)
    else:
        ld.ldk_prefill_attention(*args, window=window)
    got = out.cpu().numpy()
    ph = oracle.to_host_matrix(pool.reshape(pool.shape[0], -1)).reshape(-1)
    ref = oracle.paged_attention(q.cpu().numpy(), ph, ph[Hkv * 16 * hd:], (2 * Hkv * 16 * hd, 16 * hd, hd),
                                 table.numpy()[row_seq], [p + 1 for p in row_pos], Hkv, window=window)
    assert int(flag.item()) == 0
    err = np.max(np.abs(got - ref), axis=(1, 2)) / np.abs(ref).max()
    assert err.max() <= (1e-3 if f16 else 3e-5), (err.max(), row_pos[int(err.argmax())])


@pytest.mark.parametrize("T,N,K,epi", [(1056, 14336, 4096, "swiglu"), (2111, 4096, 4096, "add"), (1537, 5120, 5120, "store")])
def test_linear_f16_tail_keeps_both_terms(T, N, K, epi):
    """Decode rows behind whole 256-row tiles in the one-term form, at shapes where they keep both terms: every output of theirs
    within 2^-16 sum_k |w x| of float64 (two terms leave 2^-18 of an activation, the rest is float32 sums), which one fp16
    term (2^-12 of an activation) does not meet; the rows in front do show that term."""
    e = {"store": ld.LDK_STORE, "add": ld.LDK_ADD, "swiglu": ld.LDK_SWIGLU}[epi]
    rows = N * (2 if epi == "swiglu" else 1)
    W = gen.normal(43, 1, (rows, K), std=0.02, device=DEV).bfloat16()
    x, y0 = gen.normal(43, 2, (T, K), device=DEV), gen.normal(43, 3, (T, N), device=DEV)
    y, flag = y0.clone(), torch.zeros(1, dtype=torch.int32, device=DEV)
    scratch = torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, e), dtype=torch.uint8, device=DEV)
    ld.ldk_linear_f16(W, x, y, flag, e, scratch=scratch)
    assert int(flag.item()) == 0

    def worst(sel):
        xs, w = x[sel].double(), W.double()
        s, mag = xs @ w.t(), xs.abs() @ w.abs().t()
        if epi == "swiglu":      # |d(silu(a) b)| <= 1.1 |b| |da| + |silu(a)| |db|
            a, b = s[:, :N], s[:, N:]
            ref, mag = torch.nn.functional.silu(a) * b, 1.1 * b.abs() * mag[:, :N] + torch.nn.functional.silu(a).abs() * mag[:, N:]
        else:
            ref = s + (y0[sel].double() if epi == "add" else 0)
        return float((((y[sel].double() - ref).abs() - 1e-6 * ref.abs()).clamp_min(0) / mag).max())

    last = T // 256 * 256
    assert worst(slice(last, T)) <= 2.0 ** -16
    assert worst(slice(last - 64, last)) > 2.0 ** -16


@pytest.mark.parametrize("n_tiles", [65535, 65536, 65600])
def test_prefill_attention_more_tiles_than_a_grid_dimension(n_tiles):
    """As many one-row tiles as a grid's second dimension holds, and more (they go in two launches), over three cached
    sequences: every tile's row equals the row that one tile of the same position and sequence gives alone, bit for bit."""
    hd, lens = 128, [40, 7, 300]
    table, pool, _ = _attention_case(41, lens, 1, 1, hd, "bf16")
    i = torch.arange(n_tiles)
    seq = i % 3
    pos = (i * 7) % torch.tensor(lens)[seq]
    tiles = torch.stack([i, torch.ones_like(i), pos, seq], 1).int().to(DEV)
    q = gen.normal(41, 9, (1, 1, hd), device=DEV).expand(n_tiles, 1, hd).contiguous()
    out = torch.full((n_tiles, 1, hd), float("nan"), device=DEV)
    args = (device_pool(pool), table.to(DEV))
    ld.ldk_prefill_attention(q, hd, *args, tiles, 1, 1, hd, out, max(lens) - 1)
    kinds, back = torch.unique(torch.stack([pos, seq], 1), dim=0, return_inverse=True)
    few = torch.stack([torch.arange(len(kinds)), torch.ones(len(kinds)), kinds[:, 0], kinds[:, 1]], 1).int().to(DEV)
    ref = torch.full((len(kinds), 1, hd), float("nan"), device=DEV)
    for k in range(0, len(kinds), 50):
        ld.ldk_prefill_attention(q, hd, *args, few[k:k + 50].contiguous(), 1, 1, hd, ref, max(lens) - 1)
    assert torch.isfinite(out).all() and torch.equal(out, ref[back.to(DEV)])


def test_linear_rows_too_long_for_32_bit_offsets():
    """Matrix rows so long that 255 of them lie more than 4 GiB apart, at a row count that would take the big-tile kernel: first and
    last outputs against float64 (bound as in test_linear_small_batch_edges; a lane adds some 2^14 terms, the slabs' sums 2^13)."""
    T, N, K = 65, 256, (1 << 32) // 510 // 128 * 128 + 128
    torch.manual_seed(5)
    W = torch.empty(N, K, dtype=torch.bfloat16, device=DEV).normal_(0, 0.02)
    x, y = torch.randn(T, K, device=DEV), torch.full((T, N), float("nan"), device=DEV)
    ld.ldk_linear(W, x, y, ld.LDK_STORE, scratch=torch.empty(ld.ldk_linear_scratch_bytes(T, N, K, ld.LDK_STORE), dtype=torch.uint8, device=DEV))
    for n in (0, 1, 128, 254, 255):
        w = W[n].double()
        for t in (0, 31, 63, 64):
            p = x[t].double() * w
            assert abs(float(y[t, n].double() - p.sum())) <= 2.0 ** -16 * float(p.abs().sum()), (t, n)
