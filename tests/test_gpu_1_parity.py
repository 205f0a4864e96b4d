"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle on the same
seeded inputs.  Index work (slots, gathers) must be bit-exact; floating point within the
stated tolerances.  Needs a real MI355X: run with -m gpu."""
import math
import time

import numpy as np
import pytest
import torch

import chiron_oracle as orc
from helpers import as_f64, bf16_to_f32, bits, fresh_pool, gpu_setup, make_case
from test_launch_shapes import ALONE, STEP, shape
from paper_2501_08090_amd import inputs as I

pytestmark = pytest.mark.gpu

# bf16 weights/cache are identical on both sides and activations enter the matrix cores as two
# bf16 terms (relative error 2^-17 per term), so a single kernel differs from the fp32/double
# oracle by ~1e-5 of the output scale; 1e-4 leaves an order of magnitude.
KERNEL_TOL = 1e-4
# whole step: the bar is max|dlogit| <= 2e-2 * std(oracle logits) and argmax agreement >= 99% of rows
STEP_TOL = 2e-2


def B():
    from paper_2501_08090_amd import binding
    return binding


def rel_err(got, want):
    return float(np.abs(got - want).max() / (want.std() + 1e-30))


# ---- slots: append / gather are pure index work, bit-exact ---------------------------------------

@pytest.mark.parametrize("m,kind,batch", [(I.TINY, "tiny", 4), (dict(I.TINY, head_dim=128, n_kv_heads=2, n_q_heads=8), "tiny", 3)])
def test_append_gather_bit_exact(m, kind, batch):
    c = make_case(m=m, batch=batch, kind=kind, seed=11, storage="bf16")
    g = gpu_setup(c, poison=True)
    opool = fresh_pool(c)
    o = 0
    for i, L in enumerate(c.seq_lens):
        L = int(L)
        for l in range(m["n_layers"]):
            print("gather seq", i, "layer", l, "len", L, flush=True)
            k, v = g.pool.gather(l, g.block_table[i].contiguous(), L)
            ok, ov = orc.gather_kv(opool, l, c.block_table[i], L)
            assert np.array_equal(bits(k), ok) and np.array_equal(bits(v), ov)
            assert np.array_equal(bits(k), c.kv[l][0][o:o + L])
        # slots of the sequence's pages that were never written still hold the fill pattern
        npages = int(I.pages_needed([L])[0])
        k, v = g.pool.gather(0, g.block_table[i].contiguous(), npages * 16)
        assert np.all(bits(k)[L:] == 0x7FC0) and np.all(bits(v)[L:] == 0x7FC0)
        o += L


@pytest.mark.parametrize("mb", [0, 4.5])
@pytest.mark.parametrize("d,nkv", [(64, 1), (128, 8), (64, 3)])
@pytest.mark.parametrize("order", ["in order", "offset runs", "shuffled", "unaligned"])
def test_append_gather_any_order_and_alignment(d, nkv, order, mb):
    """Runs of four positions that start anywhere in the input, tokens without such a run, tokens in any order, and
    rows that are not 16-byte aligned: every value lands in its slot and nowhere else.  A few tokens (element-wise kernels), and
    with a request of 4.5 MB beside them (16 bytes a lane where rows are aligned)."""
    lens = [1, 7, 16, 35] + ([int(mb * 2 ** 20) // (4 * nkv * d) + 3] if mb else [])
    c = make_case(m=dict(I.TINY, n_layers=1, head_dim=d, n_kv_heads=nkv, n_q_heads=nkv, vocab=64, ffn=16), seed=15, storage="bf16", seq_lens=lens)
    g = gpu_setup(c)
    g.pool.memory.view(torch.int16).fill_(0x7FC0)
    idx = np.arange(sum(lens))
    if order == "offset runs":
        idx = np.concatenate([idx[1:], idx[:1]])[:-2]  # two positions stay unwritten
    elif order == "shuffled":
        idx = np.random.default_rng(5).permutation(idx)
    k, v = c.kv_t[0]
    at = torch.from_numpy(idx)
    kk, vv = k[at].cuda().contiguous(), v[at].cuda().contiguous()
    if order == "unaligned":
        kk, vv = (torch.cat([x.new_zeros(1), x.reshape(-1)])[1:].view(x.shape) for x in (kk, vv))
        assert kk.data_ptr() % 16 and kk.is_contiguous()
    print("append", d, nkv, order, flush=True)
    g.pool.append(0, kk, vv, g.block_table, torch.from_numpy(c.seq_idx[idx]).cuda(), torch.from_numpy(c.pos[idx]).cuda())
    wk, wv = np.full(k.shape, 0x7FC0, np.uint16), np.full(k.shape, 0x7FC0, np.uint16)
    wk[idx], wv[idx] = bits(k)[idx], bits(v)[idx]
    o = 0
    for i, L in enumerate(lens):
        n = int(I.pages_needed([L])[0]) * 16
        gk, gv = g.pool.gather(0, g.block_table[i].contiguous(), n)
        assert np.array_equal(bits(gk)[:L], wk[o:o + L]) and np.array_equal(bits(gv)[:L], wv[o:o + L])
        assert np.all(bits(gk)[L:] == 0x7FC0) and np.all(bits(gv)[L:] == 0x7FC0)
        b = B()
        uk, uv = (torch.zeros(L * nkv * d + 3, dtype=torch.bfloat16, device="cuda")[1:1 + L * nkv * d] for _ in range(2))
        b._check(b.load().chiron_gather_kv(g.pool._h, 0, b._ptr(g.block_table[i].contiguous()), L, b._ptr(uk), b._ptr(uv), b._stream()))
        assert np.array_equal(bits(uk).reshape(L, nkv, d), wk[o:o + L]) and np.array_equal(bits(uv).reshape(L, nkv, d), wv[o:o + L])
        o += L


def test_append_overwrites_only_its_slot():
    c = make_case(batch=3, seed=12, storage="bf16")
    g = gpu_setup(c)
    before = [[g.pool.gather(l, g.block_table[i].contiguous(), int(c.seq_lens[i])) for i in range(3)] for l in range(2)]
    nkv, d = c.m["n_kv_heads"], c.m["head_dim"]
    newk = I.normal((1, nkv, d), 1.0, 99, "newk").cuda()
    newv = I.normal((1, nkv, d), 1.0, 99, "newv").cuda()
    tgt_seq, tgt_pos = 1, int(c.seq_lens[1]) // 2
    g.pool.append(1, newk, newv, g.block_table, torch.tensor([tgt_seq], dtype=torch.int32, device="cuda"),
                  torch.tensor([tgt_pos], dtype=torch.int32, device="cuda"))
    for l in range(2):
        for i in range(3):
            k, v = g.pool.gather(l, g.block_table[i].contiguous(), int(c.seq_lens[i]))
            bk, bv = bits(before[l][i][0]).copy(), bits(before[l][i][1]).copy()
            if l == 1 and i == tgt_seq:
                bk[tgt_pos] = bits(newk)[0]
                bv[tgt_pos] = bits(newv)[0]
            assert np.array_equal(bits(k), bk) and np.array_equal(bits(v), bv)


@pytest.mark.parametrize("where", ["device", "pinned_host"])
def test_swap_out_in_relocates_a_request_bit_exactly(where):
    """Eviction to (host) memory and restore into other pages: gathers are bit-identical to the oracle's after the
    same migration, and the decode step's logits do not change by a single bit (page placement never matters)."""
    c = make_case(batch=4, seed=15, storage="bf16", pool_factor=3.0)
    g = gpu_setup(c)
    opool = fresh_pool(c)
    before = B().decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens).clone()
    # the step wrote position L of every request: rebuild the cache so that both sides hold the pre-step state
    g = gpu_setup(c)
    i = 3
    L = int(c.seq_lens[i]); npg = int(I.pages_needed([L])[0])
    nbytes = npg * g.model.kv_block_bytes()
    image = (torch.empty(nbytes, dtype=torch.uint8, device="cuda") if where == "device"
             else torch.empty(nbytes, dtype=torch.uint8, pin_memory=True))
    row = g.block_table[i].contiguous()
    g.pool.swap_out(row, npg, image)
    torch.cuda.synchronize()
    oimage = orc.swap(opool, c.block_table[i], npg)
    used = set(c.block_table[c.block_table >= 0].tolist())
    free = [b for b in range(c.num_blocks) if b not in used][:npg]
    new_row = np.full_like(c.block_table[i], -1); new_row[:npg] = free[::-1]
    # poison the old pages on the GPU (through the public append), then restore elsewhere
    nkv, d = c.m["n_kv_heads"], c.m["head_dim"]
    junk = torch.full((L, nkv, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    for l in range(c.m["n_layers"]):
        g.pool.append(l, junk, junk, g.block_table, torch.full((L,), i, dtype=torch.int32, device="cuda"),
                      torch.arange(L, dtype=torch.int32, device="cuda"))
    new_row_d = torch.from_numpy(new_row).cuda()
    g.pool.swap_in(new_row_d, npg, image)
    orc.swap(opool, new_row, npg, oimage)
    for l in range(c.m["n_layers"]):
        k, v = g.pool.gather(l, new_row_d, L)
        ok, ov = orc.gather_kv(opool, l, new_row, L)
        assert np.array_equal(bits(k), ok) and np.array_equal(bits(v), ov)
    bt2 = g.block_table.clone(); bt2[i] = new_row_d
    after = B().decode_step(g.model, g.pool, bt2, g.seq_lens, g.tokens)
    assert torch.equal(after, before)
    assert B().load().chiron_kv_swap_out(g.pool._h, None, 1, None, None) == -1


# ---- single kernels -------------------------------------------------------------------------------

@pytest.mark.parametrize("rows,n", [(1, 256), (5, 4096), (3, 8192), (2, 688)])
def test_rmsnorm(rows, n):
    rng = np.random.default_rng(rows * 1000 + n)
    h = (rng.standard_normal((rows, n)) * 3).astype(np.float32)
    gain = I.normal((n,), 0.3, 5, "gain", n, mean=1.0)
    got = B().op_rmsnorm(torch.from_numpy(h).cuda(), gain.cuda(), 1e-5).cpu().numpy()
    want = np.stack([orc.rmsnorm(h[r], I.to_numpy_storage(gain), 1e-5) for r in range(rows)])
    assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()


@pytest.mark.parametrize("M,N,K", [(1, 256, 256), (4, 512, 256), (4, 1376, 256), (4, 256, 688), (33, 96, 1040),
                                   (64, 1024, 4096), (100, 160, 512), (130, 4096, 1024), (7, 1000, 64),
                                   (400, 8192, 512), (385, 2080, 256), (70, 512, 256), (96, 1376, 4096), (65, 4096, 512),
                                   (150, 1376, 256), (270, 4096, 512), (300, 28672, 256),
                                   # wide unsliced outputs of up to 32 rows take the 16-step weight ring (256-wide chunks):
                                   # one chunk, several chunks, a ragged last chunk
                                   (8, 20000, 256), (1, 17000, 1040), (32, 16416, 784), (17, 28672, 2048)])
def test_linear(M, N, K):
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    W = I.normal((N, K), 0.05, 6, "w", N, K)
    print("linear", M, N, K, flush=True)
    lin = B().Linear(W.cuda())
    xg = torch.from_numpy(x).cuda()
    got = lin(xg).cpu().numpy()
    want = orc.linear(x, I.to_numpy_storage(W))
    assert rel_err(got, want) <= KERNEL_TOL
    # residual form: y += x W^T
    y0 = rng.standard_normal((M, N)).astype(np.float32)
    got2 = lin(xg, torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy()
    assert rel_err(got2, want + y0) <= KERNEL_TOL
    lin.close()


@pytest.mark.parametrize("M,N,K", [(3, 1, 16), (1, 17, 16), (16, 17, 256), (15, 33, 2032), (7, 48, 2304), (16, 64, 4112), (2, 8192, 272), (16, 8209, 48), (3, 100, 2048)])
def test_linear_few_rows(M, N, K):
    """Up to 16 rows: 16 or (from 8192 columns) 32 columns per workgroup, 8 waves with an eighth of K each (fewer k-steps
    than the ring holds, whole rings, a remainder behind them, a last step past K), columns past the last tile."""
    rng = np.random.default_rng(M + 3 * N + 5 * K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    W = I.normal((N, K), 0.05, 5, "wf", N, K)
    print("linear few", M, N, K, flush=True)
    lin = B().Linear(W.cuda())
    want = orc.linear(x, I.to_numpy_storage(W))
    y0 = rng.standard_normal((M, N)).astype(np.float32)
    assert rel_err(lin(torch.from_numpy(x).cuda()).cpu().numpy(), want) <= KERNEL_TOL
    assert rel_err(lin(torch.from_numpy(x).cuda(), torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy(), want + y0) <= KERNEL_TOL
    lin.close()


@pytest.mark.parametrize("M,N", [(1, 64), (5, 1024), (16, 2048), (16, 4096), (17, 48), (40, 1024), (130, 256)])
def test_linear_in_place(M, N):
    """A square matrix whose result overwrites (or is added to) its own input: no workgroup may read what another has
    already written.  Few rows, K sliced, K too short to be sliced."""
    rng = np.random.default_rng(M + 7 * N)
    x = rng.standard_normal((M, N)).astype(np.float32)
    W = I.normal((N, N), 0.05, 5, "wip", N)
    lin = B().Linear(W.cuda())
    want = orc.linear(x, I.to_numpy_storage(W))
    for accumulate in (False, True):
        print("linear in place", M, N, accumulate, flush=True)
        h = torch.from_numpy(x).cuda()
        lin(h, h, accumulate=accumulate)
        assert rel_err(h.cpu().numpy(), want + x if accumulate else want) <= KERNEL_TOL
    lin.close()


@pytest.mark.parametrize("M,K,F,N", [(1, 64, 16, 40), (16, 256, 688, 256), (5, 1040, 2064, 8208), (11, 256, 4096, 512)])
def test_swiglu_ffn_few_rows(M, K, F, N):
    """the feed-forward block whose intermediate is handed over as packed terms of M rows"""
    x, Wg, Wu, Wd, _, want = ffn_case(M, K, F, N, M + K + F)
    b = B()
    gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
    print("ffn few", M, K, F, N, flush=True)
    assert rel_err(gu.ffn(down, torch.from_numpy(x).cuda()).cpu().numpy(), want) <= KERNEL_TOL
    gu.close(); down.close()


def ffn_case(M, K, F, N, seed, scale=2.0):
    """x [M,K] fp32, Wg, Wu [F,K], Wd [N,F] bf16 and the oracle's act = silu(x Wg^T) * (x Wu^T), y = act Wd^T"""
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((M, K)) * scale).astype(np.float32)
    Wg, Wu = I.normal((F, K), 0.05, 7, "wg", seed), I.normal((F, K), 0.05, 7, "wu", seed)
    Wd = I.normal((N, F), 0.05, 7, "wd", seed)
    act = orc.swiglu(orc.linear(x, I.to_numpy_storage(Wg)), orc.linear(x, I.to_numpy_storage(Wu)))
    return x, Wg, Wu, Wd, act, orc.linear(act, I.to_numpy_storage(Wd))


@pytest.mark.parametrize("M,K,F", [(4, 256, 688), (1, 64, 16), (33, 1040, 48), (64, 512, 1408), (40, 64, 96), (96, 256, 2064),
                                   (130, 512, 704), (390, 256, 1376), (17, 2048, 14336), (300, 256, 14336),
                                   (400, 64, 14336)])
def test_gate_up_swiglu(M, K, F):
    """SwiGLU in the gate/up projection's epilogue: every column of silu(gate) * up against the oracle (a slip in the
    interleaved packing would pair a gate column with the wrong up column); widths of one 16-column group, of ragged
    counts of workgroup columns, and the 8B width; rows across the tile shapes."""
    x, Wg, Wu, _, act, _ = ffn_case(M, K, F, 16, M + K + F)
    print("gate_up_swiglu", M, K, F, flush=True)
    gu = B().GateUp(Wg.cuda(), Wu.cuda())
    got = gu.swiglu(torch.from_numpy(x).cuda()).cpu().numpy()
    assert np.all(np.isfinite(got))
    assert rel_err(got, act) <= KERNEL_TOL
    with pytest.raises(TypeError):
        gu(torch.from_numpy(x).cuda())
    gu.close()


@pytest.mark.parametrize("M,K,F,N", [(4, 256, 688, 256), (64, 256, 1408, 512), (40, 64, 64, 96), (390, 128, 704, 512), (80, 512, 704, 512),
                                     (96, 64, 64, 96), (97, 64, 688, 96), (200, 256, 2048, 1024), (513, 128, 688, 512),
                                     (600, 64, 2048, 256), (520, 64, 4096, 64)])
def test_swiglu_ffn(M, K, F, N):
    """The feed-forward block as the step runs it: gate/up with the SwiGLU epilogue, then the down projection, the
    intermediate as fp32 rows (up to 512 rows at these widths) or as tiled bf16 terms (from 513 rows on; F = 688 leaves
    K padding in the down projection's operand).  test_linear_large_batch_kernel forces the tiled form at other sizes,
    test_linear_of_every_tile from every tile."""
    x, Wg, Wu, Wd, _, want = ffn_case(M, K, F, N, M + K + F + N)
    print("swiglu_ffn", M, K, F, N, flush=True)
    gu, down = B().GateUp(Wg.cuda(), Wu.cuda()), B().Linear(Wd.cuda())
    xg = torch.from_numpy(x).cuda()
    got = gu.ffn(down, xg).cpu().numpy()
    assert rel_err(got, want) <= KERNEL_TOL
    y0 = np.random.default_rng(5).standard_normal((M, N)).astype(np.float32)
    got2 = gu.ffn(down, xg, torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy()
    assert rel_err(got2, want + y0) <= KERNEL_TOL
    gu.close(); down.close()


@pytest.mark.parametrize("M,F", [(40, 688), (1, 16), (600, 272)])
def test_swiglu_ffn_records_no_memset_into_a_graph(M, F):
    """Memset nodes have replayed wrongly here: a feed-forward block whose width is no multiple of 256 (so that the padding of
    the tiled intermediate has to be cleared) is recorded as kernels and memory nodes only.  The graph is not launched."""
    import ctypes as C
    x, Wg, Wu, Wd, _, want = ffn_case(M, 256, F, 512, M + F)
    b = B()
    gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
    xd, y = torch.from_numpy(x).cuda(), torch.empty((M, 512), device="cuda")
    b.set_tuning("linear_big_min_m", 1)  # the tiled form at any row count
    b.set_tuning("linear_ks", 4)         # (no few-row path)
    try:
        # memory full of NaN bits where the call's scratch will be
        junk = torch.full((1 << 22,), float("nan"), device="cuda")
        del junk
        gu.ffn(down, xd, y)
        torch.cuda.synchronize()
        assert rel_err(y.cpu().numpy(), want) <= KERNEL_TOL
        lib, st = b.load(), torch.cuda.Stream()
        graph, n = C.c_void_p(), C.c_size_t()
        with torch.cuda.stream(st):
            assert lib.hipStreamBeginCapture(C.c_void_p(st.cuda_stream), C.c_int(2)) == 0  # relaxed
            try:
                gu.ffn(down, xd, y)
            finally:
                assert lib.hipStreamEndCapture(C.c_void_p(st.cuda_stream), C.byref(graph)) == 0
    finally:
        b.set_tuning("linear_big_min_m", 0)
        b.set_tuning("linear_ks", 0)
    assert lib.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert lib.hipGraphGetNodes(graph, nodes, C.byref(n)) == 0
    kinds = []
    for node in nodes:
        k = C.c_int()
        assert lib.hipGraphNodeGetType(C.c_void_p(node), C.byref(k)) == 0
        kinds.append(k.value)
    assert lib.hipGraphDestroy(graph) == 0
    assert kinds.count(0) >= 2 and 2 not in kinds  # kernel nodes, no memset node
    gu.close(); down.close()


def pinned(mt=0, nf=0, ksplit=0, **more):
    """context in which projections take this tile (and none is chosen by estimate)"""
    import contextlib

    @contextlib.contextmanager
    def on():
        knobs = dict(linear_mt=mt, linear_nf=nf, linear_ksplit=ksplit, **more)
        try:
            for k, v in knobs.items():
                B().set_tuning(k, v)
            yield
        finally:
            for k in knobs:
                B().set_tuning(k, 0)
    return on()


@pytest.mark.parametrize("M,N,K,tile", [(97, 8200, 2064, (2, 2, 8)), (128, 4096, 1024, (2, 2, 8)), (100, 2080, 512, (2, 2, 8)), (129, 2080, 272, (3, 2, 4)),
                                        (250, 2144, 528, (2, 2, 8)), (384, 8224, 64, (4, 4, 8)), (384, 8224, 336, (4, 4, 8)), (500, 8192, 192, (4, 4, 8)),
                                        (387, 16400, 48, (4, 4, 8)), (387, 16400, 464, (4, 4, 8)), (97, 16352, 3088, (2, 4, 4)), (127, 8200, 6160, (2, 4, 4)),
                                        (100, 4096, 12304, (2, 4, 4)), (97, 65600, 64, (4, 4, 8)), (96, 65600, 64, (3, 2, 4)), (128, 65536, 48, (2, 4, 4))])
def test_linear_eight_waves(M, N, K, tile):
    """the eight-wave kernels, by name: 128 x 512 and 64 x 256 with several M-tiles; ragged rows, columns past
    the last tile, K below, at and past whole chunks, one chunk and several.  Beside them four-wave ones: a 96-row tile of 129 rows,
    and 64 x 512.  `tile` is what the rules from the sweeps take; the product is taken with it and with whatever shape the estimate puts in
    its place."""
    rng = np.random.default_rng(M + 3 * N + 5 * K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    W = I.normal((N, K), 0.05, 6, "w8", N, K)
    lin = B().Linear(W.cuda())
    want = orc.linear(x, I.to_numpy_storage(W))
    y0 = rng.standard_normal((M, N)).astype(np.float32)
    for mt, nf in (tile[:2], (0, 0)):
        with pinned(mt, nf):
            s = shape(N, K, M, N <= 16384, ALONE)
            print("linear eight waves", M, N, K, s.key(), flush=True)
            assert not mt or (s.mt, s.nf * s.nw // 4, s.nw) == tile
            assert rel_err(lin(torch.from_numpy(x).cuda()).cpu().numpy(), want) <= KERNEL_TOL
            assert rel_err(lin(torch.from_numpy(x).cuda(), torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy(), want + y0) <= KERNEL_TOL
    lin.close()


@pytest.mark.parametrize("mt,nf", [(1, 1), (1, 2), (2, 1), (2, 2), (2, 4), (3, 1), (3, 2), (4, 1), (4, 2), (4, 4)])
@pytest.mark.parametrize("tiles", [1, 3])
def test_linear_of_every_tile(mt, nf, tiles):
    """every tile that is built, by name: with one row tile and with several (weights with and without the streaming hint), ragged rows and columns, K of
    several chunks and a remainder, whole and in slices; alone, added to y, as gate/up (rings of 8 and 16 k-steps) and with the tiled two-term
    form written and, by the 128-row tiles, read"""
    M, K, N = 32 * mt * tiles - 7, 656, 128 * nf * 2 + 72
    x, Wg, Wu, Wd, act, y = ffn_case(M, 336, 656, N, 10 * mt + nf + tiles)
    rng = np.random.default_rng(M + N)
    b = B()
    lin, gu, xa = b.Linear(Wd.cuda()), b.GateUp(Wg.cuda(), Wu.cuda()), torch.from_numpy(act).cuda()
    y0 = rng.standard_normal((M, N)).astype(np.float32)
    for ksplit in (1, 3):
        with pinned(mt, nf, ksplit):
            s = shape(N, K, M, True, ALONE)
            assert (s.mt, s.nf * s.nw // 4, s.ksplit, s.gz) == (mt, nf, ksplit, tiles)
            assert s.nw == (8 if (mt, nf) == (4, 4) or ((mt, nf) == (2, 2) and tiles > 1) else 4)
            print("every tile", mt, nf, tiles, ksplit, flush=True)
            assert rel_err(lin(xa).cpu().numpy(), y) <= KERNEL_TOL
            assert rel_err(lin(xa, torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy(), y + y0) <= KERNEL_TOL
            assert rel_err(gu.swiglu(torch.from_numpy(x).cuda()).cpu().numpy(), act) <= KERNEL_TOL
        with pinned(mt, nf, ksplit, linear_big_min_m=1):
            assert rel_err(gu.ffn(lin, torch.from_numpy(x).cuda()).cpu().numpy(), y) <= KERNEL_TOL
    gu.close(); lin.close()


@pytest.mark.parametrize("M,N,K", [(600, 28640, 336), (300, 44000, 208), (129, 65792, 192), (1290, 12320, 656)])
def test_wide_products_with_a_halved_last_round(M, N, K):
    """128 x 512 tiles of which the last round of the chip is at most half full and taken as tiles of 256 columns: K of three chunks and more, so that
    both loops turn over their buffers; ragged rows, a last column tile that is half there (44000) and not at all for one half (65792); stored, added to
    y, and SwiGLU as fp32 rows and as tiled terms (from 513 rows on)"""
    x, Wg, Wu, Wd, act, y = ffn_case(M, K, N // 2, 96, M + N + K, scale=1.0)
    b = B()
    gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
    rng = np.random.default_rng(M + N)
    W = torch.cat([Wg, Wu])
    xg = torch.from_numpy(x).cuda()
    y0 = torch.from_numpy(rng.standard_normal((M, N)).astype(np.float32)).cuda()
    lin = b.Linear(W.cuda())
    want = orc.linear(x, I.to_numpy_storage(W))
    with pinned(4, 4, 1):
        s = shape(N, K, M, False, STEP)
        assert (s.mt, s.nf, s.nw, s.ksplit) == (4, 2, 8, 1) and s.cps >= 3
        assert s.gx * s.gz > 256 and 0 < s.gx * s.gz % 256 <= 128
        print("halved last round", M, N, K, s.gx, s.gz, flush=True)
        assert rel_err(lin(xg).cpu().numpy(), want) <= KERNEL_TOL
        assert rel_err(lin(xg, y0.clone(), accumulate=True).cpu().numpy(), want + y0.cpu().numpy()) <= KERNEL_TOL
        # silu(g) u of up to 8 million values: |d| <= 1.1 |u| |dg| + |g| |du|, as silu' <= 1.1 and |silu(g)| <= |g|, and dg and du are within
        # KERNEL_TOL of the scale of their own products, g and u (a single large u shows the error of its g in full)
        g, u = want[:, :N // 2], want[:, N // 2:]
        bound = KERNEL_TOL * want.std() * (1.1 * np.abs(u) + np.abs(g))
        assert np.all(np.abs(gu.swiglu(xg).cpu().numpy() - act) <= bound + 1e-30)
    with pinned(4, 4):
        assert rel_err(gu.ffn(down, xg).cpu().numpy(), y) <= KERNEL_TOL
    gu.close(); down.close(); lin.close()


@pytest.mark.parametrize("M,F", [(129, 16400), (200, 24576), (256, 8192)])
def test_gate_up_wide_input_row_tiles(M, F):
    """K >= 8192, unsliced: 128-row tiles past one of them where they give three quarters of the CUs a workgroup (F = 24576),
    64- and 96-row tiles otherwise"""
    K = 8192
    x = torch.from_numpy(np.random.default_rng(M + F).standard_normal((M, K)).astype(np.float32))
    Wg, Wu = I.normal((F, K), 0.01, 6, "wgw", F), I.normal((F, K), 0.01, 6, "wuw", F)
    b = B()
    print("gate/up wide", M, F, flush=True)
    gu = b.GateUp(Wg.cuda(), Wu.cuda())
    got = gu.swiglu(x.cuda()).cpu()
    gu.close()
    rows = torch.arange(0, M, 9)  # sampled rows against fp64 sums
    xg = x[rows].cuda().double()
    g, u = xg @ Wg.cuda().double().t(), xg @ Wu.cuda().double().t()
    want = (torch.nn.functional.silu(g) * u).cpu().float().numpy()
    assert rel_err(got[rows].numpy(), want) <= KERNEL_TOL


def test_linear_over_seeded_random_shapes():
    """The launch shape (rows per tile, column tiles per wave, K-slices, pre-split input) is chosen from M, N and K by
    several rules: 48 seeded random shapes, widths from a few columns to more than two workgroups per CU and rows
    across every tile boundary, each against the oracle; every third shape also as the down projection of a feed-forward
    block behind a gate/up projection with the SwiGLU epilogue."""
    rng = np.random.default_rng(2024)
    for case in range(48):
        M = int(rng.integers(1, 700))
        N = int(rng.choice([rng.integers(1, 200), rng.integers(200, 3000), rng.integers(3000, 40000)]))
        K = 16 * int(rng.integers(1, 1 + (64 if N < 3000 else 16)))
        x = rng.standard_normal((M, K)).astype(np.float32)
        W = I.normal((N, K), 0.05, 9, "wr", case)
        print("random linear", case, M, N, K, flush=True)
        lin = B().Linear(W.cuda())
        want = orc.linear(x, I.to_numpy_storage(W))
        got = lin(torch.from_numpy(x).cuda()).cpu().numpy()
        assert rel_err(got, want) <= KERNEL_TOL, (M, N, K)
        if case % 3 == 0:
            Kin = 16 * int(rng.integers(1, 9))
            xin = (rng.standard_normal((M, Kin)) * 2).astype(np.float32)
            Wg, Wu = I.normal((K, Kin), 0.05, 9, "wrg", case), I.normal((K, Kin), 0.05, 9, "wru", case)
            gu = B().GateUp(Wg.cuda(), Wu.cuda())
            got = gu.ffn(lin, torch.from_numpy(xin).cuda()).cpu().numpy()
            act = orc.swiglu(orc.linear(xin, I.to_numpy_storage(Wg)), orc.linear(xin, I.to_numpy_storage(Wu)))
            want = orc.linear(act, I.to_numpy_storage(W))
            assert rel_err(got, want) <= KERNEL_TOL, (M, N, K, Kin, "ffn")
            gu.close()
        lin.close()


@pytest.mark.parametrize("M,N,K", [(256, 512, 256), (300, 1000, 688), (513, 2080, 1040), (97, 96, 64), (640, 4096, 512)])
def test_linear_large_batch_kernel(M, N, K):
    """the large-batch path (activations pre-split into tiled bf16 terms, copied straight into LDS), forced at any M"""
    rng = np.random.default_rng(M * 5 + N * 3 + K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    W = I.normal((N, K), 0.05, 8, "wb", N, K)
    print("linear big", M, N, K, flush=True)
    b = B()
    b.set_tuning("linear_big_min_m", 1)
    b.set_tuning("linear_big_all", 1)
    try:
        lin = b.Linear(W.cuda())
        xg = torch.from_numpy(x).cuda()
        got = lin(xg).cpu().numpy()
        want = orc.linear(x, I.to_numpy_storage(W))
        assert rel_err(got, want) <= KERNEL_TOL
        y0 = rng.standard_normal((M, N)).astype(np.float32)
        got2 = lin(xg, torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy()
        assert rel_err(got2, want + y0) <= KERNEL_TOL
        lin.close()
        # the feed-forward block with its intermediate forced into the tiled form at this M: F = K is the width of
        # the gate/up output and of the down projection's input
        xs, Wg, Wu, Wd, _, want3 = ffn_case(M, 64, K, N, M + N + K)
        gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
        got3 = gu.ffn(down, torch.from_numpy(xs).cuda()).cpu().numpy()
        assert rel_err(got3, want3) <= KERNEL_TOL
        gu.close(); down.close()
    finally:
        b.set_tuning("linear_big_min_m", 0)
        b.set_tuning("linear_big_all", 0)


def test_rope_large_positions():
    rng = np.random.default_rng(21)
    pos = np.array([0, 1, 17, 4095, 32767, 131071], np.int32)
    x = rng.standard_normal((len(pos), 3, 128)).astype(np.float32)
    got = B().op_rope(torch.from_numpy(x).cuda(), torch.from_numpy(pos).cuda(), 500000.0).cpu().numpy()
    want = np.stack([orc.rope(x[r], int(pos[r]), 500000.0) for r in range(len(pos))])
    assert np.abs(got - want).max() <= 2e-6
    assert np.array_equal(got[0], x[0])


@pytest.mark.parametrize("d,nq,nkv,lens", [
    (64, 4, 2, [1, 15, 16, 17, 128]),
    (128, 32, 8, [1, 16, 33, 700, 64, 2049]),
    (128, 8, 1, [5, 300]),
    (128, 4, 4, [250]),
])
def test_paged_attention(d, nq, nkv, lens):
    m = dict(I.TINY, n_layers=2, head_dim=d, n_q_heads=nq, n_kv_heads=nkv, hidden=256)
    lens = np.array(lens, np.int32)
    # the case's seq_lens are the cached tokens; attention here spans exactly those
    c = make_case(m=m, seed=13, storage="bf16", seq_lens=lens, poison_unused=True)
    g = gpu_setup(c, poison=True)
    opool = fresh_pool(c)
    rng = np.random.default_rng(14)
    q = (rng.standard_normal((len(lens), nq * d)) * 1.3).astype(np.float32)
    for layer in (0, 1):
        print("attention d", d, "nq", nq, "nkv", nkv, "layer", layer, flush=True)
        got = B().op_paged_attention(g.model, g.pool, layer, torch.from_numpy(q).cuda(), g.block_table, g.seq_lens).cpu().numpy()
        want = np.stack([orc.paged_attention(opool, layer, c.block_table[i], int(lens[i]), q[i].reshape(nq, d)).reshape(-1)
                         for i in range(len(lens))])
        assert np.all(np.isfinite(got))
        assert np.abs(got - want).max() <= KERNEL_TOL * max(1.0, np.abs(want).max())


@pytest.mark.parametrize("d,nq,nkv,batch", [(64, 4, 2, 514), (128, 12, 3, 350), (128, 16, 1, 1030)])
def test_paged_attention_merge_of_many_rows(d, nq, nkv, batch):
    """With passes x KV heads above half a round of the grid a lane group per head folds all items of a row, four at a
    time: one to ten items of one page, and head counts that leave the last workgroup of a row partly empty."""
    lens = (1 + (np.arange(batch) * 37) % 157).astype(np.int32)
    c = make_case(m=dict(I.TINY, n_layers=1, head_dim=d, n_q_heads=nq, n_kv_heads=nkv, vocab=64, ffn=16), seed=19, storage="bf16", seq_lens=lens)
    g = gpu_setup(c)
    opool = fresh_pool(c)
    q = (np.random.default_rng(20).standard_normal((batch, nq * d)) * 1.3).astype(np.float32)
    b = B()
    print("attention merge", d, nq, nkv, batch, flush=True)
    b.set_tuning("attn_chunk_pages", 1)
    try:
        got = b.op_paged_attention(g.model, g.pool, 0, torch.from_numpy(q).cuda(), g.block_table, g.seq_lens).cpu().numpy()
    finally:
        b.set_tuning("attn_chunk_pages", 0)
    for i in range(0, batch, 7):
        want = orc.paged_attention(opool, 0, c.block_table[i], int(lens[i]), q[i].reshape(nq, d)).reshape(-1)
        assert np.abs(got[i] - want).max() <= KERNEL_TOL * max(1.0, np.abs(want).max()), i


@pytest.mark.parametrize("d,nq,nkv,batch,every", [(64, 4, 2, 514, 171), (128, 12, 3, 350, 349), (128, 16, 1, 1030, 100), (64, 4, 2, 520, 1)])
def test_paged_attention_merge_of_skewed_batches(d, nq, nkv, batch, every):
    """Many rows of one or two items and a few (every n-th request) of 17 to 70: those are dealt over the grid, a workgroup per
    row and head; if all are that long (every = 1) they are folded like the short ones."""
    rng = np.random.default_rng(23)
    lens = rng.integers(1, 30, batch)
    at = np.arange(0, batch, every)
    lens[at] = 16 * np.where(at % 2, 17, rng.integers(17, 71, len(at)))  # (pages of one item each)
    c = make_case(m=dict(I.TINY, n_layers=1, head_dim=d, n_q_heads=nq, n_kv_heads=nkv, vocab=64, ffn=16), seed=24, storage="bf16",
                  seq_lens=lens.astype(np.int32))
    g = gpu_setup(c)
    opool = fresh_pool(c)
    q = (rng.standard_normal((batch, nq * d)) * 1.3).astype(np.float32)
    b = B()
    print("attention merge, skewed", d, nq, nkv, batch, every, flush=True)
    b.set_tuning("attn_chunk_pages", 1)
    try:
        got = b.op_paged_attention(g.model, g.pool, 0, torch.from_numpy(q).cuda(), g.block_table, g.seq_lens).cpu().numpy()
    finally:
        b.set_tuning("attn_chunk_pages", 0)
    for i in sorted(set(range(0, batch, 13)) | set(at[:40].tolist())):
        want = orc.paged_attention(opool, 0, c.block_table[i], int(lens[i]), q[i].reshape(nq, d)).reshape(-1)
        assert np.abs(got[i] - want).max() <= KERNEL_TOL * max(1.0, np.abs(want).max()), i


def test_multi_token_step_of_a_skewed_batch():
    """The same with 11 new tokens per request (two token groups, the second not full): the long requests' logits in a batch of
    260 against those of a batch of their own, which merges with a workgroup per row and head."""
    T, lens = 11, np.random.default_rng(25).integers(12, 40, 260)
    long = [0, 130, 259]
    lens[long] = [700, 1100, 430]
    c = make_case(m=dict(I.TINY, vocab=64), seed=26, storage="bf16", seq_lens=lens.astype(np.int32))
    g = gpu_setup(c, max_batch=260 * T)
    b = B()
    sl = torch.from_numpy((lens - T).astype(np.int32)).cuda()
    tok = torch.from_numpy(np.random.default_rng(27).integers(0, 64, (260, T)).astype(np.int32)).cuda()
    print("multi-token step, skewed", flush=True)
    b.set_tuning("attn_chunk_pages", 1)
    try:
        got = b.decode_step_multi(g.model, g.pool, g.block_table, sl, tok)[long].cpu().numpy()
        alone = b.decode_step_multi(g.model, g.pool, g.block_table[long].contiguous(), sl[long].contiguous(), tok[long].contiguous()).cpu().numpy()
    finally:
        b.set_tuning("attn_chunk_pages", 0)
    assert np.abs(got - alone).max() <= 2e-3 * alone.std()  # other tile shapes; new K and V may round to the other bf16 neighbour


def test_projections_on_two_streams_share_the_scratch_pool():
    """K-sliced projections and feed-forward blocks take scratch from one pool per device: calls in flight on two
    streams, after a synchronisation, and after other handles of the device have gone."""
    b = B()
    rng = np.random.default_rng(33)
    x = torch.from_numpy(rng.standard_normal((70, 1024)).astype(np.float32)).cuda()
    W = [I.normal((768, 1024), 0.05, 8, "ws", i) for i in range(2)]
    Wg, Wu, Wd = (I.normal(sh, 0.05, 8, "wsf", i) for i, sh in enumerate(((512, 1024), (512, 1024), (768, 512))))
    lin = [b.Linear(w.cuda()) for w in W]
    gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
    torch.cuda.synchronize()
    want = [l(x).clone() for l in lin] + [gu.ffn(down, x).clone()]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = [[], []]
    for r in range(20):
        for k, st in enumerate(streams):
            with torch.cuda.stream(st):
                got[k].append([lin[k](x), gu.ffn(down, x)])
    torch.cuda.synchronize()
    for k in range(2):
        for y, f in got[k]:
            assert torch.equal(y, want[k]) and torch.equal(f, want[2])
    lin[1].close(); gu.close(); down.close()
    assert torch.equal(lin[0](x), want[0])
    lin[0].close()


def test_a_full_device_gets_the_scratch_pool_back():
    """The pool keeps what a feed-forward block of 4096 rows used (235 MB); an allocation of the library that fails (2^47 bytes: on
    any device) gives that back before it is reported, and the block runs again."""
    import ctypes as C
    b = B()
    x, Wg, Wu, Wd, _, want = ffn_case(8, 64, 14336, 64, 3)
    gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
    xd = torch.from_numpy(np.tile(x, (512, 1))).cuda()
    y = torch.empty((4096, 64), device="cuda")
    gu.ffn(down, xd, y)
    torch.cuda.synchronize()
    kept = torch.cuda.mem_get_info()[0]
    h = C.c_void_p()
    rc = b.load().chiron_linear_create(b._ptr(Wd.cuda()), C.c_int32(1 << 30), C.c_int32(1 << 16), b._stream(), C.byref(h))
    assert rc == -5 and not h.value  # CHIRON_ERR_OOM
    for _ in range(40):  # the GPU driver frees with some delay
        if torch.cuda.mem_get_info()[0] - kept >= 200 << 20:
            break
        time.sleep(0.05)
    else:
        pytest.fail("the pool kept its memory")
    gu.ffn(down, xd, y)
    assert rel_err(y[:8].cpu().numpy(), want) <= KERNEL_TOL and torch.equal(y[:8], y[8:16])
    gu.close(); down.close()


@pytest.mark.parametrize("batch", [1023, 2048, 2051])
def test_paged_attention_work_list_of_many_requests(batch):
    """The work list keeps the page counts of the first 2048 requests in LDS and reads the others' again; from 1025
    requests on a thread counts several."""
    lens = (1 + (np.arange(batch) * 37) % 41).astype(np.int32)
    c = make_case(m=dict(I.TINY, n_layers=1, vocab=64, ffn=16), seed=17, storage="bf16", seq_lens=lens)
    g = gpu_setup(c)
    opool = fresh_pool(c)
    q = (np.random.default_rng(18).standard_normal((batch, 4 * 64)) * 1.3).astype(np.float32)
    print("attention", batch, "requests", flush=True)
    got = B().op_paged_attention(g.model, g.pool, 0, torch.from_numpy(q).cuda(), g.block_table, g.seq_lens).cpu().numpy()
    want = np.stack([orc.paged_attention(opool, 0, c.block_table[i], int(lens[i]), q[i].reshape(4, 64)).reshape(-1) for i in range(batch)])
    assert np.abs(got - want).max() <= KERNEL_TOL * max(1.0, np.abs(want).max())


@pytest.mark.parametrize("grid,chunk", [(4, 0), (4, 3), (2, 1), (0, 5), (8, 2), (24, 1)])
def test_paged_attention_work_list_over_several_rounds(grid, chunk):
    """A small persistent grid (grid workgroups = 4*grid wave slots) makes every wave walk several items of the work
    list: its own first, then items whose indices it draws from ticket counters (one counter below 8 workgroups, eight
    from there on), records fetched one item ahead; forced chunk sizes give items of 1, 2, 3 or 5 pages with ragged
    ends.  24 requests of 1..1500 cached tokens, 4 query heads per KV head.  The call is made twice and must give the
    same bits (the counters' state between the layers of one step is covered by the multi-layer steps at batch 512)."""
    d, nq, nkv = 128, 8, 2
    rng = np.random.default_rng(41)
    lens = rng.integers(1, 1500, size=24).astype(np.int32)
    lens[:4] = [1, 16, 17, 1499]
    m = dict(I.TINY, n_layers=1, head_dim=d, n_q_heads=nq, n_kv_heads=nkv, hidden=256)
    c = make_case(m=m, seed=17, storage="bf16", seq_lens=lens, poison_unused=True)
    g = gpu_setup(c, poison=True)
    opool = fresh_pool(c)
    q = (rng.standard_normal((len(lens), nq * d)) * 1.3).astype(np.float32)
    b = B()
    b.set_tuning("attn_grid", grid)
    b.set_tuning("attn_chunk_pages", chunk)
    try:
        print("attention grid", grid, "chunk", chunk, flush=True)
        got = b.op_paged_attention(g.model, g.pool, 0, torch.from_numpy(q).cuda(), g.block_table, g.seq_lens).cpu().numpy()
        again = b.op_paged_attention(g.model, g.pool, 0, torch.from_numpy(q).cuda(), g.block_table, g.seq_lens).cpu().numpy()
    finally:
        b.set_tuning("attn_grid", 0)
        b.set_tuning("attn_chunk_pages", 0)
    want = np.stack([orc.paged_attention(opool, 0, c.block_table[i], int(lens[i]), q[i].reshape(nq, d)).reshape(-1)
                     for i in range(len(lens))])
    assert np.all(np.isfinite(got))
    assert np.abs(got - want).max() <= KERNEL_TOL * max(1.0, np.abs(want).max())
    assert np.array_equal(got, again)  # which wave takes which item does not enter the result


# ---- the whole step ---------------------------------------------------------------------------------

def norm_launches(g, step):
    """(result, launches of the norm by itself: none on the few-row path)"""
    B().kernel_timing_begin(g.model)
    try:
        out = step()
    finally:
        kt = B().kernel_timing_end(g.model)
    return out, kt["rmsnorm"][1]


def run_both(c, g=None, poison=False):
    g = g or gpu_setup(c, poison=poison)
    logits = B().decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens)
    torch.cuda.synchronize()
    opool = fresh_pool(c)
    want, slots = orc.decode_step(c.cfg, c.w, opool, c.block_table, c.seq_lens, c.tokens)
    return g, logits.cpu().numpy(), want, opool


def check_logits(got, want, min_agree=0.99):
    sig = want.std()
    err = np.abs(got - want).max() / sig
    agree = float((got.argmax(1) == want.argmax(1)).mean())
    print("max|d|/sigma = %.3e, argmax agreement = %.4f" % (err, agree), flush=True)
    assert np.all(np.isfinite(got))
    assert err <= STEP_TOL
    assert agree >= min_agree
    return err


# pages per request of lists that 32 wave slots (16 items of either KV head) hold in one round with items of more than 64 pages:
# mixed lengths, a search that ends at its lower bound (one request in 16 items of 128) and at its upper one (158), and one
# list that misses by a single item, which takes items of 64 pages drawn from the ticket counters
@pytest.mark.parametrize("pages", [[563, 75, 2063], [2048], [316, 433, 336, 5, 793, 21], [783, 65, 262, 121, 508, 780, 461]])
def test_paged_attention_one_round_of_long_items(pages):
    d, nq, nkv = 64, 4, 2
    lens = (16 * np.asarray(pages) - np.arange(len(pages)) % 16).astype(np.int32)
    c = make_case(m=dict(I.TINY, n_layers=1, head_dim=d, n_q_heads=nq, n_kv_heads=nkv, vocab=64, ffn=16), seed=29, storage="bf16", seq_lens=lens,
                  poison_unused=True)
    g = gpu_setup(c, poison=True)
    opool = fresh_pool(c)
    q = (np.random.default_rng(30).standard_normal((len(lens), nq * d)) * 1.3).astype(np.float32)
    b = B()
    b.set_tuning("attn_grid", 8)
    try:
        print("attention, one round", pages, flush=True)
        got = b.op_paged_attention(g.model, g.pool, 0, torch.from_numpy(q).cuda(), g.block_table, g.seq_lens).cpu().numpy()
    finally:
        b.set_tuning("attn_grid", 0)
    for i in range(len(lens)):
        want = orc.paged_attention(opool, 0, c.block_table[i], int(lens[i]), q[i].reshape(nq, d)).reshape(-1)
        assert np.abs(got[i] - want).max() <= KERNEL_TOL * max(1.0, np.abs(want).max()), i


def test_multi_token_step_with_long_items():
    """The same with 11 new tokens per request, two passes each (token groups of 8 and 3): items of 94 pages in one round
    of 64 slots against items of 16 pages."""
    T, lens = 11, np.array([9000, 700, 12000], np.int32)
    c = make_case(m=dict(I.TINY, vocab=64), seed=31, storage="bf16", seq_lens=lens)
    g = gpu_setup(c, max_batch=3 * T)
    b = B()
    sl = torch.from_numpy(lens - T).cuda()
    tok = torch.from_numpy(np.random.default_rng(32).integers(0, 64, (3, T)).astype(np.int32)).cuda()
    out = []
    b.set_tuning("attn_grid", 16)
    try:
        for chunk in (0, 16):
            print("multi-token step, long items, chunk", chunk, flush=True)
            b.set_tuning("attn_chunk_pages", chunk)
            out.append(b.decode_step_multi(g.model, g.pool, g.block_table, sl, tok).cpu().numpy())
    finally:
        b.set_tuning("attn_grid", 0)
        b.set_tuning("attn_chunk_pages", 0)
    assert np.all(np.isfinite(out[0]))
    assert np.abs(out[0] - out[1]).max() <= 2e-3 * out[1].std()


def step_64(c, tok, newkv):
    """(logits, k, v) of a step in 64 bits, tok [batch, T]; the attention of layer l sees the K and V that the library wrote for
    the new tokens, newkv[l] = (k, v) [batch, T, heads, d], so that a value that rounds to the other bf16 neighbour is not
    carried on; k, v [layer] are the unrounded ones"""
    m = c.m
    d, nkv, G, T = m["head_dim"], m["n_kv_heads"], m["n_q_heads"] // m["n_kv_heads"], tok.shape[1]
    t64 = lambda a: torch.from_numpy(as_f64(a))
    W = {k: ([t64(a) for a in v] if isinstance(v, list) else t64(v)) for k, v in c.w.items()}
    norm = lambda h, gain: h / torch.sqrt((h * h).mean(-1, keepdim=True) + m["rms_eps"]) * gain
    pos = torch.from_numpy(c.seq_lens.astype(np.int64))[:, None] + torch.arange(T)
    ang = pos[..., None] * m["rope_base"] ** (-2.0 * torch.arange(d // 2, dtype=torch.float64) / d)
    cs, sn = ang.cos()[:, :, None], ang.sin()[:, :, None]
    rope = lambda x: torch.cat([x[..., :d // 2] * cs - x[..., d // 2:] * sn, x[..., d // 2:] * cs + x[..., :d // 2] * sn], -1)
    ends = np.cumsum(c.seq_lens)
    h, kvs = W["embed"][torch.from_numpy(tok).long()], []
    for l in range(m["n_layers"]):
        x = norm(h, W["attn_norm"][l])
        q, k, v = ((x @ W[n][l].T).view(c.batch, T, -1, d) for n in ("wq", "wk", "wv"))
        q, k = rope(q), rope(k)
        kvs.append((k, v))
        a = torch.empty(c.batch, T, m["n_q_heads"] * d, dtype=torch.float64)
        for i, (e, n) in enumerate(zip(ends, c.seq_lens)):
            K, V = (torch.cat([t64(c.kv[l][j][e - n:e]), newkv[l][j][i].double()]) for j in (0, 1))
            for t in range(T):
                s = torch.einsum("khd,nkd->khn", q[i, t].view(nkv, G, d), K[:n + t + 1]) / math.sqrt(d)
                a[i, t] = torch.einsum("khn,nkd->khd", torch.softmax(s, -1), V[:n + t + 1]).reshape(-1)
        h = h + a @ W["wo"][l].T
        x = norm(h, W["ffn_norm"][l])
        h = h + (torch.nn.functional.silu(x @ W["w_gate"][l].T) * (x @ W["w_up"][l].T)) @ W["w_down"][l].T
    return norm(h, W["final_norm"]) @ W["lm_head"].T, kvs


@pytest.mark.parametrize("batch,T,mt", [(1, 1, 0), (11, 1, 0), (3, 5, 0), (11, 1, 1), (20, 1, 0)])
def test_step_against_64_bits(batch, T, mt):
    """Few-row path, the general path on the same rows (mt = 1), and more rows: logits and new K and V.  An activation enters
    the matrix cores with a relative error of at most 2^-17, once in each of a layer's five products and in p V, and in the
    head's: 13 of them here, 1e-4 in all (measured 1e-5).  A new K or V is that far from the 64-bit value, plus its rounding to
    bf16.  The step repeats itself bit by bit."""
    m = dict(I.TINY, n_layers=2, hidden=1040, n_q_heads=16, n_kv_heads=4, ffn=2064, vocab=1009)
    lens = np.random.default_rng(batch + T).integers(0, 200, batch).astype(np.int32)
    c = make_case(m=m, seed=44, storage="bf16", gain_jitter=0.2, seq_lens=lens)
    c.block_table, c.num_blocks = I.make_block_table(lens + T - 1, seed=44, pool_factor=2.0)
    g = gpu_setup(c, max_batch=batch * T)
    tok = I.token_ids(batch * T, m["vocab"], 7).reshape(batch, T)
    b = B()
    b.set_tuning("linear_mt", mt)
    try:
        print("64 bits", batch, T, mt, flush=True)
        step = lambda: b.decode_step_multi(g.model, g.pool, g.block_table, g.seq_lens, torch.from_numpy(tok).cuda())
        got, norms = norm_launches(g, step)
        assert (norms == 0) == (batch * T <= 16 and not mt)
        assert torch.equal(step(), got)
    finally:
        b.set_tuning("linear_mt", 0)
    kv = [[g.pool.gather(l, g.block_table[i].contiguous(), int(lens[i]) + T) for i in range(batch)] for l in range(2)]
    kv = [tuple(torch.stack([x[j][-T:] for x in row]).cpu() for j in (0, 1)) for row in kv]
    want, kvs = step_64(c, tok, kv)
    err = float((got.cpu().double() - want).norm() / want.norm())
    print("relative error of the logits %.2e" % err, flush=True)
    assert err <= 1e-4
    for have, exact in zip(kv, kvs):
        for x, y in zip(have, exact):
            assert bool(((x.double() - y).abs() <= 2.0 ** -8 * y.abs() + 1e-4 * y.std()).all())


@pytest.mark.parametrize("seed,jitter", [(0, 0.0), (1, 0.2)])
def test_decode_step_tiny_config(seed, jitter):
    """Tiny decoder (2 layers, hidden 256, 4q/2kv heads of 64, FFN 688, vocab 1024), batch 4, contexts U{16..128},
    16-token pages, shuffled block table, bf16-rounded copies of the fp32 draws on both sides."""
    c = make_case(batch=4, seed=seed, storage="bf16", gain_jitter=jitter, poison_unused=True)
    g, got, want, opool = run_both(c, poison=True)
    assert got.shape == (4, 1024)
    err = check_logits(got, want, min_agree=1.0)
    assert err <= 2e-3   # what the two-term activation split should deliver on two layers
    B().validate_step_inputs(g.model, g.pool, g.block_table, g.seq_lens, g.tokens)
    # slot contract: position p of every request now holds the new K/V (value within one bf16 ulp of the
    # oracle's, since both sides round their own fp32 k,v), every older position is bit-unchanged
    o = 0
    for i, L in enumerate(c.seq_lens):
        L = int(L)
        for l in range(c.m["n_layers"]):
            k, v = g.pool.gather(l, g.block_table[i].contiguous(), L + 1)
            ok, ov = orc.gather_kv(opool, l, c.block_table[i], L + 1)
            assert np.array_equal(bits(k)[:L], ok[:L]) and np.array_equal(bits(v)[:L], ov[:L])
            assert np.array_equal(bits(k)[:L], c.kv[l][0][o:o + L])
            for a, b in ((bits(k)[L], ok[L]), (bits(v)[L], ov[L])):
                fa, fb = bf16_to_f32(a), bf16_to_f32(b)
                # one bf16 ulp of the element, plus the fp32-level difference of the two k/v (visible where a
                # rotated element nearly cancels)
                assert np.all(np.abs(fa - fb) <= np.abs(fb) * 2.0 ** -7 + 1e-4 * np.abs(fb).max())
                assert np.mean(a == b) > 0.95
        o += L


def test_decode_step_edge_lengths_and_batch_sizes():
    # empty context, page boundaries (the new token opens a fresh page at 16 and 32), a longer one
    c = make_case(seed=3, storage="bf16", seq_lens=[0, 15, 16, 31, 32, 1, 200], poison_unused=True)
    g, got, want, _ = run_both(c, poison=True)
    check_logits(got, want, min_agree=1.0)
    # a request's logits do not depend on the rest of the batch (up to summation order)
    for b in (1, 3):
        g2 = gpu_setup(c, poison=True)
        sub = B().decode_step(g2.model, g2.pool, g2.block_table, g2.seq_lens, g2.tokens, batch=b).cpu().numpy()
        assert np.abs(sub - want[:b]).max() <= STEP_TOL * want.std()
    # batch 0 is a no-op
    B().decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens, batch=0,
                    logits=torch.empty((1, 1024), device="cuda"))


def test_decode_step_batch_permutation_and_layout():
    c = make_case(batch=6, seed=4, storage="bf16")
    g, got, want, _ = run_both(c)
    perm = np.array([4, 2, 0, 5, 1, 3])
    c2 = make_case(batch=6, seed=4, storage="bf16", shuffle=False, pool_factor=1.0)   # contiguous pages
    assert np.array_equal(c2.seq_lens, c.seq_lens)
    g2 = gpu_setup(c2)
    p = torch.from_numpy(perm).cuda()
    got2 = B().decode_step(g2.model, g2.pool, g2.block_table[p].contiguous(), g2.seq_lens[p].contiguous(),
                           g2.tokens[p].contiguous()).cpu().numpy()
    # permuted batch on a different physical layout: same logits, permuted (up to the order of partial sums)
    assert np.abs(got2 - got[perm]).max() <= 1e-4 * want.std()
    check_logits(got2, want[perm], min_agree=1.0)


def test_decode_step_medium_shape_d128():
    """4 layers of the 8B head geometry (32q/8kv heads of 128) at reduced width, batch 70 (two M-tiles, ragged),
    contexts lognormal: exercises the d=128 attention path, G=4, split contexts and M > 64."""
    m = dict(I.LLAMA_8B, name="mid", n_layers=4, hidden=1024, ffn=2816, vocab=4096, n_q_heads=32, n_kv_heads=8)
    lens = I.lognormal_lengths(70, 300, 1, 1500, np.random.default_rng(5))
    c = make_case(m=m, seed=5, storage="bf16", seq_lens=lens, poison_unused=True)
    g, got, want, _ = run_both(c, poison=True)
    check_logits(got, want, min_agree=0.99)


def test_decode_step_over_seeded_random_geometries():
    """Eight seeded random decoders: 1-3 layers, hidden and FFN widths that are multiples of 16 but of nothing larger,
    head dimension 64 or 128, 1..16 query heads per KV head, vocabularies that are not multiples of 32, batches of
    1..90 requests with 0..600 cached tokens.  Every width goes through the K padding, column masking and tile rules of
    the projections, every head grouping through its attention instance."""
    rng = np.random.default_rng(77)
    for case in range(8):
        d = 64 if case % 2 == 0 else 128
        G = int(rng.choice([1, 2, 4, 8, 16]))
        nkv = int(rng.integers(1, 4)) if G <= 4 else 1
        m = dict(I.TINY, name="rand%d" % case, n_layers=int(rng.integers(1, 4)), hidden=16 * int(rng.integers(5, 40)),
                 n_q_heads=G * nkv, n_kv_heads=nkv, head_dim=d, ffn=16 * int(rng.integers(5, 90)),
                 vocab=int(rng.integers(50, 3000)), rope_base=float(rng.choice([1e4, 5e5])))
        batch = int(rng.integers(1, 91))
        lens = rng.integers(0, 600, size=batch).astype(np.int32)
        print("geometry", case, {k: m[k] for k in ("n_layers", "hidden", "n_q_heads", "n_kv_heads", "head_dim", "ffn", "vocab")},
              "batch", batch, flush=True)
        c = make_case(m=m, seed=100 + case, storage="bf16", gain_jitter=0.1, seq_lens=lens, poison_unused=True)
        g, got, want, _ = run_both(c, poison=True)
        check_logits(got, want, min_agree=0.99)


G4_D128 = dict(I.TINY, head_dim=128, n_kv_heads=2, n_q_heads=8)
G8_D128 = dict(I.TINY, head_dim=128, n_kv_heads=1, n_q_heads=8)


@pytest.mark.parametrize("m,batch,T", [(I.TINY, 1, 1), (I.TINY, 16, 1), (G4_D128, 5, 3), (dict(I.TINY, hidden=2320, ffn=272, vocab=8400), 16, 1),
                                       (dict(G4_D128, n_q_heads=2, n_kv_heads=2, hidden=272, vocab=33000), 3, 5)])
def test_step_of_few_rows_equals_the_general_path(m, batch, T):
    """Up to 16 rows the step takes the few-row projections (norms and rotary embedding fused); a forced tile height of
    the general kernels (any knob of theirs) keeps the general path.  Same logits to fp32 rounding; new K and V
    are fp32 sums within KERNEL_TOL of their scale (what two correct kernels may be apart), rounded to bf16: few values
    differ, by one neighbour (2^-7 of the value) or, near zero, by that distance.  Past the first layer the distance is
    that of the logits: a value that fell on the other neighbour there moves an attention output by up to 2^-8 / 16 of
    the values' scale (16 positions in the shortest context), and the norm and the projections behind it by a few times that."""
    c = make_case(m=m, batch=batch, seed=41, storage="bf16", gain_jitter=0.2)
    g = gpu_setup(c, max_batch=batch * T)
    b = B()
    lens = c.seq_lens - T  # room for T new tokens in the pages that are there
    sl = torch.from_numpy(lens.astype(np.int32)).cuda()
    tok = torch.from_numpy(np.random.default_rng(3).integers(0, m["vocab"], (batch, T)).astype(np.int32)).cuda()
    out = []
    for mt in (0, 1):
        print("few rows", m["name"], batch, T, "mt", mt, flush=True)
        b.set_tuning("linear_mt", mt)
        try:
            lg, norms = norm_launches(g, lambda: b.decode_step_multi(g.model, g.pool, g.block_table, sl, tok))
        finally:
            b.set_tuning("linear_mt", 0)
        assert norms == (2 * m["n_layers"] + 1 if mt else 0)  # which path ran
        kv = [g.pool.gather(l, g.block_table[i], int(lens[i]) + T) for l in range(m["n_layers"]) for i in range(batch)]
        out.append((lg.cpu().numpy().reshape(batch * T, -1), [x.float().cpu().numpy() for p in kv for x in p]))
    (lg0, kv0), (lg1, kv1) = out
    assert np.abs(lg0 - lg1).max() <= 2e-3 * lg1.std()
    for j, (x, y) in enumerate(zip(kv0, kv1)):
        tol = KERNEL_TOL if j < 2 * batch else 2e-3
        assert np.all(np.abs(x - y) <= 2.0 ** -7 * np.abs(y) + tol * y.std())
        assert np.mean(x != y) <= 0.02


def test_the_few_row_path_ends_where_its_activations_outweigh_it():
    """480 and 320 workgroups of 5120 inputs each on 256 CUs: one row takes the few-row path, 16 rows do not.  The same holds for a
    projection by itself, which shows in nothing but time: both sides of its range against the oracle."""
    m = dict(I.TINY, name="wide", n_layers=1, hidden=5120, n_q_heads=40, n_kv_heads=40, head_dim=128, ffn=16, vocab=64)
    c = make_case(m=m, seed=43, storage="bf16", seq_lens=np.arange(20, 36, dtype=np.int32))
    g = gpu_setup(c)
    b = B()
    out = []
    for n in (16, 1):
        print("range of the few-row path", n, flush=True)
        lg, norms = norm_launches(g, lambda: b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens, batch=n))
        assert norms == (3 if n == 16 else 0)
        out.append(lg[0].cpu().numpy())
    assert np.abs(out[0] - out[1]).max() <= 2e-3 * out[0].std()
    for M, N, K in ((8, 4096, 14336), (16, 4096, 14336), (1, 256, 28672), (16, 10240, 4096)):
        x = np.random.default_rng(M + N).standard_normal((M, K)).astype(np.float32)
        W = I.normal((N, K), 0.02, 5, "wr", N, K)
        lin = b.Linear(W.cuda())
        want = orc.linear(x[:2], I.to_numpy_storage(W))
        assert rel_err(lin(torch.from_numpy(x).cuda()).cpu().numpy()[:2], want) <= KERNEL_TOL
        lin.close()


@pytest.mark.parametrize("m,T", [(I.TINY, 2), (I.TINY, 4), (I.TINY, 8), (I.TINY, 9), (I.TINY, 17), (G4_D128, 4), (G4_D128, 3),
                                 (G4_D128, 5), (G4_D128, 8), (G4_D128, 11), (G8_D128, 2), (G8_D128, 5)])
def test_multi_token_step(m, T):
    """q_len > 1 (speculative-decoding verify shape): causal over the block, all T tokens' K/V appended.
    As many tokens as fit the 16 operand columns (16 / heads-per-KV-head) share one pass over the request's pages
    (operand columns token*G + head); longer blocks take several passes, the last one ragged (9 = 8+1, 17 = 8+8+1,
    11 = 4+4+3, 5 = 2+2+1).  Lengths 15, 31, 63 put the first new token at the end of a page / of a work item, so
    that later tokens open a page or an item in which the earlier ones see nothing."""
    lens = [14, 15, 31, 63, 60, 0, 127, 1]
    c = make_case(m=m, seed=16, storage="bf16", gain_jitter=0.1, seq_lens=lens, pool_factor=3.0)
    toks = I.token_ids(len(lens) * T, c.m["vocab"], 6).reshape(len(lens), T)
    bt, nb = I.make_block_table(np.asarray(lens) + T - 1, seed=16, pool_factor=3.0)
    c.block_table, c.num_blocks = bt, nb
    g = gpu_setup(c, max_batch=len(lens) * T, poison=True)
    B().validate_step_inputs(g.model, g.pool, g.block_table, g.seq_lens, torch.from_numpy(toks).cuda())
    got = B().decode_step_multi(g.model, g.pool, g.block_table, g.seq_lens, torch.from_numpy(toks).cuda()).cpu().numpy()
    opool = fresh_pool(c)
    want = orc.decode_step_multi(c.cfg, c.w, opool, bt, c.seq_lens, toks)
    assert got.shape == (len(lens), T, c.m["vocab"])
    check_logits(got.reshape(-1, c.m["vocab"]), want.reshape(-1, c.m["vocab"]), min_agree=1.0)
    # the T new positions of every request hold the oracle's k, v up to one bf16 ulp; older ones are untouched
    o = 0
    for i, L in enumerate(lens):
        k, v = g.pool.gather(1, g.block_table[i].contiguous(), L + T)
        ok, ov = orc.gather_kv(opool, 1, bt[i], L + T)
        assert np.array_equal(bits(k)[:L], ok[:L]) and np.array_equal(bits(v)[:L], ov[:L])
        fa, fb = bf16_to_f32(bits(k)[L:]), bf16_to_f32(ok[L:])
        assert np.all(np.abs(fa - fb) <= np.abs(fb) * 2.0 ** -7 + 1e-3 * np.abs(fb).max())
        o += L
    with pytest.raises(B().ChironError) as e:
        B().decode_step_multi(g.model, g.pool, g.block_table, g.seq_lens, torch.zeros((len(lens), T + 1), dtype=torch.int32, device="cuda"))
    assert e.value.code == -3


def test_a_request_of_nan_leaves_nothing_behind_in_the_split_input():
    """With every projection's input split into tiled terms, the workspace that holds them also holds the feed-forward
    intermediate, whose padding (width 688 of 768) the down projection multiplies by zero: what another projection left there must
    not be NaN.  A request whose embedding is NaN spoils its own logits and no others, in that step and in the next."""
    c = make_case(m=dict(I.TINY, vocab=64), batch=100, kind="tiny", seed=45, storage="bf16")
    bad = 70  # its terms lie where the padding of the first 32 rows is read
    c.w_t["embed"][63] = float("nan")
    c.tokens = np.where(c.tokens == 63, 0, c.tokens).astype(np.int32)
    g = gpu_setup(c)
    b = B()
    spoiled = g.tokens.clone()
    spoiled[bad] = 63
    b.set_tuning("linear_big_all", 1)
    b.set_tuning("linear_big_min_m", 1)
    try:
        print("nan in the split input", flush=True)
        first = b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens).cpu()
        nan = b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, spoiled).cpu()
        again = b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens).cpu()
        b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, spoiled)
        b.set_tuning("linear_big_all", 0)  # only the intermediate is split from here on
        plain = b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens).cpu()
    finally:
        b.set_tuning("linear_big_all", 0)
        b.set_tuning("linear_big_min_m", 0)
    others = [i for i in range(100) if i != bad]
    assert torch.isfinite(first).all() and torch.isnan(nan[bad]).all()
    assert torch.equal(nan[others], first[others])
    assert torch.equal(again, first)
    assert (plain - first).abs().max() <= 2e-3 * first.std()  # other tile shapes


def test_continuous_batching_over_several_iterations():
    """The calls in the use the paper describes (Continuous Batching: requests join and leave the running batch between
    iterations; the queue and its lengths are the caller's): eight requests start, every iteration feeds each running
    request the token the oracle's greedy choice gave it and advances its length, some finish and others take
    their place, lengths cross page boundaries.  Both sides run the same schedule from the same cache content;
    every iteration's logits are compared."""
    lens0 = np.array([13, 15, 30, 47, 5, 64, 0, 95], np.int32)
    n_iter, grow = 7, 8
    c = make_case(seed=21, storage="bf16", gain_jitter=0.1, seq_lens=lens0, pool_factor=3.0)
    bt, nb = I.make_block_table(lens0 + grow, seed=21, pool_factor=3.0)   # pages for the tokens still to come
    c.block_table, c.num_blocks = bt, nb
    g = gpu_setup(c, poison=True)
    opool = fresh_pool(c)
    lens = lens0.copy()
    toks = c.tokens.copy()
    running = list(range(8))
    for it in range(n_iter):
        if it == 2:
            running = [0, 2, 3, 5, 7]          # three requests finish
        if it == 4:
            running = [7, 1, 0, 4, 5, 6]       # two waiting ones (their caches kept) join, order changes
        idx = np.asarray(running)
        B().validate_step_inputs(g.model, g.pool, g.block_table[idx].contiguous(), torch.from_numpy(lens[idx]).cuda(),
                                 torch.from_numpy(toks[idx]).cuda())
        got = B().decode_step(g.model, g.pool, g.block_table[idx].contiguous(), torch.from_numpy(lens[idx]).cuda(),
                              torch.from_numpy(toks[idx]).cuda()).cpu().numpy()
        want, _ = orc.decode_step(c.cfg, c.w, opool, np.ascontiguousarray(bt[idx]), lens[idx], toks[idx])
        print("iteration", it, "batch", running, flush=True)
        check_logits(got, want, min_agree=1.0)
        toks[idx] = want.argmax(1).astype(np.int32)   # greedy continuation, the same on both sides
        lens[idx] += 1
    assert lens.max() <= (lens0 + grow).max()
    # the caches agree afterwards: old content bit-exact, generated positions to one bf16 ulp
    for i in range(8):
        k, v = g.pool.gather(1, g.block_table[i].contiguous(), int(lens[i]))
        ok, ov = orc.gather_kv(opool, 1, bt[i], int(lens[i]))
        L0 = int(lens0[i])
        assert np.array_equal(bits(k)[:L0], ok[:L0]) and np.array_equal(bits(v)[:L0], ov[:L0])
        fa, fb = bf16_to_f32(bits(k)[L0:]), bf16_to_f32(ok[L0:])
        if fb.size:
            assert np.all(np.abs(fa - fb) <= np.abs(fb) * 2.0 ** -6 + 2e-3 * np.abs(fb).max())


def test_repeat_step_is_idempotent_and_profile_runs():
    c = make_case(batch=4, seed=6, storage="bf16")
    g, got, want, _ = run_both(c)
    again = B().decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens).cpu().numpy()
    assert np.abs(again - got).max() <= 1e-4 * want.std()
    pts = B().step_latency_profile(g.model, g.pool, g.block_table, g.seq_lens, g.tokens, [1, 2, 4], warmup=1, iters=3)
    assert [p["batch"] for p in pts] == [1, 2, 4]
    for p in pts:
        assert p["lat_ms_median"] > 0 and p["lat_ms_p99"] >= p["lat_ms_median"] and p["tokens_per_s"] > 0


def test_decode_step_replays_from_a_hip_graph():
    """The step only enqueues kernels, so it can be recorded into a HIP graph.  Three replays, each after eager work of
    the program's own on the same model (a step over another batch size, a host synchronisation) and into a logits
    buffer overwritten in between, must give the bits of the eager step.  A small attention grid makes the waves draw
    work items from the ticket counters, which only kernels of the step itself put back to zero."""
    m = dict(I.LLAMA_8B, name="mid", n_layers=3, hidden=1024, ffn=2816, vocab=4096, n_q_heads=32, n_kv_heads=8)
    lens = I.lognormal_lengths(70, 300, 1, 1500, np.random.default_rng(8))
    c = make_case(m=m, seed=8, storage="bf16", seq_lens=lens, poison_unused=True)
    g = gpu_setup(c, poison=True)
    b = B()
    b.set_tuning("attn_grid", 16)
    try:
        logits = torch.empty((70, 4096), dtype=torch.float32, device="cuda")
        step = lambda: b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens, logits=logits, batch=70)
        step()
        torch.cuda.synchronize()
        eager = logits.clone()
        assert torch.isfinite(eager).all()
        side = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            step()
        torch.cuda.synchronize()
        for replay in range(3):
            print("graph replay", replay, flush=True)
            other = b.decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens, batch=5 + replay)
            torch.cuda.synchronize()
            assert (other - eager[:5 + replay]).abs().max() <= 1e-2 * eager.std()  # other tile shapes: not the same bits
            logits.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(logits, eager), replay
    finally:
        b.set_tuning("attn_grid", 0)


def test_error_paths_on_device():
    c = make_case(batch=4, seed=7, storage="bf16")
    g = gpu_setup(c)
    Bd = B()
    with pytest.raises(Bd.ChironError) as e:
        five = lambda t: torch.cat([t, t[:1]]).contiguous()
        Bd.decode_step(g.model, g.pool, five(g.block_table), five(g.seq_lens), five(g.tokens), batch=5,
                       logits=torch.empty((5, 1024), device="cuda"))
    assert e.value.code == -3
    # the binding itself refuses a block table whose row stride is not the model's, or with too few rows
    with pytest.raises(ValueError):
        Bd.decode_step(g.model, g.pool, g.block_table[:, :-1].contiguous(), g.seq_lens, g.tokens)
    with pytest.raises(ValueError):
        Bd.decode_step(g.model, g.pool, g.block_table[:3].contiguous(), g.seq_lens, g.tokens)
    bad = g.block_table.clone(); bad[2, 0] = g.pool.num_blocks + 3
    with pytest.raises(Bd.ChironError) as e:
        Bd.validate_step_inputs(g.model, g.pool, bad, g.seq_lens, g.tokens)
    assert e.value.code == -4
    badtok = g.tokens.clone(); badtok[1] = 1024
    with pytest.raises(Bd.ChironError) as e:
        Bd.validate_step_inputs(g.model, g.pool, g.block_table, g.seq_lens, badtok)
    assert e.value.code == -7
    # the fused gate/up matrix: widths, pairing and use are checked on the host before anything is launched
    import ctypes as C
    W = I.normal((48, 64), 0.05, 7, "e_w").cuda()
    with pytest.raises(Bd.ChironError) as e:
        Bd.GateUp(W[:40].contiguous(), W[:40].contiguous())  # 40 columns: not a multiple of 16
    assert e.value.code == -2
    gu, plain, narrow = Bd.GateUp(W, W), Bd.Linear(I.normal((32, 48), 0.05, 7, "e_d").cuda()), Bd.Linear(I.normal((32, 64), 0.05, 7, "e_n").cuda())
    x = torch.zeros((3, 64), dtype=torch.float32, device="cuda")
    y = torch.zeros((3, 96), dtype=torch.float32, device="cuda")
    lib = Bd.load()
    ptr = lambda t: C.c_void_p(t.data_ptr())
    assert lib.chiron_op_linear(gu._h, ptr(x), C.c_int32(3), ptr(y), C.c_int32(0), None) == -1      # no plain product of it
    assert lib.chiron_op_gate_up_swiglu(plain._h, ptr(x), C.c_int32(3), ptr(y), None) == -1         # not a gate/up matrix
    with pytest.raises(Bd.ChironError) as e:
        gu.ffn(narrow, x)                                                                            # 48 columns into 64 inputs
    assert e.value.code == -2
    with pytest.raises(Bd.ChironError) as e:
        gu.ffn(gu, x)                                                                                # a gate/up matrix as the down projection
    assert e.value.code == -1
    assert gu.ffn(plain, x).shape == (3, 32) and float(gu.ffn(plain, x).abs().max()) == 0.0        # silu(0) * 0 = 0
    for l in (gu, plain, narrow):
        l.close()


@pytest.mark.parametrize("M,N,K", [(33, 512, 512), (384, 4096, 2048), (500, 2722, 464), (1455, 448, 1040), (160, 3000, 4096), (97, 6144, 512), (385, 6144, 4112),
                                   (640, 8224, 1040), (1025, 3072, 2064), (512, 8192, 48), (40, 2048, 2048), (686, 1955, 1136), (2000, 96, 6160),
                                   (600, 28640, 80), (1290, 12300, 48)])  # 128 x 512 tiles with the last round in halves
def test_linear_shapes_by_estimate(M, N, K):
    """widths and row counts between those that the launch shapes were swept at, where the estimated time decides: slices or none, ragged
    rows and columns; alone, added to y, and as the two halves of a feed-forward block (K of which is the narrow side).  Which tile it
    takes is its own affair: test_linear_of_every_tile has every one by name."""
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    x = rng.standard_normal((M, K)).astype(np.float32)
    W = I.normal((N, K), 0.05, 12, "wse", N, K)
    print("linear by estimate", M, N, K, flush=True)
    lin = B().Linear(W.cuda())
    want = orc.linear(x, I.to_numpy_storage(W))
    y0 = rng.standard_normal((M, N)).astype(np.float32)
    assert rel_err(lin(torch.from_numpy(x).cuda()).cpu().numpy(), want) <= KERNEL_TOL
    assert rel_err(lin(torch.from_numpy(x).cuda(), torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy(), want + y0) <= KERNEL_TOL
    lin.close()
    F, H = N // 16 * 16, min(K, 528)
    xs, Wg, Wu, Wd, _, want = ffn_case(M, H, F, 272, M + N)
    gu, down = B().GateUp(Wg.cuda(), Wu.cuda()), B().Linear(Wd.cuda())
    assert rel_err(gu.ffn(down, torch.from_numpy(xs).cuda()).cpu().numpy(), want) <= KERNEL_TOL
    gu.close(); down.close()


@pytest.mark.parametrize("M,K,F,N", [(1, 16, 16, 16), (16, 272, 4096, 4112), (3, 2064, 8192, 8192), (9, 1040, 4112, 100), (16, 2048, 8208, 9216), (12, 2320, 48, 5120)])
def test_few_rows_gate_up_and_two_column_tiles(M, K, F, N):
    """gate/up by the few-row kernel with SwiGLU in its epilogue (up to one round of 32-column tiles, 4096 columns, two at K >= 2048,
    and what lies past either), and outputs of 4097 .. 8192 columns, whose workgroups take two column tiles"""
    x, Wg, Wu, Wd, _, want = ffn_case(M, K, F, N, M + K + F)
    b = B()
    gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
    print("few gate/up", M, K, F, N, flush=True)
    assert rel_err(gu.ffn(down, torch.from_numpy(x).cuda()).cpu().numpy(), want) <= KERNEL_TOL
    gu.close(); down.close()


@pytest.mark.parametrize("M,K,F,N", [(17, 16, 16, 17), (32, 272, 688, 4096), (31, 1040, 48, 4112), (17, 2064, 4096, 2048), (32, 4096, 16, 96), (24, 5008, 16, 48)])
def test_few_rows_two_row_tiles(M, K, F, N):
    """17 .. 32 rows of a projection and a feed-forward block: one and two column tiles, whole rings of k-steps, a remainder, a last
    step past K, and widths past the range, against the oracle"""
    x, Wg, Wu, Wd, _, want = ffn_case(M, K, F, N, M + K + F)
    b = B()
    gu, down, lin = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda()), b.Linear(Wg.cuda())
    print("two row tiles", M, K, F, N, flush=True)
    assert rel_err(gu.ffn(down, torch.from_numpy(x).cuda()).cpu().numpy(), want) <= KERNEL_TOL
    y0 = np.random.default_rng(M).standard_normal((M, F)).astype(np.float32)
    wg = orc.linear(x, I.to_numpy_storage(Wg))
    assert rel_err(lin(torch.from_numpy(x).cuda()).cpu().numpy(), wg) <= KERNEL_TOL
    assert rel_err(lin(torch.from_numpy(x).cuda(), torch.from_numpy(y0).cuda(), accumulate=True).cpu().numpy(), wg + y0) <= KERNEL_TOL
    gu.close(); down.close(); lin.close()


@pytest.mark.parametrize("over,batch,T,norms", [({}, 17, 1, 1), (dict(hidden=1040, ffn=2832, vocab=16416), 16, 2, 1),
                                                (dict(hidden=272, n_kv_heads=4), 31, 1, 1), (dict(hidden=2048, ffn=5632), 32, 1, 3)])
def test_step_of_two_row_tiles(over, batch, T, norms):
    """steps of 17 .. 32 rows against the oracle: layers by the few-row kernel and a head behind a norm of its own, a width past that range,
    and each by the general path, to which the distance is that of fp32 rounding"""
    c = make_case(m=dict(I.TINY, n_layers=1, **over), batch=batch, kind="tiny", seed=53, storage="bf16", gain_jitter=0.2)
    lens = (c.seq_lens - T).astype(np.int32)
    c.seq_lens = lens  # room for T new tokens in the pages that are there
    c.seq_idx, c.pos = I.prefill_index(lens)
    c.kv_t = [I.make_kv_layer(c.m, int(lens.sum()), 0, seed=53, dtype=torch.bfloat16)]
    c.kv = [(I.to_numpy_storage(k), I.to_numpy_storage(v)) for k, v in c.kv_t]
    g = gpu_setup(c, max_batch=batch * T)
    b = B()
    toks = np.random.default_rng(3).integers(0, c.m["vocab"], (batch, T)).astype(np.int32)
    want = orc.decode_step_multi(c.cfg, c.w, fresh_pool(c), c.block_table, lens, toks).reshape(batch * T, -1)
    out = []
    for mt in (0, 1):
        print("two row tiles", over, batch, T, "mt", mt, flush=True)
        with pinned(mt):
            lg, n = norm_launches(g, lambda: b.decode_step_multi(g.model, g.pool, g.block_table, g.seq_lens, torch.from_numpy(toks).cuda()))
        assert n == (3 if mt else norms)
        out.append(lg.cpu().numpy().reshape(batch * T, -1))
        check_logits(out[-1], want, min_agree=1.0 - 1.0 / batch)
    assert np.abs(out[0] - out[1]).max() <= 2e-3 * out[1].std()


def test_the_two_term_form_can_be_asked_for_at_few_rows():
    """linear_big_min_m within 17 .. 32 rows: from there on a feed-forward block takes the tiled two-term form, and a step the path that may
    (a model made for so few rows has no workspace for it), not the few-row kernel"""
    c = make_case(m=dict(I.TINY, n_layers=1), batch=20, kind="tiny", seed=59, storage="bf16", gain_jitter=0.2)
    g = gpu_setup(c)
    x, Wg, Wu, Wd, _, want_ffn = ffn_case(20, 272, 688, 256, 5)
    b = B()
    gu, down = b.GateUp(Wg.cuda(), Wu.cuda()), b.Linear(Wd.cuda())
    for start, norms in ((0, 1), (21, 1), (20, 3)):
        print("two-term form from", start, flush=True)
        b.set_tuning("linear_big_min_m", start)
        try:
            (_, got, want, _), n = norm_launches(g, lambda: run_both(c, g))
            y = gu.ffn(down, torch.from_numpy(x).cuda()).cpu().numpy()
        finally:
            b.set_tuning("linear_big_min_m", 0)
        assert n == norms
        check_logits(got, want, min_agree=0.95)
        assert rel_err(y, want_ffn) <= KERNEL_TOL
    gu.close(); down.close()


@pytest.mark.parametrize("over,batch", [(dict(vocab=8192), 16), (dict(vocab=8208), 3), (dict(hidden=2064, ffn=4112, vocab=16384), 9), (dict(hidden=4624, ffn=32, vocab=96), 2)])
def test_step_of_few_rows_with_narrow_gate_up_and_head(over, batch):
    """steps whose gate/up and head are products of the few-row kernel too (one round of 32-column tiles, two at K >= 2048), and the
    widths behind them, against the oracle"""
    c = make_case(m=dict(I.TINY, n_layers=1, **over), batch=batch, kind="tiny", seed=47, storage="bf16", gain_jitter=0.2)
    print("few head", over, batch, flush=True)
    g = gpu_setup(c)
    (_, got, want, _), norms = norm_launches(g, lambda: run_both(c, g))
    assert norms == 0  # the few-row path
    check_logits(got, want, min_agree=1.0 - 1.0 / batch)


@pytest.mark.parametrize("m,batch", [(I.TINY, 1), (I.TINY, 16), (I.TINY, 32), (G4_D128, 5)])
def test_few_row_rotation_rounds_one_product(m, batch):
    """The QKV projection of few rows rotates with one product rounded and the other inside a fused multiply-add.  Every rotary pair
    is an exact number of 24 bits (three bf16 weights against inputs of one) that its angle all but cancels, so what is left is the
    rounding itself: the new K has to be the bf16 value of fma(x, cos, -+round(y sin))."""
    m = dict(m, n_layers=1, rms_eps=1e-12)
    H, d, nkv = m["hidden"], m["head_dim"], m["n_kv_heads"]
    half, pos = d // 2, 77
    rng = np.random.default_rng(5)
    ang = pos * float(m["rope_base"]) ** (-2.0 * np.arange(half) / d)
    cs, sn = np.cos(ang).astype(np.float32), np.sin(ang).astype(np.float32)
    x = rng.uniform(1, 2, (nkv, half)).astype(np.float32)
    y = np.empty_like(x)
    y[::2] = x[::2].astype(np.float64) * cs / sn   # x cos - y sin is next to nothing (the pair's first half)
    y[1::2] = -x[1::2].astype(np.float64) * sn / cs  # y cos + x sin is (its second half)
    want_k = np.concatenate([x, y], 1)  # [nkv, d], before the rotation
    c = make_case(m=m, kind="tiny", seed=3, storage="bf16", seq_lens=[pos] * batch)
    wk = torch.zeros((nkv * d, H))
    rest = torch.from_numpy(want_k.reshape(-1).copy())
    for t in range(3):
        wk[:, t] = rest.to(torch.bfloat16).float()
        rest = rest - wk[:, t]
    assert not rest.any()
    c.w_t["wk"] = [wk.to(torch.bfloat16)]
    for n in ("embed", "final_norm"):
        c.w_t[n] = torch.ones_like(c.w_t[n])
    c.w_t["attn_norm"] = [torch.ones_like(c.w_t["attn_norm"][0])]
    g = gpu_setup(c)
    print("rotation of few rows", batch, flush=True)
    _, norms = norm_launches(g, lambda: B().decode_step(g.model, g.pool, g.block_table, g.seq_lens, g.tokens))
    assert norms == (batch > 16)  # the few-row path

    def fma(a, cos, prod):  # exact products of 48 bits, a sum of 64
        return (a.astype(np.longdouble) * cos + prod.astype(np.longdouble)).astype(np.float32)
    want = np.concatenate([fma(x, cs, -(y * sn)), fma(y, cs, x * sn)], 1)
    want = torch.from_numpy(want).to(torch.bfloat16)
    split = torch.from_numpy(np.concatenate([x * cs - y * sn, y * cs + x * sn], 1)).to(torch.bfloat16)
    assert float((split != want).float().mean()) > 0.2  # (two rounded products would show)
    for i in range(batch):
        k, _ = g.pool.gather(0, g.block_table[i].contiguous(), pos + 1)
        assert np.array_equal(bits(k[pos]), bits(want)), i
