"""Kernels at the edges of their tiles, tables and dispatch ranges, against the oracle or a plain fp32 reference."""
import ctypes as C

import numpy as np
import pytest
import torch

import csd_inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_11462_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("n", [2, 3, 1024, 1025, 2049, 8191, 8192])
@pytest.mark.parametrize("text", ["one_token", "two_tokens", "few", "all_distinct", "bad_ids"])
def test_bigram_fit_tables(P, n, text):
    """The hash tables of the fit: every pair in one slot, every pair in its own, positions at and across a thread's
    share, ids outside the vocabulary (their pairs do not count).  Whole numbers: bit-exact."""
    from oracle import csd_oracle as O
    V = 9000
    r = np.random.RandomState(n)
    s = {"one_token": lambda: np.full(n, 5), "two_tokens": lambda: r.randint(0, 2, n), "few": lambda: r.randint(0, 40, n),
         "all_distinct": lambda: r.permutation(V)[:n], "bad_ids": lambda: r.randint(-3, 30, n)}[text]().astype(np.int32)
    vocab = 25 if text == "bad_ids" else V
    default = I.default_next_table(vocab, 3)
    if text == "bad_ids":
        want, best = default.numpy().copy(), {}
        ok = [(int(a), int(b)) for a, b in zip(s[:-1], s[1:]) if 0 <= a < vocab and 0 <= b < vocab]
        count = {x: ok.count(x) for x in set(ok)}
        for a, b in ok:                                      # in order: among equal counts the pair seen latest stays
            if count[a, b] >= best.get(a, 0):
                best[a], want[a] = count[a, b], b
    else:
        want = O.bigram_fit(s, vocab, default.numpy())
    got = P.bigram_fit(torch.from_numpy(s).cuda(), vocab, default.cuda().clone())
    assert np.array_equal(got.cpu().numpy(), want)


BF = I.ModelShape("edge_dh64", 0, "bf16", 2, 256, 4, 64, 512, 1024)
BF128 = I.ModelShape("edge_dh128", 0, "bf16", 2, 256, 2, 128, 480, 1040)


@pytest.mark.parametrize("n,room", [(1, 0), (2, 254), (256, 0), (256, 1), (511, 1), (513, 0), (1024, 300), (4096, 1), (4097, 0), (8192, 5), (8193, 0), (9000, 60), (1, 3000), (200, 1848),
                                    (200, 1849), (2048, 0), (2048, 1), (2049, 0)])
@pytest.mark.parametrize("max_match", [0, 3])
def test_draft_of_long_and_short_sequences(P, n, room, max_match):
    """Either side of what one workgroup size or the other takes, in tokens and in room for them, and of what LDS holds; drafts given and drafts
    appended to the sequences (a sequence without room for them is left alone)."""
    from oracle import csd_oracle as O
    vocab, k = 50, 9
    rng = np.random.default_rng(n + room)
    ctx = rng.integers(0, vocab, (2, n + room)).astype(np.int32)
    ctx[1, :n] = np.arange(n) % 49                           # a long period; and a suffix that is nowhere else
    ctx[1, n - 1] = 49
    table = rng.integers(0, vocab, vocab).astype(np.int32)
    got, length = P.bigram_draft(torch.from_numpy(ctx).cuda(), torch.full((2,), n, dtype=torch.int32, device="cuda"), torch.from_numpy(table).cuda(), k,
                                 max_match=max_match)
    want, want_len = O.bigram_draft(ctx, [n, n], table, k, max_match=max_match)
    assert np.array_equal(got.cpu().numpy(), want) and np.array_equal(length.cpu().numpy(), want_len)
    dev, dev_len = torch.from_numpy(ctx).cuda(), torch.full((2,), n, dtype=torch.int32, device="cuda")
    P.bigram_draft_append(dev, dev_len, torch.from_numpy(table).cuda(), k, max_match=max_match)
    if n + k < ctx.shape[1]:
        ctx[:, n:n + k] = want
    assert np.array_equal(dev.cpu().numpy(), ctx) and (dev_len == (n + k if n + k < ctx.shape[1] else n)).all()


@pytest.mark.parametrize("shape", [BF, BF128], ids=["dh64", "dh128"])
@pytest.mark.parametrize("B,m", [(1, 145), (1, 192), (1, 193), (1, 256), (1, 257), (1, 288), (1, 289), (2, 100), (3, 173)])
def test_tall_blocks(P, shape, B, m):
    """The GEMMs over many rows: one row more than the row-split form takes, whole and ragged blocks of 96 and of 128 rows, rows of several
    sequences in one row tile, column tiles that do not fill a workgroup.  Tolerances: the project's (bf16)."""
    from gpu_util import make_pair, prefill_both, tol_ok
    gm, om = make_pair(shape, 17, B, 40 + m, m, std=0.05)
    toks = I.token_ids(B * (m + 30), shape.vocab, 17, 1).reshape(B, m + 30)
    prefill_both(gm, om, toks[:, :30], 15)
    cl = np.asarray([30 - 7 * b for b in range(B)], np.int32)
    block = np.stack([toks[b, cl[b]:cl[b] + m].numpy() for b in range(B)]).astype(np.int32)
    tr = torch.zeros((shape.n_layers + 1, B * m, shape.d_model), dtype=torch.float32, device="cuda")
    gm.set_trace(tr)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    gm.set_trace(None)
    ref, otr = om.verify_block(block, cl, trace=True)
    for l in range(shape.n_layers + 1):
        g = tr.cpu().numpy()[l, :m].astype(np.float64)
        assert np.linalg.norm(g - otr[l]) < 5e-3 * np.linalg.norm(otr[l])
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), ref, 2e-2, 1e-2)
    assert ok, f"max abs err {err}"
    for b in range(B):
        for got, want in zip(gm.kv_read(1, b, 0, int(cl[b]) + m), om.kv_read(1, b, 0, int(cl[b]) + m)):
            ok, err = tol_ok(got.cpu().numpy().astype(np.float64), want, 2e-2, 1e-2)
            assert ok, f"cache rows of sequence {b}: max abs err {err}"


@pytest.mark.parametrize("m", [192, 256, 384, 512])
def test_tall_tile_forms(P, m):
    """Matrices wide enough that the plan takes wide tiles of several heights, and two workgroups per compute unit (the
    shapes above all go to the narrowest).  Tolerances: the project's (bf16)."""
    from gpu_util import make_pair, tol_ok
    shape = I.ModelShape("edge_forms", 0, "bf16", 1, 512, 16, 128, 6144, 32000)
    gm, om = make_pair(shape, 19, 1, m + 3, m, std=0.05)
    block = I.token_ids(m, shape.vocab, 19, 1).reshape(1, m).numpy().astype(np.int32)
    cl = np.zeros(1, np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


def _tall_plan(P, N, K, rows, split):
    """(column tiles, row tiles, stages, K splits) of a GEMM over many rows; split: it writes partial sums, in as many splits as
    the matrix has been packed for at most."""
    S = 1
    while split and N // 16 * S < 2048 and K // 32 // (2 * S) >= 8 and S < 8:
        S *= 2
    v = [C.c_int32() for _ in range(4)]
    assert P.lib().csd_debug_tall_plan(N, K, rows, S, *[C.byref(x) for x in v]) == 0
    return tuple(x.value for x in v)


def _check_cache(gm, om, layers, b, n):
    from gpu_util import tol_ok
    for l in range(layers):
        for got, want in zip(gm.kv_read(l, b, 0, n), om.kv_read(l, b, 0, n)):
            ok, err = tol_ok(got.cpu().numpy().astype(np.float64), want, 2e-2, 1e-2)
            assert ok, f"cache rows of sequence {b}, layer {l}: max abs err {err}"


@pytest.mark.parametrize("dims,m,t,want", [
    ((256, 2, 64, 512, 1024), 154, 37, {"qkv": (4, 2, 4), "gu": (4, 2, 4)}),
    ((512, 32, 128, 6144, 16384), 146, 201, {"qkv": (4, 3, 4), "gu": (4, 3, 4), "lm": (4, 3, 4), "o": (4, 2, 4, 8)}),
    ((512, 32, 128, 6144, 4096), 201, 64, {"qkv": (6, 2, 3), "gu": (6, 2, 3), "lm": (4, 2, 4)}),
    ((768, 24, 128, 8192, 16384), 473, 15, {"qkv": (6, 3, 3), "gu": (6, 3, 2), "lm": (6, 3, 2), "down": (4, 3, 4, 8)}),
    ((512, 2, 128, 6144, 32000), 325, 500, {"gu": (6, 3, 3), "lm": (6, 4, 2)}),
    ((1024, 32, 128, 6144, 1024), 487, 33, {"qkv": (6, 4, 3), "gu": (6, 4, 3)}),
    ((512, 4, 64, 11008, 1024), 451, 300, {"gu": (6, 4, 2)}),
    ((768, 32, 128, 512, 1024), 527, 9, {"qkv": (6, 3, 2)}),
    ((512, 64, 128, 512, 512), 385, 21, {"qkv": (6, 4, 2)}),
    ((2048, 1, 64, 4096, 512), 516, 5, {"down": (4, 4, 4, 3)})], ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else None)
def test_tall_tile_form_of_every_epilogue(P, dims, m, t, want):
    """Every pair of tile form and epilogue that matrices of ordinary shapes lead to, by the plan's own word: ragged row counts
    over a cache that is not empty, logits and cache rows.  Tolerances: the project's (bf16)."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    d, H, dh, F, V = dims
    hd = H * dh
    plans = {"qkv": (3 * hd, d, m, False), "o": (d, hd, m, True), "gu": (2 * F, d, m, False), "down": (d, F, m, True), "lm": (V, d, m, False)}
    for k, form in want.items():
        assert _tall_plan(P, *plans[k])[:len(form)] == form, k
    shape = I.ModelShape("edge_forms", 0, "bf16", 1, d, H, dh, F, V)
    gm, om = make_pair(shape, 19, 1, t + m + 3, m, std=0.05)
    import_synthetic_kv(gm, om, shape, t, 19)
    block = I.token_ids(m, shape.vocab, 19, 1).reshape(1, m).numpy().astype(np.int32)
    cl = np.full(1, t, np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"
    _check_cache(gm, om, 1, 0, t + m)


@pytest.mark.parametrize("dims,B,m,want", [
    ((256, 2, 64, 512, 1024), 2, 73, {(4, 2, 4)}),
    ((512, 32, 128, 4096, 32128), 1, 321, {(4, 3, 4), (6, 3, 3), (6, 4, 2)}),
    ((1024, 32, 128, 8192, 32128), 1, 208, {(4, 4, 4), (6, 2, 3), (6, 3, 2)}),
    ((1024, 32, 128, 512, 1024), 1, 497, {(6, 4, 3)}),
    ((256, 16, 64, 512, 1024), 1, 203, {(4, 2, 4)})], ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else None)
def test_tall_blocks_of_the_encoder_decoder(P, dims, B, m, want):
    """arch 1 blocks of more than 144 rows: every GEMM writes partial sums, in every form; attention with the distance bias over
    many row tiles and cached rows (the last shape on single key tiles per request)."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    d, H, dh, F, V = dims
    hd, M = H * dh, B * m
    assert want <= {_tall_plan(P, N, K, M, True)[:3] for N, K in ((3 * hd, d), (d, hd), (hd, d), (2 * F, d), (d, F), (V, d))}
    t = 161
    shape = I.ModelShape("edge_t5_tall", 1, "bf16", 1, d, H, dh, F, V, rms_eps=1e-6, enc_len=70)
    gm, om = make_pair(shape, 53, B, 760, m, std=0.05)
    enc = I.encoder_output(shape, B, 53)
    gm.cross_kv_init(enc.cuda())
    om.cross_kv_init(enc.numpy())
    import_synthetic_kv(gm, om, shape, t, 53, B=B)
    block = I.token_ids(M, V, 53, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([t - 30 * b for b in range(B)], np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"
    for b in range(B):
        _check_cache(gm, om, 1, b, int(cl[b]) + m)


@pytest.mark.parametrize("d,H,dh,B,enc_len,form", [(512, 32, 128, 1, 257, (4, 3, 4)), (1024, 32, 128, 1, 385, (4, 4, 4)),
                                                   (1024, 32, 128, 2, 251, (4, 4, 4))])
def test_cross_projection_tile_forms(P, d, H, dh, B, enc_len, form):
    """The encoder projection in the taller tiles, ragged; (4, 2, 4) is what test_cross_projection_rows takes."""
    from gpu_util import make_pair, tol_ok
    assert _tall_plan(P, 2 * H * dh, d, B * enc_len, False)[:3] == form
    shape = I.ModelShape("edge_cross", 1, "bf16", 1, d, H, dh, 256, 512, rms_eps=1e-6, enc_len=enc_len)
    gm, om = make_pair(shape, 59, B, 32, 8, std=0.05)
    enc = I.encoder_output(shape, B, 59)
    gm.cross_kv_init(enc.cuda())
    om.cross_kv_init(enc.numpy())
    block = I.token_ids(B * 5, shape.vocab, 59, 1).reshape(B, 5).numpy().astype(np.int32)
    cl = np.zeros(B, np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("H,dh,m,t,max_seq", [(12, 64, 200, 0, 1024), (12, 64, 331, 431, 1024), (16, 64, 512, 477, 1024), (12, 128, 200, 311, 1024),
                                              (16, 128, 512, 389, 1024)])
def test_attention_of_tall_blocks(P, H, dh, m, t, max_seq):
    """So many row tiles that a wave requests one key tile at a time: row tiles that see few of the chunk's keys, several chunks,
    an odd number of cached rows, one row in the last tile."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    assert H * ((m + 15) // 16) * (max_seq // 128) > 1024
    shape = I.ModelShape("edge_tall_attn", 0, "bf16", 1, 256, H, dh, 128, 512)
    gm, om = make_pair(shape, 61, 1, max_seq, m, std=0.05)
    if t:
        import_synthetic_kv(gm, om, shape, t, 61)
    block = I.token_ids(m, shape.vocab, 61, 1).reshape(1, m).numpy().astype(np.int32)
    cl = np.full(1, t, np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("H,dh", [(12, 64), (8, 128)])
@pytest.mark.parametrize("B,m", [(8, 40), (3, 64), (6, 25)])
def test_tree_blocks_of_many_rows(P, H, dh, B, m):
    """Tree blocks of several sequences, more than 144 rows in all: rotation by depth in the epilogue of the tall GEMM, ancestor masks of
    several sequences in one launch, ragged cached lengths, logits and cache rows."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    shape = I.ModelShape("edge_tree", 0, "bf16", 1, 256, H, dh, 512, 1024)
    gm, om = make_pair(shape, 67, B, 512, m, std=0.05)
    import_synthetic_kv(gm, om, shape, 333, 67, B=B)
    r = np.random.RandomState(m)
    parent = np.stack([np.asarray([-1] + [r.randint(max(0, i - 7), i) for i in range(1, m)]) for _ in range(B)]).astype(np.int32)
    block = I.token_ids(B * m, shape.vocab, 67, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([333 - 41 * b for b in range(B)], np.int32)
    lg = gm.verify_tree(torch.from_numpy(block).cuda(), torch.from_numpy(parent).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_tree(block, parent, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"
    for b in (0, B - 1):
        _check_cache(gm, om, 1, b, int(cl[b]) + m)


@pytest.mark.parametrize("dh,path", [(64, "multikernel"), (128, "multikernel"), (32, "default")])
@pytest.mark.parametrize("B,m", [(1, 150), (2, 130)])
def test_tall_blocks_with_epilogue_kernels(P, monkeypatch, dh, path, B, m):
    """More than 144 rows where the GEMMs write partial sums for epilogue kernels: the forward with one kernel per operation when
    it is asked for, and models whose head size leaves the attention to the generic kernel."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    monkeypatch.setenv("CSD_PATH", path)
    shape = I.ModelShape("edge_unfused", 0, "bf16", 2, 256, 256 // dh, dh, 512, 1024)
    gm, om = make_pair(shape, 71, B, m + 60, m, std=0.05)
    import_synthetic_kv(gm, om, shape, 51, 71, B=B)
    block = I.token_ids(B * m, shape.vocab, 71, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([51 - 20 * b for b in range(B)], np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"
    for b in range(B):
        _check_cache(gm, om, 2, b, int(cl[b]) + m)


@pytest.mark.parametrize("m", [20, 145])
def test_planes_of_more_than_two_gib(P, m):
    """Room for 4096 rows of 196608 features: both planes of the feed-forward input take 3.2 GB.  The lower plane carries the bits
    behind the first eight: without it the feed-forward sums are off by about 2^-9 of their size, with it by 2^-17, and a K or V
    element rounded to the other side adds 1e-5 or so."""
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GiB of device memory")
    shape = I.ModelShape("edge_wide", 0, "bf16", 1, 32, 1, 64, 196608, 64)
    from oracle import csd_oracle as O
    w = I.make_weights(shape, 47, device="cuda", std=0.05)
    gm = P.Model(shape, w, max_batch=8, max_seq=512, max_block=512)
    om = O.Model(shape, [x.cpu() for x in w], max_batch=1, max_seq=512, max_block=m)
    assert gm.path(1, m) == 0
    block = I.token_ids(m, shape.vocab, 47, 1).reshape(1, m).numpy().astype(np.int32)
    cl = np.zeros(1, np.int32)
    got = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda()).cpu().numpy().astype(np.float64)
    ref = om.verify_block(block, cl)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print("m", m, "relative error", err)
    gm.close()
    assert err < 1e-4


def _head_alone(P, K, V, rows, emb, lm, gain=None):
    """Logits of a model of one layer that adds nothing to its input: the LM head over the embedding rows 0 .. rows - 1."""
    shape = I.ModelShape("edge_head", 0, "bf16", 1, K, 1, 64, 64, V)
    z = lambda r, c: torch.zeros((r, c), dtype=torch.bfloat16, device="cuda")
    one = torch.ones(K, device="cuda")
    gm = P.Model(shape, [emb, one, z(K, 64), z(K, 64), z(K, 64), z(64, K), one, z(K, 64), z(K, 64), z(64, K), one if gain is None else gain, lm],
                 max_batch=1, max_seq=rows, max_block=rows)
    out = gm.verify_block(torch.arange(rows, dtype=torch.int32, device="cuda")[None], torch.zeros(1, dtype=torch.int32, device="cuda"))[0]
    gm.close()
    return out


@pytest.mark.parametrize("K,V,m", [(4096, 4096, 145), (4096, 4096, 512), (4096, 22016, 384), (4096, 22016, 512), (4096, 32000, 512),
                                   (768, 32000, 300), (1024, 4096, 200), (16384, 1024, 160), (16384, 12304, 512)])
def test_tall_sums_are_no_further_from_64_bits_than_row_split_ones(P, K, V, m):
    """Sums over K of the GEMM over many rows (accumulators beside a second set of sums; the form that sets upper halves aside:
    22016 columns at 512 rows) against 64 bits, beside the same rows on the row-split form.  The embedding rows are bf16, so the
    planes hold them exactly and what is left is the rounding of the sums, 2 to 5 units of 2^-24 of their size here; the scale of a
    row (one rounded number) is taken out.  Two draws of a row set differ by 1 % at most; one chain through all of K is 40 % to
    190 % above the row-split form.  That form by itself: a chain of K / 32 steps, whose sums grow as the square root, each rounded by 0.29 to 0.58 units
    of its size, ends within 0.58 sqrt(K / 64) of the last one's size, and the splits leave shorter ones; a sum that misses one step of K / 32 is off by 10^5 units."""
    g = torch.Generator(device="cuda").manual_seed(K + V)
    emb = torch.empty((V, K), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    lm = torch.empty((K, V), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)

    def error(rows):
        x = emb[:rows].double()
        ref = (x @ lm.double()) * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5)
        got = _head_alone(P, K, V, rows, emb, lm).double()
        got *= ((got * ref).sum(-1) / (got * got).sum(-1))[:, None]
        return ((got - ref).norm() / ref.norm()).item() * 2 ** 24

    split, tall = error(128), error(m)
    print(K, V, m, "row-split", split, "tall", tall)
    assert split < 1 + 0.58 * (K / 64) ** 0.5
    assert tall < 1.03 * split


def _rows_plan(P, N, K, rows):
    v = [C.c_int32(), C.c_int32()]
    assert P.lib().csd_debug_gemm_plan(N, K, rows, 8, *[C.byref(x) for x in v]) == 0
    return tuple(x.value for x in v)


@pytest.mark.parametrize("K,V,plan", [(96, 528, (6, 1)), (544, 12304, (8, 2)), (4096, 4096, (8, 8)), (4096, 22016, (11, 2)), (4096, 12288, (12, 4)),
                                      (768, 32000, (16, 2))])
@pytest.mark.parametrize("m", [33, 48, 49, 64, 65, 96, 97, 128, 129, 144])
def test_row_split_sums(P, K, V, plan, m):
    """The GEMM over 33 to 144 rows in each of its forms: the five widths, one to three row tiles on three or four waves with the first and last
    row count of each, K slices shorter than the stages in flight, slices that end inside a turn, and ragged column groups.  A sum of K
    exact products in 32 bits is within K 2^-23 of the sum of their sizes, the scale of the row and the partial sums add a few units."""
    assert _rows_plan(P, V, K, m) == plan
    g = torch.Generator(device="cuda").manual_seed(K + m)
    emb = torch.empty((V, K), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    lm = torch.empty((K, V), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    x = emb[:m].double()
    rstd = torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5)
    ref, size = (x @ lm.double()) * rstd, (x.abs() @ lm.double().abs()) * rstd
    got = _head_alone(P, K, V, m, emb, lm).double()
    assert ((got - ref).abs() <= (K + 16) * 2.0 ** -23 * size).all()


@pytest.mark.parametrize("steps", [1, 2, 4, 5, 6, 7, 8, 9, 10, 11])
@pytest.mark.parametrize("m", [40, 64, 72, 96, 104, 136])
def test_row_split_sums_of_every_remainder(P, steps, m):
    """Slices of K of every length modulo the four k-steps in flight, from one k-step on, with and without a whole turn before the last."""
    K = 32 * steps
    assert _rows_plan(P, 528, K, m) == (6, 1)
    test_row_split_sums(P, K, 528, (6, 1), m)


@pytest.mark.parametrize("K,V", [(64, 528), (768, 4112), (4096, 8208)])
@pytest.mark.parametrize("m", [1, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32])
def test_few_row_sums(P, K, V, m):
    """The GEMM over up to 32 rows at either side of half a row tile, where one fragment holds both planes of the last rows, with inputs
    that need the lo plane (rows times a gain of 24 bits).  The planes hold an input to 2^-17 of its size; a sum of K products of either
    plane in 32 bits is within K 2^-23 of the sum of their sizes."""
    g = torch.Generator(device="cuda").manual_seed(K + m)
    emb = torch.empty((V, K), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    lm = torch.empty((K, V), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    gain = torch.rand(K, generator=g, device="cuda") + 0.5
    x = emb[:m].double()
    rstd = torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5)
    x = x * gain.double()
    ref, size = (x @ lm.double()) * rstd, (x.abs() @ lm.double().abs()) * rstd
    got = _head_alone(P, K, V, m, emb, lm, gain).double()
    assert ((got - ref).abs() <= ((K + 16) * 2.0 ** -23 + 2.0 ** -17) * size).all()


@pytest.mark.parametrize("arch,dh", [(0, 64), (1, 64), (0, 128)])
@pytest.mark.parametrize("B,m", [(1, 8), (1, 9), (4, 2), (3, 8), (5, 5)])
def test_blocks_of_half_row_tiles(P, arch, dh, B, m):
    """Every epilogue over 8, 9, 24 and 25 rows, of one sequence and of several, on the forward with its epilogues inside the GEMMs."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    shape = I.ModelShape("edge_half", arch, "bf16", 2, 192, 3, dh, 320, 512, rms_eps=1e-6 if arch else 1e-5, enc_len=20 if arch else 0)
    gm, om = make_pair(shape, 47, B, 96, m, std=0.05)
    import_synthetic_kv(gm, om, shape, 40, 47, B=B)
    if arch:
        enc = I.encoder_output(shape, B, 47)
        gm.cross_kv_init(enc.cuda())
        om.cross_kv_init(enc.numpy())
    block = I.token_ids(B * m, shape.vocab, 47, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([40 - 3 * b for b in range(B)], np.int32)
    assert gm.path(B, m) == 1
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"
    for b in range(B):
        for got, want in zip(gm.kv_read(1, b, 0, int(cl[b]) + m), om.kv_read(1, b, 0, int(cl[b]) + m)):
            ok, err = tol_ok(got.cpu().numpy().astype(np.float64), want, 2e-2, 1e-2)
            assert ok, f"cache rows of sequence {b}: max abs err {err}"


@pytest.mark.parametrize("V,m", [(22016, 512), (4096, 512)])
def test_tall_sums_that_overflow(P, V, m):
    """Infinite products, sums that leave the range within a part of K and only when parts are added, infinities of both signs: the
    same infinities and NaN as on the row-split form, and no other column touched."""
    K = 4096
    g = torch.Generator(device="cuda").manual_seed(7)
    emb = torch.empty((V, K), dtype=torch.bfloat16, device="cuda").normal_(0, 1e15, generator=g)
    lm = torch.empty((K, V), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    emb[:, [5, 9, 3000, 4000]] = 1e15
    for col, at in enumerate([{5: 1e25}, {4000: -1e25}, {5: 1e25, 4000: -1e25}, {5: 2.5e23, 9: 2.5e23}, {5: 2.5e23, 4000: 2.5e23},
                              {5: -2.5e23, 3000: -2.5e23}, {5: 2.5e23, 4000: -2.5e23}, {5: 3.3e23}]):
        for k, x in at.items():
            lm[k, col * 7] = x
    split, tall = _head_alone(P, K, V, 128, emb, lm), _head_alone(P, K, V, m, emb, lm)[:128]
    assert torch.equal(torch.isnan(split), torch.isnan(tall)) and torch.equal(torch.isinf(split), torch.isinf(tall))
    ok = torch.isfinite(split)
    assert torch.equal(split[~ok].sign().nan_to_num(9), tall[~ok].sign().nan_to_num(9))
    assert not ok[:, [0, 7, 14, 21, 28, 35]].any() and ok[:, [42, 49]].all() and ok[:, 50:].all()
    assert ((split - tall)[ok].abs() <= 1e-5 * split[ok].abs() + 1e-3).all()


@pytest.mark.parametrize("B,enc_len", [(1, 1), (1, 31), (1, 96), (1, 97), (1, 130), (2, 300), (3, 171)])
def test_cross_projection_rows(P, B, enc_len):
    """Encoder rows of several sequences in one pass: a single row, ragged row tiles and row blocks, sequences that cross the
    limit of 512 rows per pass."""
    _check_cross_projection(P, B, enc_len, 8)


@pytest.mark.parametrize("B,enc_len,max_block", [(1, 16, 64), (1, 33, 64), (1, 64, 64), (1, 64, 63), (1, 65, 80), (1, 128, 140), (1, 129, 140), (2, 30, 64)])
def test_cross_projection_of_few_rows(P, B, enc_len, max_block):
    """One sequence whose rows fit a decoder block: the GEMMs that stream the matrices (a whole row tile, the first count of the
    row-split form, the last one for a matrix of this size); one row more than a block, than those rows, and a second sequence: the tall form."""
    _check_cross_projection(P, B, enc_len, max_block)


def _check_cross_projection(P, B, enc_len, max_block):
    from gpu_util import make_pair, tol_ok
    shape = I.ModelShape("edge_t5", 1, "bf16", 2, 256, 4, 64, 512, 1024, rms_eps=1e-6, enc_len=enc_len)
    gm, om = make_pair(shape, 29, B, max(32, max_block), max_block, std=0.05)
    enc = I.encoder_output(shape, B, 29)
    gm.cross_kv_init(enc.cuda())
    om.cross_kv_init(enc.numpy())
    block = I.token_ids(B * 5, shape.vocab, 29, 1).reshape(B, 5).numpy().astype(np.int32)
    cl = np.zeros(B, np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("dims", [(48, 3, 16, 100, 301), (64, 4, 16, 256, 512), (33, 3, 2, 65, 70), (40, 1, 130, 7, 129), (300, 5, 64, 90, 65)],
                         ids=lambda d: "-".join(map(str, d)))
@pytest.mark.parametrize("B,m,t", [(1, 1, 1), (2, 4, 30), (1, 9, 400), (3, 17, 63)])
@pytest.mark.parametrize("form", ["by_rule", "five_launches"])
def test_fp32_forward(P, dims, B, m, t, form):
    """The fp32 GEMMs (K slices shorter than a turn, ragged column groups and rotary pairs, rows across workgroups) and the
    generic attention (heads narrower and wider than the groups of its threads, few and many keys).  They run for every model while the
    profile is on; by the rule, some of these models take the form of a workgroup per block row."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    d, H, dh, F, V = dims
    shape = I.ModelShape("edge_fp32", 0, "fp32", 2, d, H, dh, F, V)
    gm, om = make_pair(shape, 31, B, t + m + 3, m, std=0.1)
    gm.prof_enable(form == "five_launches")
    import_synthetic_kv(gm, om, shape, t, 31, B=B)
    block = I.token_ids(B * m, V, 31, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([max(0, t - 5 * b) for b in range(B)], np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 1e-4, 1e-4)
    assert ok, f"max abs err {err}"
    for b in range(B):
        for got, want in zip(gm.kv_read(1, b, 0, int(cl[b]) + m), om.kv_read(1, b, 0, int(cl[b]) + m)):
            assert tol_ok(got.cpu().numpy().astype(np.float64), want, 1e-4, 1e-4)[0]


@pytest.mark.parametrize("dims,B,m,t,max_seq", [
    ((128, 4, 12, 40, 200), 2, 5, 31, 64), ((40, 1, 130, 9, 129), 1, 3, 70, 128), ((32, 2, 10, 512, 1024), 3, 4, 9, 32), ((16, 1, 6, 8, 16), 1, 2, 0, 8),
    ((32, 2, 16, 24, 50), 4, 64, 10, 80), ((32, 2, 16, 24, 50), 4, 65, 10, 80), ((32, 4, 8, 24, 50), 1, 3, 2600, 2688), ((32, 4, 8, 24, 50), 1, 3, 2750, 2816),
    ((40, 1, 130, 9, 129), 1, 3, 50, 64), ((32, 4, 16, 24, 50), 1, 3, 2680, 2688), ((32, 1, 16, 24, 50), 1, 3, 10930, 10944), ((16, 16, 16, 24, 50), 1, 3, 50, 64),
    ((32, 8, 16, 24, 50), 2, 9, 180, 192), ((32, 3, 30, 24, 50), 2, 9, 110, 128),
    ((64, 1, 24, 32, 64), 1, 3, 20, 64), ((64, 4, 16, 32, 66), 1, 3, 20, 64), ((40, 2, 16, 34, 68), 2, 3, 20, 64), ((96, 4, 16, 31, 60), 1, 3, 20, 64),
    ((64, 3, 20, 146, 512), 1, 3, 20, 64), ((64, 3, 20, 136, 512), 1, 3, 20, 64), ((64, 1, 76, 146, 300), 2, 3, 20, 64), ((16, 1, 6, 256, 512), 1, 3, 20, 64),
    ((24, 6, 16, 192, 384), 1, 3, 20, 64)],
    ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else None)
def test_small_fp32_models(P, dims, B, m, t, max_seq):
    """The forward of a workgroup per block row at the edges of what it takes: most values per thread in each product, 1024 and 16 columns, products
    that are and are not read four columns per thread (64 columns and more, a multiple of 4, 36 slices of two products or 18 of one), heads whose keys are not read 16 values at a time, 256 rows and more, the most scores in LDS, the most features times keys of either kind of head, and more."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    d, H, dh, F, V = dims
    shape = I.ModelShape("edge_small", 0, "fp32", 2, d, H, dh, F, V)
    gm, om = make_pair(shape, 33, B, max_seq, m, std=0.1)
    if t:
        import_synthetic_kv(gm, om, shape, t, 33, B=B)
    block = I.token_ids(B * m, V, 33, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([max(0, t - 3 * b) for b in range(B)], np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 1e-4, 1e-4)
    assert ok, f"max abs err {err}"
    for b in range(B):
        for got, want in zip(gm.kv_read(1, b, 0, int(cl[b]) + m), om.kv_read(1, b, 0, int(cl[b]) + m)):
            assert tol_ok(got.cpu().numpy().astype(np.float64), want, 1e-4, 1e-4)[0]


@pytest.mark.parametrize("V", [18428, 18432, 18436, 32764, 32766, 32768, 32772])
@pytest.mark.parametrize("kind", ["plain", "zero_residual", "large", "empty"])
def test_accept_at_the_longest_row_in_registers(P, V, kind):
    """Either side of the vocabularies that a workgroup holds in registers, and what it hands on to the general way: a residual without weight,
    weights above 256, a row of zeros.  Whole numbers, decided by exact sums."""
    from oracle import csd_oracle as O
    B, k = 3, 2
    g = torch.Generator().manual_seed(V)
    p = torch.softmax(2.0 * torch.randn((B, k + 1, V), generator=g), -1)
    q = torch.softmax(2.0 * torch.randn((B, k, V), generator=g), -1)
    draft = torch.stack([torch.tensor([0, V - 1]), torch.tensor([V // 2, 3]), torch.tensor([V - 1, 255])]).int()
    if kind == "zero_residual":
        q = 2.0 * p[:, :k]                                   # (every draft is rejected: the uniforms are 0.5 and more)
    elif kind == "large":
        p = p * 3e4
        p[0, :, V - 1] = 300.0
    elif kind == "empty":
        p[1:] = 0.0
    u_acc, u_s = torch.rand((B, k), generator=g) * 0.5 + 0.5, torch.rand(B, generator=g)
    for dense in (q, None):
        if dense is None and kind == "large":
            continue
        n, tok = P.accept(p.cuda(), None if dense is None else dense.cuda(), draft.cuda(), u_acc.cuda(), u_s.cuda(), 1.0, 0)
        s = 1 if kind == "empty" else B                      # (the oracle refuses a row of zeros; here its token is -1)
        wn, wt = O.accept(p[:s].numpy(), None if dense is None else dense[:s].numpy(), draft[:s].numpy(), u_acc[:s].numpy(), u_s[:s].numpy(), 1.0, 0)
        n, tok = n.cpu().numpy(), tok.cpu().numpy()
        assert np.array_equal(n[:s], wn) and np.array_equal(tok[:s], wt), (kind, dense is None)
        assert (n[s:] == 0).all() and (tok[s:] == -1).all()


@pytest.mark.parametrize("V", [18432, 32000, 32768])
@pytest.mark.parametrize("lenience", [1.0, 4.0, 256.0])
def test_accept_of_rows_with_little_weight(P, V, lenience):
    """Rows whose groups of 256 tokens are left out where they are below 2^-40: weight at the edges of groups, values on either side of the
    line before and after the lenience, rejected drafts with and without draft distributions.  Whole numbers, decided by exact sums."""
    from oracle import csd_oracle as O
    B, k = 4, 2
    g = torch.Generator().manual_seed(V)
    small = torch.tensor([0.0, 2.0 ** -41, 2.0 ** -40 / 256, 2.0 ** -40 * (1 - 2.0 ** -24), 2.0 ** -40, 2.0 ** -39])
    p = small[torch.randint(0, 6, (B, k + 1, V), generator=g)]
    p[1, :, 2048:] = 2.0 ** -41                              # whole groups below the line; and above it
    p[2, :, 2048:] = 2.0 ** -38
    p[3] = 0.0
    for b in range(B):
        for i, v in enumerate([0, 255, 256, 1023, 2047, 2048, V // 2, V - 257, V - 1]):
            p[b, :, v] = 0.1 + 0.01 * i
    q = torch.where(torch.rand((B, k, V), generator=g) < 0.5, torch.zeros(()), p[:, :k] * 0.5)
    draft = torch.tensor([[255, V - 1], [7, 256], [V - 1, 0], [2048, 9]]).int()
    for b in range(B):
        for i in range(k):
            q[b, i, draft[b, i]] = 300.0                     # rejected at any lenience
    u_acc, u_s = torch.rand((B, k), generator=g) * 0.25 + 0.75, torch.rand(B, generator=g)
    for dense in (q, None):
        n, tok = P.accept(p.cuda(), None if dense is None else dense.cuda(), draft.cuda(), u_acc.cuda(), u_s.cuda(), lenience, 0)
        wn, wt = O.accept(p.numpy(), None if dense is None else dense.numpy(), draft.numpy(), u_acc.numpy(), u_s.numpy(), lenience, 0)
        assert np.array_equal(n.cpu().numpy(), wn) and np.array_equal(tok.cpu().numpy(), wt)


@pytest.mark.parametrize("V", [1, 3, 4, 254, 256, 260, 4096, 12284, 12288, 12292, 32764, 32766, 32768, 32772])
def test_arg_max_of_rows_with_nan_and_without_finite_values(P, V):
    """The greedy rule's own token, in registers and in the general way: NaN never wins, the lowest index among equals does, a row of -inf gives its first
    token that is not NaN, a row of NaN the first token."""
    g = torch.Generator().manual_seed(V)
    rows = torch.randn((9, V), generator=g)
    rows[1] = float("nan")
    rows[2] = float("-inf")
    rows[3] = float("-inf")
    rows[3, :V // 2] = float("nan")
    rows[4, torch.randperm(V, generator=g)[:V // 2]] = float("nan")
    rows[5, [V // 3, V - 1]] = float("inf")
    rows[6, V // 2:] = rows[6].max() + 1.0
    rows[7, :V - 1] = float("nan")
    rows[8] = float("nan")
    rows[8, V // 2] = float("-inf")
    most = torch.where(rows.isnan(), torch.tensor(float("-inf")), rows).max(1, keepdim=True).values
    want = (rows == most).numpy().argmax(1).tolist()         # (NaN equals nothing; numpy gives the first)
    # two reviewer rows per sequence: a draft that is not the arg-max, so the first row decides; then drafts that are, so the second does
    p = torch.stack([rows, rows.roll(1, 0)], 1).contiguous().cuda()
    u, us = torch.zeros((9, 1), device="cuda"), torch.zeros(9, device="cuda")
    miss = torch.full((9, 1), V, dtype=torch.int32, device="cuda")
    n, tok = P.accept(p, None, miss, u, us, 1.0, 1)
    assert n.tolist() == [0] * 9 and tok.tolist() == want
    n, tok = P.accept(p, None, torch.tensor(want, dtype=torch.int32, device="cuda")[:, None].contiguous(), u, us, 1.0, 1)
    assert n.tolist() == [1] * 9 and tok.tolist() == want[-1:] + want[:-1]


@pytest.mark.parametrize("H,dh,max_seq,row_form", [
    (4, 16, 2688, True), (4, 16, 2689, False), (1, 64, 10944, True), (1, 64, 10945, False), (2, 32, 1024, True), (8, 16, 192, True), (8, 16, 193, False),
    (3, 32, 256, True), (3, 32, 257, False), (3, 64, 128, True), (3, 64, 129, False), (16, 16, 64, True), (16, 16, 65, False), (2, 10, 576, True),
    (2, 10, 577, False), (3, 30, 128, True), (3, 30, 129, False), (8, 8, 192, True), (8, 8, 193, False), (1, 300, 64, False)])
def test_small_fp32_models_with_long_caches(P, H, dh, max_seq, row_form):
    """The forward of a workgroup per block row is taken where it is the faster one with a full cache: heads x features x keys bounded, the bound half as
    large for heads whose keys are not read 16 values at a time.  While the profile is on, the other form runs: where that is the form in
    any case, the logits are the same bit for bit."""
    shape = I.ModelShape("edge_rule", 0, "fp32", 2, 24, H, dh, 40, 300)
    gm = P.Model(shape, I.make_weights(shape, 9, device="cuda", std=0.3), max_batch=1, max_seq=max_seq, max_block=8)
    block, cl = I.token_ids(8, 300, 9, 1).reshape(1, 8).to(torch.int32).cuda(), torch.zeros(1, dtype=torch.int32, device="cuda")
    plain = gm.verify_block(block, cl)
    gm.prof_enable(True)
    other = gm.verify_block(block, cl)
    assert torch.equal(plain, other) == (not row_form)
    assert ((plain - other).abs() <= 1e-4 + 1e-4 * plain.abs()).all()


def test_profile_of_an_fp32_forward(P):
    """Launches per kernel class of the fp32 forward: four GEMMs and one attention per layer, the LM head, the embedding."""
    shape = I.ModelShape("edge_prof", 0, "fp32", 3, 64, 4, 16, 128, 80)
    gm = P.Model(shape, I.make_weights(shape, 5, device="cuda", std=0.1), max_batch=1, max_seq=32, max_block=4)
    gm.prof_enable(True)
    for _ in range(2):
        gm.verify_block(torch.ones((1, 3), dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    got = [gm.prof_read(c) for c in range(3)]
    assert [n for _, n in got] == [2 * 13, 2 * 3, 2] and all(ms > 0 for ms, _ in got)


def test_generic_attention_longest_sequence(P):
    """The longest sequence that a model on the generic attention accepts: 64 KB of scores and query."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    shape = I.ModelShape("edge_long", 0, "fp32", 1, 64, 1, 64, 32, 40)
    gm, om = make_pair(shape, 3, 1, 16384 - 64, 2, std=0.1)
    import_synthetic_kv(gm, om, shape, 16300, 3)
    block, cl = np.asarray([[5, 9]], np.int32), np.asarray([16300], np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 1e-4, 1e-4)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("max_seq,m,t", [(2048, 3, 2040), (2112, 16, 2060), (4224, 5, 4200)])
def test_small_block_attention_over_many_chunks(P, dh, max_seq, m, t):
    """16 chunks and more: the merge takes the chunk states of a head 16 at a time."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    shape = I.ModelShape("edge_chunks", 0, "bf16", 1, 256, 2, dh, 256, 512)
    gm, om = make_pair(shape, 43, 1, max_seq, m, std=0.05)
    import_synthetic_kv(gm, om, shape, t, 43)
    block = I.token_ids(m, shape.vocab, 43, 1).reshape(1, m).numpy().astype(np.int32)
    cl = np.full(1, t, np.int32)
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("arch,dh", [(0, 64), (0, 128), (1, 64), (1, 128)])
@pytest.mark.parametrize("max_seq,B,m,t", [(64, 1, 1, 1), (64, 2, 8, 31), (192, 1, 16, 128), (448, 2, 5, 443), (512, 1, 1, 0), (576, 1, 7, 512),
                                           (832, 2, 3, 829), (896, 1, 4, 600)])
def test_small_block_attention(P, arch, dh, max_seq, B, m, t):
    """The attention of blocks of up to 16 rows on either side of the cache lengths where one workgroup per head gives way to
    chunks: one tile and less, a tile per wave and one key more, waves without a tile, several turns, a full cache."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    shape = I.ModelShape("edge_attn", arch, "bf16", 1, 256, 2, dh, 256, 512, rms_eps=1e-6 if arch else 1e-5,
                         enc_len=max(1, min(t, 520)) if arch else 0)
    gm, om = make_pair(shape, 37, B, max_seq, m, std=0.05)
    if t:
        import_synthetic_kv(gm, om, shape, t, 37, B=B)
    if arch:
        enc = I.encoder_output(shape, B, 37)
        gm.cross_kv_init(enc.cuda())
        om.cross_kv_init(enc.numpy())
    block = I.token_ids(B * m, shape.vocab, 37, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([max(0, t - 40 * b) for b in range(B)], np.int32)
    assert gm.path(B, m) == 1
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("arch,dh", [(0, 64), (0, 128), (1, 64)])
@pytest.mark.parametrize("max_seq,B,m,t", [(128, 8, 4, 90), (128, 9, 3, 90), (128, 32, 1, 120), (384, 9, 3, 300), (384, 32, 1, 17), (448, 1, 5, 440),
                                           (448, 2, 5, 440), (448, 8, 1, 447), (512, 2, 3, 450)])
def test_small_block_attention_of_many_heads(P, arch, dh, max_seq, B, m, t):
    """Caches short enough for one workgroup per head, with as many (sequence, head) pairs as compute units and with more, where
    the chunked kernels take over; and either side of the two limits for heads of 128, below and from 64 pairs on."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    shape = I.ModelShape("edge_heads", arch, "bf16", 1, 64, 32, dh, 64, 512, rms_eps=1e-6 if arch else 1e-5, enc_len=70 if arch else 0)
    gm, om = make_pair(shape, 43, B, max_seq, m, std=0.05)
    import_synthetic_kv(gm, om, shape, t, 43, B=B)
    if arch:
        enc = I.encoder_output(shape, B, 43)
        gm.cross_kv_init(enc.cuda())
        om.cross_kv_init(enc.numpy())
    block = I.token_ids(B * m, shape.vocab, 43, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([max(0, t - 3 * b) for b in range(B)], np.int32)
    assert gm.path(B, m) == 1
    lg = gm.verify_block(torch.from_numpy(block).cuda(), torch.from_numpy(cl).cuda())
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("max_seq,m,t", [(192, 9, 150), (192, 40, 150), (704, 17, 640), (2048, 33, 1900), (512, 150, 300)])
def test_attention_output_is_rounded_once(P, dh, max_seq, m, t):
    """Rows of a zero embedding: every visible key has the score 0, so row i's output is the sum of the cached values over the
    t + i + 1 keys it sees (the block's own values are 0).  The values are whole numbers, their sums exact, so what the output
    projection (a unit matrix) adds to the zero residual is one correctly rounded quotient, in two bf16 planes, to the last bit."""
    d = 64
    shape = I.ModelShape("edge_quot", 0, "bf16", 1, d, d // dh if dh < d else 1, dh, 32, 32)
    z = lambda r, c: torch.zeros((r, c), dtype=torch.bfloat16, device="cuda")
    one = torch.ones(d, device="cuda")
    wo = z(dh, d)
    wo[:d] = torch.eye(d, device="cuda")
    gm = P.Model(shape, [z(32, d), one, z(d, dh), z(d, dh), z(d, dh), wo, one, z(d, 32), z(d, 32), z(32, d), one, z(d, 32)],
                 max_batch=1, max_seq=max_seq, max_block=m)
    v = torch.randint(-60, 61, (t, dh), device="cuda").float()
    v[:, :32] = torch.arange(1, 33, device="cuda").float()   # exact quotients among the results
    gm.kv_write(0, 0, 0, torch.randn((t, dh), device="cuda"), v)
    tr = torch.zeros((2, m, d), device="cuda")
    gm.set_trace(tr)
    gm.verify_block(torch.zeros((1, m), dtype=torch.int32, device="cuda"), torch.tensor([t], dtype=torch.int32, device="cuda"))
    gm.set_trace(None)
    q = (v.double().sum(0)[None, :d] / torch.arange(t + 1, t + m + 1, device="cuda")[:, None].double()).float()
    hi = q.bfloat16().float()
    want = hi + (q - hi).bfloat16().float()
    gm.close()
    print("differ", (tr[1] != want).sum().item(), "of", want.numel())
    assert torch.equal(tr[1], want)


@pytest.mark.parametrize("arch,dh,tree", [(0, 64, False), (0, 128, False), (1, 64, False), (1, 128, False), (0, 64, True), (0, 128, True)])
@pytest.mark.parametrize("B,H,m,t", [(20, 64, 1, 250), (13, 96, 2, 200)])
def test_small_block_attention_of_more_waves_than_simds(P, arch, dh, tree, B, H, m, t):
    """More (sequence, head) pairs than SIMDs, one row tile each: the form with registers for two waves per SIMD."""
    from gpu_util import import_synthetic_kv, make_pair, tol_ok
    shape = I.ModelShape("edge_waves", arch, "bf16", 1, 64, H, dh, 64, 512, rms_eps=1e-6 if arch else 1e-5, enc_len=70 if arch else 0)
    gm, om = make_pair(shape, 73, B, 256, m, std=0.05)
    import_synthetic_kv(gm, om, shape, t, 73, B=B)
    if arch:
        enc = I.encoder_output(shape, B, 73)
        gm.cross_kv_init(enc.cuda())
        om.cross_kv_init(enc.numpy())
    block = I.token_ids(B * m, shape.vocab, 73, 1).reshape(B, m).numpy().astype(np.int32)
    cl = np.asarray([t - 9 * b for b in range(B)], np.int32)
    dev = [torch.from_numpy(x).cuda() for x in (block, np.tile(np.arange(-1, m - 1, dtype=np.int32), (B, 1)), cl)]
    lg = gm.verify_tree(*dev) if tree else gm.verify_block(dev[0], dev[2])
    ok, err = tol_ok(lg.cpu().numpy().astype(np.float64), om.verify_block(block, cl), 2e-2, 1e-2)
    assert ok, f"max abs err {err}"


@pytest.mark.parametrize("V", [4, 512, 2048, 2052, 8192, 8196, 32768])
@pytest.mark.parametrize("mode", [0, 1])
def test_review_of_all_rows_equals_softmax_then_accept(P, V, mode):
    """Vocabularies at the limits of the values a thread holds: the fused review decides as the two kernels, bit for bit."""
    shape = I.ModelShape("edge_review", 0, "fp32", 1, 16, 1, 16, 16, V)
    gm = P.Model(shape, I.make_weights(shape, 41, device="cuda", std=0.3), max_batch=2, max_seq=16, max_block=6)
    g = torch.Generator(device="cuda").manual_seed(V)
    block = torch.randint(0, V, (2, 6), generator=g, device="cuda", dtype=torch.int32)
    cl = torch.zeros(2, dtype=torch.int32, device="cuda")
    for dense in (False, True):
        q = torch.softmax(torch.randn((2, 5, V), generator=g, device="cuda"), -1) if dense else None
        ua, us = torch.rand((2, 5), generator=g, device="cuda"), torch.rand(2, generator=g, device="cuda")
        probs = torch.empty((2, 6, V), device="cuda")
        n, x = gm.verify_accept(block, cl, ua, us, q=q, mode=mode, probs=probs)
        lg, p = gm.verify_block(block, cl, want_probs=True)
        n2, x2 = P.accept(lg if mode else p, q, block[:, 1:].contiguous(), ua, us, mode=mode)
        assert torch.equal(n, n2) and torch.equal(x, x2)
        assert torch.equal(probs, p)


@pytest.mark.parametrize("V", [512, 8192, 32000])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("std", [0.3, 2.0, 6.0])
def test_review_of_confident_rows_equals_softmax_then_accept(P, V, mode, std):
    """Rows of which some groups, most or nearly all are too far below the maximum to carry weight, without probabilities asked for: the fused review,
    which leaves such groups out, decides as the two kernels, bit for bit, at any lenience."""
    shape = I.ModelShape("edge_review", 0, "fp32", 1, 16, 1, 16, 16, V)
    gm = P.Model(shape, I.make_weights(shape, 43, device="cuda", std=std), max_batch=2, max_seq=16, max_block=6)
    g = torch.Generator(device="cuda").manual_seed(V)
    cl = torch.zeros(2, dtype=torch.int32, device="cuda")
    for lenience in (1.0, 3.0, 256.0):
        for dense in (False, True):
            block = torch.randint(0, V, (2, 6), generator=g, device="cuda", dtype=torch.int32)
            q = torch.softmax(6.0 * torch.randn((2, 5, V), generator=g, device="cuda"), -1) if dense else None
            ua, us = torch.rand((2, 5), generator=g, device="cuda"), torch.rand(2, generator=g, device="cuda")
            n, x = gm.verify_accept(block, cl, ua, us, q=q, mode=mode, lenience=lenience)
            lg, p = gm.verify_block(block, cl, want_probs=True)
            n2, x2 = P.accept(lg if mode and lenience == 1.0 else p, q, block[:, 1:].contiguous(), ua, us, lenience=lenience, mode=mode)
            assert torch.equal(n, n2) and torch.equal(x, x2)


@pytest.mark.parametrize("V", [512, 8192, 32000])
@pytest.mark.parametrize("temperature", [1e-2, 1e-4, 1e-6, 3e-7, 1e-7, 3e-8, 1e-8, 1e-9])
def test_review_at_small_temperatures_equals_softmax_then_accept(P, V, temperature):
    """Scaled logits of 2^9 to 2^37, up to where the distance of two neighbouring 32-bit numbers passes every margin below the maximum: with and without
    drafts, without probabilities asked for, the fused review decides as the two kernels, bit for bit, and emits a token."""
    shape = I.ModelShape("edge_review", 0, "fp32", 1, 16, 1, 16, 16, V)
    gm = P.Model(shape, I.make_weights(shape, 43, device="cuda", std=2.0), max_batch=2, max_seq=16, max_block=6)
    g = torch.Generator(device="cuda").manual_seed(V)
    cl = torch.zeros(2, dtype=torch.int32, device="cuda")
    for m in (1, 6):
        block = torch.randint(0, V, (2, m), generator=g, device="cuda", dtype=torch.int32)
        for i in range(m):                                   # one sequence's drafts are all kept
            lg, p = gm.verify_block(block, cl, want_probs=True, temperature=temperature)
            if i + 1 < m:
                block[0, i + 1] = lg[0, i].argmax()
        assert (lg.max(-1).values > 4.0).all() and (lg.max(-1).values < 100.0).all()
        for lenience in (1.0, 256.0):
            for dense in (False, True) if m > 1 else (False,):
                q = torch.softmax(6.0 * torch.randn((2, m - 1, V), generator=g, device="cuda"), -1) if dense else None
                ua, us = torch.rand((2, m - 1), generator=g, device="cuda"), torch.rand(2, generator=g, device="cuda")
                n, x = gm.verify_accept(block, cl, ua, us, q=q, lenience=lenience, temperature=temperature)
                n2, x2 = P.accept(p, q, block[:, 1:].contiguous(), ua, us, lenience=lenience)
                assert torch.equal(n, n2) and torch.equal(x, x2) and (x >= 0).all()
