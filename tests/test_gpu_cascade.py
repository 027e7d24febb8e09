"""The cascade generation loop (Algorithm 1) on the GPU.

What the paper fixes (Sections 2, 3.1, 5.1): with temperature 0 and no lenience where the target
reviews, cascaded decoding emits exactly the target's own greedy continuation, whatever the draft
levels, K and the lenience between draft levels are; a draft identical to its reviewer is accepted
whole.  Both are checked on the GPU's own outputs (cascade vs plain decoding with the same kernels),
and the fp32 configuration also against the CPU oracle's cascade driver."""
import itertools

import os

import numpy as np
import pytest
import torch

import csd_inputs as I

pytestmark = pytest.mark.gpu

TARGET = I.ModelShape("t", 0, "fp32", 2, 64, 4, 16, 256, 512)
DRAFT1 = I.ModelShape("d1", 0, "fp32", 1, 32, 2, 16, 64, 512)
DRAFT2 = I.ModelShape("d2", 0, "fp32", 1, 16, 2, 8, 32, 512)
TARGET_BF = I.ModelShape("tb", 0, "bf16", 2, 256, 4, 64, 512, 1024)
DRAFT_BF = I.ModelShape("db", 0, "bf16", 1, 256, 4, 64, 512, 1024)
MAX_CTX = 160


def _gpu_level(shape, seed, std):
    import paper_2312_11462_amd as P
    from paper_2312_11462_amd.cascade import Level
    w = I.make_weights(shape, seed, device="cuda", std=std)
    return Level(P.Model(shape, w, max_batch=1, max_seq=MAX_CTX, max_block=16), 16)


def _prompt(vocab, seed):
    p = I.token_ids(24, vocab, seed, 1).tolist()
    return p[:12] + p[:12]            # a repeated phrase so that Max-Gram has matches


def _table(prompt, vocab):
    import paper_2312_11462_amd as P
    t = I.default_next_table(vocab, 1).cuda()
    P.bigram_fit(torch.tensor(prompt, dtype=torch.int32).cuda(), vocab, t)
    return t


@pytest.mark.parametrize("K,lenience,n_drafts", [
    ([[4]], 1.0, 0),
    ([[2, 6], [0, 6]], 1.0, 1),
    ([[2, 6], [0, 6]], 3.0, 1),
    ([[2, 2, 4], [0, 1, 3], [0, 0, 3]], 2.0, 2),
])
def test_greedy_cascade_equals_target_greedy_fp32_and_matches_the_oracle_driver(K, lenience, n_drafts):
    from paper_2312_11462_amd.cascade import Cascade, autoregressive
    from oracle import csd_oracle as O
    from oracle import cascade as OC
    prompt = _prompt(512, 21)
    table = _table(prompt, 512)
    shapes = [TARGET, DRAFT1, DRAFT2][:n_drafts + 1]
    levels = [_gpu_level(s, 1 + i, 0.2) for i, s in enumerate(shapes)]
    want = autoregressive(levels[0], prompt, 40, MAX_CTX)
    got, steps = Cascade(levels, table, K, MAX_CTX, lenience=lenience, mode=1).generate(prompt, 40)
    assert got == want
    assert steps <= 40
    # the CPU oracle's driver on the same weights emits the same tokens (fp64 vs fp32 arg-maxes agree
    # at this weight scale)
    olevels = []
    for i, s in enumerate(shapes):
        w = I.make_weights(s, 1 + i, std=0.2)
        lv = OC.Level(O.Model(s, w, max_batch=1, max_seq=MAX_CTX, max_block=16), 16)
        lv._keep = w
        olevels.append(lv)
    otable = O.bigram_fit(np.array(prompt, np.int32), 512, I.default_next_table(512, 1).numpy())
    assert np.array_equal(otable, table.cpu().numpy())
    ogot, osteps = OC.cascade_generate(olevels, otable, prompt, 40, K, lenience=lenience, mode=1)
    assert got == ogot and steps == osteps


def test_greedy_cascade_bf16_on_the_default_forward():
    """bf16 models whose blocks (<= 16 rows) take the forward with the epilogues inside its GEMM kernels: the
    cascade still reproduces the target's greedy continuation, because reviewer and plain decoding run the
    same kernels."""
    from paper_2312_11462_amd.cascade import Cascade, autoregressive
    prompt = _prompt(1024, 31)
    table = _table(prompt, 1024)
    target, draft = _gpu_level(TARGET_BF, 5, 0.05), _gpu_level(DRAFT_BF, 6, 0.05)
    assert target.model.path(1, 9) == 1 and draft.model.path(1, 7) == 1
    want = autoregressive(target, prompt, 32, MAX_CTX)
    got, steps = Cascade([target, draft], table, [[2, 6], [0, 6]], MAX_CTX, lenience=2.0, mode=1).generate(prompt, 32)
    # block shape changes the summation order inside the kernels; an arg-max tie within rounding could
    # legitimately differ, so report rather than hide: the seeded models here have no such tie
    assert got == want


def test_identical_draft_is_accepted_whole():
    from paper_2312_11462_amd.cascade import Cascade, autoregressive
    prompt = I.token_ids(10, 512, 22, 1).tolist()
    table = I.default_next_table(512, 1).cuda()
    target, twin = _gpu_level(TARGET, 1, 0.2), _gpu_level(TARGET, 1, 0.2)
    want = autoregressive(target, prompt, 24, MAX_CTX)
    got, steps = Cascade([target, twin], table, [[3, 0], [0, 1]], MAX_CTX, mode=1).generate(prompt, 24)
    assert got == want
    assert steps <= 24 // 4 + 1        # every target review keeps the twin's 3 drafts and adds one token


def test_sampling_cascade_is_reproducible_and_emits_valid_tokens():
    from paper_2312_11462_amd.cascade import Cascade
    prompt = I.token_ids(16, 512, 23, 1).tolist()
    table = I.default_next_table(512, 1).cuda()
    levels = [_gpu_level(TARGET, 1, 0.2), _gpu_level(DRAFT1, 2, 0.2)]
    outs = []
    for _ in range(2):
        u = iter(I.uniforms(4000, 77, 3).tolist())
        got, _ = Cascade(levels, table, [[3, 3], [0, 2]], MAX_CTX, lenience=2.0, mode=0).generate(prompt, 30, u)
        outs.append(got)
    assert outs[0] == outs[1]
    assert all(0 <= t < 512 for t in outs[0])


class _FixedGpuLevel:
    """A level whose next-token distribution does not depend on the context (same interface as Level): its
    logits and fp32 probabilities are inputs, identical on both sides, so the GPU driver and the oracle
    driver must then agree token for token in sampling mode (csd_accept is bit-exact on equal inputs)."""

    class _M:
        def __init__(self, vocab):
            self.shape = I.ModelShape("fixed", 0, "fp32", 1, 16, 1, 16, 16, vocab)

    def __init__(self, logits, probs):
        self.lg = torch.tensor(logits, dtype=torch.float32).cuda()
        self.pr = torch.tensor(probs, dtype=torch.float32).cuda()
        self.model = self._M(len(probs))
        self.cached = 0

    def rows_from(self, ctx, n_tokens, first_row, want_probs=False, temperature=1.0):
        n = n_tokens - first_row
        return self.lg.repeat(n, 1), (self.pr.repeat(n, 1) if want_probs else None)


class _FixedOracleLevel:
    def __init__(self, logits):
        self.logits = np.asarray(logits, np.float64)
        self.cached = 0

    def rows_from(self, seq, first_row):
        return np.tile(self.logits, (len(seq) - first_row, 1))


def _u24(seed):
    rs = np.random.RandomState(seed)
    while True:
        for u in rs.randint(0, 1 << 24, size=4096):
            yield float(u) / float(1 << 24)


@pytest.mark.parametrize("K,lenience", [
    ([[3, 2, 0], [0, 0, 0], [0, 0, 0]], 1.0),        # horizontal: 3 tokens of level 1, 2 of level 2
    ([[4, 0, 0], [0, 3, 0], [0, 0, 0]], 1.0),        # vertical: level 1 reviews level 2's drafts
    ([[2, 1, 3], [0, 2, 2], [0, 0, 2]], 2.5),        # both, with Max-Gram drafts and lenience between draft levels
])
def test_sampling_cascade_matches_the_oracle_driver_token_for_token(K, lenience):
    from paper_2312_11462_amd.cascade import Cascade
    from oracle import csd_oracle as O
    from oracle import cascade as OC
    V, n_new = 37, 1500
    rs = np.random.RandomState(5)
    logits = [np.log(rs.dirichlet(np.full(V, a))) for a in (0.6, 0.8, 2.0)]
    probs = [O.probs_f32(lg[None])[0] for lg in logits]
    logits32 = [np.asarray(lg, np.float32) for lg in logits]
    prompt = _prompt(V, 3)
    table = _table(prompt, V)
    glevels = [_FixedGpuLevel(lg, pr) for lg, pr in zip(logits32, probs)]
    got, steps = Cascade(glevels, table, K, n_new + 64, lenience=lenience, mode=0).generate(prompt, n_new, _u24(17))
    olevels = [_FixedOracleLevel(lg.astype(np.float64)) for lg in logits32]
    otable = O.bigram_fit(np.array(prompt, np.int32), V, I.default_next_table(V, 1).numpy())
    assert np.array_equal(otable, table.cpu().numpy())
    ogot, osteps = OC.cascade_generate(olevels, otable, prompt, n_new, K, lenience=lenience, mode=0, uniforms=_u24(17))
    assert steps == osteps
    assert got == ogot


# ------------------------------------------------------------------ device-resident control

def _oracle_steps(olevels, otable, prompt, K, lenience, mode, n_steps, uniform_at=None):
    from oracle import cascade as OC
    seq = list(prompt)
    for lv in olevels:
        lv.cached = 0
    for _ in range(n_steps):
        toks, _ = OC._step(olevels, otable, seq, K, lenience, mode, None, True, 0, uniform_at, 0)
        seq += toks
    return seq


@pytest.mark.parametrize("K,lenience,n_drafts", [
    ([[4]], 1.0, 0),
    ([[2, 6], [0, 6]], 1.0, 1),
    ([[2, 3], [0, 4]], 3.0, 1),
    ([[2, 2, 3], [0, 1, 3], [0, 0, 3]], 2.0, 2),
    ([[4, 0], [0, 0]], 1.0, 1),     # plain speculative decoding: four one-row forwards of the draft model, then the review
])
def test_resident_cascade_greedy_equals_the_oracle_driver_step_for_step(K, lenience, n_drafts):
    """Algorithm 1 as a chain of enqueues with device-resident control (no host synchronisation inside or between
    steps): after 10 steps the kept sequence equals the oracle driver's after 10 steps, and the target's own greedy
    continuation."""
    from paper_2312_11462_amd.cascade import ResidentCascade, autoregressive
    from oracle import csd_oracle as O
    from oracle import cascade as OC
    prompt = _prompt(512, 21)
    table = _table(prompt, 512)
    shapes = [TARGET, DRAFT1, DRAFT2][:n_drafts + 1]
    levels = [_gpu_level(s, 1 + i, 0.2) for i, s in enumerate(shapes)]
    rc = ResidentCascade(levels, table, K, MAX_CTX, lenience=lenience, mode=1)
    rc.start(prompt)
    for _ in range(10):
        rc.step()
    got = rc.tokens()
    assert all(int(st.item()) in (0, 1) for st in rc.status)
    olevels = []
    for i, s in enumerate(shapes):
        w = I.make_weights(s, 1 + i, device="cpu", std=0.2)
        olevels.append(OC.Level(O.Model(s, w, max_batch=1, max_seq=MAX_CTX, max_block=16), 16))
    otable = O.bigram_fit(np.array(prompt, np.int32), 512, I.default_next_table(512, 1).numpy())
    want = _oracle_steps(olevels, otable, prompt, K, lenience, 1, 10)
    assert got == want
    assert got[len(prompt):] == autoregressive(levels[0], prompt, len(got) - len(prompt), MAX_CTX)


class _FixedResidentLevel:
    """A level whose reviewer rows are inputs (the same fp32 distribution in every row): csd_review_ctx then runs
    no forward, only the device-resident accept and commit."""

    def __init__(self, probs, vocab, max_block=16):
        import paper_2312_11462_amd as P
        shape = I.ModelShape("fixed", 0, "fp32", 1, 16, 1, 16, 16, vocab)
        self.model = P.Model(shape, I.make_weights(shape, 1, device="cuda"), max_batch=1, max_seq=64, max_block=max_block)
        self.max_block = max_block
        self.ext_rows = torch.tensor(np.tile(probs, (max_block, 1))[None], dtype=torch.float32).cuda().contiguous()


@pytest.mark.parametrize("K,lenience", [
    ([[3, 2, 0], [0, 0, 0], [0, 0, 0]], 1.0),        # horizontal: 3 tokens of level 1, 2 of level 2
    ([[4, 0, 0], [0, 3, 0], [0, 0, 0]], 1.0),        # vertical: level 1 reviews level 2's drafts
    ([[2, 1, 3], [0, 2, 2], [0, 0, 2]], 2.5),        # both, with Max-Gram drafts and lenience between draft levels
])
def test_resident_cascade_sampling_matches_the_oracle_driver_token_for_token(K, lenience):
    """Sampling mode with levels whose distributions are inputs, uniforms taken by position on both sides: dense
    draft distributions handed upward on the device, Max-Gram positions one-hot, gated worst-case rounds."""
    from paper_2312_11462_amd.cascade import ResidentCascade
    from oracle import csd_oracle as O
    V, n_steps, max_ctx = 37, 60, 1024
    rs = np.random.RandomState(5)
    logits = [np.log(rs.dirichlet(np.full(V, a))) for a in (0.6, 0.8, 2.0)]
    probs = [O.probs_f32(lg[None])[0] for lg in logits]
    logits32 = [np.asarray(lg, np.float32) for lg in logits]
    prompt = _prompt(V, 3)
    table = _table(prompt, V)
    glevels = [_FixedResidentLevel(pr, V) for pr in probs]
    rc = ResidentCascade(glevels, table, K, max_ctx, lenience=lenience, mode=0)
    u = np.random.RandomState(17).randint(0, 1 << 24, size=(3, 2, max_ctx)).astype(np.float32) / np.float32(1 << 24)
    for i in range(3):
        rc.u_acc[i].copy_(torch.tensor(u[i, 0][None]))
        rc.u_samp[i].copy_(torch.tensor(u[i, 1][None]))
    rc.start(prompt)
    for _ in range(n_steps):
        rc.step()
    got = rc.tokens()
    assert all(int(st.item()) in (0, 1) for st in rc.status)
    olevels = [_FixedOracleLevel(lg.astype(np.float64)) for lg in logits32]
    otable = O.bigram_fit(np.array(prompt, np.int32), V, I.default_next_table(V, 1).numpy())
    want = _oracle_steps(olevels, otable, prompt, K, lenience, 0, n_steps, lambda d, kind, pos: float(u[d, kind, pos]))
    assert got == want
    assert len(got) - len(prompt) >= n_steps


# (sequences, rows a call has room for): one row tile with the two planes in a fragment each, and in one; two row tiles, the last one half
ROOMS = [(1, 16), (2, 16), (3, 16), (1, 8), (2, 12)]


@pytest.mark.parametrize("B,room", ROOMS)
@pytest.mark.parametrize("H,dh,max_seq", [(4, 64, 192), (4, 64, 1088), (2, 128, 192), (2, 128, 1088)])
def test_review_of_fewer_rows_than_the_call_has_room_for(H, dh, max_seq, B, room):
    """csd_review_ctx with room for 8 to 16 rows reviews 6, 1 and 4 of them, after a call in which every sequence is skipped and together with a skipped
    one: what the unused rows and the cache behind the used ones hold (NaN here) reaches nothing, and a plain review of
    exactly those rows decides the same."""
    import paper_2312_11462_amd as P
    shape = I.ModelShape("live", 0, "bf16", 2, 256, H, dh, 512, 1024)
    w = I.make_weights(shape, 5, device="cuda", std=0.05)
    gm = P.Model(shape, w, max_batch=B, max_seq=max_seq, max_block=16)
    ref = P.Model(shape, w, max_batch=B, max_seq=max_seq, max_block=16)
    gm.kv.view(torch.uint8).fill_(0xFF)
    t, i32 = 20, dict(dtype=torch.int32, device="cuda")
    tok = torch.stack([I.token_ids(48, shape.vocab, 5, b) for b in range(B)]).to(torch.int32).cuda()
    for m in (gm, ref):
        for pos in (0, 10):
            m.verify_block(tok[:, pos:pos + 10].contiguous(), torch.full((B,), pos, **i32))
    cache, length = torch.full((B,), t, **i32), torch.full((B,), t, **i32)
    ctx, skip = tok.clone(), torch.full((B,), -1, **i32)
    status, n_acc, nxt = (torch.zeros(B, **i32) for _ in range(3))

    def review(prefix):
        gm.review_ctx(ctx, length, cache, prefix, room, status, n_accepted=n_acc, next_token=nxt, mode=1)

    for rows in (6, 1, 4):
        start = cache.clone()
        length.copy_(start + rows)
        review(skip)
        assert (status == 1).all() and torch.equal(length, start + rows) and torch.equal(cache, start)
        block = torch.stack([ctx[b, int(start[b]):int(start[b]) + rows] for b in range(B)]).contiguous()
        n_ref, nxt_ref = ref.verify_accept(block, start, None, None, mode=1)
        for turn in range(B):                                # all but one sequence skipped, one after the other
            review(torch.where(torch.arange(B, device="cuda") == turn, start + 1, skip))
            assert int(status[turn]) == 0 and int(n_acc[turn]) == int(n_ref[turn]) and int(nxt[turn]) == int(nxt_ref[turn])
            length[turn] = cache[turn] + 1
        assert torch.equal(cache, start + 1 + n_ref)
    gm.close()
    ref.close()


@pytest.mark.parametrize("mode,lenience", [(0, 1.0), (0, 2.0), (1, 1.0), (1, 2.0)])
@pytest.mark.parametrize("B,room", [x for x in ROOMS if x[0] < 3])
@pytest.mark.parametrize("arch,H,dh,max_seq", [(0, 4, 64, 192), (0, 2, 128, 1088), (1, 4, 64, 192), (1, 4, 64, 1088), (1, 2, 128, 192), (1, 2, 128, 1088)])
def test_review_after_nan_everywhere(arch, H, dh, max_seq, B, room, mode, lenience, dims=(256, 512, 1024)):
    """csd_review_ctx with room for 8 to 16 rows after a call that left NaN in every buffer of the model and in the cache behind the kept rows: reviews of
    fewer rows, after a call in which every sequence is skipped and beside a skipped one, decide as a plain review of exactly those rows does, and the
    rows they hand on are its probabilities.  Both architectures, self- and cross-attention in either form for short blocks."""
    import paper_2312_11462_amd as P
    shape = I.ModelShape("live", arch, "bf16", 2, dims[0], H, dh, dims[1], dims[2], rms_eps=1e-6 if arch else 1e-5, enc_len=90 if arch else 0)
    w = I.make_weights(shape, 5, device="cuda", std=0.05)
    gm = P.Model(shape, w, max_batch=B, max_seq=max_seq, max_block=16)
    ref = P.Model(shape, w, max_batch=B, max_seq=max_seq, max_block=16)
    t, i32, V = 20, dict(dtype=torch.int32, device="cuda"), shape.vocab
    tok = torch.stack([I.token_ids(48, V, 5, b) for b in range(B)]).to(torch.int32).cuda()
    gm.kv.view(torch.uint8).fill_(0xFF)
    probs = torch.empty((B, 16, V), device="cuda")
    gm.verify_accept(tok[:, :16].contiguous(), torch.full((B,), 100, **i32), None, None, mode=1)
    gm.verify_block(tok[:, :16].contiguous(), torch.full((B,), 100, **i32), logits=probs, probs=probs)
    assert probs.isnan().all()
    gm.kv.view(torch.uint8).fill_(0xFF)
    for m in (gm, ref):
        if arch:
            m.cross_kv_init(I.encoder_output(shape, B, 5).cuda())
        for pos in (0, 10):
            m.verify_block(tok[:, pos:pos + 10].contiguous(), torch.full((B,), pos, **i32))
    cache, length = torch.full((B,), t, **i32), torch.full((B,), t, **i32)
    ctx, skip = tok.clone(), torch.full((B,), -1, **i32)
    status, n_acc, nxt = (torch.zeros(B, **i32) for _ in range(3))
    u_acc, u_samp = I.uniforms(B * 48, 5, 1).reshape(B, 48).cuda(), I.uniforms(B * 48, 5, 2).reshape(B, 48).cuda()
    u_acc[:, ::2] = 0.0                                      # (kept whatever their probability)
    out_q, base = torch.full((B, 48, V), float("nan"), device="cuda"), torch.zeros(B, **i32)

    def review(prefix):
        gm.review_ctx(ctx, length, cache, prefix, room, status, u_acc_tab=u_acc, u_samp_tab=u_samp, out_q_tab=out_q, out_base=base, n_accepted=n_acc,
                      next_token=nxt, mode=mode, lenience=lenience)

    for rows in (6, 1, 4):
        start = cache.clone()
        length.copy_(start + rows)
        review(skip)
        assert (status == 1).all() and torch.equal(length, start + rows) and torch.equal(cache, start)
        at = start.long()[:, None] + 1 + torch.arange(rows, device="cuda")
        block = torch.gather(ctx, 1, at - 1).contiguous()
        p_ref = torch.empty((B, rows, V), device="cuda")
        n_ref, nxt_ref = ref.verify_accept(block, start, torch.gather(u_acc, 1, at[:, :-1]).contiguous(), torch.gather(u_samp, 1, at[:, :1])[:, 0].contiguous(),
                                           mode=mode, lenience=lenience, probs=p_ref)
        for turn in range(B):                                # all but one sequence skipped, one after the other
            review(torch.where(torch.arange(B, device="cuda") == turn, start + 1, skip))
            n = int(n_ref[turn])
            assert int(status[turn]) == 0 and int(n_acc[turn]) == n and int(nxt[turn]) == int(nxt_ref[turn])
            if mode == 0:
                first = int(start[turn]) + 1
                assert torch.allclose(out_q[turn, first:first + n + 1], p_ref[turn, :n + 1], rtol=2e-2, atol=1e-6)
            length[turn] = cache[turn] + 1
        assert torch.equal(cache, start + 1 + n_ref)
    gm.close()
    ref.close()


@pytest.mark.parametrize("room", [8, 16])
@pytest.mark.parametrize("arch,H,dh,dims", [(0, 32, 128, (4096, 11008, 32000)), (1, 64, 64, (4096, 10240, 32128)), (0, 12, 64, (768, 3072, 32000))])
def test_review_after_nan_everywhere_with_wide_matrices(arch, H, dh, dims, room):
    """The same for the widths of the benchmark shapes' matrices: two to eight tiles per workgroup, long and short sums."""
    test_review_after_nan_everywhere(arch, H, dh, 192, 1, room, 0, 1.0, dims)
