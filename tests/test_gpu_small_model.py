"""Small RMSNorm models, whose norms and residual stream are folded into the projections: logits and cache rows against the
CPU oracle where the tiling changes, and where the rows leave the range in which a folded norm is exact."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import minions_oracle as orc
from paper_2402_15678_amd import synth
from tests import util

pytestmark = pytest.mark.gpu

NARROW = synth.ModelDesc(synth.ARCH_LLAMA, synth.DT_BF16, 2, 256, 4, 4, 64, 512, 500, 512)
WIDE = synth.ModelDesc(synth.ARCH_LLAMA, synth.DT_BF16, 2, 1024, 16, 8, 64, 3584, 500, 512)     # most norm columns
LONG = synth.ModelDesc(synth.ARCH_LLAMA, synth.DT_BF16, 2, 896, 14, 14, 64, 3968, 500, 512)      # k ranges that leave a wave short, or none
GROUPED = synth.ModelDesc(synth.ARCH_LLAMA, synth.DT_BF16, 2, 768, 6, 2, 128, 896, 500, 512)


def _folded(desc, rows):
    from paper_2402_15678_amd import binding
    return bool(binding.lib._ZN2mn16gemm_small_modelEiiiiii(rows, desc.n_qkv, desc.d_model, desc.n_heads * desc.head_dim, desc.w1_rows, desc.d_ffn) & 1)


def _check(desc, W, ctx, ks, seed, tol):
    from paper_2402_15678_amd import binding, harness
    ctx, ks = np.asarray(ctx, np.int32), np.asarray(ks, np.int32)
    B, k_max = len(ctx), max(1, int(ks.max()))
    model = harness.DeviceModel.from_host(desc, W)
    kvh = synth.make_paged_kv(desc, ctx, ks, seed)
    kvd = harness.DeviceKV.from_host(desc, kvh)
    g = synth.stream(seed, 1)
    last = g.integers(0, desc.vocab, size=B).astype(np.int32)
    voted = g.integers(0, desc.vocab, size=(B, k_max)).astype(np.int32)
    dev = lambda a: torch.tensor(np.asarray(a, np.int32), device="cuda:0")
    ses = harness.VerifySession(model, kvd, B, k_max, 1, int((ctx + ks + 1).max()), max_rows=int((ks + 1).sum()), want_logits=True)
    t_last, t_k, t_voted = dev(last), dev(ks), dev(voted)
    caches = util.oracle_caches(desc, kvh)
    toks = [[int(last[b])] + voted[b, :ks[b]].tolist() for b in range(B)]
    want = np.concatenate(orc.decoder_step(desc, util.weights_f64(W), toks, caches))
    got = []
    for _ in range(2):                       # (the second pass finds the first one's statistics in the workspace)
        binding.mn_profile_enable(model.ctx, True)
        ses.forward(t_last, t_k, ks.tolist(), voted=t_voted)
        torch.cuda.synchronize()
        assert ses.dev_status.item() == 0
        launches = {k: n for k, (_, n) in binding.mn_profile_collect(model.ctx).items()}
        folded = _folded(desc, int((ks + 1).sum()))  # (the whole condition, the fused append included, holds in these tests)
        assert launches["norm"] == (2 if folded else 2 * desc.n_layers + 1) and launches["gemm"] == 4 * desc.n_layers + 1
        assert not (folded and launches["rope_append"])
        got.append(ses.logits.cpu().numpy().copy())
    assert np.array_equal(got[0], got[1])
    assert np.abs(got[0] - want).max() < tol, np.abs(got[0] - want).max()
    off = size = 0.0                         # of the rows that the last layer appended
    for l in range(desc.n_layers):
        kp, vp = kvd.download(l)
        img = synth.PagedKV(16, kp.shape[0], kvh.block_tables.shape[1], kvh.block_tables, None, {l: kp}, {l: vp})
        for b in range(B):
            K, V = synth.gather_sequence_kv(img, l, b, int(ctx[b] + ks[b] + 1))
            assert max(np.abs(K - caches[b].K[l]).max(), np.abs(V - caches[b].V[l]).max()) < tol
            if l == desc.n_layers - 1:
                for have, ref in ((K, caches[b].K[l]), (V, caches[b].V[l])):
                    off += float(((have - ref)[ctx[b]:] ** 2).sum())
                    size += float((ref[ctx[b]:] ** 2).sum())
    return got[0], (off / size) ** 0.5


@pytest.mark.parametrize("desc", [NARROW, WIDE, LONG, GROUPED], ids=["d256", "d1024", "d896", "d768-gqa"])
@pytest.mark.parametrize("rows", [1, 8, 9, 15, 16, 17, 25, 32, 33, 48, 95, 113])
def test_folded_norms_match_oracle(desc, rows):
    """Up to half a tile of rows, a whole one (in halves), its edges, two, three and more, with a last tile that is not full."""
    assert _folded(desc, rows)
    B = -(-rows // 4)
    ks = [3] * (B - 1) + [rows - 4 * (B - 1) - 1]
    ctx = [(37 * b + 5) % 90 for b in range(B)]
    _check(desc, synth.make_weights(desc, 91), ctx, ks, 92, util.TOL[desc.dtype])


@pytest.mark.parametrize("rows,folded", [(640, True), (641, False)])
def test_most_rows_of_folded_norms(rows, folded):
    assert _folded(NARROW, rows) == folded
    ks = [15] * 40 + [0] * (rows - 640)
    _check(NARROW, synth.make_weights(NARROW, 91), [b % 50 for b in range(len(ks))], ks, 93, util.TOL[synth.DT_BF16])


@pytest.mark.parametrize("rows", [25, 33, 48, 113])
def test_rows_of_every_tiling_that_grow(rows):
    """All rows outgrow their scale in front of every projection that folds a norm (see below), in row groups of two and three tiles."""
    W = synth.make_weights(NARROW, 91)
    W["tok_emb"] = W["tok_emb"] * 2.0 ** -10
    for L in W["layers"]:
        L["wo"] = L["wo"] * 2.0 ** 12
        L["w2"] = L["w2"] * 2.0 ** 13
    assert _folded(NARROW, rows)
    B = -(-rows // 4)
    _check(NARROW, W, [(37 * b + 5) % 90 for b in range(B)], [3] * (B - 1) + [rows - 4 * (B - 1) - 1], 94, util.TOL[synth.DT_BF16])


def test_rows_that_grow_or_shrink_between_two_norms():
    """The scale that a row is stored with comes from its norm before: rows that outgrow it (projections 2^12 and 2^13
    times their size on embeddings 2^-10 of theirs) or all but vanish (an output projection that takes the row back to 2^-7 of itself) are
    normalised from the fp32 rows instead, to the same tolerance."""
    W = synth.make_weights(NARROW, 91)
    W["tok_emb"] = W["tok_emb"] * 2.0 ** -10
    for L in W["layers"]:
        L["wo"] = L["wo"] * 2.0 ** 12
        L["w2"] = L["w2"] * 2.0 ** 13        # (as much from the FFN, which reads the folded norm)
    _check(NARROW, W, [20, 0, 33, 7], [3, 2, 0, 3], 94, util.TOL[synth.DT_BF16])

    desc = dataclasses.replace(NARROW, n_layers=1, d_model=128, n_heads=2, n_kv_heads=2, norm_eps=1e-9)
    W = synth.make_weights(desc, 95)
    W["tok_emb"] = (np.sign(W["tok_emb"]) + (W["tok_emb"] == 0)).astype(np.float32) * 2.0 ** -6
    L = W["layers"][0]
    L["ln1_g"] = np.ones_like(L["ln1_g"])
    L["wqkv"] = L["wqkv"].copy()
    L["wqkv"][256:384] = np.eye(128, dtype=np.float32)             # values = the normalised row, and no other key to see
    L["wo"] = -np.eye(128, dtype=np.float32) * np.float32(2.0 ** -6 * (1 - 2.0 ** -7))
    _check(desc, W, [0] * 5, [0] * 5, 96, util.TOL[synth.DT_BF16])


@pytest.mark.parametrize("rows", [5, 12, 33])
@pytest.mark.parametrize("gain,channel", [(2.0 ** -12, 1.0), (2.0 ** -10, 64.0)], ids=["small-gains", "dominant-channel"])
def test_small_normalised_rows_keep_their_bits(gain, channel, rows):
    """Norms whose output is small everywhere (gains of 2^-12, the matrices behind them 2^12 times theirs) or in all columns but one
    (a channel 64 times the others', as trained models have them, with its gain taken back): the last layer's new keys and values,
    which are the projection of a folded norm, are off by what rounding to fp16 gives.  That is 2^-12.2 of a value in the mean
    (a step of 2^-11 to 2^-10 of it, over sqrt(12)) at each of seven places (embedding's norm, values, attention and its output, FFN
    norm, activation, last norm, pages), sqrt(7) 2^-12.2 together: below 2^-10."""
    desc = NARROW
    W = synth.make_weights(desc, 97)
    W["tok_emb"] = W["tok_emb"].copy()
    W["tok_emb"][:, 7] *= channel
    for L in W["layers"]:
        for norm, matrix in (("ln1_g", "wqkv"), ("ln2_g", "w1")):
            L[norm] = L[norm] * np.float32(gain)
            L[norm][7] /= np.float32(channel)
            L[matrix] = L[matrix] * np.float32(1.0 / gain)
    B = -(-rows // 4)
    ks = [3] * (B - 1) + [rows - 4 * (B - 1) - 1]
    assert _folded(desc, rows)
    rel = _check(desc, W, [(37 * b + 5) % 90 for b in range(B)], ks, 98, util.TOL[desc.dtype])[1]
    assert rel < 2.0 ** -10, rel


def _logits(desc, W, ctx, ks, last, voted):
    from paper_2402_15678_amd import harness
    ctx, ks = np.asarray(ctx, np.int32), np.asarray(ks, np.int32)
    B, k_max = len(ctx), int(ks.max())
    model = harness.DeviceModel.from_host(desc, W)
    kvh = synth.make_paged_kv(desc, ctx, ks, 99)
    kvd = harness.DeviceKV.from_host(desc, kvh)
    dev = lambda a: torch.tensor(np.asarray(a, np.int32), device="cuda:0")
    ses = harness.VerifySession(model, kvd, B, k_max, 1, int((ctx + ks + 1).max()), max_rows=int((ks + 1).sum()), want_logits=True)
    t_last, t_k, t_voted = dev(last), dev(ks), dev(voted)
    ses.forward(t_last, t_k, ks.tolist(), voted=t_voted)
    torch.cuda.synchronize()
    assert ses.dev_status.item() == 0
    toks = [[int(last[b])] + voted[b, :ks[b]].tolist() for b in range(B)]
    want = np.concatenate(orc.decoder_step(desc, util.weights_f64(W), toks, util.oracle_caches(desc, kvh)))
    got = ses.logits.cpu().numpy()
    assert np.abs(got - want).max() < util.TOL[desc.dtype], np.abs(got - want).max()
    return got


@pytest.mark.parametrize("rows", [5, 12, 25, 33, 48, 113])
@pytest.mark.parametrize("grown_by", ["attention", "ffn"])
def test_marked_rows_leave_their_neighbours_alone(grown_by, rows):
    """Sequences 1 and 6 (where there is one) take tokens whose embeddings are 2^-18 of the others', so that their rows outgrow the
    scale they were stored with (in front of gate||up or of the next QKV) while their neighbours' do not: every logit is right, and
    the neighbours' are bit for bit those of the batch in which these sequences take ordinary tokens."""
    desc = dataclasses.replace(NARROW, norm_eps=1e-16)
    assert _folded(desc, rows)
    W = synth.make_weights(desc, 91)
    W["tok_emb"] = W["tok_emb"].copy()
    W["tok_emb"][400:] *= np.float32(2.0 ** -18)
    if grown_by == "ffn":
        W["layers"][0]["wo"] = np.zeros_like(W["layers"][0]["wo"])
    B = -(-rows // 4)
    ks = [3] * (B - 1) + [rows - 4 * (B - 1) - 1]
    ctx = [(37 * b + 5) % 90 for b in range(B)]
    g = synth.stream(99, 2)
    last, voted = g.integers(0, 400, size=B), g.integers(0, 400, size=(B, 3))
    plain = _logits(desc, W, ctx, ks, last, voted)
    small = [b for b in (1, 6) if b < B]
    last[small] = g.integers(400, 500, size=len(small))
    voted[small] = g.integers(400, 500, size=(len(small), 3))
    mixed = _logits(desc, W, ctx, ks, last, voted)
    other = np.repeat([b not in small for b in range(B)], np.asarray(ks) + 1)
    assert np.array_equal(mixed[other], plain[other])


@pytest.mark.parametrize("desc", [NARROW, GROUPED], ids=["hd64", "hd128"])
@pytest.mark.parametrize("copies", [1, 5], ids=["8-waves", "4-waves"])
def test_fused_append_over_tiles_per_wave(desc, copies):
    """The few-row attention kernel that appends: waves with no tile, one, two (both ends of the pass over two) and up to six, and
    new rows that start, end or straddle a tile; with 8 waves (up to 256 workgroups) and with 4."""
    desc = dataclasses.replace(desc, max_pos=1664)
    ctx = [0, 1, 29, 31, 32, 61, 255, 256, 286, 509, 512, 767, 770, 1023, 1024, 1054, 1279, 1310, 1535, 1570][:20 if copies == 1 else 13]
    ks = [(3 * i) % 4 for i in range(len(ctx))]
    if copies > 1 and desc.n_kv_heads == 2:  # (more than 256 workgroups of two KV heads)
        copies = 10
    ctx, ks = ctx * copies, ks * copies
    assert (len(ctx) * desc.n_kv_heads > 256) == (copies > 1)
    _check(desc, synth.make_weights(desc, 91), ctx, ks, 95, util.TOL[desc.dtype])
