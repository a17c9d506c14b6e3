"""fp32 models against the CPU oracle where their kernels change: the norm folded into the projection behind it (narrow rows, few
rows), the append folded into the attention kernel (few rows per sequence), pieces per row of the projections, page sizes."""
import numpy as np
import pytest
import torch

from oracle import minions_oracle as orc
from paper_2402_15678_amd import synth
from tests import util

pytestmark = pytest.mark.gpu


def _check(desc, ctx, ks, block_size=16, seed=71):
    from paper_2402_15678_amd import binding, harness
    ctx, ks = np.asarray(ctx, np.int32), np.asarray(ks, np.int32)
    B, k_max = len(ctx), max(1, int(ks.max()))
    W = synth.make_weights(desc, seed)
    model = harness.DeviceModel.from_host(desc, W)
    kvh = synth.make_paged_kv(desc, ctx, ks, seed, block_size=block_size)
    kvd = harness.DeviceKV.from_host(desc, kvh)
    g = synth.stream(seed, 1)
    last = g.integers(0, desc.vocab, size=B).astype(np.int32)
    voted = g.integers(0, desc.vocab, size=(B, k_max)).astype(np.int32)
    dev = lambda a: torch.tensor(np.asarray(a, np.int32), device="cuda:0")
    ses = harness.VerifySession(model, kvd, B, k_max, 1, int((ctx + ks + 1).max()), max_rows=int((ks + 1).sum()), want_logits=True)
    t_last, t_k, t_voted = dev(last), dev(ks), dev(voted)
    caches = util.oracle_caches(desc, kvh)
    toks = [[int(last[b])] + voted[b, :ks[b]].tolist() for b in range(B)]
    want = np.concatenate(orc.decoder_step(desc, W, toks, caches))
    binding.mn_profile_enable(model.ctx, True)
    ses.forward(t_last, t_k, ks.tolist(), voted=t_voted)
    torch.cuda.synchronize()
    launches = {k: n for k, (_, n) in binding.mn_profile_collect(model.ctx).items()}
    assert ses.dev_status.item() == 0
    tol = util.TOL[synth.DT_F32]
    assert np.abs(ses.logits.cpu().numpy() - want).max() < tol
    greedy = np.concatenate([ses.greedy.cpu().numpy()[b, :ks[b] + 1] for b in range(B)])
    assert all(util.near_tie_ok(want[i], greedy[i], tol) for i in range(len(greedy)))
    for l in range(desc.n_layers):
        kp, vp = kvd.download(l)
        img = synth.PagedKV(block_size, kp.shape[0], kvh.block_tables.shape[1], kvh.block_tables, None, {l: kp}, {l: vp})
        for b in range(B):
            K, V = synth.gather_sequence_kv(img, l, b, int(ctx[b] + ks[b] + 1))
            assert max(np.abs(K - caches[b].K[l]).max(), np.abs(V - caches[b].V[l]).max()) < tol
    return launches


def _opt(d, heads, hd, ffn):
    return synth.ModelDesc(synth.ARCH_OPT, synth.DT_F32, 2, d, heads, heads, hd, ffn, max(1001, 3 * d + 1), 1300)  # (the QKV sums lie where the scores will)


@pytest.mark.parametrize("d,heads,hd,ffn", [(64, 8, 8, 64), (256, 4, 64, 320), (320, 5, 64, 576), (512, 4, 128, 1024), (576, 9, 64, 320), (1024, 4, 256, 1088), (1088, 17, 64, 256)])
def test_widths(d, heads, hd, ffn):
    """One, two and four pieces per row, rows that are no whole number of them; norms are launches beyond two pieces."""
    assert _check(_opt(d, heads, hd, ffn), [40, 0, 3], [4, 1, 7])["norm"] == (0 if d <= 512 else 5)


@pytest.mark.parametrize("rows", [1, 8, 9, 64, 65])
def test_rows(rows):
    """Row groups of 8, the most rows of a folded norm and one more."""
    ks = [7] * (rows // 8) + ([rows % 8 - 1] if rows % 8 else [])
    assert _check(_opt(256, 4, 64, 256), [11 * b % 70 for b in range(len(ks))], ks)["norm"] == (0 if rows <= 64 else 5)


@pytest.mark.parametrize("k", [15, 16, 17])
@pytest.mark.parametrize("block_size", [1, 5, 16])
def test_appended_rows(k, block_size):
    """17 rows of a sequence are the most that the attention kernel appends; contexts below, at and beyond a chunk of 256 keys
    (16 of them with 1024 threads), pages whose values come in fours and pages whose do not."""
    _check(_opt(256, 4, 64, 256), [0, 250, 16, 256 - k], [k, 2, 0, k], block_size)
    _check(_opt(256, 4, 64, 256), [1100, 3], [k, 1], block_size)


@pytest.mark.parametrize("hd", [8, 16])
@pytest.mark.parametrize("k", [4, 20])
def test_narrow_heads_long_contexts(hd, k):
    """Chunks of 256 and 1024 keys whose groups of four are fewer than the threads' pieces of them: none counts twice."""
    _check(_opt(128, 128 // hd, hd, 64), [252, 300, 1], [k, 0, 1])
    _check(_opt(64, 64 // hd, hd, 64), [1100, 3], [k, 1])


def test_rotary_and_head_groups():
    desc = synth.ModelDesc(synth.ARCH_LLAMA, synth.DT_F32, 2, 256, 8, 2, 32, 256, 1001, 600)
    _check(desc, [33, 0, 300], [4, 16, 1])
    _check(desc, [33, 0], [4, 20], 8)
