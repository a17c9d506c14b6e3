"""The streaming projection at 97 to 144 rows (seven, eight and nine row tiles, a last one that is not full) through the component
entry point: automatic and given splits (8: five to eight waves per workgroup) against an fp64 product, partial columns of the packed
matrix included; and waves of 16 columns."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import minions_oracle as orc
from paper_2402_15678_amd import synth
from tests import util

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [97, 112, 113, 128, 129, 144])
@pytest.mark.parametrize("N,K,split", [(1000, 1024, 0), (5120, 2176, 0), (6152, 512, 1), (2304, 768, 3), (33000, 256, 0),
                                       (5120, 2048, 8), (6144, 2048, 8), (7168, 2048, 8), (8192, 2048, 8), (10240, 2048, 8), (5000, 2176, 9), (5120, 1024, 8), (768, 768, 6)])
def test_rows_and_splits(rows, N, K, split):
    from paper_2402_15678_amd import binding, harness
    g = torch.Generator(device="cuda").manual_seed(rows * 131 + N)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    a = torch.randn((rows, K), generator=g, device="cuda").half()
    bias = torch.randn((N,), generator=g, device="cuda")
    packed = harness.pack_matrix(w, 0)
    out = torch.full((rows, N), float("nan"), device="cuda")
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    binding.mn_proj_gemm(None, a.data_ptr(), packed.data_ptr(), bias.data_ptr(), out.data_ptr(), rows, N, K, split, ws.data_ptr(),
                         ws.numel(), harness.stream_ptr())
    want = a.double() @ w.double().t() + bias.double()
    # fp16 products are exact in fp32, K of them summed in fp32: 2^-24 of the sum of magnitudes per step, sqrt(K) steps of it at most
    bound = 2.0 ** -24 * float(np.sqrt(K)) * (a.double().abs() @ w.double().abs().t() + bias.double().abs()) + 1e-6
    assert bool(((out.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("rows", [1, 16, 17, 40, 64, 65])
@pytest.mark.parametrize("N,K", [(16400, 256), (16500, 384), (20480, 128), (20481, 256), (16384, 256)])
def test_sixteen_column_slices(rows, N, K):
    """Unsplit matrices of 513 to 640 32-column slices, and one of each next to them (rows and columns)."""
    test_rows_and_splits(rows, N, K, 1)


@pytest.mark.parametrize("rows", [1, 17, 40, 65, 96, 144])
def test_sixteen_column_slices_with_relu(rows):
    _check_step(synth.ModelDesc(synth.ARCH_OPT, synth.DT_BF16, 1, 512, 8, 8, 64, 16512, 500, 256), rows)


@pytest.mark.parametrize("rows", [97, 104, 112, 113, 128, 144])
@pytest.mark.parametrize("arch", [synth.ARCH_OPT, synth.ARCH_LLAMA])
def test_step_at_its_own_splits(arch, rows):
    """Inside a step these rows may take more splits than the entry points ask room for (the output projection of this width two instead
    of none): scores and cache rows of a layer against the CPU oracle."""
    from paper_2402_15678_amd import binding
    desc = synth.ModelDesc(arch, synth.DT_BF16, 1, 2048, 16, 16 if arch == synth.ARCH_OPT else 4, 128, 8192, 500, 256)
    pick, step = binding.lib._ZN2mn15gemm_pick_splitEiiii, binding.lib._ZN2mn15gemm_step_splitEiiiim
    room = ctypes.c_size_t(4 * rows * desc.d_ffn)    # (what gate||up or the first FFN matrix alone make of it)
    assert pick(rows, 2048, 2048, desc.dtype) == 1 and step(rows, 2048, 2048, desc.dtype, room) == 2
    _check_step(desc, rows)


def _check_step(desc, rows):
    from paper_2402_15678_amd import harness
    ks = np.asarray([7] * (rows // 8 - 1) + [7 + rows % 8] if rows >= 8 else [rows - 1], np.int32)
    B, k_max = len(ks), max(1, int(ks.max()))
    ctx = np.asarray([(29 * b + 3) % 60 for b in range(B)], np.int32)
    W = synth.make_weights(desc, 61)
    model = harness.DeviceModel.from_host(desc, W)
    kvh = synth.make_paged_kv(desc, ctx, ks, 62)
    kvd = harness.DeviceKV.from_host(desc, kvh)
    g = synth.stream(62, 1)
    last = g.integers(0, desc.vocab, size=B).astype(np.int32)
    voted = g.integers(0, desc.vocab, size=(B, k_max)).astype(np.int32)
    dev = lambda a: torch.tensor(np.asarray(a, np.int32), device="cuda:0")
    ses = harness.VerifySession(model, kvd, B, k_max, 1, int((ctx + ks + 1).max()), max_rows=rows, want_logits=True)
    t_last, t_k, t_voted = dev(last), dev(ks), dev(voted)
    caches = util.oracle_caches(desc, kvh)
    toks = [[int(last[b])] + voted[b, :ks[b]].tolist() for b in range(B)]
    want = np.concatenate(orc.decoder_step(desc, util.weights_f64(W), toks, caches))
    ses.forward(t_last, t_k, ks.tolist(), voted=t_voted)
    torch.cuda.synchronize()
    assert ses.dev_status.item() == 0
    tol = util.TOL[desc.dtype]
    assert np.abs(ses.logits.cpu().numpy() - want).max() < tol
    kp, vp = kvd.download(0)
    img = synth.PagedKV(16, kp.shape[0], kvh.block_tables.shape[1], kvh.block_tables, None, {0: kp}, {0: vp})
    for b in range(B):
        K, V = synth.gather_sequence_kv(img, 0, b, int(ctx[b] + ks[b] + 1))
        assert max(np.abs(K - caches[b].K[0]).max(), np.abs(V - caches[b].V[0]).max()) < tol
