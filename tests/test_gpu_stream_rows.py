"""The streaming projection at 97 to 144 rows (seven, eight and nine row tiles, a last one that is not full) through the component
entry point: automatic and given splits (8: five to eight waves per workgroup) against an fp64 product, partial columns of the packed
matrix included."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [97, 112, 113, 128, 129, 144])
@pytest.mark.parametrize("N,K,split", [(1000, 1024, 0), (5120, 2176, 0), (6152, 512, 1), (2304, 768, 3), (33000, 256, 0),
                                       (5120, 2048, 8), (6144, 2048, 8), (7168, 2048, 8), (8192, 2048, 8), (10240, 2048, 8), (5000, 2176, 9), (5120, 1024, 8), (768, 768, 6)])
def test_rows_and_splits(rows, N, K, split):
    from paper_2402_15678_amd import binding, harness, synth
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
