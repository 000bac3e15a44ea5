"""GPU parity of the per-layer products over the tile shapes their grids choose: the queries
with their input norm (wide, narrow, and large tiles with a norm launch of their own) and the
stand-in block's output projection (narrow, 128 x 64, 128 x 128 and 256 x 256 tiles), at
ragged token counts.

With one layer, a prefill's states are its embeddings, so its cache is that of the first pool
and one pass is h = X + W_o o with o = layer_attend over that cache: h is checked against the
float64 product of the library's own o, and o against layer_step's, whose queries come from
the large tiles. Both sides round at the same points (bf16 results of fp32 sums), so a result
is off by its own rounding, 2^-9, plus that of sums in another order: 2^-8 in all."""
import pytest
import torch

from tests.parity import wm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,Hq,Hkv,d", [(1, 37, 64, 2, 1, 64), (2, 100, 96, 3, 3, 96),
                                            (3, 333, 512, 6, 3, 96), (3, 333, 256, 4, 2, 64),
                                            (4, 1030, 512, 6, 3, 96), (4, 1030, 512, 8, 8, 64),
                                            (4, 1024, 1024, 12, 3, 96),
                                            (5, 1111, 2048, 32, 4, 64)])
def test_one_layer_pass(wm, B, T, D, Hq, Hkv, d):
    print("one layer B%d T%d D%d %d/%d heads of %d" % (B, T, D, Hq, Hkv, d), flush=True)
    gen = torch.Generator().manual_seed(77)

    def normal(*shape, std=1.0, mean=0.0):
        return torch.empty(shape).normal_(mean, std, generator=gen).bfloat16().cuda()

    P = {"g_pre": normal(2, 1, D, std=0.1, mean=1.0), "W_alpha": normal(2, 1, D, std=0.002),
         "b_alpha": torch.ones(2, 1).bfloat16().cuda(), "g_mid": normal(2, 1, D, std=0.1, mean=1.0),
         "Wk": normal(1, Hkv * d, D, std=0.05), "Wv": normal(1, Hkv * d, D, std=0.05),
         "g_knorm": normal(1, d, std=0.1, mean=1.0), "Kd": normal(1, Hkv, d),
         "Vd": normal(1, Hkv, d), "g_in": normal(1, D, std=0.1, mean=1.0),
         "Wq": normal(1, Hq * d, D, std=0.05), "g_qnorm": normal(1, d, std=0.1, mean=1.0)}
    X, W_o = normal(B, T, D), normal(1, D, Hq * d, std=0.05)
    dims = wm.make_dims(B, T, 1, 1, D, Hq, Hkv, d, S_cap=T, dtype=wm.BF16)
    Kc = torch.zeros((1, B, Hkv, T, d), dtype=torch.bfloat16, device="cuda")
    Vc = torch.zeros_like(Kc)
    H = torch.empty((B, T, 1, D), dtype=torch.bfloat16, device="cuda")
    top = torch.full((B, T, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.prefill_passes(dims, P, W_o, X, [0], 1, Kc, Vc, H, h_top=top)
    O = torch.full((1, B, T, Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ctx = torch.zeros(B, dtype=torch.int32, device="cuda")
    wm.layer_attend(dims, P, 0, X[:, :, None].contiguous(), [0], ctx, Kc, Vc, O[0])
    K2, V2, O2 = torch.zeros_like(Kc), torch.zeros_like(Vc), torch.empty_like(O)
    wm.layer_step(dims, P, X[:, :, None].contiguous(), [0], ctx, K2, V2, O2)
    torch.cuda.synchronize()

    def off(a, b):
        a, b = a.double(), b.double()
        assert torch.isfinite(a).all()
        return ((a - b).norm() / b.norm()).item()

    assert torch.equal(H[:, :, 0], X)
    assert off(O, O2) <= 2 ** -8
    ref = X.double().cpu() + O[0].double().cpu() @ W_o[0].double().cpu().t()
    assert off(top.cpu(), ref) <= 2 ** -8
