"""GPU parity of the per-layer products over the tile shapes their grids choose: the queries
with their input norm (narrow and wide tiles that sum the squares of the rows they read, large
tiles with a norm launch of their own) and the stand-in block's output projection (narrow,
128 x 64, 128 x 128 and 256 x 256 tiles), at ragged token counts.

With one layer, a prefill's states are its embeddings, so one pass is h = X + W_o o with o =
layer_attend over the cache that pool makes of them. The queries show in o:
rows at both ends of every sequence and on both sides of every tile boundary are computed again
in float64 from X and the library's own cache rows, and held to the bf16 bounds row by row. h is
checked in every element against X + W_o o for the library's own o: an fp32 sum rounded once to
bf16 (2^-8 of the value), with W_o wide enough that X does not hide the product."""
import pytest
import torch

from tests.parity import check_close, wm  # noqa: F401

pytestmark = pytest.mark.gpu

EPS, THETA = 1e-6, 1e6


def _rms(x, g):
    return g * x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS)


def _attend_row(P, x, i, K, V, Hq, Hkv, d):
    """Output row [Hq d] of the token with embedding x at position i, float64; K, V [Hkv, S, d]."""
    q = (P["Wq"][0] @ _rms(x, P["g_in"][0])).reshape(Hq, d)
    q = _rms(q, P["g_qnorm"][0])
    f = i * THETA ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    a, b = q[:, :d // 2], q[:, d // 2:]
    q = torch.cat([a * f.cos() - b * f.sin(), b * f.cos() + a * f.sin()], 1)
    kv = torch.arange(Hq, device=x.device) // (Hq // Hkv)
    Kd, Vd = P["Kd"][0][:, None], P["Vd"][0][:, None]
    K, V = torch.cat([Kd, K[:, :i]], 1)[kv], torch.cat([Vd, V[:, :i]], 1)[kv]  # the dummy first
    w = torch.softmax((K @ q[:, :, None])[:, :, 0] / d ** 0.5, 1)
    return (w[:, None] @ V)[:, 0].reshape(-1)


@pytest.mark.parametrize("B,T,D,Hq,Hkv,d", [
    # queries / output projection (channels x tokens of a block)
    (1, 37, 64, 2, 1, 64),        # narrow 64 x 64 / narrow 64 x 64
    (2, 100, 96, 3, 3, 96),       # narrow 96 x 64 / narrow
    (3, 333, 512, 6, 3, 96),      # narrow 96 x 64 / narrow
    (3, 333, 256, 4, 2, 64),      # narrow 64 x 64 / narrow
    (4, 1030, 512, 6, 3, 96),     # narrow 96 x 64 / 128 x 64
    (4, 1030, 512, 8, 8, 64),     # wide 128 x 64 / 128 x 64
    (4, 1024, 1024, 12, 3, 96),   # wide 288 x 64 / 128 x 128
    (4, 1670, 512, 12, 3, 96),    # large 192 x 256, norm apart / 128 x 64
    (5, 1111, 2048, 32, 4, 64)])  # large 256 x 256, norm apart / 256 x 256
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
    X, W_o = normal(B, T, D), normal(1, D, Hq * d, std=0.5)
    dims = wm.make_dims(B, T, 1, 1, D, Hq, Hkv, d, S_cap=T, dtype=wm.BF16, eps=EPS,
                        rope_theta=THETA)
    Kc = torch.zeros((1, B, Hkv, T, d), dtype=torch.bfloat16, device="cuda")
    Vc = torch.zeros_like(Kc)
    H = torch.empty((B, T, 1, D), dtype=torch.bfloat16, device="cuda")
    top = torch.full((B, T, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.prefill_passes(dims, P, W_o, X, [0], 1, Kc, Vc, H, h_top=top)
    # the layer attended the cache of the first pool (the pass's own takes the rows' norms from
    # the layer's queries, which may round otherwise)
    ctx = torch.zeros(B, dtype=torch.int32, device="cuda")
    wm.pool(dims, P, X[:, :, None].contiguous(), ctx, Kc, Vc)
    O = torch.full((1, B, T, Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.layer_attend(dims, P, 0, X[:, :, None].contiguous(), [0], ctx, Kc, Vc, O[0])
    torch.cuda.synchronize()
    assert torch.equal(H[:, :, 0], X)
    assert torch.isfinite(O.float()).all()

    # tokens at the ends of the sequences and on both sides of the tiles' boundaries
    N, ends = B * T, {0, B * T - 1}
    for b in range(B):
        ends |= {b * T, b * T + T - 1}
    for tile in (64, 256):
        for n in range(tile, N, max(1, N // tile // 6) * tile):
            ends |= {n - 1, n}
        ends |= {N // tile * tile - 1, min(N // tile * tile, N - 1)}
    P64 = {n: t.double() for n, t in P.items()}
    K64, V64 = Kc[0].double(), Vc[0].double()
    for n in sorted(ends):
        b, i = n // T, n % T
        ref = _attend_row(P64, X[b, i].double(), i, K64[b], V64[b], Hq, Hkv, d)
        check_close(O[0, b, i], ref.cpu().numpy(), "bf16", "o of sequence %d, position %d" % (b, i))

    ref = X.double() + O[0].double() @ W_o[0].double().t()
    off = (top.double() - ref).abs() - 2.0 ** -8 * ref.abs()
    # what is left: the fp32 sum of Hq d terms, 2^-24 of the terms for each step at most
    terms = X.double().abs() + O[0].double().abs() @ W_o[0].double().abs().t()
    assert bool((off <= 2.0 ** -24 * Hq * d * terms).all()), float((off / terms).max())


@pytest.mark.parametrize("D", [512, 2048, 4608])
@pytest.mark.parametrize("d,Hq", [(64, 4), (96, 3)])
def test_own_norm_keeps_fp32(wm, d, Hq, D):
    """The norm that a product makes of the rows it reads (1 / RMS, left at the head of the
    workspace) against float64. Roundings of 2^-24 in the sum: five for 16 squares (four for
    eight, one where two eights join), three for the sums' own with the rounding of each carried
    along, one where the halves of a row join, two for the mean and eps; half of these eleven
    pass the root, which adds its own and the division's. Squares added one after the other are
    off by 20 such roundings at D = 2048 and 50 at 4608."""
    B, L = 80, 2
    gen = torch.Generator().manual_seed(9)

    def normal(*shape):
        return torch.empty(shape).normal_(generator=gen).bfloat16().cuda()

    print("own norm D%d d%d" % (D, d), flush=True)
    P = {n: torch.zeros(8, dtype=torch.bfloat16, device="cuda") for n in wm.PARAM_NAMES}
    P.update(Kd=normal(1, Hq, d), Vd=normal(1, Hq, d), g_in=normal(L, D), Wq=normal(L, Hq * d, D),
             g_qnorm=normal(L, d))
    H = normal(B, 5, L, D)
    dims = wm.make_dims(B, 5, L, 1, D, Hq, Hq, d, S_cap=64, dtype=wm.BF16, eps=EPS)
    Kc = torch.zeros((1, B, Hq, 64, d), dtype=torch.bfloat16, device="cuda")
    O = torch.empty((B, 5, Hq * d), dtype=torch.bfloat16, device="cuda")
    ws = wm.workspace(dims, wm.OP_LAYER_ATTEND)
    ctx = torch.zeros(B, dtype=torch.int32, device="cuda")
    wm.layer_attend(dims, P, 1, H, [0, 0], ctx, Kc, torch.zeros_like(Kc), O, ws=ws)
    torch.cuda.synchronize()
    got = ws[:4 * B * 5 * L].view(torch.float32).reshape(B, 5, L)[:, :, 1].double()
    x = H[:, :, 1].double()
    ref = torch.rsqrt((x * x).mean(-1) + EPS)
    worst = float((got / ref - 1).abs().max())
    print("worst %.2g" % worst)
    assert worst <= 8 * 2.0 ** -24, worst
