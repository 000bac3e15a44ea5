"""GPU parity of the bf16 decode attention on the matrix cores (Section 3.1 Step 3, Section
3.2) at the edges of its tiles: 32 rows (consumers x grouped heads x new tokens) per tile,
32-slot blocks dealt to one, two or four waves, splits of at least 256 slots, and ragged sequences that
leave waves and whole splits without a slot. Against the oracle, with the repository's bf16
bounds."""
import pytest
import torch

import oracle
from tests import synth
from tests.parity import (_bias, _check_cache, _dev, _f64, _gdims, _odims,  # noqa: F401
                          check_close, wm)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96])
@pytest.mark.parametrize("mask_mode", [0, 1])
@pytest.mark.parametrize("L,Hq,Hkv,T_new", [(1, 2, 2, 1),     # 1 row
                                            (4, 6, 3, 4),     # 32 rows: a full tile
                                            (11, 3, 1, 1),    # 33 rows: one in a second tile
                                            (5, 16, 2, 2)])   # 80 rows: three tiles
@pytest.mark.parametrize("ctx", [0, 1, 31, 33, 128, 129, 257, 1100])
def test_decode_row_and_slot_edges(wm, d, mask_mode, L, Hq, Hkv, T_new, ctx):
    B = 3
    w = synth.small("dec_d%d" % d, B=B, T_new=T_new, L=L, k=1, D=64, Hq=Hq, Hkv=Hkv, d=d,
                    ctx=ctx + T_new, dtype="bf16", chan_map=[0] * L)
    print("decode d%d mask%d L%d Hq%d T%d ctx%d" % (d, mask_mode, L, Hq, T_new, ctx), flush=True)
    P = synth.make_params(w, _bias(w))
    Q = synth.make_queries(w)
    Kc, Vc = synth.make_cache_cpu(w, fill=0.0)
    ctx_len = torch.tensor([ctx, ctx // 2, 0], dtype=torch.int32)
    ref = oracle.channel_attend(_odims(w, mask_mode=mask_mode), P, Q, w.chan_map,
                                ctx_len.numpy(), _f64(Kc), _f64(Vc))
    O = torch.full((L, B, T_new, Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.channel_attend(_gdims(wm, w, mask_mode=mask_mode, ctx_max=ctx), _dev(P), Q.cuda(),
                      w.chan_map, ctx_len.cuda(), Kc.cuda(), Vc.cuda(), O)
    torch.cuda.synchronize()
    check_close(O, ref, "bf16", "decode d%d mask%d rows %d ctx %d"
                % (d, mask_mode, L * Hq // Hkv * T_new, ctx))


@pytest.mark.parametrize("d", [64, 96])
@pytest.mark.parametrize("mode", ["linear", "softmax", "static", "nofeedback"])
@pytest.mark.parametrize("B,T_new,D,p,ctx", [(1, 1, 32, 1, 0),      # waves without a share of K
                                             (5, 1, 160, 2, 37),   # a part batch of columns
                                             (31, 1, 64, 1, 70),
                                             (8, 4, 544, 3, 70),   # 32 tokens
                                             (11, 3, 96, 1, 9)])   # 33: the many-token path
def test_few_token_step(wm, d, mode, B, T_new, D, p, ctx):
    """The few-token pool and queries (router, mix, K/V and query projections of at most 32
    bf16 tokens) through the fused step, at uneven widths, against the oracle."""
    L = 4 if mode == "nofeedback" else 5
    k = L if mode == "nofeedback" else 3
    w = synth.small("few_%s" % mode, B=B, T_new=T_new, L=L, k=k, D=D, Hq=4, Hkv=2, d=d, ctx=ctx,
                    dtype="bf16", p=p)
    print("few tokens d%d %s B%d T%d D%d p%d" % (d, mode, B, T_new, D, p), flush=True)
    P = synth.make_params(w, torch.as_tensor(_bias(w)) + 0.2, gains="random")
    H = synth.make_states(w)
    K0, V0 = synth.make_cache_cpu(w)
    ctx_len = synth.make_ctx_len(w, ragged=True)
    opts = dict(mix_mode=1 if mode == "softmax" else 0,
                router_mode={"static": 1, "nofeedback": 2}.get(mode, 0))
    Ko, Vo = _f64(K0).copy(), _f64(V0).copy()
    Oo = oracle.layer_step(_odims(w, **opts), P, H, w.chan_map, ctx_len.numpy(), Ko, Vo)
    Kg, Vg = K0.cuda(), V0.cuda()
    O = torch.full((w.L, B, T_new, w.Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.layer_step(_gdims(wm, w, **opts), _dev(P), H.cuda(), w.chan_map, ctx_len.cuda(), Kg, Vg, O)
    torch.cuda.synchronize()
    _check_cache(Kg, Ko, K0, w, ctx_len.numpy(), "bf16", "K")
    _check_cache(Vg, Vo, V0, w, ctx_len.numpy(), "bf16", "V")
    check_close(O, Oo, "bf16", "few-token step %s" % mode)


# (d, k, Hq, Hkv, B, T_new, ctx, waves a workgroup)
STREAM_CASES = [(96, 8, 6, 3, 8, 4, 4000, 2), (64, 6, 8, 8, 16, 1, 2000, 2),
                (64, 12, 16, 16, 28, 1, 100, 1), (96, 12, 16, 16, 20, 2, 98, 1)]


@pytest.mark.parametrize("docs", [False, True])
@pytest.mark.parametrize("d,k,Hq,Hkv,B,T_new,ctx,waves", STREAM_CASES)
def test_streamed_cache(wm, d, k, Hq, Hkv, B, T_new, ctx, waves, docs):
    """Caches just past 128 MB, whose slots are copied without keeping them in the caches
    (non-temporal), with and without documents, by workgroups of two waves and (walks of at
    most 128 slots) one: the first and the last sequence against the oracle."""
    w = synth.small("stream_d%d" % d, B=B, T_new=T_new, L=k, k=k, D=64, Hq=Hq, Hkv=Hkv, d=d,
                    ctx=ctx + T_new, dtype="bf16")
    print("streamed cache d%d k%d B%d T%d ctx%d docs %s" % (d, k, B, T_new, ctx, docs), flush=True)
    kend = ctx + T_new
    assert 4 * k * B * Hkv * kend * d >= 128 << 20
    length, slices = 4096, k * B * Hkv
    while length > 256 and slices * -(-kend // length) < 512:
        length //= 2
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    wgs = slices * -(-kend // length)
    four = wgs <= cus if d == 96 else wgs <= 2 * cus or (wgs > 5 * cus and min(kend, length) >= 1024)
    assert waves == (1 if min(kend, length) <= 128 else 4 if four else 2)
    P = synth.make_params(w, _bias(w))
    Q = synth.make_queries(w)
    Kc, Vc = synth.make_cache_device(w, fill=0.0)
    ctx_len = torch.tensor([ctx - 7 * (b % 5) for b in range(B)], dtype=torch.int32)
    doc = synth.make_doc_start(w, ctx_len, mean_len=61.0) if docs else None
    O = torch.full((k, B, T_new, Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.channel_attend(_gdims(wm, w, ctx_max=ctx), _dev(P), Q.cuda(), w.chan_map, ctx_len.cuda(),
                      Kc, Vc, O, doc_start=doc.cuda() if docs else None)
    torch.cuda.synchronize()
    at = [0, B - 1]
    ref = oracle.channel_attend(_odims(w, B=2), P, Q[:, at], w.chan_map, ctx_len[at].numpy(),
                                _f64(Kc[:, at]), _f64(Vc[:, at]),
                                doc_start=doc[at].numpy() if docs else None)
    check_close(O[:, at], ref, "bf16", "streamed d%d B%d docs %s" % (d, B, docs))


@pytest.mark.parametrize("k", [1, 12])
@pytest.mark.parametrize("B,ctx", [(1, 8191), (2, 4000)])
def test_one_layer_splits_its_own_channel(wm, k, B, ctx):
    """One layer reads one channel of the cache: its slots are split for that channel's
    workgroups alone (until there are 512 of them, at 256 slots or more each), however many
    channels have no reader in the call. The ranges are counted by the partial states written
    into a workspace of all ones."""
    L, Hq, d = 12, 16, 64
    w = synth.small("one_layer", B=B, T_new=1, L=L, k=k, D=64, Hq=Hq, Hkv=Hq, d=d, ctx=ctx + 1,
                    dtype="bf16", chan_map=[0] * L)
    print("one layer of %d channels, B%d ctx%d" % (k, B, ctx), flush=True)
    P = _dev(synth.make_params(w, _bias(w)))
    H = synth.make_states(w).cuda()
    Kc, Vc = synth.make_cache_device(w, fill=0.0)
    ctx_len = torch.full((B,), ctx, dtype=torch.int32, device="cuda")
    dims = _gdims(wm, w, ctx_max=ctx)
    ws = torch.full((wm.workspace_size(dims, wm.OP_LAYER_ATTEND),), 255, dtype=torch.uint8,
                    device="cuda")
    O = torch.full((B, 1, Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.layer_attend(dims, P, 0, H, w.chan_map, ctx_len, Kc, Vc, O, ws=ws)
    torch.cuda.synchronize()
    assert torch.isfinite(O.float()).all()
    words = int((ws.view(torch.int32) != -1).sum()) - B * Hq * d // 2  # less the queries
    nsplit, rest = divmod(words, B * Hq * (d + 2))
    assert rest == 0
    length = 4096
    while length > 256 and B * Hq * -(-(ctx + 1) // length) < 512:
        length //= 2
    assert nsplit == -(-(ctx + 1) // length), (nsplit, length)


@pytest.mark.parametrize("d", [64, 96])
def test_weights_keep_fp32(wm, d):
    """Two slots whose values nearly cancel under the weights 1 and exp(s): the output shows the
    weights' own error. Bound: the bf16 rounding of the result, 2^-8 of it, and 2^-20 of the
    terms' sum, what a score of at most 1 in fp32 (2^-24 for each of its few roundings) and an
    exponential good to 2^-23 allow; weights of 16 bits are off by up to 2^-17."""
    L, Hq = 16, 2
    w = synth.small("cancel", B=1, T_new=1, L=L, k=1, D=64, Hq=Hq, Hkv=1, d=d, ctx=2,
                    dtype="bf16", chan_map=[0] * L)
    print("weights d%d" % d, flush=True)
    P = synth.make_params(w, _bias(w))
    Kc, Vc = synth.make_cache_cpu(w, fill=0.0)
    gen = torch.Generator().manual_seed(5)
    rows = L * Hq
    Q = torch.randn(L, 1, Hq, 1, d, generator=gen).bfloat16()
    Kc[:, :, :, 0] = 0
    k1 = torch.randn(d, generator=gen).bfloat16()
    # scores in (-0.65, -0.02): the query's part along the key replaced
    q64, k64 = Q.double().reshape(rows, d), k1.double()
    want = torch.linspace(-0.65, -0.02, rows, dtype=torch.float64)
    q64 = q64 - (q64 @ k64)[:, None] * k64 / (k64 @ k64)
    q64 = q64 + (want * d ** 0.5 / (k64 @ k64))[:, None] * k64
    Q = q64.reshape(Q.shape).bfloat16()
    p1 = torch.exp(Q.double().reshape(rows, d) @ k64 / d ** 0.5)
    Kc[0, 0, 0, 1] = k1
    # channel j cancels for row j mod rows: the bf16 pair of [1, 2) closest to p1 y = x
    grid = 1 + torch.arange(128, dtype=torch.float64) / 128
    for j in range(d):
        off = (p1[j % rows] * grid[:, None] - grid[None, :]).abs()
        i = int(off.argmin())
        Vc[0, 0, 0, 0, j] = -float(grid[i % 128])
        Vc[0, 0, 0, 1, j] = float(grid[i // 128])
    x, y = Vc[0, 0, 0, 0].double(), Vc[0, 0, 0, 1].double()
    ref = (x + p1[:, None] * y) / (1 + p1[:, None])
    terms = (x.abs() + p1[:, None] * y.abs()) / (1 + p1[:, None])
    O = torch.full((L, 1, 1, Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    wm.channel_attend(_gdims(wm, w, mask_mode=1, ctx_max=1), _dev(P), Q.cuda(), w.chan_map,
                      torch.tensor([1], dtype=torch.int32).cuda(), Kc.cuda(), Vc.cuda(), O)
    torch.cuda.synchronize()
    off = (O.double().cpu().reshape(rows, d) - ref).abs() - 2.0 ** -8 * ref.abs()
    worst = float((off / terms).max())
    print("worst %.3g of the terms" % worst)
    assert worst <= 2.0 ** -20, worst


@pytest.mark.parametrize("d", [64, 96])
@pytest.mark.parametrize("D", [64, 544])
def test_few_token_mid_norm_is_the_many_token_one(wm, d, D):
    """The mid norm's sum of squares is that of the fp32 mixed channels, as with many tokens,
    not of their bf16 copies. Every mixed element is +-(1 + 11/128)(1 + 6/128), which bf16
    rounds up by 3.3e-3: the value rows of 8 tokens and of the same tokens among 40 have the
    same norm to the rounding of their elements, 2^-8 / sqrt(the elements), not 3.3e-3 apart."""
    rows = {}
    for B in (8, 40):
        w = synth.small("mid_norm", B=B, T_new=1, L=1, k=1, D=D, Hq=2, Hkv=2, d=d, ctx=1,
                        dtype="bf16", chan_map=[0])
        print("mid norm d%d D%d N%d" % (d, D, B), flush=True)
        P = synth.make_params(w, torch.ones(1))
        P["b_alpha"] = torch.full_like(P["b_alpha"], 1 + 11 / 128)
        P["g_pre"] = torch.full_like(P["g_pre"], 1 + 6 / 128)
        gen = torch.Generator().manual_seed(3)
        H = torch.randint(0, 2, (8, 1, 1, D), generator=gen).bfloat16() * 2 - 1
        H = H.repeat(B // 8, 1, 1, 1)
        Kc, Vc = synth.make_cache_cpu(w, fill=0.0)
        Kg, Vg = Kc.cuda(), Vc.cuda()
        wm.pool(_gdims(wm, w, router_mode=1, ctx_max=0), _dev(P), H.cuda(),
                torch.zeros(B, dtype=torch.int32, device="cuda"), Kg, Vg)
        torch.cuda.synchronize()
        rows[B] = Vg[0, :8, :, 0].double().cpu()
    ratio = float(rows[8].norm() / rows[40].norm())
    assert abs(ratio - 1) <= 2 ** -8 / rows[8].numel() ** 0.5, ratio
