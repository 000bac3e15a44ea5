"""GPU parity of the full-sequence attention for few rows, where a workgroup takes 32 query
rows and its four waves cut the slots between them (32-slot blocks in turn, one ring each,
states merged at the end), and for the strided groups of larger grids, where it takes 64 queries of
two heads: partial and single-row last tiles, sequences whose short contexts
leave waves without a block, remainders of blocks, contiguous tokens and strided groups, both
masks, one and two query heads per KV head, peaked scores whose references differ between the
waves of one row. A walk past that kernel's range keeps the split ranges covered.

The operands and the rounding points are those of the 128-query tiles (bf16 weights against
fp32 sums), so the tolerance is theirs (parity.check_close)."""
import pytest
import torch

import oracle
from oracle import backward as ob
from tests import synth
from tests.parity import _bias, _dev, _f64, _gdims, _odims, check_close, wm  # noqa: F401

pytestmark = pytest.mark.gpu


def _case(wm, d, Hq, Hkv, T_new, ctx, ctx_len, g, q, mask_mode, peak, L=2):
    span = q + g * (T_new - 1) + 1
    w = synth.small("tile_d%d" % d, B=len(ctx_len), T_new=T_new, L=L, k=1, D=64, Hq=Hq, Hkv=Hkv,
                    d=d, ctx=ctx + span, dtype="bf16", chan_map=[0] * L)
    print("tiles d%d %d/%d T%d ctx%d g%d q%d mask%d peaked %s"
          % (d, Hq, Hkv, T_new, ctx, g, q, mask_mode, peak), flush=True)
    P = synth.make_params(w, _bias(w))
    if peak:
        Q, Kc, Vc = synth.make_peaked_attention(w, rise=60.0, period=256)
    else:
        Q = synth.make_queries(w)
        Kc, Vc = synth.make_cache_cpu(w)
    lens = torch.tensor(ctx_len, dtype=torch.int32)
    od = _odims(w, mask_mode=mask_mode)
    if g == 1:
        ref = oracle.channel_attend(od, P, Q, w.chan_map, lens.numpy(), _f64(Kc), _f64(Vc))
    else:
        ref = ob.attend(od, ob._t(P["Kd"]), ob._t(P["Vd"]), ob._t(Q), w.chan_map,
                        torch.as_tensor(lens.numpy(), dtype=torch.long), ob._t(Kc), ob._t(Vc),
                        (g, q)).detach().numpy()
    O = torch.full((w.L, w.B, T_new, Hq * d), float("nan"), dtype=torch.bfloat16, device="cuda")
    dims = _gdims(wm, w, mask_mode=mask_mode, ctx_max=ctx, groups=g, group=q)
    wm.channel_attend(dims, _dev(P), Q.cuda(), w.chan_map, lens.cuda(), Kc.cuda(), Vc.cuda(), O)
    torch.cuda.synchronize()
    check_close(O, ref, "bf16", "tiles d%d T%d ctx%d g%d" % (d, T_new, ctx, g))
    return (T_new + 31) // 32 * Hq * w.L * w.B, ctx + span


@pytest.mark.parametrize("d,Hq,Hkv", [(64, 4, 2), (96, 6, 3), (96, 2, 2)])
@pytest.mark.parametrize("mask_mode", [0, 1])
@pytest.mark.parametrize("T_new,ctx,g,q,peak", [(5, 700, 1, 0, False), (33, 600, 1, 0, True),
                                                (64, 509, 3, 2, False), (65, 120, 8, 5, False)])
def test_few_rows(wm, d, Hq, Hkv, mask_mode, T_new, ctx, g, q, peak):
    tiles, slots = _case(wm, d, Hq, Hkv, T_new, ctx, [ctx, ctx // 3, 0], g, q, mask_mode, peak)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert tiles <= cus and 512 <= slots <= 3072, (tiles, slots)


@pytest.mark.parametrize("d,Hq,Hkv", [(64, 4, 2), (96, 6, 3)])
def test_split_ranges_past_the_tiles_walk(wm, d, Hq, Hkv):
    _, slots = _case(wm, d, Hq, Hkv, 40, 3300, [3300, 900], 1, 0, 0, False)
    assert slots > 3072 and slots // 64 >= 32


@pytest.mark.parametrize("d,Hq,Hkv,L,B,order", [(96, 6, 3, 3, 8, "bands"), (96, 6, 3, 5, 8, "bands"),
                                                (64, 4, 2, 3, 8, "bands"),
                                                (96, 6, 3, 5, 7, "tiles"),
                                                (64, 4, 2, 5, 7, "tiles"),
                                                (96, 6, 3, 11, 8, "queue"),
                                                (64, 4, 2, 25, 8, "queue")])
def test_strided_groups_of_two_heads(wm, d, Hq, Hkv, L, B, order):
    """Pairs of heads that divide among the 8 XCDs (a band of them each, longest tiles first) and
    that do not (tile order), and more tiles than the CUs hold at once (the work queue); the
    last tile of 100 queries is partial."""
    T_new = 100
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows, slots = _case(wm, d, Hq, Hkv, T_new, 40, [40, 0, 7, 33, 1, 2, 39, 20][:B], 4, 3, 0,
                        False, L=L)
    tiles = (T_new + 127) // 128 * Hq * B * L
    resident = cus * (3 if d == 64 else 2)
    # neither the few-row tiles (one per CU at most) nor split ranges (from 32 blocks of 64)
    assert rows > cus and slots < 2048
    units = Hq // 2 * B * L
    assert order == ("queue" if tiles > resident else "tiles" if units % 8 else "bands")
