"""GPU parity of the bf16 decode attention on the matrix cores (Section 3.1 Step 3, Section
3.2) at the edges of its tiles: 32 rows (consumers x grouped heads x new tokens) per tile,
32-slot blocks dealt to four waves, splits of at least 256 slots, and ragged sequences that
leave waves and whole splits without a slot. Against the oracle, with the repository's bf16
bounds."""
import pytest
import torch

import oracle
from tests import synth
from tests.parity import _bias, _dev, _f64, _gdims, _odims, check_close, wm  # noqa: F401

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
