"""The wave-private attention kernel with eight waves per workgroup: fewer steps than waves, as many, one more; units that are
split among workgroups and units that are not; 16 and 32 rows; ragged ends and shared segments; and the shapes next to them
that keep four waves.  Against the oracle (tolerance of the attention tests), twice: a call repeats itself bit for bit."""
import pytest
import torch

from dsbd_synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("cfg,kw", [
    ("c2", dict(L=0, Hq=8, Hkv=8)),                                     # the tree's own step alone
    ("c2", dict(L=7 * 32, Hq=8, Hkv=8)),                                # a step for every wave
    ("c2", dict(L=8 * 32 + 1, Hq=8, Hkv=8)),                            # two steps for two of them
    ("c2", dict(L=320, Hq=4, Hkv=4)),                                   # 16 units of 11 steps: eight waves; of 12: four
    ("c2", dict(L=330, Hq=4, Hkv=4)),
    ("c2", dict(L=22 * 32, Hq=16, Hkv=16)),                             # 64 units, the last length that is not split ...
    ("c2", dict(L=31 * 32 - 5, Hq=16, Hkv=16)),                         # ... and one that is (33 steps, two pieces and a merge)
    ("c3", dict(L=700, shared_len=333, Hq=32, Hkv=32)),                 # 256 units: one workgroup per compute unit, no merge
    ("c3", dict(L=700, shared_len=333, Hq=25, Hkv=25)),                 # 200 units
    ("c3", dict(L=300, shared_len=101, Hq=16, Hkv=8)),                  # 30 rows: eight waves with 64 channels only
    ("c4", dict(L=(33, 900), n_prompts=8, W=(1, 4), tree_nodes=(2, 8), Hq=4, Hkv=4)),       # unequal lengths
])
def test_eight_waves_per_workgroup(cfg, kw, D):
    import gpu_util as gu
    w = make_workload(cfg, V=64, D=D, **kw)
    d = gu.DeviceWorkload(w)
    out, lse, fault = d.attention()
    again, lse2, _ = d.attention()
    torch.cuda.synchronize()
    assert int(fault.item()) == 0
    gu.compare_attention(w, out, lse, *gu.oracle_attention(w))
    assert torch.equal(out, again) and torch.equal(lse, lse2)
