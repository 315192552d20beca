"""The layer walk where its exchanges and draws can go wrong: chain entries that nobody collects in their layer (narrow
layers pass before the entry on its way arrives), one to many workgroups, slices in the LDS, in both homes and in the
workspace.  Against the oracle, bit for bit but for near ties."""
import pytest

from dsbd_synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [1, 2, 7, 64])
@pytest.mark.parametrize("cfg,kw,W_L,t", [
    ("c5", dict(L=8, V=1500, Hq=4, Hkv=4), 1, -1.0),      # the first acceptance ends a layer: five layers, entries left open
    ("c5", dict(L=8, V=1500, Hq=4, Hkv=4), 3, -1.0),
    ("c3", dict(L=8, V=3001, Hq=4, Hkv=4), 0, -1.0),      # layers that fall short: residual and fill draws in one pass
    ("c3", dict(L=8, V=3001, Hq=4, Hkv=4), 0, 0.6),
])
def test_layers_with_open_chain_entries(cfg, kw, W_L, t, G, knobs):
    import gpu_util as gu
    knobs.set("DSBD_VERIFY_G", G)
    w = make_workload(cfg, **kw)
    d = gu.DeviceWorkload(w)
    for _ in range(2):                                    # (the second call finds the first one's accumulator values)
        res, _ = d.verify_select(W_L=W_L, t=t)
    assert int(res.fault.item()) == 0
    gu.compare_verify(res, gu.oracle_verify(w, W_L=W_L, t=t), w)


@pytest.mark.parametrize("lds", [0, 100, 1 << 20])
@pytest.mark.parametrize("G,W_L", [(1, 0), (3, 16), (8, 0)])
def test_draws_from_slices_in_either_home(G, W_L, lds, knobs):
    import gpu_util as gu
    knobs.set("DSBD_VERIFY_G", G)
    knobs.set("DSBD_VERIFY_LDS_SLICE", lds)
    w = make_workload("c2", L=8, V=777, Hq=4, Hkv=4)
    d = gu.DeviceWorkload(w)
    res, _ = d.verify_select(W_L=W_L, t=-1.0)             # (W_L 16: one draw from the residual, many fills)
    assert int(res.fault.item()) == 0
    gu.compare_verify(res, gu.oracle_verify(w, W_L=W_L), w)
