"""Draft steps whose drawing workgroups stand behind the chunks' in one launch, against the two-launch form (which calls under
capture take), against waiting workgroups that take every chunk themselves, and against the oracle."""
import numpy as np
import pytest
import torch

from dsbd_synth import uniform01_f32

pytestmark = pytest.mark.gpu


def _inputs(beams, V, W_S, seed):
    rng = np.random.Generator(np.random.Philox(key=[seed, 5]))
    off = np.concatenate([[0], np.cumsum(beams)]).astype(np.int32)
    z = (rng.standard_normal((int(off[-1]), V), dtype=np.float32) * np.float32(3.0))
    return off, z, -3.0 * rng.random(int(off[-1])), uniform01_f32(len(beams) * W_S, seed, 201).reshape(len(beams), W_S)


SHAPES = [
    ([1], 1, 1), ([3], 700, 4), ([8], 1025, 16), ([16], 32000, 16),
    ([5], 128256, 12),                     # chunks of 2048
    ([2], 300001, 8),                      # chunks of several tiles, a ragged last one
    ([2, 0, 3, 1], 5000, 8),               # a prompt without beams
    ([1] * 40, 3001, 6),                   # 240 drawing workgroups, and 40 warped ones
    ([8, 3], 285975, 4),                   # 3145725 logits, the most of a warped step in one launch ...
    ([16], 196609, 4),                     # ... and 3145744, in two
]


@pytest.mark.parametrize("top_k,top_p", [(0, 1.0), (10, 0.8), (32, 1.0)])
@pytest.mark.parametrize("beams,V,W_S", SHAPES)
def test_one_launch_or_two(beams, V, W_S, top_k, top_p, knobs):
    import paper_2409_16560_amd as dsbd
    from oracle import draft as o_draft
    off, z, cum, u = _inputs(beams, V, W_S, V + W_S)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (off, z, cum, u)]
    kw = dict(max_prompt_beams=max(beams), top_k=top_k, top_p=top_p)
    call = lambda **k: dsbd.dsbd_draft_layer(*dev, W_S, **kw, **k)      # noqa: E731
    one = [t.clone() for t in call()]
    assert int(one[3].item()) == 0
    knobs.set("DSBD_DRAFT_WAIT_US", 0)
    alone = [t.clone() for t in call()]
    knobs.set("DSBD_DRAFT_WAIT_US", 100000)
    for got, want in zip(alone, one):
        assert torch.equal(got, want)
    # under capture, replayed three times with eager work (and new slots in the eager call's workspace) in between
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(s), torch.cuda.graph(g, stream=s):
        two = call(stream=s)
    for scale in (1.0, 0.5, 1.0):
        dev[1].copy_(torch.from_numpy(z * np.float32(scale)))
        eager = [t.clone() for t in call()]
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for got, want in zip(two[:3], eager[:3]):
            assert torch.equal(got, want), scale
        _ = torch.randn(1 << 16, device="cuda").square().sum().item()
    for p in range(len(beams)):
        if beams[p] == 0:
            assert bool((one[0][p] == -1).all())
            continue
        par, tok, lp = o_draft.draft_layer(z[off[p]:off[p + 1]], cum[off[p]:off[p + 1]], u[p], top_k=top_k, top_p=float(np.float32(top_p)))
        assert np.array_equal(one[0][p].cpu().numpy() - off[p], par) and np.array_equal(one[1][p].cpu().numpy(), tok)
        assert np.allclose(one[2][p].cpu().numpy(), lp, rtol=0, atol=1e-9)


def test_draft_steps_beside_verifications_on_another_stream():
    """Neither side's waiting workgroups keep the other's from finishing."""
    import gpu_util as gu
    import paper_2409_16560_amd as dsbd
    from dsbd_synth import make_workload
    w = make_workload("c5", L=1, Hq=1, Hkv=1, D=64, V=20000)
    d = gu.DeviceWorkload(w)
    off, z, cum, u = _inputs([8], 128256, 16, 9)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (off, z, cum, u)]
    alone = [t.clone() for t in dsbd.dsbd_draft_layer(*dev, 16, max_prompt_beams=8, top_k=10, top_p=0.8)]
    want = d.verify(t=0.8)
    torch.cuda.synchronize()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    drafts, checks = [], []
    for _ in range(6):
        with torch.cuda.stream(sa):
            checks.append(d.verify(t=0.8, stream=sa))
        with torch.cuda.stream(sb):
            drafts.append(dsbd.dsbd_draft_layer(*dev, 16, max_prompt_beams=8, top_k=10, top_p=0.8, stream=sb))
    torch.cuda.synchronize()
    for got in drafts:
        assert all(torch.equal(a, b) for a, b in zip(got, alone))
    for got in checks:
        assert int(got.fault.item()) == 0 and torch.equal(got.out_token, want.out_token) and torch.equal(got.node_status, want.node_status)
