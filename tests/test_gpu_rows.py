"""The row records behind warped verifications, where their cuts can go wrong: rows shorter than a tile, ragged last tiles
and chunks, rows of several tiles per chunk, as many entries as there are tokens, crowds of equal logits, one model in both
roles.  Against the oracle, bit for bit but for near ties; the fp32 row outputs against 64 bits."""
import dataclasses

import numpy as np
import pytest

from dsbd_synth import make_workload

pytestmark = pytest.mark.gpu


def _check(w, top_k, top_p, t):
    import gpu_util as gu
    d = gu.DeviceWorkload(w)
    res, _ = d.verify_select(t=t, top_k=top_k, top_p=top_p)
    assert int(res.fault.item()) == 0
    gu.compare_verify(res, gu.oracle_verify(w, t=t, top_k=top_k, top_p=top_p), w)
    for z, lse, logp in ((w.logits_p, res.lse_target, res.node_logp_target), (w.logits_q, res.lse_draft, res.node_logp_draft)):
        z = z.astype(np.float64)
        m = z.max(axis=1, keepdims=True)
        want = m[:, 0] + np.log(np.exp(z - m).sum(axis=1))
        # (one rounding to fp32 of a value computed in fp64: half an ulp, 6e-8 relative)
        np.testing.assert_allclose(lse.cpu().numpy(), want, rtol=6.5e-8, atol=1e-12)
        child = np.nonzero(w.parent >= 0)[0]
        want = z[w.parent[child], w.token[child]] - want[w.parent[child]]
        np.testing.assert_allclose(logp.cpu().numpy()[child], want, rtol=6.5e-8, atol=1e-9)


@pytest.mark.parametrize("fast", [1, 0])
@pytest.mark.parametrize("V,top_k,top_p", [
    (1, 1, 1.0), (3, 32, 0.9), (63, 10, 0.8), (1023, 32, 1.0), (1024, 5, 0.8), (1025, 10, 0.8), (2049, 32, 0.95),
    (4099, 2, 0.8), (32001, 10, 0.8),
    # around the lengths where the parts of a row change
    (4096, 32, 0.95), (4097, 32, 0.95), (16384, 32, 0.95), (16385, 32, 0.95), (65536, 32, 0.95), (65537, 32, 0.95),
])
def test_rows_of_any_length(V, top_k, top_p, fast, knobs):
    knobs.set("DSBD_WARP_FAST", fast)
    w = make_workload("c2", L=8, V=V, Hq=4, Hkv=4, draft_top_k=min(4, V))
    for t in (-1.0, 0.7):
        _check(w, top_k, top_p, t)


@pytest.mark.parametrize("fast", [1, 0])
@pytest.mark.parametrize("V", [131073, 270001])            # two and three tiles of 1024 in the last chunks, ragged ends
def test_rows_of_several_tiles_per_chunk(V, fast, knobs):
    knobs.set("DSBD_WARP_FAST", fast)
    w = make_workload("c1", L=8, V=V, draft_top_k=4)
    # the leading entries also where a chunk's second half, a row's last tile and its last token are
    lead = np.array([0, 1023, 1024, 2047, 2048, 3071, V - 1025, V - 1])
    w.logits_p[:, lead] += 12.0
    w.logits_q[:, lead] += 12.0
    _check(w, 16, 0.9, -1.0)


@pytest.mark.parametrize("fast", [1, 0])
@pytest.mark.parametrize("V", [300, 5000, 40000])
def test_rows_with_crowds_of_equal_logits(V, fast, knobs):
    """More entries at the bound than are ranked directly (5000, 40000), masked tokens among them."""
    knobs.set("DSBD_WARP_FAST", fast)
    w = make_workload("c1", L=8, V=V, draft_top_k=4)
    zp, zq = np.round(w.logits_p / 8) * 8, np.zeros_like(w.logits_q)
    keep = w.token[w.token >= 0]
    mask = np.zeros(V, dtype=bool)
    mask[::3] = True
    mask[keep] = False
    zp[:, mask] = -np.inf
    zq[:, mask] = -np.inf
    w = dataclasses.replace(w, logits_p=zp.astype(np.float32), logits_q=zq.astype(np.float32))
    _check(w, 10, 0.8, -1.0)
    _check(w, 32, 1.0, 0.5)


@pytest.mark.parametrize("fast", [1, 0])
@pytest.mark.parametrize("V", [300, 4097, 40000, 140000])
def test_different_logits_with_equal_joint_entries(V, fast, knobs):
    """Logits around zero that differ by less than fp64 resolves in exp(z - max): equal entries, ordered by token.  (Magnitude
    1e-18 against maxima of 0.5 and 2.)"""
    import gpu_util as gu
    knobs.set("DSBD_WARP_FAST", fast)
    w = make_workload("c2", L=1, V=4, Hq=1, Hkv=1, D=64)
    rng, N = np.random.default_rng(1), len(w.parent)
    token = np.array([5, V - 1], dtype=np.int32)[rng.integers(0, 2, N)]
    zp, zq = (rng.standard_normal((2, N, V)) * 1e-18).astype(np.float32)
    for z, top in ((zp, 0.5), (zq, 2.0)):
        z[:, [5, V - 1]] = top
    w = dataclasses.replace(w, logits_p=zp, logits_q=zq, token=token)
    for top_k, top_p in ((32, 1.0), (32, 0.95), (20, 1.0)):
        d = gu.DeviceWorkload(w)
        res, _ = d.verify_select(t=-1.0, top_k=top_k, top_p=top_p)
        assert int(res.fault.item()) == 0
        gu.compare_verify(res, gu.oracle_verify(w, t=-1.0, top_k=top_k, top_p=top_p), w)


def test_one_model_in_both_roles():
    import gpu_util as gu
    w = make_workload("c2", L=8, V=3001, Hq=4, Hkv=4, draft_top_k=4)
    w = dataclasses.replace(w, logits_q=w.logits_p, beam_logp_q=w.beam_logp_p)
    d = gu.DeviceWorkload(w)
    d.logits_q, d.blq = d.logits_p, d.blp
    res, _ = d.verify_select(t=-1.0, top_k=10, top_p=0.8)
    assert int(res.fault.item()) == 0
    gu.compare_verify(res, gu.oracle_verify(w, top_k=10, top_p=0.8), w)


@pytest.mark.parametrize("V,top_k,n_prompts,nodes,entry_bytes", [
    (200, 32, 600, (12, 16), 8), (1000, 32, 600, (12, 16), 8), (1500, 32, 600, (12, 16), 8),
    # ... nor would records with tokens alone fit: records without entries
    (24, 10, 1134, (60, 64), 1), (300, 14, 900, (60, 64), 2), (3, 32, 1600, (60, 64), 1),
])
def test_compact_records_of_large_batches(V, top_k, n_prompts, nodes, entry_bytes):
    """Batches whose records with logits would outgrow 32 MiB keep 8- or 16-bit tokens instead, or no entries."""
    import gpu_util as gu
    import paper_2409_16560_amd as dsbd
    base = make_workload("c4", n_prompts=n_prompts, W=(8, 8), tree_nodes=nodes, L=1, Hq=1, Hkv=1, D=64, V=4, seed=5)
    N, rng = len(base.parent), np.random.default_rng(3)
    zp = rng.standard_normal((N, V), dtype=np.float32) * 3
    zq = zp + rng.standard_normal((N, V), dtype=np.float32) * np.float32(0.5)
    if V > 4:          # (every third row: all but a few logits so close to zero that their entries are equal)
        zp[::3, 4:] *= np.float32(1e-19)
        zq[::3, 4:] *= np.float32(1e-19)
        zp[::3, :4] = zq[::3, :4] = (0.25, 0.5, 0.375, 0.125)
    par = np.maximum(base.parent, 0)
    kth = min(3, V - 1)
    token = np.argpartition(-zq[par], kth, axis=1)[np.arange(N), rng.integers(0, kth + 1, N)].astype(np.int32)
    w = dataclasses.replace(base, logits_p=zp, logits_q=zq, token=token)
    d = gu.DeviceWorkload(w)
    assert N * 2 * ((16 + entry_bytes * min(top_k, V) + 7) // 8 * 8) > 32 << 20    # what the records would take
    assert dsbd.dsbd_verify_forest_workspace_bytes(d.forest, V, 0, 1, w.W_cap, -1.0, top_k, 0.9) <= 32 << 20
    res, _ = d.verify_select(t=0.6, top_k=top_k, top_p=0.9)
    assert int(res.fault.item()) == 0
    # (the first prompts only: the oracle takes milliseconds for each)
    P, T = 12, int(np.searchsorted(w.tree_prompt, 12))
    n = int(w.tree_off[T])
    first = dataclasses.replace(
        w, n_prompts=P, n_trees=T, n_nodes=n, tree_prompt=w.tree_prompt[:T], tree_off=w.tree_off[:T + 1], parent=w.parent[:n], token=token[:n], logits_p=zp[:n],
        logits_q=zq[:n], beam_logp_p=w.beam_logp_p[:T], beam_logp_q=w.beam_logp_q[:T], u_accept=w.u_accept[:n],
        u_resid=w.u_resid[:P], u_fill=w.u_fill[:P])
    ref = gu.oracle_verify(first, t=0.6, top_k=top_k, top_p=0.9)
    for k in ("l_last", "n_out"):
        assert np.array_equal(getattr(res, k).cpu().numpy()[:P], ref[k])
    assert np.array_equal(res.node_status.cpu().numpy()[:n], ref["node_status"])
    for p in range(P):
        m = int(ref["n_out"][p])
        assert np.array_equal(res.out_token.cpu().numpy()[p, :m], ref["out_token"][p, :m])
        assert np.array_equal(res.out_parent.cpu().numpy()[p, :m], ref["out_parent"][p, :m])


@pytest.mark.parametrize("V", [300, 5000, 140000])
@pytest.mark.parametrize("top_k", [0, 10])
def test_without_row_outputs_only_the_layers_rows_are_reported(V, top_k):
    """All four per-node outputs left out: NaN and +Inf are reported for the rows of beams that enter a layer alone, rows of
    nothing but -Inf and masked drafted tokens not at all; with an output, every row's are."""
    import torch
    import gpu_util as gu
    import paper_2409_16560_amd as dsbd
    w = make_workload("c2", L=8, V=V, Hq=4, Hkv=4, draft_top_k=4)
    d = gu.DeviceWorkload(w)
    kw = dict(t=-1.0, top_k=top_k, top_p=0.9 if top_k else 1.0)
    names = ("lse_target", "lse_draft", "node_logp_target", "node_logp_draft")
    whole = ("node_status", "l_last", "layer_width", "n_out", "out_parent", "out_token", "out_node")

    def call(outputs):
        res = dsbd.VerifyResult.allocate(d.forest, w.W_cap)
        kept = {n: getattr(res, n) for n in names}
        for n in names:
            if n not in outputs:
                setattr(res, n, None)
        d.verify(result=res, **kw)
        torch.cuda.synchronize()
        del kept
        return res
    clean = call(())
    assert int(clean.fault.item()) == 0
    status = clean.node_status.cpu().numpy()
    unused = [n for n in range(w.n_nodes) if status[n] not in (dsbd.DSBD_ROOT, dsbd.DSBD_ACCEPTED)]
    assert unused                                                    # (nodes that are not accepted enter no layer)
    first_child = int(np.nonzero(np.asarray(w.parent) >= 0)[0][0])
    masked = (int(w.parent[first_child]), int(w.token[first_child]))
    for bad, used in (((unused[-1], 7, float("nan")), False), ((unused[0], V - 1, float("inf")), False),
                      ((unused[0], slice(None), -float("inf")), False), ((masked[0], masked[1], -float("inf")), False),
                      ((0, V // 2, float("nan")), True), ((0, V - 1, float("inf")), True)):
        for z in (d.logits_p, d.logits_q):
            row = z[bad[0]].clone()
            z[bad[0], bad[1]] = bad[2]
            res = call(())
            assert int(res.fault.item()) == (dsbd.DSBD_FAULT_NONFINITE if used else 0), (bad, used)
            if not used and bad[0] in unused:
                for n in whole:
                    assert torch.equal(getattr(res, n), getattr(clean, n)), (bad, n)
            assert int(call(names).fault.item()) & dsbd.DSBD_FAULT_NONFINITE, bad
            z[bad[0]] = row


def test_a_warped_verification_as_a_process_s_first_call():
    """The most dynamic LDS a warped call asks for (64 beams, 32 entries each) without any other call in front."""
    import subprocess
    import sys
    import gpu_util as gu
    w = make_workload("c2", W_cap=64, L=8, V=300, Hq=4, Hkv=4, draft_top_k=4)
    code = ("import conftest, json, torch\n"
            "from dsbd_synth import make_workload\n"
            "from dsbd_synth.device import DeviceWorkload\n"
            "w = make_workload('c2', W_cap=64, L=8, V=300, Hq=4, Hkv=4, draft_top_k=4)\n"
            "r = DeviceWorkload(w).verify(t=-1.0, top_k=32, top_p=0.9)\n"
            "print(json.dumps([int(r.fault.item()), r.n_out.tolist(), r.out_token.tolist(), r.node_status.tolist()]))\n")
    out = subprocess.run([sys.executable, "-c", code], cwd=__file__.rsplit("/", 1)[0], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr[-2000:]
    import json
    fault, n_out, token, status = json.loads(out.stdout.strip().splitlines()[-1])
    ref = gu.oracle_verify(w, t=-1.0, top_k=32, top_p=0.9)
    assert fault == 0 and n_out == ref["n_out"].tolist() and status == ref["node_status"].tolist()
    assert [r[:n] for r, n in zip(token, n_out)] == [r[:n] for r, n in zip(ref["out_token"].tolist(), n_out)]


def test_more_rows_than_a_launch_takes():
    """16.8 million rows (with 256 threads each more than the 2^32 of a launch): the first and the last prompts as if alone."""
    import torch
    import paper_2409_16560_amd as dsbd
    P, W, n, V, W_cap = 16400, 8, 64, 4, 8
    T, N = P * W, P * W * n
    assert 2 * N * 256 > 1 << 32
    gen = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *s, dt=torch.float32: torch.rand(*s, generator=gen, device="cuda", dtype=dt)      # noqa: E731
    token = torch.randint(0, V, (N,), generator=gen, device="cuda", dtype=torch.int32)
    zp = rand(N, V) * 4
    arrays = [(zp, W * n), (zp + rand(N, V), W * n), (-rand(T, dt=torch.float64), W), (-rand(T, dt=torch.float64), W), (rand(N), W * n),
              (rand(P, n + 1), 1), (rand(P, n + 1, W_cap), 1)]

    def call(p0, p1):
        m = p1 - p0
        forest = dsbd.Forest(np.repeat(np.arange(m), W).astype(np.int32), (np.arange(m * W + 1) * n).astype(np.int32),
                             np.where(np.arange(m * W * n) % n == 0, -1, np.arange(m * W * n) - 1).astype(np.int32),
                             token[p0 * W * n:p1 * W * n].contiguous(), n_prompts=m, max_tree_nodes=n, max_depth=n - 1,
                             max_prompt_trees=W, device="cuda")
        res = dsbd.dsbd_verify_forest(forest, *[x[p0 * k:p1 * k].contiguous() for x, k in arrays], W_cap=W_cap, top_k=3, top_p=0.9)
        torch.cuda.synchronize()
        assert int(res.fault.item()) == 0
        return res
    whole = call(0, P)
    for p0, p1 in ((0, 3), (P - 3, P)):
        part = call(p0, p1)
        for name in ("l_last", "n_out", "layer_width"):
            assert torch.equal(getattr(whole, name)[p0:p1], getattr(part, name)), name
        for name in ("node_status", "lse_target", "lse_draft", "node_logp_target", "node_logp_draft"):
            assert torch.equal(getattr(whole, name)[p0 * W * n:p1 * W * n], getattr(part, name)), name
        for p in range(p1 - p0):
            k = int(part.n_out[p])
            for name in ("out_token", "out_logp_target"):
                assert torch.equal(getattr(whole, name)[p0 + p, :k], getattr(part, name)[p, :k]), name
