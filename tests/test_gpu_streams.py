"""Verifications issued from several streams without synchronisation in between.  The layer kernel is persistent and
needs its workgroups resident together, so the library orders its layer launches across streams by itself; each call
must return what the same call returns alone."""
import numpy as np
import pytest
import torch

from dsbd_synth import make_workload

pytestmark = pytest.mark.gpu

NAMES = ("node_status", "l_last", "layer_width", "n_out", "out_parent", "out_token", "out_node", "near_tie_count",
         "out_logp_target", "out_logp_draft", "lse_target", "lse_draft", "node_logp_target", "node_logp_draft")


def test_verifications_on_two_streams_do_not_disturb_each_other():
    import gpu_util as gu
    from dsbd_synth.device import DeviceWorkload
    wa = make_workload("c5", L=1, Hq=1, Hkv=1, D=64, V=20000)
    wb = make_workload("c4", L=1, Hq=1, Hkv=1, D=64, V=6000, n_prompts=5, seed=7)
    da, db = DeviceWorkload(wa), DeviceWorkload(wb)
    alone_a, alone_b = da.verify(t=-1.0), db.verify(t=0.8)
    torch.cuda.synchronize()
    gu.compare_verify(alone_a, gu.oracle_verify(wa, t=-1.0), wa)
    gu.compare_verify(alone_b, gu.oracle_verify(wb, t=0.8), wb)
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    sa.wait_stream(torch.cuda.current_stream())
    sb.wait_stream(torch.cuda.current_stream())
    got = []
    for _ in range(4):
        with torch.cuda.stream(sa):
            got.append((da.verify(t=-1.0, stream=sa), alone_a))
        with torch.cuda.stream(sb):
            got.append((db.verify(t=0.8, stream=sb), alone_b))
    torch.cuda.synchronize()
    g = lambda x: x.cpu().numpy()
    for i, (res, ref) in enumerate(got):
        assert int(g(res.fault)[0]) == 0, i
        for name in NAMES:
            assert np.array_equal(g(getattr(res, name)), g(getattr(ref, name))), (i, name)


def _static_calls():
    """Three calls that share the library's static scratch array (two of them warped: rows' records, then layers), and what
    each returns alone."""
    import paper_2409_16560_amd as dsbd
    from dsbd_synth.device import DeviceWorkload
    dsbd.dsbd_init()
    calls = []
    for w, kw in ((make_workload("c5", L=1, Hq=1, Hkv=1, D=64, V=20000, draft_top_k=4), dict(t=-1.0, top_k=10, top_p=0.9)),
                  (make_workload("c4", L=1, Hq=1, Hkv=1, D=64, V=6000, n_prompts=5, seed=7), dict(t=0.8)),
                  (make_workload("c3", L=1, Hq=1, Hkv=1, D=64, V=30000, draft_top_k=4), dict(t=0.6, top_k=32, top_p=1.0))):
        d = DeviceWorkload(w)

        def call(stream, d=d, w=w, kw=kw):
            res = dsbd.VerifyResult.allocate(d.forest, w.W_cap, stream)
            dsbd.dsbd_verify_forest_static(d.forest, d.logits_p, d.logits_q, d.blp, d.blq, d.u_accept, d.u_resid, d.u_fill, res,
                                           W_cap=w.W_cap, stream=stream, **kw)
            return res
        ref = d.verify(**kw)
        torch.cuda.synchronize()
        calls.append((call, ref))
    return calls


def _same(got):
    g = lambda x: x.cpu().numpy()      # noqa: E731
    for i, (res, ref) in enumerate(got):
        assert int(g(res.fault)[0]) == 0, i
        for name in NAMES:
            assert np.array_equal(g(getattr(res, name)), g(getattr(ref, name))), (i, name)


def test_static_calls_on_two_streams_take_turns_on_the_scratch_array():
    """Warped and plain calls without synchronisation in between: each waits for the one before to be done with the array."""
    calls, streams = _static_calls(), [torch.cuda.Stream(), torch.cuda.Stream()]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    got = []
    for i in range(12):
        s, (call, ref) = streams[i % 2], calls[i % 3]
        with torch.cuda.stream(s):
            got.append((call(s), ref))
    torch.cuda.synchronize()
    _same(got)


def test_static_calls_of_two_threads_on_one_stream_are_enqueued_whole():
    """A warped call is several kernels on one workspace: another thread's call must not get in between."""
    import threading
    calls, stream = _static_calls(), torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    got, errors = [[], []], []

    def work(k):
        try:
            with torch.cuda.stream(stream):
                for _ in range(20):
                    call, ref = calls[2 * k]
                    got[k].append((call(stream), ref))
        except Exception as e:      # noqa: BLE001
            errors.append(e)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors
    _same(got[0] + got[1])
