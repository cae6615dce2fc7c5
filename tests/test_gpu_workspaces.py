"""The binding's kept workspaces: calls of one operation on two streams, or from two threads, are not
ordered to each other and must not share one; a captured call must not lose its own when a later call
needs a larger one. Results are compared bit for bit with the same calls run one after the other."""

import threading

import numpy as np
import pytest

from synth import ffn_weights, decode_inputs, calibration_inputs, attn_inputs
from gpu_util import say, dev_bf16, dev_f32, dev_i32, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def calls():
    """name -> a function of (index 0 or 1, keywords) that makes the call on that input."""
    import paper_2409_03856_amd as sr
    d, f = 1024, 4000
    W = [dev_bf16(w) for w in ffn_weights(1, d, f, d ** -0.5)]
    x = [dev_f32(decode_inputs(2 + i, 9, d)) for i in range(2)]
    xc = [dev_f32(calibration_inputs(4 + i, 70, d)) for i in range(2)]
    at = []
    for i in range(2):
        q, kn, vn, kc, vc = attn_inputs(6 + i, 2, 3, 8, 2, 64, 3000)
        at.append([dev_f32(q)] + [dev_bf16(b) for b in (kn, vn, kc, vc)] + [dev_i32(np.array([2900 - i, 1500]))])
    return {
        "cats": lambda i, **kw: sr.sirius_ffn_cats(x[i], *W, 0.2, want_active=False, **kw)[0],
        "topk": lambda i, **kw: sr.sirius_ffn_topk(x[i], *W, 1700, want_active=False, **kw)[0],
        "dense": lambda i, **kw: sr.sirius_ffn_dense(x[i], *W, **kw),
        "calibrate": lambda i, **kw: sr.sirius_cats_calibrate(xc[i], W[0], 0.5, **kw),
        "attention": lambda i, **kw: sr.sirius_attn_kv(*at[i], **kw),
    }


NAMES = ("cats", "topk", "dense", "calibrate", "attention")


def test_one_workspace_per_thread_and_stream():
    import torch
    import paper_2409_03856_amd as sr
    from paper_2409_03856_amd import _lib
    size = (_lib.OP_FFN_CATS, 4, 1024, 4000)
    ptr = lambda: _lib.workspace(*size).data_ptr()
    here = ptr()
    assert ptr() == here
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        there = ptr()
        assert ptr() == there
    assert there != here and ptr() == here
    other = []
    t = threading.Thread(target=lambda: other.append(_lib.workspace(*size)))
    t.start()
    t.join()
    assert other[0].data_ptr() not in (here, there)
    # the number kept is bounded
    with torch.cuda.stream(s):
        for op in range(10):
            for i in range(12):
                with torch.cuda.stream(torch.cuda.Stream()):
                    ptr()
    assert len(_lib._workspaces.bufs) <= _lib._WS_MOST


@pytest.mark.parametrize("name", NAMES)
def test_two_streams(calls, name):
    import torch
    say(f"two streams: {name}")
    call = calls[name]
    want = [host(call(i)) for i in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for explicit in (False, True):
        got = [[], []]
        for _ in range(30):
            for i, s in enumerate(streams):
                if explicit:
                    got[i].append(call(i, stream=s))
                else:
                    with torch.cuda.stream(s):
                        got[i].append(call(i))
        torch.cuda.synchronize()
        for i in range(2):
            for g in got[i]:
                assert np.array_equal(host(g), want[i])


@pytest.mark.parametrize("name", NAMES)
def test_two_threads_on_one_stream(calls, name):
    say(f"two threads: {name}")
    call = calls[name]
    want = [host(call(i)) for i in range(2)]
    got = [[], []]
    threads = [threading.Thread(target=lambda i=i: got[i].extend(call(i) for _ in range(60))) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(got[i]) == 60
        for g in got[i]:
            assert np.array_equal(host(g), want[i])


def test_captured_call_keeps_its_workspace():
    """A captured call, then a larger call on the same stream, which replaces the kept workspace, and
    tensors that take the memory it gave back: every replay still gives the eager result."""
    import torch
    import paper_2409_03856_amd as sr
    d, f = 1024, 4000
    W = [dev_bf16(w) for w in ffn_weights(1, d, f, d ** -0.5)]
    x, big = dev_f32(decode_inputs(2, 9, d)), dev_f32(decode_inputs(3, 64, d))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        want = sr.sirius_ffn_cats(x, *W, 0.2, want_active=False)[0]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            y = sr.sirius_ffn_cats(x, *W, 0.2, want_active=False)[0]
        sr.sirius_ffn_cats(big, *W, 0.2, want_active=False)
        held = [torch.full((1 << 18,), 7.0, device="cuda") for _ in range(64)]
        for rep in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want), rep
        for h in held:
            assert bool((h == 7.0).all())
