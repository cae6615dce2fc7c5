"""GPU parity: batch-1 decode on both sides of every row class (chunks of 512 columns per lane: 4, 6, 8, 10, 12, 14, 16).

Each width is compared with the fp64 oracle at the repository's fp32-path tolerance (1e-4 x RMS: exact products, fp32
sums of at most d_model terms), with the threshold, top-k and dense forms of the pass, RMSNorm and residual.
"""

import numpy as np
import pytest

import oracle
from synth import ffn_weights, decode_inputs
from gpu_util import say, dev_bf16, dev_f32, host, check_ffn, check_cats_sets, check_topk_sets, FP32_PATH_TOL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sr():
    import paper_2409_03856_amd as sr
    sr.lib()
    return sr


@pytest.mark.parametrize("d,f", [(2048, 515), (2056, 515), (3072, 300), (3080, 300), (4104, 257), (5120, 1030),
                                 (5128, 300), (6144, 515), (6152, 257), (7168, 300), (7176, 300), (8184, 257)])
def test_every_mode(sr, d, f):
    say(f"batch-1 row class d={d} f={f}")
    wg, wu, wd = ffn_weights(5000 + d + f, d, f, 1.0 / np.sqrt(d))
    W = tuple(dev_bf16(w) for w in (wg, wu, wd))
    x = decode_inputs(5100 + d, 1, d) * 3.0
    res = decode_inputs(5200 + d, 1, d)
    xn = oracle.rmsnorm(x, 1e-5)
    kw = dict(norm_eps=1e-5, resid=dev_f32(res))
    t = float(np.median(np.abs(oracle.gate_activations(xn, wg))))
    y, idx, cnt = sr.sirius_ffn_cats(dev_f32(x), *W, t, **kw)
    sets, _ = check_cats_sets(xn, wg, t, host(idx), host(cnt))
    check_ffn(host(y), oracle.ffn_masked(xn, wg, wu, wd, sets), resid=res, tol=FP32_PATH_TOL)
    yneg, _, cneg = sr.sirius_ffn_cats(dev_f32(x), *W, -1.0, **kw)
    assert np.all(host(cneg) == f)
    yd = sr.sirius_ffn_dense(dev_f32(x), *W, **kw)
    assert np.array_equal(host(yd), host(yneg))  # a row's sum is the same in both forms: bitwise
    check_ffn(host(yd), oracle.ffn_dense(xn, wg, wu, wd), resid=res, tol=FP32_PATH_TOL)
    k = max(1, f // 3)
    y, idx, cnt = sr.sirius_ffn_topk(dev_f32(x), *W, k, **kw)
    sets, _ = check_topk_sets(xn, wg, k, host(idx), host(cnt))
    check_ffn(host(y), oracle.ffn_masked(xn, wg, wu, wd, sets), resid=res, tol=FP32_PATH_TOL)
