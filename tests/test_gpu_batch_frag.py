"""GPU parity: the operand-order gate/up kernels of batched FFN calls at the edges of their tiles.

Odd and even numbers of 256-column blocks below and above the load depth (256, 512, 768, 2048),
token counts on both sides of every 16-token tile, segments of every position class (16, 32, 48 and
64 positions; row counts on both sides of one full round of 256 segments), ragged last segments.
Every mode is compared with the fp64 oracle at the repository's fp32-path tolerance (1e-4 x RMS;
the kernel's own error is below 1e-6 x RMS: exact products, fp32 sums of at most d_model terms).
"""

import numpy as np
import pytest

import oracle
from synth import ffn_weights, decode_inputs
from gpu_util import (say, dev_bf16, dev_f32, host, check_ffn, check_cats_sets, check_topk_sets,
                      rounded_bf16, FP32_PATH_TOL)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sr():
    import paper_2409_03856_amd as sr
    sr.lib()
    return sr


@pytest.mark.parametrize("d,f,bsz", [(256, 1, 2), (256, 1025, 5), (512, 4099, 3), (512, 14336, 16), (256, 14337, 17),
                                     (768, 8193, 33), (768, 9001, 7), (256, 12289, 48), (512, 24571, 49),
                                     (256, 12288, 64), (2048, 4097, 15), (1280, 3584, 64),
                                     (1536, 12289, 9), (2048, 14337, 20)])
def test_every_mode(sr, d, f, bsz):
    say(f"operand-order batch d={d} f={f} B={bsz}")
    wg, wu, wd = ffn_weights(3000 + d + f + bsz, d, f, 1.0 / np.sqrt(d))
    W = tuple(dev_bf16(w) for w in (wg, wu, wd))
    x = decode_inputs(3100 + bsz, bsz, d)
    t = float(np.median(np.abs(oracle.gate_activations(x, wg))))
    y, idx, cnt = sr.sirius_ffn_cats(dev_f32(x), *W, t)
    sets, _ = check_cats_sets(x, wg, t, host(idx), host(cnt))
    check_ffn(host(y), oracle.ffn_masked(x, wg, wu, wd, sets), tol=FP32_PATH_TOL)
    yneg, ineg, cneg = sr.sirius_ffn_cats(dev_f32(x), *W, -1.0)
    assert np.all(host(cneg) == f)
    assert np.array_equal(host(ineg), np.tile(np.arange(f, dtype=np.int32), (bsz, 1)))
    check_ffn(host(yneg), oracle.ffn_dense(x, wg, wu, wd), tol=FP32_PATH_TOL)
    yd = host(sr.sirius_ffn_dense(dev_f32(x), *W))
    if bsz < 8:  # same kernel, same sums: bitwise
        assert np.array_equal(yd, host(yneg))
    else:
        check_ffn(yd, oracle.ffn_dense(rounded_bf16(x), wg, wu, wd), tol=FP32_PATH_TOL)
    k = max(1, f // 3)
    y, idx, cnt = sr.sirius_ffn_topk(dev_f32(x), *W, k)
    sets, _ = check_topk_sets(x, wg, k, host(idx), host(cnt))
    check_ffn(host(y), oracle.ffn_masked(x, wg, wu, wd, sets), tol=FP32_PATH_TOL)


@pytest.mark.parametrize("d", [2048, 1280])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.float32(3.4e38)])
def test_infinite_input_is_the_same_at_every_batch(sr, d, value):
    """One infinite (or nearly infinite) input element: the activations that it makes infinite are kept,
    in the calls of at most 4 tokens (unit kernels where d_model is a multiple of 2048) as in those of
    5 and more and of one; the other tokens are untouched."""
    f = 300
    say(f"infinite input d={d} value={value}")
    wg, wu, wd = ffn_weights(4000 + d, d, f, 1.0 / np.sqrt(d))
    W = tuple(dev_bf16(w) for w in (wg, wu, wd))
    x = decode_inputs(4100, 5, d)
    t = float(np.median(np.abs(oracle.gate_activations(x, wg))))
    clean = [host(a) for a in sr.sirius_ffn_cats(dev_f32(x), *W, t)]
    x[2, 9] = value
    one = [host(a) for a in sr.sirius_ffn_cats(dev_f32(x[2:3]), *W, t)]
    for b in (3, 4, 5):
        y, idx, cnt = (host(a) for a in sr.sirius_ffn_cats(dev_f32(x[:b]), *W, t))
        assert cnt[2] == one[2][0] and np.array_equal(idx[2, :cnt[2]], one[1][0, :cnt[2]]), b
        for m in (0, 1):
            assert cnt[m] == clean[2][m] and np.array_equal(idx[m, :cnt[m]], clean[1][m, :cnt[m]])
            assert np.all(np.isfinite(y[m]))


def test_bf16_rounding_at_the_top_of_the_range(sr):
    """The dense pass of 8 or more tokens rounds its input to bf16: a value above the largest bf16 by
    half a step is an infinity there, at a width of the unit kernels and at one of the others."""
    for d in (2048, 1280):
        wg, wu, wd = ffn_weights(4200 + d, d, 64, 1.0 / np.sqrt(d))
        x = np.zeros((8, d), dtype=np.float32)
        x[:, 0] = 3.4e38
        wg[:, 0] = wu[:, 0] = 0x0D80  # 2^-100: finite products for any finite input
        say(f"bf16 rounding at the top d={d}")
        y = host(sr.sirius_ffn_dense(dev_f32(x), *(dev_bf16(w) for w in (wg, wu, wd))))
        assert not np.any(np.isfinite(y))
