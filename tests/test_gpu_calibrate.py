"""GPU parity of the threshold calibration at the edges of its tiles (64 inputs x 128 neurons, 64
columns per stage, 1024 inputs per launch) and of its radix select: ranks at both ends, ties,
zeros, infinities. Tolerance: the nearest-rank value moves by no more than the largest error of an
activation, fp32 sums of at most 8192 exact products: 1e-5 relative plus 2e-6 of the gate's spread
(values near zero)."""

import numpy as np
import pytest

import oracle
from synth import ffn_weights, calibration_inputs
from gpu_util import say, dev_bf16, dev_f32, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sr():
    import paper_2409_03856_amd as sr
    sr.lib()
    return sr


@pytest.mark.parametrize("d,f,n", [(8, 1, 1), (72, 127, 63), (264, 129, 65), (4104, 100, 64), (256, 700, 1100),
                                   (8192, 260, 3), (8192, 260, 2), (4096, 131, 4), (4104, 131, 4), (5456, 77, 3), (16, 9, 5)])
def test_edges(sr, d, f, n):
    say(f"calibrate d={d} f={f} N={n}")
    wg, _, _ = ffn_weights(800 + d, d, f, 1.0 / np.sqrt(d))
    x = calibration_inputs(800 + d, n, d)
    xd, wd = dev_f32(x), dev_bf16(wg)
    v = np.sort(np.abs(oracle.gate_activations(x, wg)).ravel())
    for q in (1e-9, 0.25, 0.5, 0.9, 1.0):
        want = v[min(max(int(np.ceil(q * v.size)), 1), v.size) - 1]
        got = float(host(sr.sirius_cats_calibrate(xd, wd, q))[0])
        assert abs(got - want) <= 1e-5 * want + 2e-6, (q, got, want)


def test_ties_zeros_and_infinities(sr):
    """Equal rows give equal values (one long run of ties), zero rows give zeros, and an input that
    holds an infinity takes the highest ranks only."""
    d, f, n = 264, 1000, 40
    wg, _, _ = ffn_weights(900, d, f, 1.0 / np.sqrt(d))
    wg[:400] = 0
    wg[400:900] = wg[400]
    x = np.repeat(calibration_inputs(900, 1, d), n, axis=0)
    v = np.sort(np.abs(oracle.gate_activations(x, wg)).ravel())
    for q in (0.1, 0.4, 0.41, 0.6, 0.95):
        want = v[int(np.ceil(q * v.size)) - 1]
        got = float(host(sr.sirius_cats_calibrate(dev_f32(x), dev_bf16(wg), q))[0])
        assert abs(got - want) <= 1e-5 * want + (2e-6 if want > 0 else 0), (q, got, want)
    clean = calibration_inputs(901, n, d)
    wg, _, _ = ffn_weights(901, d, f, 1.0 / np.sqrt(d))
    bad = np.concatenate([clean, clean[:1]])
    bad[n, 7] = np.inf
    t = float(host(sr.sirius_cats_calibrate(dev_f32(clean), dev_bf16(wg), 0.5))[0])
    # the same rank among the clean values: all of the bad input's f activations lie above it
    tb = float(host(sr.sirius_cats_calibrate(dev_f32(bad), dev_bf16(wg), 0.5 * n / (n + 1)))[0])
    assert t == tb


@pytest.mark.parametrize("n", [3, 5, 70])
def test_infinite_weights(sr, n):
    """A gate weight that is an infinity gives an infinite activation where the gate is positive (its
    SiLU is NaN where it is negative, and NaN ranks above the infinities): every rank below them is the
    finite activations', the ranks from there on are infinities, then NaN."""
    d, f = 264, 300
    say(f"calibrate with infinite weights N={n}")
    wg, _, _ = ffn_weights(950, d, f, 1.0 / np.sqrt(d))
    x = calibration_inputs(950, n, d)
    wd = dev_bf16(wg)
    wd[3, 7], wd[299, 100], wd[150, 0] = float("inf"), float("-inf"), float("inf")
    finite = np.sort(np.abs(oracle.gate_activations(x, np.delete(wg, [3, 150, 299], axis=0))).ravel())
    up = int(np.sum(x[:, 7] > 0) + np.sum(x[:, 100] < 0) + np.sum(x[:, 0] > 0))
    total = n * f
    at = lambda rank: float(host(sr.sirius_cats_calibrate(dev_f32(x), wd, (rank - 0.5) / total))[0])  # 1-based, ascending
    assert 0 < up < 3 * n
    for rank in (1, finite.size // 2, finite.size):
        assert abs(at(rank) - finite[rank - 1]) <= 1e-5 * finite[rank - 1] + 2e-6
    assert np.isposinf(at(finite.size + 1)) and np.isposinf(at(finite.size + up))
    assert np.isnan(at(finite.size + up + 1)) and np.isnan(at(total))


@pytest.mark.parametrize("d,n,few", [(4096, 4, True), (8192, 2, True), (256, 1, True), (4104, 4, False), (8192, 3, False),
                                     (256, 5, False)])
def test_few_inputs_are_not_padded_to_tiles(sr, d, n, few):
    """At most four inputs of 64 KiB in all take the vector kernel: no launch that splits them for MFMA."""
    import torch
    f = 300
    say(f"calibration route d={d} N={n}")
    wg, _, _ = ffn_weights(970, d, f, 1.0 / np.sqrt(d))
    x, w = dev_f32(calibration_inputs(970, n, d)), dev_bf16(wg)
    sr.sirius_cats_calibrate(x, w, 0.5)
    sr.sirius_profile_reset()
    sr.sirius_profile_enable(True)
    try:
        sr.sirius_cats_calibrate(x, w, 0.5)
        torch.cuda.synchronize()
        prep = sr.sirius_profile_query("calib_prep")[1]
    finally:
        sr.sirius_profile_enable(False)
        sr.sirius_profile_reset()
    assert prep == (0 if few else 1)
