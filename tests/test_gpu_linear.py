"""GPU parity of the chunk projections (q/k/v with the norm, output projection with the residual,
LM head) at the edges of their tiles: widths that fill no K step or block, row counts that fill no
16- or 64-row tile, and 1, 2, 3 and 4 token tiles with remainders. A one-layer decoder whose sparse
pass keeps every neuron has fp32 FFN inputs at any token count, so the fp32 tolerance of the
forward passes holds: max-abs error <= 1e-4 x RMS of the oracle's logits (fp32 accumulation of at
most 1e4 terms, about 1e-6 observed); cache rows within one bf16 step plus 1e-5 x RMS."""

import numpy as np
import pytest

from oracle import loop
from synth import ModelShape, model_weights, prompt_tokens
from gpu_util import say, dev_bf16, dev_i32, host

pytestmark = pytest.mark.gpu

# (d_model, heads, kv heads, head_dim, vocab, tokens)
CASES = [
    (256, 4, 2, 64, 1000, 2),      # whole tiles, one block of columns
    (264, 3, 1, 40, 5, 16),        # K tail inside a step, q/k/v boundaries inside a row tile
    (1032, 5, 5, 24, 77, 17),      # two token tiles, more than one block
    (520, 2, 1, 128, 12289, 33),   # the 64-row form with one row in its last tile, three token tiles
    (776, 4, 4, 32, 12352, 64),    # four token tiles, whole 64-row tiles
    (2056, 2, 2, 8, 12300, 9),     # K tail in the fifth 512-column block
    (1032, 3, 1, 24, 2031, 2),     # two tokens: every product of at most two million weights
    (1032, 3, 1, 24, 2033, 2),     # the LM head above them
    (2048, 5, 5, 56, 77, 2),       # the widest rows of the pair kernel
    (8, 1, 1, 8, 3, 2),            # the narrowest
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}-h{c[1]}x{c[3]}-v{c[4]}-n{c[5]}")
def test_chunk_projections(case):
    import torch
    import paper_2409_03856_amd as sr
    d, h, hkv, hd, v, n = case
    say(f"chunk projections {case}")
    s = ModelShape("edge", 1, d, 96, h, hkv, hd, v, 96, 6.0)
    bits = model_weights(31 + d, s)
    m = loop.model_from_bits(bits, h, hkv, hd, np.full(1, -1.0))
    gm = sr.Model({k: dev_bf16(b) for k, b in bits.items()}, h, hkv, hd, 96, [-1.0])
    pos = torch.zeros(1, dtype=torch.int32, device="cuda")
    cache = loop.new_cache(m, 96)
    for p, k in ((0, 7), (7, n)):  # a context, then the chunk
        pos.fill_(p)
        toks = prompt_tokens(3 + p, k, v)
        lg, _, _ = sr.sirius_model_forward(gm, dev_i32(toks), pos, True)
        want, _ = loop.forward(m, toks, cache, p, True)
        err = np.max(np.abs(host(lg) - want)) / np.sqrt(np.mean(want * want))
        say(f"  {k} tokens: logits error {err:.2e} x RMS")
        assert err <= 1e-4
    for g, o in ((gm.k_cache, cache[0][0]), (gm.v_cache, cache[0][1])):
        want = o[0, :7 + n]
        step = np.abs(want) * 2.0 ** -7 + 1e-5 * np.sqrt(np.mean(want * want))
        assert np.all(np.abs(host(g[0].float())[:7 + n] - want) <= step)


@pytest.mark.parametrize("d,v,n", [(264, 700, 3), (1032, 12301, 18)])
def test_infinite_weights(d, v, n):
    """A weight that is an infinity gives the infinity (or, with one of the other sign or a NaN in its
    row, the NaN) that the whole fp32 values give, as the one-token passes do; other outputs stay as
    they were. In the LM head, and in the key and value projections (their cache rows)."""
    import torch
    import paper_2409_03856_amd as sr
    h, hkv, hd, inf = 3, 1, 40, np.float32(np.inf)
    say(f"infinite weights d={d} v={v} n={n}")
    s = ModelShape("inf", 1, d, 96, h, hkv, hd, v, 96, 6.0)
    w = {k: dev_bf16(b) for k, b in model_weights(77, s).items()}
    toks = dev_i32(prompt_tokens(5, n, v))

    def passes(weights):
        m = sr.Model(weights, h, hkv, hd, 96, [-1.0])
        pos = torch.zeros(1, dtype=torch.int32, device="cuda")
        lg, _, _ = sr.sirius_model_forward(m, toks, pos, True)
        one = sr.Model(weights, h, hkv, hd, 96, [-1.0])
        rows = []
        for i in range(n):
            pos.fill_(i)
            rows.append(host(sr.sirius_model_forward(one, toks[i:i + 1], pos, True)[0])[0])
        return host(lg), np.stack(rows), m, one

    clean, _, _, _ = passes(w)
    bad = dict(w)
    bad["lm_head"] = w["lm_head"].clone()
    for j, cols in ((0, {1: inf}), (17, {d - 1: -inf}), (v - 1, {8: inf, 9: inf}), (40, {3: inf, 4: -inf}),
                    (41, {2: np.nan}), (100, {c: inf for c in range(d)})):
        for c, x in cols.items():
            bad["lm_head"][j, c] = float(x)
    got, want, _, _ = passes(bad)
    rows = np.array([0, 17, v - 1, 40, 41, 100])
    assert np.array_equal(got[:, rows], want[:, rows], equal_nan=True)
    assert np.all(np.isinf(got[:, [0, 17]])) and np.all(np.isnan(got[:, [41, 100]]))
    keep = np.setdiff1d(np.arange(v), rows)
    assert np.array_equal(got[:, keep], clean[:, keep])
    bad = dict(w)
    for k, x in (("wk", inf), ("wv", -inf)):
        bad[k] = w[k].clone()
        bad[k][0, 5, 7] = float(x)
    _, _, m, one = passes(bad)
    for a, b in ((m.k_cache, one.k_cache), (m.v_cache, one.v_cache)):
        a, b = host(a[0, :n].float())[:, 0], host(b[0, :n].float())[:, 0]
        assert np.all(np.isinf(a[:, 5])) and np.array_equal(a[:, 5], b[:, 5])
        assert np.all(np.isfinite(np.delete(a, 5, 1)))


def test_two_tokens_of_a_small_layer_take_one_launch_per_product():
    """Products of up to two million weights for two tokens are one launch each; the others keep the
    operand preparation in front."""
    import torch
    import paper_2409_03856_amd as sr
    say("launches of a two-token pass")
    s = ModelShape("pair", 2, 256, 300, 4, 2, 64, 9000, 64, 6.0)
    m = sr.Model({k: dev_bf16(b) for k, b in model_weights(5, s).items()}, 4, 2, 64, 64, [0.1] * 2)
    pos = torch.zeros(1, dtype=torch.int32, device="cuda")
    toks = dev_i32(prompt_tokens(5, 2, 9000))
    sr.sirius_model_forward(m, toks, pos, False)
    sr.sirius_profile_reset()
    sr.sirius_profile_enable(True)
    try:
        sr.sirius_model_forward(m, toks, pos, False)
        torch.cuda.synchronize()
        count = {k: sr.sirius_profile_query(k)[1] for k in ("linear_prep", "linear_mfma", "embed")}
    finally:
        sr.sirius_profile_enable(False)
        sr.sirius_profile_reset()
    assert count == {"linear_prep": 1, "linear_mfma": 1, "embed": 1}
