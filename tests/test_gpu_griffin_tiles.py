"""GPU parity of the prompt statistic over every tile that its size rule can choose: token counts and
widths that leave ragged last tiles, one token, a K tail, both variants. Scores within 2e-5 of the
oracle's (fp32 products and SiLU, fp64 sums: the tolerance of the selection tests), plus 1e-6 for the
few neurons whose products cancel: a sum of 72 products of size 0.1 to 0.2 rounds by up to
72 x 2^-24 x 0.2 = 9e-7 whatever is left of it."""

import numpy as np
import pytest

import oracle
from synth import ffn_weights, griffin_prompt
from gpu_util import say, dev_bf16, host

pytestmark = pytest.mark.gpu

# tokens, d_ff: 256 x 112, 192 x 112, 128 x 112, 64 x 112, 256 x 64, 192 x 64, 128 x 64 and 64 x 64 tiles
CASES = [(391, 9623), (264, 8194), (578, 3277), (1, 14214), (388, 4182), (131, 4216), (67, 3570), (50, 300)]


@pytest.mark.parametrize("normalize", [False, True])
@pytest.mark.parametrize("t,f", CASES)
def test_scores(t, f, normalize):
    import paper_2409_03856_amd as sr
    d, k = 72, max(1, f // 3)
    say(f"griffin tile T={t} F={f} normalize={normalize}")
    wg, wu, wd = ffn_weights(40 + t, d, f, 1.0 / np.sqrt(d))
    xp = griffin_prompt(40 + t, t, d)
    sel, scores, wgc, _, _ = sr.sirius_griffin_select(dev_bf16(xp), *[dev_bf16(w) for w in (wg, wu, wd)], k,
                                                      normalize_tokens=normalize)
    scores, sel = host(scores), host(sel)
    np.testing.assert_allclose(scores, oracle.griffin_scores(xp, wg, wu, normalize), rtol=2e-5, atol=1e-6)
    # index work on the returned scores: exactly their top k, ascending
    assert np.array_equal(sel, np.sort(np.argsort(-scores, kind="stable")[:k]))
    assert np.array_equal(host(wgc), wg[sel])
