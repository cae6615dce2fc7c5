"""GPU parity of the drafting step where its lists change form: widths on both sides of the list
lengths 4, 8 and 16, rows that end inside a thread's run and off the 16-byte grid, rows of more than
64 segments (several lists per lane), infinities, and ties across segments. Compared with the oracle
as the tree tests do (pairs exact where scores differ by more than 1e-5)."""

import numpy as np
import pytest

from synth import tree_build_inputs
from gpu_util import say, dev_f32, host, check_tree_build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wc,width,vocab", [(2, 4, 2051), (3, 5, 131072), (2, 8, 131073), (1, 9, 600001),
                                            (3, 16, 280005), (16, 3, 4099), (1, 1, 524293),
                                            (16, 16, 4097), (2, 9, 131072), (1, 16, 37)])
def test_lists(wc, width, vocab):
    import paper_2409_03856_amd as sr
    say(f"tree lists Wc={wc} W={width} V={vocab}")
    lg, cum = tree_build_inputs(vocab + width, 2, wc, vocab, 3.0)
    tok, par, out = (host(t) for t in sr.sirius_tree_build_step(dev_f32(lg), width, dev_f32(cum), 0.8))
    for b in range(2):
        check_tree_build(lg[b], cum[b], width, 0.8, tok[b], par[b], out[b])


def test_infinite_logits_and_ties_across_many_segments():
    import paper_2409_03856_amd as sr
    v = 400000
    lg = np.full((1, 2, v), -np.inf, dtype=np.float32)
    for i, t in enumerate((399999, 5, 263000, 130000, 8191, 8192)):
        lg[0, 0, t] = 1.0
        lg[0, 1, t] = float(i)
    cum = np.array([[0.0, -50.0]], dtype=np.float32)
    tok, par, out = (host(t) for t in sr.sirius_tree_build_step(dev_f32(lg), 7, dev_f32(cum)))
    assert tok[0].tolist() == [5, 8191, 8192, 130000, 263000, 399999, 8192]
    assert par[0].tolist() == [0] * 6 + [1]
    np.testing.assert_allclose(out[0, :6], -np.log(6.0), rtol=1e-6)
