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
