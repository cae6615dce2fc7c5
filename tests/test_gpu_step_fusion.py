"""One-token passes form their rows in the next projection's launch (the drafted token's embedding, the
residual with the FFN's partials) where sizes allow. On both sides of each size rule the results are
those of the separate launches bit for bit: a pass that also returns the kept lists keeps the separate
FFN sum, and a loop of single passes drafts with torch's argmax."""

import numpy as np
import pytest

from synth import ModelShape, model_weights, prompt_tokens
from gpu_util import say, dev_bf16, dev_i32, host

pytestmark = pytest.mark.gpu

# layers, d_model, d_ff, heads, kv heads, head_dim, vocab
CASES = [
    (2, 256, 688, 4, 2, 64, 1000),     # both: the draft and the partials
    (3, 512, 300, 8, 2, 64, 2600),     # the widest row that takes partials, eight pairs per thread
    (2, 512, 2600, 4, 4, 32, 700),     # more partials than the rule takes
    (2, 520, 400, 2, 1, 40, 333),      # wider than the rule takes
    (2, 136, 90, 3, 1, 24, 9000),      # few rows per launch: a larger vocabulary inside the draft rule
    (1, 72, 17, 1, 1, 8, 60001),       # one partial row group, 24 rows: the largest vocabulary inside it
    (2, 264, 1500, 2, 2, 128, 5),      # a vocabulary of five
    (2, 256, 688, 8, 4, 64, 8192),     # the draft rule's last vocabulary at 1024 rows, partials taken
    (2, 256, 688, 8, 4, 64, 8193),     # and the first past it: every draft a launch of its own
    (1, 520, 400, 8, 4, 64, 12000),    # past it, rows too wide for partials
]


def drafts_folded(case):
    """Each workgroup of the first projection (4 rows each, 2048 at most) reads all the logits: 8 MiB in all."""
    _, _, _, h, hkv, hd, v = case
    return 4 * v * min(-(-(h + 2 * hkv) * hd // 4), 2048) <= 8 << 20


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_drafts_on_both_sides_of_the_logits_rule(case):
    """Past the rule a period's n drafts are n launches; inside it the last one alone."""
    import torch
    import paper_2409_03856_amd as sr
    layers, d, f, h, hkv, hd, v = case
    assert drafts_folded(case) == (case not in CASES[-2:])
    s = ModelShape("fusion", layers, d, f, h, hkv, hd, v, 64, 6.0)
    m = sr.Model({k: dev_bf16(b) for k, b in model_weights(3, s).items()}, h, hkv, hd, 64, [0.2] * layers)
    n = 4
    call = lambda: sr.sirius_generate(m, torch.zeros(n + 1, dtype=torch.int32, device="cuda"),
                                      torch.zeros(1, dtype=torch.int32, device="cuda"), n, 0.1, 1)
    call()
    sr.sirius_profile_reset()
    sr.sirius_profile_enable(True)
    try:
        call()
        torch.cuda.synchronize()
        launches = sr.sirius_profile_query("draft_tail")[1]
    finally:
        sr.sirius_profile_enable(False)
        sr.sirius_profile_reset()
    assert launches == (1 if drafts_folded(case) else n)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_same_bits_as_separate_launches(case):
    import torch
    import paper_2409_03856_amd as sr
    layers, d, f, h, hkv, hd, v = case
    say(f"step fusion {case}")
    s = ModelShape("fusion", layers, d, f, h, hkv, hd, v, 64, 6.0)
    w = {k: dev_bf16(b) for k, b in model_weights(d + f, s).items()}
    models = [sr.Model(w, h, hkv, hd, 64, [0.2] * layers) for _ in range(3)]
    prompt = prompt_tokens(9, 6, v)
    pos = torch.zeros(1, dtype=torch.int32, device="cuda")
    for m in models:
        sr.sirius_model_forward(m, dev_i32(prompt), pos, False)
    # one token, with and without the lists
    pos.fill_(6)
    a, _, _ = sr.sirius_model_forward(models[0], dev_i32(prompt[:1]), pos, True)
    b, idx, cnt = sr.sirius_model_forward(models[1], dev_i32(prompt[:1]), pos, True, want_active=True)
    assert np.array_equal(host(a), host(b)) and np.all(host(cnt) <= f)
    # a period by generate, with and without the lists, and by single passes
    n = 5
    runs = []
    for m, active in ((models[0], False), (models[1], True)):
        seq = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
        seq[0] = int(prompt[2])
        p = torch.full((1,), 6, dtype=torch.int32, device="cuda")
        out, cnt, tr = sr.sirius_generate(m, seq, p, n, 0.1, 1, trace=True, trace_active=active)
        runs.append([host(x) for x in (out, cnt, p, seq[:1], tr["drafted"], tr["accept_len"], tr["q"], m.k_cache.float(),
                                       m.v_cache.float())])
    for x, y in zip(*runs):
        assert np.array_equal(x, y)
    toks = [int(prompt[2])]
    for i in range(n):
        pos.fill_(6 + i)
        lg, _, _ = sr.sirius_model_forward(models[2], dev_i32(np.array([toks[i]], np.int32)), pos, True, want_active=True)
        toks.append(int(torch.argmax(lg[0])))
    assert runs[0][4][0].tolist() == toks[1:]


def test_dense_one_token_pass_and_unknown_token():
    """A full-model pass of one token takes the same launches; an id outside the vocabulary embeds as
    zeros, so its logits are those of a zero row (all equal to W_lm's product with 0)."""
    import torch
    import paper_2409_03856_amd as sr
    s = ModelShape("fusion", 2, 256, 300, 4, 2, 64, 500, 64, 6.0)
    m = sr.Model({k: dev_bf16(b) for k, b in model_weights(5, s).items()}, 4, 2, 64, 64, [0.1] * 2)
    pos = torch.zeros(1, dtype=torch.int32, device="cuda")
    for bad in (-1, 500):
        lg, _, _ = sr.sirius_model_forward(m, dev_i32(np.array([bad], np.int32)), pos, False)
        assert np.all(host(lg) == 0)
    one, _, _ = sr.sirius_model_forward(m, dev_i32(np.array([7], np.int32)), pos, False)
    two, _, _ = sr.sirius_model_forward(m, dev_i32(np.array([7, 8], np.int32)), pos, False)
    a, b = host(one)[0], host(two)[0]
    assert np.max(np.abs(a - b)) <= 1e-4 * np.sqrt(np.mean(b * b))


@pytest.mark.parametrize("d,f,vocab,sums", [(256, 688, 1000, 0), (256, 688, 1536, 0), (256, 688, 1537, 1),
                                            (256, 688, 32000, 1), (512, 1024, 1000, 2)])
def test_partials_are_folded_into_few_rows_only(d, f, vocab, sums):
    """The 128 workgroups of a launch that adds the FFN's partials itself serve at most 1536 output rows:
    the LM head of a larger vocabulary follows a separate sum (one per FFN whose partials are summed so),
    and partials that would be read for 1.5 us and more are summed once."""
    import torch
    import paper_2409_03856_amd as sr
    say(f"fold of partials d={d} f={f} v={vocab}")
    s = ModelShape("fusion", 2, d, f, 4, 2, 64, vocab, 64, 6.0)
    m = sr.Model({k: dev_bf16(b) for k, b in model_weights(5, s).items()}, 4, 2, 64, 64, [0.1] * 2)
    pos = torch.zeros(1, dtype=torch.int32, device="cuda")
    tok = dev_i32(np.array([3], np.int32))
    sr.sirius_model_forward(m, tok, pos, True)
    sr.sirius_profile_reset()
    sr.sirius_profile_enable(True)
    try:
        sr.sirius_model_forward(m, tok, pos, True)
        torch.cuda.synchronize()
        n = sr.sirius_profile_query("cats_reduce")[1]
    finally:
        sr.sirius_profile_enable(False)
        sr.sirius_profile_reset()
    assert n == sums
