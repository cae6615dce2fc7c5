"""GPU parity of the shared-cache attention at the edges of its MFMA tiles: 1, 2 and 4 query tiles
with remainders and a second row group, head dimensions that fill no 32-wide step, contexts that
end on and beside a 32-position block, a tile or a chunk, one and many chunks, and entries whose
context leaves most chunks empty. Tolerance: that of the attention tests, 1e-4 x RMS of the fp64
output (fp32 products; about 1e-6 observed)."""

import numpy as np
import pytest

import oracle
from synth import attn_inputs
from gpu_util import say, dev_bf16, dev_f32, dev_i32, host

pytestmark = pytest.mark.gpu

# B, n, H, Hkv, head_dim, Lmax, positions
CASES = [
    (1, 1, 2, 2, 8, 300, [0]),                     # one row, first position, several chunks allowed
    (2, 3, 4, 2, 40, 1000, [5, 997]),              # empty chunks in one entry, the full cache in the other
    (1, 16, 2, 2, 72, 700, [511]),                 # exactly one query tile; 527 positions
    (1, 17, 1, 1, 96, 700, [127]),                 # 17 rows: the second tile holds one
    (1, 16, 2, 1, 128, 256, [31]),                 # 32 rows, one chunk (direct), 47 positions
    (2, 33, 1, 1, 56, 256, [0, 223]),              # 33 rows: four tiles, the third holds one; direct
    (1, 33, 4, 2, 128, 400, [367]),                # 66 rows: a second row group of two
    (3, 8, 8, 1, 128, 2100, [63, 1024, 2092]),     # 64 rows; beside tile and chunk ends
    (1, 8, 8, 1, 64, 2100, [2048]),                # the 64-wide form with four tiles
    (1, 1, 16, 1, 128, 5000, [4000]),              # 16 rows of one token, position groups merged
    (70, 1, 8, 8, 32, 300, list(range(0, 280, 4))),  # one chunk per entry in a cache above 256 rows
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(x) for x in c[:6]))
def test_tiles(case):
    import paper_2409_03856_amd as sr
    b, n, h, hkv, hd, lmax, pos = case
    say(f"attention {case[:6]}")
    q, kn, vn, kc, vc = attn_inputs(900 + h * n + hd, b, n, h, hkv, hd, lmax)
    q *= 3.0  # peaked rows: the running maximum moves
    Kc, Vc = dev_bf16(kc), dev_bf16(vc)
    out = host(sr.sirius_attn_kv(dev_f32(q), dev_bf16(kn), dev_bf16(vn), Kc, Vc, dev_i32(np.asarray(pos))))
    want, _, _ = oracle.attn_kv(q, kn, vn, kc, vc, pos)
    rms = np.sqrt(np.mean(want * want))
    assert np.max(np.abs(out - want)) <= 1e-4 * rms
    for i, p in enumerate(pos):
        kc[i, p:p + n], vc[i, p:p + n] = kn[i], vn[i]
    assert np.array_equal(host(Kc), kc) and np.array_equal(host(Vc), vc)
    # an entry that does not fit leaves the cache as it was and gives NaN
    bad = np.asarray(pos)
    bad[0] = lmax - n + 1
    o2 = host(sr.sirius_attn_kv(dev_f32(q), dev_bf16(kn), dev_bf16(vn), Kc, Vc, dev_i32(bad)))
    assert np.all(np.isnan(o2[0])) and np.array_equal(o2[1:], out[1:])
    assert np.array_equal(host(Kc), kc) and np.array_equal(host(Vc), vc)


def _widen(bits):
    return (np.asarray(bits).astype(np.uint32) << 16).view(np.float32)


# B, n, H, Hkv, head_dim, Lmax, position: one, two and four query tiles, one chunk and several
@pytest.mark.parametrize("case", [(1, 1, 4, 1, 64, 200, 150), (1, 1, 8, 2, 128, 3000, 2500), (1, 5, 4, 1, 72, 900, 700),
                                  (1, 16, 4, 1, 128, 2000, 1500), (1, 20, 2, 1, 40, 250, 200)],
                         ids=lambda c: "-".join(str(x) for x in c))
def test_infinite_keys_and_values(case):
    """Infinities in the cache give what whole fp32 products give. A value row with an infinity: that
    infinity in its column for every token that sees the row. A key that makes a score -infinity or
    NaN: the position weighs nothing. One that makes it +infinity: NaN. Tokens that do not see the
    position, and heads beside it, stay as they were (1e-5 x RMS: fp32 sums in another order)."""
    import paper_2409_03856_amd as sr
    b, n, h, hkv, hd, lmax, p = case
    say(f"attention with infinities {case}")
    g = h // hkv
    q, kn, vn, kc, vc = attn_inputs(77 + hd, b, n, h, hkv, hd, lmax)
    q *= 3.0
    q[0, 0, :g, 3] = 0.0  # a NaN score: 0 times an infinity

    def run(kn, vn, kc, vc):
        return host(sr.sirius_attn_kv(dev_f32(q), dev_bf16(kn), dev_bf16(vn), dev_bf16(kc), dev_bf16(vc),
                                      dev_i32(np.array([p]))))[0]

    clean = run(kn, vn, kc, vc)
    scale = np.sqrt(np.mean(clean * clean))
    pinf, ninf = 0x7F80, 0xFF80
    # values: column 5 of a cached row that holds each row's maximum weight or not
    v2 = vc.copy()
    v2[0, p // 2, 0, 5] = ninf
    got = run(kn, vn, kc, v2)
    assert np.all(np.isneginf(got[:, :g, 5]))
    keep = np.ones(hd, bool)
    keep[5] = False
    assert np.max(np.abs(got[:, :g][..., keep] - clean[:, :g][..., keep])) <= 1e-5 * scale
    assert np.array_equal(got[:, g:], clean[:, g:])
    # the chunk's last new value row: seen by the last token only
    vn2 = vn.copy()
    vn2[0, n - 1, 0, 0] = pinf
    got = run(kn, vn2, kc, vc)
    assert np.all(np.isposinf(got[n - 1, :g, 0]))
    assert np.max(np.abs(got[:n - 1] - clean[:n - 1]), initial=0.0) <= 1e-5 * scale
    # keys: the sign of the query's column decides, and a zero there gives NaN: no weight
    k2 = kc.copy()
    k2[0, p // 3, 0, 3] = pinf
    got = run(kn, vn, k2, vc)
    qs = q[0, :, :g, 3]
    assert np.all(np.isnan(got[:, :g][qs > 0]))
    kf, vf = _widen(kc), _widen(vc)
    kf[0, p:p + n], vf[0, p:p + n] = _widen(kn[0]), _widen(vn[0])
    for i in range(n):
        rows = [r for r in range(p + i + 1) if r != p // 3]
        for j in range(g):
            if qs[i, j] > 0:
                continue
            s = kf[0, rows, 0].astype(np.float64) @ q[0, i, j].astype(np.float64) / np.sqrt(hd)
            w = np.exp(s - s.max())
            want = (w / w.sum()) @ vf[0, rows, 0].astype(np.float64)
            assert np.max(np.abs(got[i, j] - want)) <= 1e-4 * scale
    assert np.array_equal(got[:, g:], clean[:, g:])
