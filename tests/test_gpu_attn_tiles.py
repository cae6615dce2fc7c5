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
