"""The decode's three workgroup shapes (8, 4 and 2 waves) at the edges of their rules: cache
capacities one row below and above the most rows that one workgroup takes (640 rows for at
most 64 problems, 1024 for at most 256, 384 else), problem counts on both sides of those
lines, contexts that leave waves without a tile, and one split more or less.  bf16 tolerance of
the other decode tests; the bound on the contexts must not change a bit of the result."""
import numpy as np
import pytest

import oracle
from paper_2607_08186_amd import synth
from tests import gpu_helpers as G
from tests.test_gpu_decode import INTRA, LOCAL, MIX, _inputs, _run

pytestmark = pytest.mark.gpu

# B, Lcap, n, Hq, Hkv, D, mode, window, contexts (tokens before the new one)
CASES = [
    (2, 640, 4, 8, 4, 128, INTRA, 0, [639, 255]),       # 32 problems, 8 waves
    (2, 641, 4, 8, 4, 128, INTRA, 0, [640, 384]),       # one row more: split
    (2, 160, 4, 16, 2, 64, MIX, 0, [159, 7]),           # 640 rows of all streams
    (2, 161, 4, 16, 2, 64, MIX, 0, [160, 95]),
    (17, 1024, 4, 8, 1, 32, INTRA, 0, [1023, 0, 768] + [31] * 14),   # 68 problems, 8 waves
    (17, 1025, 4, 8, 1, 32, INTRA, 0, [1024, 383, 384] + [40] * 14),
    (65, 256, 1, 4, 4, 64, MIX, 0, [255] * 3 + [1] * 62),            # 260 problems, 2 waves
    (3, 900, 4, 8, 2, 128, LOCAL, 500, [899, 130, 0]),  # a window's rows decide, not the cache
    (3, 900, 4, 8, 2, 128, LOCAL, 605, [899, 160, 10]),
    (1, 1700, 2, 4, 1, 128, MIX, 0, [1699]),            # 4 waves, 14 splits
    (38, 1100, 1, 16, 16, 64, MIX, 0, [1099, 1023, 1024, 700] + [3] * 34),  # 608 problems: parts of 1024
    (31, 600, 1, 16, 16, 128, MIX, 0, [599, 384] + [5] * 29),               # 496: whole
    (72, 520, 1, 16, 16, 32, MIX, 0, [519, 385, 384] + [9] * 69),           # 1152: parts of 256
]


@pytest.mark.parametrize("case", CASES, ids=[str(c[:8]) for c in CASES])
def test_decode_grids(case):
    B, Lcap, n, Hq, Hkv, D, mode, w, ctx = case
    seed = synth.seed_for("decode-grids", str(case))
    print(f"decode grids case={case} seed={seed}", flush=True)
    ins = _inputs(seed, B, Lcap, n, Hq, Hkv, D)
    o, lse = _run(ins, ctx, mode, w)
    ro, rl = oracle.sfa_decode(ins["q"], ins["k"], ins["v"], ctx, n=n, mode=mode,
                               scale=D ** -0.5, window=w)
    G.assert_close_fwd(o, lse, ro, rl, "bf16", str(case))
    # every sequence again, shorter contexts first: the same cache with a lower bound
    low = [min(c, max(ctx) // 3) for c in ctx]
    a, b = _run(ins, low, mode, w), _run(ins, low, mode, w, max_ctx=Lcap - 1)
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


@pytest.mark.parametrize("mode,w", [(MIX, 0), (INTRA, 0), (LOCAL, 300)])
def test_decode_context_outside_the_bound(mode, w):
    """A context below 0 or past the bound counts as the nearest one inside: grid and workspace
    are made for the bound, and nothing beyond them is read or written."""
    B, Lcap, n, Hq, Hkv, D = 3, 900, 4, 8, 2, 64
    ins = _inputs(synth.seed_for("decode-outside", mode), B, Lcap, n, Hq, Hkv, D)
    a = _run(ins, [-3, 899, 100], mode, w, max_ctx=500)
    b = _run(ins, [0, 500, 100], mode, w, max_ctx=500)
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])
    assert np.all(np.isfinite(a[0]))
