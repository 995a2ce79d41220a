"""The decode's workgroup shapes (eight waves up to 256 problems at D=128 and 64 else, four
beyond) and splits at the edges of their rules: contexts one row below and above the most rows
that one workgroup takes (640 rows for at most 64 problems, 1024 for at most 256, 384 else),
problem counts on both sides of those lines, contexts that leave waves without a tile, and one
split more or less.  bf16 tolerance of the other decode tests; neither the bound on the contexts
nor the cache's capacity may change a bit of the result."""
import numpy as np
import pytest

import oracle
from paper_2607_08186_amd import synth
from tests import gpu_helpers as G
from tests.test_gpu_decode import INTRA, LOCAL, MIX, _inputs, _run

pytestmark = pytest.mark.gpu

# B, Lcap, n, Hq, Hkv, D, mode, window, contexts (tokens before the new one)
CASES = [
    (2, 640, 4, 8, 4, 128, INTRA, 0, [639, 255]),       # 32 problems, whole
    (2, 641, 4, 8, 4, 128, INTRA, 0, [640, 384]),       # one row more: split
    (2, 160, 4, 16, 2, 64, MIX, 0, [159, 7]),           # 640 rows of all streams
    (2, 161, 4, 16, 2, 64, MIX, 0, [160, 95]),
    (17, 1024, 4, 8, 1, 32, INTRA, 0, [1023, 0, 768] + [31] * 14),   # 68 problems, whole
    (17, 1025, 4, 8, 1, 32, INTRA, 0, [1024, 383, 384] + [40] * 14),
    (65, 256, 1, 4, 4, 64, MIX, 0, [255] * 3 + [1] * 62),            # 260 problems
    (3, 900, 4, 8, 2, 128, LOCAL, 500, [899, 130, 0]),  # a window's rows decide, not the cache
    (3, 900, 4, 8, 2, 128, LOCAL, 605, [899, 160, 10]),
    (1, 1700, 2, 4, 1, 128, MIX, 0, [1699]),            # 14 splits
    (38, 1100, 1, 16, 16, 64, MIX, 0, [1099, 1023, 1024, 700] + [3] * 34),  # 608 problems: parts of 1024
    (31, 600, 1, 16, 16, 128, MIX, 0, [599, 384] + [5] * 29),               # 496 problems: whole
    (72, 520, 1, 16, 16, 32, MIX, 0, [519, 385, 384] + [9] * 69),           # 1152 problems: whole
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


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("rows", [32, 64, 320, 31, 60])
def test_decode_last_rows_of_a_tile(rows, D):
    """All of a query's weight lies on one of the last rows of the last tile, whole (no mask, the
    shortest way from the scores' product to their first read) or ragged: those rows' scores
    are the last registers that the product writes."""
    B, n, Hq, Hkv, scale = 4, 1, 4, 1, D ** -0.5
    ins = _inputs(synth.seed_for("decode-last", rows, D), B, rows, n, Hq, Hkv, D)
    for b, back in enumerate((0, 1, 4, 5)):
        x = 8 * synth.bf16_bits_to_f32(ins["q"][b].reshape(-1)[:D])
        ins["k"][b, rows - 1 - back, 0] = synth.to_bf16_bits(x)
    o, lse = _run(ins, [rows - 1] * B, MIX, 0)
    ro, rl = oracle.sfa_decode(ins["q"], ins["k"], ins["v"], [rows - 1] * B, n=n, mode=MIX, scale=scale, window=0)
    G.assert_close_fwd(o, lse, ro, rl, "bf16", str((rows, D)))


# B, n, Hq, Hkv, D, mode, window, contexts: problems on both sides of the lines of the rule
SHAPES = [
    (2, 4, 8, 4, 128, INTRA, 0, [639, 500]),            # 32 problems: whole, eight waves
    (1, 4, 16, 4, 128, MIX, 0, [777]),                  # 4 problems: as many parts as rows allow
    (16, 1, 16, 16, 128, MIX, 0, [1499, 1024, 1023, 30] + [800] * 12),    # 256 problems
    (17, 1, 16, 16, 128, MIX, 0, [2500, 2049, 2048, 385] + [384] * 13),   # 272: parts of 2048
    (9, 1, 16, 16, 128, MIX, 0, [4200, 4095, 5] + [100] * 6),             # 144: whole up to 4096
    (5, 1, 16, 16, 64, MIX, 0, [1500, 1025, 640, 0, 7]),                  # 80, four waves
    (17, 1, 16, 16, 64, MIX, 0, [1500, 1025, 640] + [3] * 14),            # 272: parts of 1024
    (5, 2, 16, 16, 32, INTRA, 0, [1500, 1025, 640, 0, 7]),                # heads taken by eights
    (3, 3, 6, 3, 32, MIX, 0, [700, 5, 300]),                              # 3 heads: one by one
    (2, 4, 8, 2, 64, LOCAL, 700, [1100, 200]),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s[:7]) for s in SHAPES])
def test_decode_capacity_and_bound_change_no_bit(shape):
    """The same sequences in a tight cache, in one of twice the rows and in one of 5000 tokens, each
    under a tight and a loose bound: every result has the same bits, and the tight one is right."""
    B, n, Hq, Hkv, D, mode, w, ctx = shape
    seed = synth.seed_for("decode-capacity", str(shape))
    print(f"decode capacity shape={shape} seed={seed}", flush=True)
    tight = max(ctx) + 1
    ins = _inputs(seed, B, tight, n, Hq, Hkv, D)
    want = _run(ins, ctx, mode, w)
    pick = sorted({int(np.argmax(ctx)), int(np.argmin(ctx)), B // 2})
    ro, rl = oracle.sfa_decode(ins["q"][pick], ins["k"][pick], ins["v"][pick], [ctx[b] for b in pick],
                               n=n, mode=mode, scale=D ** -0.5, window=w)
    G.assert_close_fwd(want[0][pick], want[1][pick], ro, rl, "bf16", str(shape))
    for cap in (2 * tight, 5000):
        roomy = dict(ins)
        for x in ("k", "v"):
            roomy[x] = np.zeros((B, n * cap, Hkv, D), dtype=ins[x].dtype)
            roomy[x][:, :n * tight] = ins[x]
        for bound in (None, cap - 1):
            got = _run(roomy, ctx, mode, w, max_ctx=bound)
            np.testing.assert_array_equal(want[0], got[0])
            np.testing.assert_array_equal(want[1], got[1])
