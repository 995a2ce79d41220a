"""fp32 layers at the edges of their 16- and 32-row tiles, in both tile widths, and rows
with infinities or NaN that a causal mask hides from other rows.

Tolerance against the fp64 oracle: the repository's fp32 bar (1e-4), which these sums of at
most a few hundred fp32 terms meet with three orders to spare."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_08186_amd as hd
from paper_2607_08186_amd import synth

from gpu_helpers import run_sfa, to_dev, to_host64

pytestmark = pytest.mark.gpu

INTRA, MIX, LOCAL = hd.HD_SFA_INTRA, hd.HD_SFA_MIX, hd.HD_SFA_LOCAL


# B, L, n, Hq, Hkv, D, mode, window: row counts 1, 15..17, 31..33 and 47..49 per problem, a
# window inside one tile, at a tile's edge and past the sequence, and enough problems
# for the wide tiles (the last four)
@pytest.mark.parametrize("B,L,n,Hq,Hkv,D,mode,window", [
    (1, 1, 1, 1, 1, 32, MIX, None), (1, 1, 3, 2, 1, 64, INTRA, None), (2, 15, 1, 2, 2, 128, MIX, None),
    (1, 16, 2, 4, 2, 32, INTRA, None), (1, 17, 3, 3, 1, 64, MIX, None), (1, 31, 1, 2, 1, 128, MIX, None),
    (1, 33, 2, 2, 1, 32, LOCAL, 1), (1, 49, 1, 2, 2, 64, LOCAL, 16), (1, 47, 2, 2, 1, 128, LOCAL, 33),
    (1, 48, 1, 2, 1, 64, LOCAL, 500), (4, 33, 8, 32, 8, 32, INTRA, None), (4, 65, 8, 16, 8, 64, LOCAL, 40),
    (8, 17, 8, 8, 8, 128, INTRA, None), (8, 31, 4, 32, 16, 64, MIX, None)])
def test_tile_edges(B, L, n, Hq, Hkv, D, mode, window):
    scale = D ** -0.5
    ins = synth.sfa_inputs(B, L, n, Hq, Hkv, D, seed=synth.seed_for(f"f32-tiles-{B}-{L}-{n}-{D}"), dtype="f32")
    out = run_sfa(ins, n, mode, scale, window=window)
    kw = dict(L=L, n=n, mode=mode, scale=scale)
    if window is not None:
        kw["window"] = window
    ro, rlse = oracle.sfa_fwd(ins["q"], ins["k"], ins["v"], **kw)
    grads = oracle.sfa_bwd(ins["q"], ins["k"], ins["v"], ins["dout"], **kw)
    assert np.abs(to_host64(out["o"]) - ro).max() <= 1e-4
    assert np.abs(to_host64(out["lse"]) - rlse).max() <= 1e-4
    for name, ref in zip(("dq", "dk", "dv"), grads):
        err = np.abs(to_host64(out[name]) - ref).max()
        # where every row sees one key, dq and dk are zero and dP - Delta leaves the rounding
        # of two fp32 sums of D unit products: sqrt(D) * sqrt(D) * 2^-24 typically, 8e-6 at
        # D = 128, times |k| scale of about a few tenths
        assert err <= max(1e-4 * np.abs(ref).max(), 1e-5), (name, err)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("copies", [1, 40])  # 40 problems and more: the wide tiles
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_hidden_nonfinite_rows(D, copies, bad):
    """A non-finite key or value reaches only the queries that see it, a non-finite query or
    upstream row only the keys it sees: every other row keeps its bits."""
    L, at, scale = 71, 37, D ** -0.5
    ins = synth.sfa_inputs(copies, L, 1, 8, 8, D, seed=synth.seed_for(f"f32-nonfinite-{D}"), dtype="f32")

    def both(t):
        o, lse = hd.sfa_forward(t["q"], t["k"], t["v"], n=1, mode=MIX, scale=scale)
        dq, dk, dv = hd.sfa_backward(t["q"], t["k"], t["v"], o, lse, t["dout"], n=1, mode=MIX, scale=scale)
        return dict(o=o, dq=dq, dk=dk, dv=dv)

    clean = {k: to_dev(ins[k]) for k in ("q", "k", "v", "dout")}
    want = both(clean)
    for name in ("k", "v"):
        t = dict(clean, **{name: clean[name].clone()})
        t[name][:, at, :, D // 2] = bad
        got = both(t)
        for x in ("o", "dq"):
            assert torch.equal(got[x][:, :at], want[x][:, :at]), (name, x)
        if name == "v" or bad != bad:  # an infinite key may leave a score of -inf, weight zero
            assert not torch.isfinite(got["o"][:, at:]).all(-1).any(), name
    for name in ("q", "dout"):
        t = dict(clean, **{name: clean[name].clone()})
        t[name][:, at, :, D // 2] = bad
        got = both(t)
        for x in ("dk", "dv"):
            assert torch.equal(got[x][:, at + 1:], want[x][:, at + 1:]), (name, x)
        for x in ("o", "dq"):
            assert torch.equal(got[x][:, :at], want[x][:, :at]), (name, x)
            assert torch.equal(got[x][:, at + 1:], want[x][:, at + 1:]), (name, x)
        if name == "dout" or bad != bad:
            assert not torch.isfinite(got["dv"][:, :at + 1]).all(-1).any(), name
