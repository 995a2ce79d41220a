"""The bf16 backward's block shapes for small and large grids at the edges of their tiles:
64-key dK/dV workgroups and key-split 128-row dQ blocks (few heads), 128-key and 256-row ones
(many heads); on grids between them the long key sweeps cut at a CU's mean share.  Lengths around 64, 128 and 256, an upper half tile without a key, windows
that reach one half of a key tile only, final-stream layers, and the smallest workspace
(query bands), whose dQ must equal the one-pass one bit for bit.  bf16 tolerances of the other
backward tests."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_08186_amd as hd
from paper_2607_08186_amd import synth
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

INTRA, MIX, LOCAL = 0, 1, 2
HEADS = {"small": (1, 4, 2), "large": (2, 160, 80), "mid16": (2, 16, 8), "mid60": (5, 12, 12), "mid64": (8, 8, 8)}


def _check(heads, D, L, n, mode, window, final):
    B, Hq, Hkv = HEADS[heads]
    what = (heads, D, L, n, mode, window, final)
    ins = synth.sfa_inputs(B, L, n, Hq, Hkv, D, seed=synth.seed_for("bwd-grids", *what), dtype="bf16",
                           qkv_std=2 ** -0.5)
    scale = D ** -0.5
    if final:
        ins = dict(ins, q=np.ascontiguousarray(ins["q"][:, n - 1::n]),
                   dout=np.ascontiguousarray(ins["dout"][:, n - 1::n]))
    q, k, v, do = (G.to_dev(ins[x]) for x in ("q", "k", "v", "dout"))
    dt = hd.HD_DTYPE_BF16
    if final:
        w = window if mode == LOCAL else 0
        o, lse = hd.sfa_final_forward(q, k, v, n=n, scale=scale, window=w)
        low = hd.hd_sfa_bwd_final_min_workspace_bytes(B, L, n, Hq, Hkv, D, w, dt)

        def bwd(**kw):
            return hd.sfa_final_backward(q, k, v, o, lse, do, n=n, scale=scale, window=w, **kw)
    else:
        w = window if mode == LOCAL else None
        o, lse = hd.sfa_forward(q, k, v, n=n, mode=mode, scale=scale, window=w)
        low = (hd.hd_sfa_bwd_local_min_workspace_bytes(B, L, n, Hq, Hkv, D, window, dt) if mode == LOCAL
               else hd.hd_sfa_bwd_min_workspace_bytes(B, L, n, Hq, Hkv, D, mode, dt))

        def bwd(**kw):
            return hd.sfa_backward(q, k, v, o, lse, do, n=n, mode=mode, scale=scale, window=w, **kw)
    got = bwd()
    banded = bwd(workspace_bytes=low)
    torch.cuda.synchronize()
    kw = dict(final=True) if final else {}
    ref = oracle.sfa_bwd(ins["q"], ins["k"], ins["v"], ins["dout"], L=L, n=n, mode=mode, scale=scale,
                         window=window, **kw)
    for name, a, r in zip(("dq", "dk", "dv"), got, ref):
        G.assert_close_grad(G.to_host64(a), r, "bf16", name, str(what))
    assert torch.equal(banded[0], got[0])
    for name, a, r in zip(("dk", "dv"), banded[1:], ref[1:]):
        G.assert_close_grad(G.to_host64(a), r, "bf16", "banded " + name, str(what))


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("L,n,mode,window", [
    (2, 1, MIX, 0), (63, 1, MIX, 0), (65, 2, INTRA, 0), (128, 1, MIX, 0), (129, 1, MIX, 0), (193, 1, MIX, 0),
    (300, 2, MIX, 0), (385, 1, LOCAL, 2), (385, 1, LOCAL, 65), (150, 2, LOCAL, 130)])
def test_small_grids(D, L, n, mode, window):
    _check("small", D, L, n, mode, window, False)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("L,n,mode,window", [(65, 1, MIX, 0), (129, 1, INTRA, 0), (130, 1, LOCAL, 66)])
def test_large_grids(D, L, n, mode, window):
    _check("large", D, L, n, mode, window, False)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("L,n,mode,window", [(2, 5, MIX, 0), (70, 3, MIX, 0), (140, 4, LOCAL, 3), (300, 2, LOCAL, 70)])
def test_small_final_grids(D, L, n, mode, window):
    _check("small", D, L, n, mode, window, True)


# 16, 60 or 64 key problems: the long sweeps are cut at the mean share of 256 CUs (remainders from
# one query tile up), or in halves where most lie below it or all are about as long
@pytest.mark.parametrize("D", [32, 128])
@pytest.mark.parametrize("heads,L,n,mode,window", [
    ("mid64", 640, 1, MIX, 0), ("mid64", 513, 1, MIX, 0), ("mid60", 577, 1, MIX, 0), ("mid60", 960, 1, LOCAL, 300),
    ("mid16", 1100, 1, MIX, 0), ("mid16", 560, 2, LOCAL, 500), ("mid16", 640, 2, INTRA, 0)])
def test_mid_grids(heads, D, L, n, mode, window):
    _check(heads, D, L, n, mode, window, False)
