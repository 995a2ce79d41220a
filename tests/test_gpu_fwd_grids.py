"""The bf16 forward's two block shapes at the edges of their tiles: 128-row blocks whose keys
the two wave groups split (grids of at most 128 256-row blocks), and 256-row blocks (more),
which at D = 64 run one or two per CU by the grid's size.  Row counts around 128 and 256,
key-tile counts odd and even, one tile only (the second group then has none), windows that
leave a group without a visible key; all masks and head dims.  bf16 tolerance of the other
forward tests."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_08186_amd as hd
from paper_2607_08186_amd import synth
from tests import gpu_helpers as G

pytestmark = pytest.mark.gpu

INTRA, MIX, LOCAL = 0, 1, 2


def _check(B, L, n, Hq, Hkv, D, mode, window, final):
    seed = synth.seed_for("fwd-grids", B, L, n, Hq, Hkv, D, mode, window, final)
    ins = synth.sfa_inputs(B, L, n, Hq, Hkv, D, seed=seed, dtype="bf16", qkv_std=2 ** -0.5)
    q, k, v = (G.to_dev(ins[x]) for x in ("q", "k", "v"))
    scale = D ** -0.5
    kw = dict(L=L, n=n, mode=mode, scale=scale, window=window)
    if final:
        qf = np.ascontiguousarray(ins["q"][:, n - 1::n])
        o, lse = hd.sfa_final_forward(G.to_dev(qf), k, v, n=n, scale=scale,
                                      window=window if mode == LOCAL else 0)
        ro, rl = oracle.sfa_fwd(qf, ins["k"], ins["v"], final=True, **kw)
    else:
        o, lse = hd.sfa_forward(q, k, v, n=n, mode=mode, scale=scale,
                                window=window if mode == LOCAL else None)
        ro, rl = oracle.sfa_fwd(ins["q"], ins["k"], ins["v"], **kw)
    torch.cuda.synchronize()
    G.assert_close_fwd(G.to_host64(o), G.to_host64(lse), ro, rl, "bf16",
                       f"{(B, L, n, Hq, Hkv, D, mode, window, final)}")


# heads: few blocks (keys split), many, and at D = 64 more than 512
HEADS = {"split": (1, 4, 2), "blocks": (3, 48, 2), "many": (3, 192, 1)}


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("heads", ["split", "blocks"])
@pytest.mark.parametrize("L,n,mode,window", [
    (1, 1, MIX, 0), (63, 1, MIX, 0), (65, 2, INTRA, 0), (127, 1, MIX, 0), (128, 1, MIX, 0), (129, 1, MIX, 0),
    (193, 1, MIX, 0), (257, 1, MIX, 0), (100, 3, MIX, 0), (385, 1, LOCAL, 1), (385, 1, LOCAL, 64),
    (320, 1, LOCAL, 65), (150, 2, LOCAL, 130)])
def test_blocks(heads, D, L, n, mode, window):
    B, Hq, Hkv = HEADS[heads]
    _check(B, L, n, Hq, Hkv, D, mode, window, False)


@pytest.mark.parametrize("L", [40, 130, 300])
def test_one_or_two_blocks_per_cu(L):
    _check(*HEADS["many"][:1], L, 1, *HEADS["many"][1:], 64, MIX, 0, False)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("heads", ["split", "blocks"])
@pytest.mark.parametrize("L,n,mode,window", [(1, 5, MIX, 0), (31, 3, MIX, 0), (129, 2, MIX, 0), (140, 4, LOCAL, 3),
                                             (260, 2, LOCAL, 70)])
def test_final_blocks(heads, D, L, n, mode, window):
    B, Hq, Hkv = HEADS[heads]
    _check(B, L, n, Hq, Hkv, D, mode, window, True)
