"""The bf16 forward's block shapes at the edges of their tiles: 128-row blocks whose keys the two
wave groups split (at most 192 256-row blocks, and more than 128 keys or a final-stream layer),
and 256-row blocks (more of them), which at D = 64 run one (up to 512) or two per CU.  Row counts
around 128 and 256, key-tile counts odd and even, one tile only (the second group then has
none), windows that leave a group without a visible key; all masks and head dims.  bf16
tolerance of the other forward tests."""
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


# heads: few blocks (keys split), whole blocks, and at D = 64 two of them per CU
HEADS = {"split": (1, 4, 2), "blocks": (4, 50, 2), "many": (3, 192, 1)}


def _blocks(heads, rows, n=1, mode=MIX):
    """The 256-row blocks of a grid: on the side of the shapes' lines that `heads` is for."""
    B, Hq, _ = HEADS[heads]
    blocks = B * Hq * (n if mode == INTRA else 1) * -(-(rows if mode == INTRA else rows * n) // 256)
    assert {"split": blocks <= 192, "blocks": blocks > 192, "many": blocks > 512}[heads], blocks
    return blocks


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("heads", ["split", "blocks"])
@pytest.mark.parametrize("L,n,mode,window", [
    (1, 1, MIX, 0), (63, 1, MIX, 0), (65, 2, INTRA, 0), (127, 1, MIX, 0), (128, 1, MIX, 0), (129, 1, MIX, 0),
    (193, 1, MIX, 0), (257, 1, MIX, 0), (100, 3, MIX, 0), (385, 1, LOCAL, 1), (385, 1, LOCAL, 64),
    (320, 1, LOCAL, 65), (150, 2, LOCAL, 130)])
def test_blocks(heads, D, L, n, mode, window):
    _blocks(heads, L, n, mode)
    B, Hq, Hkv = HEADS[heads]
    _check(B, L, n, Hq, Hkv, D, mode, window, False)


@pytest.mark.parametrize("L", [40, 130, 300])
def test_one_or_two_blocks_per_cu(L):
    _blocks("many", L)
    _check(*HEADS["many"][:1], L, 1, *HEADS["many"][1:], 64, MIX, 0, False)


@pytest.mark.parametrize("L,n,mode,window,final", [
    (1, 2, INTRA, 0, False), (65, 2, INTRA, 0, False), (257, 1, INTRA, 0, False), (193, 1, LOCAL, 64, False),
    (130, 2, LOCAL, 65, False), (385, 1, LOCAL, 1, False), (1, 5, MIX, 0, True), (129, 2, MIX, 0, True),
    (140, 3, LOCAL, 3, True), (260, 2, LOCAL, 70, True)])
def test_two_blocks_per_cu(L, n, mode, window, final):
    """D = 64, more than 512 blocks, held to 128 registers: masks and final-stream queries."""
    _blocks("many", L, 1 if final else n, mode)
    B, Hq, Hkv = HEADS["many"]
    _check(B, L, n, Hq, Hkv, 64, mode, window, final)


@pytest.mark.parametrize("B,L,n,mode,window,final", [(8, 250, 1, MIX, 0, False), (8, 257, 1, MIX, 0, False),
                                                     (8, 300, 1, LOCAL, 65, False), (8, 64, 2, INTRA, 0, False),
                                                     (7, 130, 3, MIX, 0, True)])
def test_one_block_per_cu(B, L, n, mode, window, final):
    """D = 64, from 193 to 512 blocks."""
    rows = L if final or mode == INTRA else L * n
    assert 192 < B * 32 * (n if mode == INTRA else 1) * -(-rows // 256) <= 512
    _check(B, L, n, 32, 2, 64, mode, window, final)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("B,L,n,mode,window,final", [
    (1, 129, 1, MIX, 0, False), (1, 128, 1, MIX, 0, False),           # one key tile per group, or more
    (5, 250, 1, MIX, 0, False), (5, 250, 1, LOCAL, 90, False),        # 160 blocks, 320 of 128 rows
    (1, 1281, 1, MIX, 0, False), (1, 1281, 1, LOCAL, 300, False),     # 192 blocks, 352 of 128 rows
    (5, 129, 2, LOCAL, 60, True), (6, 60, 2, MIX, 0, True)])
def test_split_or_whole_rounds(D, B, L, n, mode, window, final):
    """At most 192 blocks of 256 rows that make more or fewer than 256 of 128."""
    _check(B, L, n, 32, 8, D, mode, window, final)


@pytest.mark.parametrize("D", [32, 64, 128])
@pytest.mark.parametrize("heads", ["split", "blocks"])
@pytest.mark.parametrize("L,n,mode,window", [(1, 5, MIX, 0), (31, 3, MIX, 0), (129, 2, MIX, 0), (140, 4, LOCAL, 3),
                                             (260, 2, LOCAL, 70)])
def test_final_blocks(heads, D, L, n, mode, window):
    _blocks(heads, L)
    B, Hq, Hkv = HEADS[heads]
    _check(B, L, n, Hq, Hkv, D, mode, window, True)
