"""Expansion backward where its row-wise work split can go wrong: runs of equal ids at and
around the 4 and 16 rows a wave loads at once and the 16 rows of a run that four waves
split, runs that start and end at the edges of those groups, rows of odd widths, and the token
counts where the sort changes.

Distinct ids must be bit-exact, rows within the rounding bound of an fp32 sum in token
order (see test_gpu_embed_bwd)."""
import numpy as np
import pytest

from paper_2607_08186_amd import synth
from tests.test_gpu_embed_bwd import _check, _dout

pytestmark = pytest.mark.gpu


def _runs(seed, lengths, V, bad=0):
    """Token ids whose sorted order has runs of the given lengths, and `bad` invalid ones."""
    rng = np.random.default_rng(seed)
    ids = np.repeat(np.sort(rng.choice(V, len(lengths), replace=False)), lengths)
    ids = np.concatenate([ids, np.full(bad, V)]).astype(np.int32)
    return rng.permutation(ids).reshape(1, -1)


LENGTHS = {
    "around16": [1, 15, 16, 17, 31, 32, 33, 1, 1, 14, 2, 64, 65, 5],
    "aligned": [16, 16, 32, 8, 8, 48, 16],
    "one_long": [3, 700, 1],
    "around_split": [2, 18, 1, 19, 20, 3, 21, 34, 35, 36, 37, 66, 70, 1, 130, 131],
    "singles": [1] * 37,
}


@pytest.mark.parametrize("bad", [0, 1, 20])
@pytest.mark.parametrize("Dm,dtype", [(8, "bf16"), (520, "bf16"), (1026, "bf16"), (67, "bf16"),
                                      (520, "f32"), (130, "f32"), (129, "f32")])
@pytest.mark.parametrize("name", sorted(LENGTHS))
def test_run_lengths(name, Dm, dtype, bad):
    seed = synth.seed_for("embed_runs", name, Dm, dtype, bad)
    ids = _runs(seed, LENGTHS[name], 900, bad)
    _check(ids, _dout(seed + 1, 1, 3 * ids.shape[1], Dm, dtype), 900)


@pytest.mark.parametrize("M,V", [(8192, 2 ** 19 - 1), (8192, 2 ** 19), (8193, 151936), (9216, 511), (18433, 512), (20480, 2 ** 18),
                                 (40000, 2 ** 27 + 5), (131072, 3000), (131073, 3000), (131073, 151936),
                                 (131073, 2 ** 27 + 5)])
def test_sort_sizes(M, V):
    """Counting sort up to 8192 tokens (packed keys for V < 2^19), 9-bit digits up to 131072 (one to four passes, by
    V), 8-bit ones with device-wide scans beyond (two, three and four passes: results in either buffer pair); a
    tenth of the ids outside [0, V)."""
    seed = synth.seed_for("embed_sort_sizes", M, V)
    rng = np.random.default_rng(seed)
    ids = (V * rng.random(M) ** 3).astype(np.int64)
    ids[rng.random(M) < 0.1] = -1
    _check(ids.astype(np.int32).reshape(1, M), _dout(seed + 1, 1, M, 8, "bf16"), V)
