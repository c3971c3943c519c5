"""The index builder's passes at the sizes and score distributions where they change course: one launch
against several, key ranges that fit their lists, that are split once more, and that never fit (runs
of equal scores), odd block counts.  Bit-exact against the oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from gpu_util import assert_index_equal, download_index, make_session, upload_scores

pytestmark = pytest.mark.gpu
T, IS, BC = 0, 1, 2


def _scores(kind, rng, shape):
    if kind == "spread":    # many octaves: short boundary lists
        return np.exp(rng.normal(-7, 2, shape)).astype(np.float32)
    if kind == "narrow":    # one part in a thousand: a boundary bin with almost every key
        return (2.0 ** -9 * (1 + 1e-3 * rng.random(shape))).astype(np.float32)
    if kind == "equal":     # a list can never hold the ties
        return np.full(shape, 2.0 ** -10, np.float32)
    if kind == "few":       # three values
        return (rng.integers(1, 4, shape) * 2.0 ** -11).astype(np.float32)
    if kind == "tiny":      # below the histogram's lowest octave, zeros and denormals among them
        return np.where(rng.random(shape) < 0.3, 0, np.exp2(rng.uniform(-140, -26, shape))).astype(np.float32)
    raise AssertionError(kind)


# around the switch to several launches (182^2 > 32768 map entries, > 32768 keys) and the smallest maps
@pytest.mark.parametrize("N,b", [(64, 64), (192, 64), (4096, 64), (11584, 64), (11648, 64), (16448, 64),
                                 (32768, 128), (32896, 128)])
@pytest.mark.parametrize("kind", ["spread", "narrow", "equal", "few", "tiny"])
def test_index_passes_bit_exact(N, b, kind):
    print(f"case index passes N={N} b={b} {kind}", flush=True)
    Hq, nb, w = 3, N // b, min(64, N)
    rng = np.random.default_rng(N + len(kind))
    v, s = _scores(kind, rng, (Hq, N)), _scores(kind, rng, (Hq, N))
    blk = np.tril(_scores(kind, rng, (Hq, nb, nb)))
    all_blocks = nb * (nb + 1) // 2
    for select, kb in ((0, nb + (all_blocks - nb) // 3), (2, nb + (all_blocks - nb) // 7), (1, nb + (all_blocks - nb) // 5)):
        bud = orc.Budgets(1, min(2, nb), max(1, N // 9), max(1, N // 100), kb, block_select=select)
        ses = make_session(Hq, 1, N, b, w, bud)
        upload_scores(ses, v, s, blk)
        for ov in (None, [IS, BC, T]):
            ses.build_index(ov)
            assert_index_equal(download_index(ses), orc.build_index(v, s, blk, N, b, w, bud, override=ov))
