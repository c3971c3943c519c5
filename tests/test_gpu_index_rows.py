"""The per-row block rule where its search changes course: maps at the edges of the 256 keys a wave loads
at a time and of the kernel's register sizes (nb = 256, 1024), scores between which the search by halves stops
early, and runs of equal ones in which it does not.  Bit-exact against the oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from gpu_util import assert_index_equal, download_index, make_session, upload_scores

pytestmark = pytest.mark.gpu
BC = 2


def _map(kind, rng, nb):
    if kind == "spread":    # many octaves
        x = np.exp(rng.normal(-7, 2, (nb, nb)))
    elif kind == "ulps":    # neighbouring values: ties, and a search down to the last bit
        x = (np.float32(2.0 ** -9).view(np.uint32) + rng.integers(0, 3, (nb, nb), dtype=np.uint32)).view(np.float32)
    elif kind == "zeros":   # ties at 0 and denormals beside them
        x = np.where(rng.random((nb, nb)) < 0.7, 0, np.exp2(rng.uniform(-149, 0, (nb, nb))))
    else:                   # every row flat, the rows different
        x = np.broadcast_to(1 / np.arange(1, nb + 1)[:, None], (nb, nb))
    return np.tril(x.astype(np.float32))


@pytest.mark.parametrize("nb", [1, 2, 5, 63, 255, 256, 257, 261, 1023, 1026, 2049])
def test_rows_bit_exact(nb):
    print(f"case index rows nb={nb}", flush=True)
    b, kinds = 64, ["spread", "ulps", "zeros", "flat"]
    N, Hq = nb * b, len(kinds)
    rng = np.random.default_rng(nb)
    v, s = rng.random((Hq, N), np.float32), rng.random((Hq, N), np.float32)
    blk = np.stack([_map(k, rng, nb) for k in kinds])
    all_blocks = nb * (nb + 1) // 2
    # one block of a row, a seventh, all but a hundredth, all
    for kb in sorted({nb, nb + (all_blocks - nb) // 7, all_blocks - all_blocks // 100, all_blocks}):
        bud = orc.Budgets(1, 1, 1, 1, kb, block_select=1)
        ses = make_session(Hq, 1, N, b, min(64, N), bud)
        upload_scores(ses, v, s, blk)
        ses.build_index([BC] * Hq)
        assert_index_equal(download_index(ses), orc.build_index(v, s, blk, N, b, min(64, N), bud, override=[BC] * Hq))
