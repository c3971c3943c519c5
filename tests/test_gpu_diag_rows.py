"""Block-granular diagonals where their rows are written by the launch that places the lists (v and s of one segment,
32768 keys: up to 512 row blocks of 64) and where by a launch of their own (more keys, per-row blocks of several
segments, budgets beyond a list): offsets around block edges, words of 32 blocks and the last row.  Bit-exact."""
import numpy as np
import pytest

from oracle import oracle as orc
from gpu_util import assert_index_equal, download_index, make_session, upload_scores

pytestmark = pytest.mark.gpu
T, IS, BC = 0, 1, 2


#                                      N       b   k_s    options
@pytest.mark.parametrize("N,b,ks,options", [(64, 64, 64, dict()), (128, 128, 1, dict()), (2112, 64, 5, dict(block_select=1)),
                                            (2048, 64, 2048, dict()), (11648, 64, 40, dict(block_select=1)),
                                            (32768, 64, 40, dict()), (32768, 64, 16384, dict(block_select=2)),
                                            (32768, 64, 300, dict(block_select=1)), (32768, 128, 16385, dict()),
                                            (32896, 128, 300, dict()), (262144, 64, 40, dict())])
def test_rows_of_diagonals_bit_exact(N, b, ks, options):
    print(f"case diag rows N={N} b={b} ks={ks} {options}", flush=True)
    Hq, nb = 3, N // b
    rng = np.random.default_rng(N + ks)
    v = rng.random((Hq, N), dtype=np.float32)
    s = rng.random((Hq, N), dtype=np.float32)
    edges = [e for o in (0, b, 31 * b, 32 * b, 33 * b, 64 * b, N - b, N) for e in (o - 1, o, o + 1) if 0 <= e < N]
    s[1, edges] += 1.0                    # these first
    s[2, : min(N, 3 * b)] += 1.0          # neighbours: most fall into the same blocks
    blk = np.tril(rng.random((Hq, nb, nb), dtype=np.float32))
    bud = orc.Budgets(1, min(2, nb), min(N, 16), ks, min(2 * nb, nb * (nb + 1) // 2), probe_v=1, probe_s=1, diagonal_select=1, **options)
    ses = make_session(Hq, 1, N, b, 64, bud)
    upload_scores(ses, v, s, blk)
    for ov in ([IS] * Hq, [T, IS, BC]):
        ses.build_index(ov)
        assert_index_equal(download_index(ses), orc.build_index(v, s, blk, N, b, 64, bud, override=ov))
