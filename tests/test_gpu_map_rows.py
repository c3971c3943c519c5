"""The block map where a workgroup takes 4, 8 or 16 row blocks of a strip: block counts around multiples of them, and
numbers of strips on either side of the lines between them (b = 64: 64 and 128 strips with 256 compute units, b = 128
twice as many).  Against the fp64 oracle."""
import numpy as np
import pytest

from harness import gen
from oracle import oracle as orc
import paper_2412_06198_amd as sa
from gpu_util import dev_bf16, download_scores

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,nb,b", [(2, nb, 64) for nb in (2, 3, 4, 5, 8, 11, 12, 13, 16, 17, 21, 25, 31, 33)] +
                                    [(2, 6, 128), (2, 19, 128), (32, 30, 64), (33, 30, 64), (64, 29, 64), (65, 29, 64),
                                     (127, 18, 128), (128, 7, 128)])
def test_block_map_rows(Hq, nb, b):
    print(f"case map rows heads={Hq} nb={nb} b={b}", flush=True)
    N = nb * b
    Q, K, _ = gen.random_qkv(Hq, 1, N, 128, seed=nb + Hq)
    ses = sa.Session(Hq, 1, N, b, 64, keep=0.5)
    ses.blk.fill_(-1.0)
    ses.estimate(dev_bf16(Q), dev_bf16(K))
    for got, want in zip(download_scores(ses), orc.estimate(Q, K, b, 64)):  # the tolerance of every score check
        assert (np.abs(got - want) <= 1e-3 * np.abs(want) + 1e-6 * 64).all()
