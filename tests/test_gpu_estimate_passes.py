"""The estimator at the sizes where its launches change shape: registers per strip of the block map (512,
1024, 2048 and 4096 blocks), chunk lengths and counts of the window passes, head groups of one to
eight, ragged ends.  Against the fp64 oracle."""
import numpy as np
import pytest

from harness import gen
from oracle import oracle as orc
import paper_2412_06198_amd as sa
from gpu_util import dev_bf16, download_scores

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,N,b,w", [
    (1, 1, 64, 64, 64), (3, 1, 192, 64, 5), (8, 8, 1088, 64, 64), (8, 1, 4224, 128, 33),
    (16, 8, 8192, 64, 64), (5, 5, 33088, 64, 64),      # 517 blocks
    (2, 1, 65600, 64, 64), (1, 1, 131072, 64, 64),     # 1025 and 2048 blocks, one walk of K
    (1, 1, 131200, 64, 17), (2, 2, 262144, 64, 64),    # 2050 and 4096 blocks
])
def test_scores_match_oracle_at_the_edges(Hq, Hkv, N, b, w):
    print(f"case estimate passes {Hq}/{Hkv} N={N} b={b} w={w}", flush=True)
    Q, K, _ = gen.random_qkv(Hq, Hkv, N, 128, seed=N + Hq)
    ses = sa.Session(Hq, Hkv, N, b, w, keep=0.2)
    ses.v.fill_(-1.0), ses.s.fill_(-1.0), ses.blk.fill_(-1.0)
    ses.estimate(dev_bf16(Q), dev_bf16(K))
    for got, want in zip(download_scores(ses), orc.estimate(Q, K, b, w)):
        assert (np.abs(got - want) <= 1e-3 * np.abs(want) + 1e-6 * w).all()


def test_logits_far_apart():
    # rows whose largest logits come late and exceed the first ones by hundreds: the running reference of
    # the first pass has to move
    print("case estimate far apart", flush=True)
    N, b, w = 2048, 64, 64
    Q, K, _ = gen.random_qkv(4, 1, N, 128, seed=3)
    f = gen.bf16_bits_to_f32(K)
    f[:, :700] *= 0.01
    f[:, 1500:1520] *= 60.0
    K = gen.f32_to_bf16_bits(f)
    ses = sa.Session(4, 1, N, b, w, keep=0.2)
    ses.estimate(dev_bf16(Q), dev_bf16(K))
    for got, want in zip(download_scores(ses), orc.estimate(Q, K, b, w)):
        assert (np.abs(got - want) <= 1e-3 * np.abs(want) + 1e-5 * w).all()
