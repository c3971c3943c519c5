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
        assert (np.abs(got - want) <= 1e-3 * np.abs(want) + 1e-6 * w).all()


@pytest.mark.parametrize("octaves", [20, 29, 45, 56])
def test_a_reference_far_below_the_row_costs_no_precision(octaves):
    # The first 32 keys of the only chunk lie `octaves` and a bit (each window row and head differently) below keys
    # 40, 50 and 60, which share a row's weight: at their offsets s holds nothing else of a row but 2^-octaves.
    # Two exponentials and a logarithm of one unit in the last place each, 2^-23 of the weight, and as much again for
    # the sums.  A reference that stayed at the first keys adds the rounding of log2(sum) there: half a unit in the
    # last place of `octaves`, times ln 2, is 6.6e-7 from 16 octaves and 1.3e-6 from 32 on.
    print(f"case estimate reference octaves={octaves}", flush=True)
    Hq, N, w, scale = 32, 128, 8, 0.5
    Q, K = np.zeros((Hq, N, 128), np.float32), np.zeros((1, N, 128), np.float32)
    Q[:, :, 0] = (octaves + np.random.default_rng(octaves).random((Hq, N))) / (scale * np.log2(np.e))
    K[0, :, 0] = -1.0
    K[0, [40, 50, 60], 0] = 0.0
    Q, K = gen.f32_to_bf16_bits(Q), gen.f32_to_bf16_bits(K)
    ses = sa.Session(Hq, 1, N, 64, w, keep=0.5, softmax_scale=scale)
    ses.estimate(dev_bf16(Q), dev_bf16(K))
    _, s, _ = download_scores(ses)
    _, want, _ = orc.estimate(Q, K, 64, w, scale=scale)
    at = np.concatenate([np.arange(N - w, N) - key for key in (40, 50, 60)])
    err = np.abs(s[:, at] - want[:, at]) / want[:, at]
    print(f"largest relative error {err.max():.2e}")
    assert err.max() <= 4 * 2.0 ** -23
