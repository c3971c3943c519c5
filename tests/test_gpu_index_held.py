"""The index where workgroups hold whole arrays or segments of them: sizes around a unit per wave (4096 keys), a
segment (32768) and the last size taken (8 segments of v and s, 16 of the block map), budgets up to what a list
takes, scores whose lists overflow (ties, a few neighbouring values), probes over several segments.
Bit-exact against the oracle; the sizes and budgets just beyond take the general passes."""
import numpy as np
import pytest

from oracle import oracle as orc
from gpu_util import (assert_index_equal, dev_bf16, download_index, download_scores, make_session, upload_scores)
from harness import gen

pytestmark = pytest.mark.gpu
T, IS, BC = 0, 1, 2


def _scores(kind, rng, shape):
    if kind == "spread":
        return np.exp(rng.normal(-7, 2, shape)).astype(np.float32)
    if kind == "ulps":      # six neighbouring values: a list's worth of ties inside one bin
        return (np.float32(2.0 ** -9).view(np.uint32) + rng.integers(0, 6, shape, dtype=np.uint32)).view(np.float32)
    if kind == "narrow":    # different values, all in one bin
        return (2.0 ** -9 * (1 + 1e-3 * rng.random(shape))).astype(np.float32)
    return np.where(rng.random(shape) < 0.9, 0, np.exp2(rng.uniform(-140, 6, shape))).astype(np.float32)


#        N       b   k_v    k_s    share of the map's blocks, probes, options
CASES = [(4096, 64, 4096, 1, 1.0, 4, dict()),
         (4160, 64, 4160, 4159, 0.9, 9, dict(block_select=2)),
         (11648, 64, 100, 11648, 0.499, 64, dict(diagonal_select=1)),       # 182 blocks: 16471 candidates, 8192 listed
         (11712, 64, 11712, 3, 0.01, 1, dict(block_select=1)),
         (32768, 128, 16384, 300, 0.25, 64, dict()),                        # as many columns as a list takes
         (32832, 64, 16384, 16, 0.05, 32, dict(block_select=1)),            # a second segment of v and s
         (32832, 64, 4000, 200, 0.06, 32, dict(block_select=2)),
         (65536, 64, 3000, 16384, 0.0039, 32, dict(diagonal_select=1)),     # 16 segments of the map: 2048 of each
         (65664, 128, 10922, 40, 0.015, 21, dict()),                        # a third segment
         (131072, 128, 2000, 8192, 0.003, 16, dict(block_select=2)),
         (262144, 128, 4096, 77, 0.5, 8, dict(block_select=1)),             # eight segments
         (262144, 128, 4097, 77, 0.5, 8, dict(block_select=1))]             # general passes


@pytest.mark.parametrize("N,b,kv,ks,share,probe,options", CASES)
def test_held_arrays_bit_exact(N, b, kv, ks, share, probe, options):
    print(f"case index held N={N} b={b} kv={kv} ks={ks} share={share} probe={probe} {options}", flush=True)
    kinds, nb = ["spread", "ulps", "narrow", "sparse"], N // b
    Hq = len(kinds)
    rng = np.random.default_rng(N + kv)
    v = np.stack([_scores(k, rng, N) for k in kinds])
    s = np.stack([_scores(k, rng, N) for k in kinds[::-1]])
    blk = np.stack([np.tril(_scores(k, rng, (nb, nb))) for k in kinds])
    kb = nb + int(share * nb * (nb - 1) // 2)
    bud = orc.Budgets(1, 2, kv, ks, kb, probe_v=probe, probe_s=max(1, probe // 2), **options)
    ses = make_session(Hq, 1, N, b, 64, bud)
    upload_scores(ses, v, s, blk)
    for ov in (None, [IS] * Hq, [BC] * Hq):
        ses.build_index(ov)
        assert_index_equal(download_index(ses), orc.build_index(v, s, blk, N, b, 64, bud, override=ov))


@pytest.mark.parametrize("N,options", [(4096, dict()), (33024, dict(diagonal_select=1)), (33024, dict(block_select=1))])
def test_held_one_call_and_lazy_block_map(N, options):
    # the stages in separate launches: the patterns come from the launch before the block map's
    print(f"case index held lazy N={N} {options}", flush=True)
    b, Hq, Hkv = 128, 4, 1
    data = gen.generate(gen.scaled(gen.WORKLOADS["cfg3"], name="t", n_q_heads=Hq, n_kv_heads=Hkv, seq_len=N, block=b,
                                   seed=N, n_hot=8, hot_block=b, keep=0.1))
    Q, K = dev_bf16(data["Q"]), dev_bf16(data["K"])
    bud = orc.Budgets(1, 2, N // 40, N // 50, N // b + 3000 * (N > 5000), probe_v=8, probe_s=8, **options)
    two = make_session(Hq, Hkv, N, b, 64, bud)
    two.estimate(Q, K)
    v, s, blk = download_scores(two)
    for lazy in (0, 1):
        ses = make_session(Hq, Hkv, N, b, 64, bud, lazy_block_map=lazy)
        for ov in (None, [BC, T, IS, BC]):
            ses.estimate_and_index(Q, K, ov)
            assert_index_equal(download_index(ses), orc.build_index(v, s, blk, N, b, 64, bud, override=ov))
