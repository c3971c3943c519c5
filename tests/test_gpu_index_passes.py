"""The index builder's passes at the sizes and score distributions where they change course: one launch
against several, key ranges that fit their lists, that are split once more, and that never fit (runs
of equal scores), odd block counts.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

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


def _long_scores(kind, rng, shape):
    if kind == "ulps":      # a handful of neighbouring values: a range of few different keys, none of which fits a list
        return (np.float32(2.0 ** -9).view(np.uint32) + rng.integers(0, 6, shape, dtype=np.uint32)).view(np.float32)
    if kind == "wide":      # the same over the 128 keys that the refine pass leaves of a bin, and beyond both ends
        return (np.float32(2.0 ** -9).view(np.uint32) + rng.integers(0, 300, shape, dtype=np.uint32)).view(np.float32)
    if kind == "zeros":     # one entry in a hundred is not 0
        return np.where(rng.random(shape, np.float32) < 0.99, 0, np.exp(rng.standard_normal(shape, np.float32) - 7)).astype(np.float32)
    if kind == "below":     # different values in an eighth of an octave below the histogram's lowest one
        return (np.float32(2.0 ** -40) * (1 + 0.08 * rng.random(shape, np.float32))).astype(np.float32)
    return _scores(kind, rng, shape)


# as many ties as a long prompt can have: the lists cannot take them, and one workgroup must not have to
@pytest.mark.parametrize("N,b,kind,select", [(131072, 128, k, s) for k in ("equal", "few", "ulps", "wide", "zeros", "below")
                                             for s in (0, 2)] + [(66624, 64, "ulps", 0), (262144, 64, "ulps", 2),
                                                                 (262144, 64, "zeros", 0), (262144, 64, "equal", 0)])
def test_long_runs_bit_exact(N, b, kind, select):
    print(f"case index long runs N={N} b={b} {kind} select={select}", flush=True)
    Hq, nb = 2, N // b
    rng = np.random.default_rng(N + len(kind))
    v, s = _long_scores(kind, rng, (Hq, N)), _long_scores(kind, rng, (Hq, N))
    blk = np.tril(_long_scores(kind, rng, (Hq, nb, nb)))
    if kind == "equal" and select == 2:  # flat softmax rows: equal but for the rounding of the key
        blk = np.tril(np.broadcast_to(1 / np.arange(1, nb + 1, dtype=np.float32)[:, None], (Hq, nb, nb)))
    # probes as many as the lists of v and s cannot take either
    bud = orc.Budgets(1, 2, N // 9, N // 100, nb + nb * (nb - 1) // 2 // 7, probe_v=4500, probe_s=N // 9, block_select=select)
    ses = make_session(Hq, 1, N, b, 64, bud)
    upload_scores(ses, v, s, blk)
    for ov in (None, [IS, BC]):
        ses.build_index(ov)
        assert_index_equal(download_index(ses), orc.build_index(v, s, blk, N, b, 64, bud, override=ov))


def test_long_runs_take_a_few_passes():
    # five launches whatever the scores are: long runs of ties cost a pass or two more, not a walk by one workgroup
    # (which took 12 to 60 times as long as scores without ties)
    N, b, Hq = 131072, 128, 8
    nb = N // b
    ses = make_session(Hq, 1, N, b, 64, orc.Budgets(1, 2, N // 33, N // 4000, nb * (nb + 1) // 64))
    g = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda *s: torch.exp(2 * torch.randn(s, generator=g, device="cuda") - 7)
    tri = torch.ones((nb, nb), device="cuda").tril()

    def best():
        times = []
        for _ in range(7):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(5):
                ses.build_index(None)
            t1.record()
            torch.cuda.synchronize()
            times.append(t0.elapsed_time(t1))
        return min(times)

    def fill(flat_vs=False, flat_blk=False, zeros=False):
        ses.v.copy_(rand(Hq, N)), ses.s.copy_(rand(Hq, N)), ses.blk.copy_(rand(Hq, nb, nb) * tri)
        if flat_vs: ses.v.fill_(2.0 ** -10), ses.s.fill_(2.0 ** -10)
        if flat_blk: ses.blk.copy_(2.0 ** -10 * tri.expand(Hq, nb, nb))
        if zeros: ses.blk.mul_(torch.rand((Hq, nb, nb), generator=g, device="cuda") < 0.01)

    fill()
    spread = best()
    for kind in ("flat_vs", "flat_blk", "zeros"):
        fill(**{kind: True})
        t = best()
        print(f"{kind}: {t / spread:.2f} times as long as scores without ties", flush=True)
        assert t <= 4 * spread, (kind, t, spread)
