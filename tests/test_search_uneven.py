"""The offline search over numbers of heads that no batch divides evenly: how many heads a batch takes, and that a head of
any batch gets what it gets alone."""
import pytest
import torch

import paper_2412_06198_amd as sa


def _scratch(Hq, Hkv, N):
    cfg = sa.SaConfig(n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, seq_len=N, block=64, last_q=64)
    ctx = sa.sa_create(sa.sa_default_budgets(cfg, 0.3))
    try:
        return sa.sa_search_scratch_bytes(ctx)
    finally:
        sa.sa_destroy(ctx)


# prime numbers of heads and of KV heads beyond a batch's 32 heads; the scratch is that of at least half as many
@pytest.mark.parametrize("Hq,Hkv,like", [(37, 1, (16, 1)), (37, 37, (16, 16)), (74, 2, (16, 1)), (39, 13, (15, 5)),
                                         (33, 3, (11, 1)), (127, 127, (16, 16))])
def test_batches_stay_large(Hq, Hkv, like):
    assert _scratch(Hq, Hkv, 1024) >= _scratch(*like, 1024)
    assert _scratch(Hq, Hkv, 65536) <= 2 << 30


def _search(ses, Q, K, V, frac):
    ses.estimate(Q, K)
    N = ses.cfg.seq_len
    return ses.search_patterns(Q, K, V, int(frac * N * (N + 1) / 2), N)


# the last batch smaller: of one group, of every group, of all KV heads; 8256: a step of the refinement per launch
@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,N,b", [(37, 1, 320, 64), (74, 2, 256, 128), (37, 37, 320, 64), (39, 13, 448, 64),
                                        (33, 33, 8256, 64)])
def test_heads_of_uneven_batches(Hq, Hkv, N, b):
    print(f"case search uneven {Hq}/{Hkv} N={N} b={b}", flush=True)
    g = Hq // Hkv
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((h, N, 128), generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    got = _search(sa.Session(Hq, Hkv, N, b, 64, keep=0.3), Q, K, V, 0.4)
    for h in {0, 1, g - 1, 16, Hq // 2, Hq // 2 + 1, Hq - 2, Hq - 1}:
        kv = slice(h // g, h // g + 1)
        assert _search(sa.Session(1, 1, N, b, 64, keep=0.3), Q[h:h + 1], K[kv], V[kv], 0.4)[0] == got[h], h
