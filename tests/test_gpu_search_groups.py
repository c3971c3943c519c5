"""The offline search where a batch takes part of a KV group (heads times indices beyond the head limit), and the
bisection that evaluates three sizes a step, against the oracle's that evaluates one."""
import numpy as np
import pytest
import torch

import paper_2412_06198_amd as sa
from harness import gen
from oracle import search as srch
from gpu_util import dev_bf16, download_scores

pytestmark = pytest.mark.gpu


def _search(ses, Q, K, V, frac):
    ses.estimate(Q, K)
    N = ses.cfg.seq_len
    return ses.search_patterns(Q, K, V, int(frac * N * (N + 1) / 2), N)


@pytest.mark.parametrize("Hq,Hkv,N,b", [(40, 1, 512, 64), (128, 1, 256, 128), (66, 2, 320, 64), (37, 1, 192, 64)])
def test_parts_of_a_group(Hq, Hkv, N, b):
    print(f"case search groups {Hq}/{Hkv} N={N} b={b}", flush=True)
    g = Hq // Hkv
    gen_ = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((h, N, 128), generator=gen_, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    got = _search(sa.Session(Hq, Hkv, N, b, min(64, N), keep=0.3), Q, K, V, 0.4)
    for h in {0, 1, Hq // 2, Hq - 2, Hq - 1}:
        kv = slice(h // g, h // g + 1)
        assert _search(sa.Session(1, 1, N, b, min(64, N), keep=0.3), Q[h:h + 1], K[kv], V[kv], 0.4)[0] == got[h], h


@pytest.mark.parametrize("N", [64, 128, 192, 576])  # 2, 4, 6 and 18 sizes: no halving, one, some
@pytest.mark.parametrize("eps", [0, 400])
def test_steps_of_the_bisection(N, eps):
    print(f"case search steps N={N} eps={eps}", flush=True)
    H, b, w = 2, 64, 32
    Q, K, V = gen.random_qkv(H, 1, N, 128, seed=N + eps)
    ses = sa.Session(H, 1, N, b, w, keep=0.3)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    ses.estimate(Qd, Kd)
    v, s, blk = download_scores(ses)
    for frac in (0.0, 0.05, 0.2, 0.45, 0.6, 0.7, 0.8, 0.9, 0.97, 1.0):
        target = int(frac * N * (N + 1) / 2)
        res = ses.search_patterns(Qd, Kd, Vd, target, eps)
        ref = srch.search_patterns(Q, K, V, v, s, blk, b, w, ses.cfg.sink_blocks, target, eps)
        for g, r in zip(res, ref):
            assert g["param"] == r["param"] and g["pairs"] == r["pairs"], (frac, g, r)
