"""The offline search over batches of heads: what a head gets must not depend on the heads beside it,
on the batch it falls into or on the layout of Q, K and V."""
import pytest
import torch

import paper_2412_06198_amd as sa

pytestmark = pytest.mark.gpu


def _search(ses, Q, K, V, frac):
    ses.estimate(Q, K)
    N = ses.cfg.seq_len
    return ses.search_patterns(Q, K, V, int(frac * N * (N + 1) / 2), N)


# (40, 40, 65536): more heads than a batch holds; (12, 2): two KV groups; the rest: edges of the size ranges
@pytest.mark.parametrize("Hq,Hkv,N,b,frac", [(40, 40, 65536, 128, 0.04), (12, 2, 4160, 64, 0.2), (3, 1, 64, 64, 0.5),
                                             (4, 4, 384, 128, 1.0), (4, 2, 1088, 64, 0.0)])
def test_heads_are_searched_independently(Hq, Hkv, N, b, frac):
    print(f"case search batches {Hq}/{Hkv} N={N} b={b} {frac}", flush=True)
    g = Hq // Hkv
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((h, N, 128), generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    got = _search(sa.Session(Hq, Hkv, N, b, min(64, N), keep=0.2), Q, K, V, frac)
    for h in {0, Hq // 2, Hq - 1}:
        one = sa.Session(1, 1, N, b, min(64, N), keep=0.2)
        kv = slice(h // g, h // g + 1)
        assert _search(one, Q[h:h + 1], K[kv], V[kv], frac)[0] == got[h], h


def test_search_reads_strided_layouts():
    print("case search strided", flush=True)
    Hq, Hkv, N = 4, 2, 1024
    gen = torch.Generator(device="cuda").manual_seed(7)
    Q, K, V = (torch.randn((N, h, 128), generator=gen, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    inter = sa.Session(Hq, Hkv, N, 64, 64, keep=0.2, q_head_stride=128, q_row_stride=Hq * 128, kv_head_stride=128,
                       kv_row_stride=Hkv * 128)
    plain = sa.Session(Hq, Hkv, N, 64, 64, keep=0.2)
    got = _search(inter, Q, K, V, 0.25)
    want = _search(plain, *(x.transpose(0, 1).contiguous() for x in (Q, K, V)), 0.25)
    assert got == want
