"""Items shared by two groups of waves: few heads of short prompts (and, where the band covers the sequence, twice as
many).  Arbitrary indices, so that a group is left with no tile, no diagonal or nothing at all, lists of odd and
even length meet gather tiles at either place, and rows end inside a row block; against the oracle."""
import numpy as np
import pytest
import torch

import paper_2412_06198_amd as sa
from harness import gen
from oracle import oracle as orc
from gpu_util import check_attention, dev_bf16, host_f64, make_session, random_index, upload_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,b,k_v,k_s", [(64, 64, 1, 1), (128, 128, 64, 1), (192, 64, 65, 3), (448, 64, 130, 70),
                                         (640, 128, 200, 2), (1088, 64, 257, 129), (2048, 64, 64, 0)])
def test_arbitrary_indices(N, b, k_v, k_s):
    print(f"case split items N={N} b={b} columns {k_v} diagonals {k_s}", flush=True)
    Hq, Hkv, nb = 8, 2, N // b
    rng = np.random.default_rng(N + k_v)
    cap = nb * (nb + 1) // 2 + nb
    ses = make_session(Hq, Hkv, N, b, min(64, N), orc.Budgets(1, 1, k_v, max(k_s, 1), cap - nb))
    cap = ses.index_tensors()[6].shape[1]
    index = random_index(rng, Hq, N, b, k_v, max(k_s, 1), max(cap, nb * (nb + 1)))
    index.blkcols = index.blkcols[:, :cap]
    for h in range(2):  # one tile or none per row block, and nothing else
        index.n_cols[h] = index.n_offs[h] = 0
        index.blkcols[h] = -1
        index.blkcols[h, :nb] = np.arange(nb)
        index.rowptr[h] = np.arange(nb + 1) if h else 0
    upload_index(ses, index)
    Q, K, V = gen.random_qkv(Hq, Hkv, N, 128, seed=N)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    O, counted = torch.full_like(Qd, 7.0), torch.full_like(Qd, 7.0)
    for _ in range(2):  # the second call meets what the first left in the workspace
        ses.prefill(Qd, Kd, Vd, O)
    _, kept = ses.prefill_counted(Qd, Kd, Vd, counted)
    torch.cuda.synchronize()
    check_attention(host_f64(O), orc.masked_rows(Q, K, V, b, index)[0], f"split {N}")
    assert torch.equal(O, counted)
    assert kept == sum(orc.mask_count(N, b, h, index) for h in range(Hq))


# at and beyond the number of items up to which they are shared; with the band over the sequence up to twice that
@pytest.mark.parametrize("Hq,dense", [(0, False), (1, False), (0, True), (1, True)])
def test_limits(Hq, dense):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    N, b = 1024, 64
    nb, Hq = N // b, min((2 if dense else 1) * n_cu // 8 + Hq, 128)
    print(f"case split items limits heads={Hq} dense={dense}", flush=True)
    Q, K, V = gen.random_qkv(Hq, 1, N, 128, seed=Hq)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    more = dict(local_blocks=nb, k_blocks=nb * (nb + 1) // 2) if dense else dict()
    ses = sa.Session(Hq, 1, N, b, 64, keep=0.4, **more)
    ses.estimate(Qd, Kd)
    ses.build_index([sa.SA_TRIANGULAR] * Hq if dense else None)
    O = torch.empty_like(Qd)
    ses.prefill(Qd, Kd, Vd, O)
    torch.cuda.synchronize()
    index = orc.Index(*[t.cpu().numpy() for t in ses.index_tensors()])
    check_attention(host_f64(O), orc.masked_rows(Q, K, V, b, index)[0], f"limits {Hq}")
