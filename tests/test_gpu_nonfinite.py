"""NaN and infinities in K, NaN in Q: a query whose softmax takes one in must show it, whatever part of the index keeps the key
(a block, a column, a diagonal), and no other query may; against a softmax in fp64."""
import numpy as np
import pytest
import torch

from harness import gen
from helpers import f64, numpy_mask
from oracle import oracle as orc
from gpu_util import check_attention, dev_bf16, host_f64, make_session, upload_index

pytestmark = pytest.mark.gpu


# few heads: two groups of waves share an item; 72 heads of four row blocks: more items than compute units
@pytest.mark.parametrize("H", [2, 72])
@pytest.mark.parametrize("value", ["nan", "inf"])
@pytest.mark.parametrize("by", ["diagonal", "block", "column"])
def test_key_rows(H, value, by):
    print(f"case non-finite keys {by} {value} heads {H}", flush=True)
    N, b, key = 448, 64, 70
    nb = N // b
    cols = [5, key, 200] if by == "column" else [5, 200]
    # beside its own block, queries 130, 170 and 381 keep the key through offsets 60, 100 and 311
    offs = [60, 100, 311] if by == "diagonal" else [33, 100]
    blocks = [sorted({R} | ({1} if by == "block" and R in (3, 6) else set())) for R in range(nb)]
    blk = np.concatenate(blocks).astype(np.int32)
    index = orc.Index(np.full(H, 1, np.int32), np.full(H, len(cols), np.int32), np.tile(np.array(cols, np.int32), (H, 1)),
                      np.full(H, len(offs), np.int32), np.tile(np.array(offs, np.int32), (H, 1)),
                      np.tile(np.concatenate([[0], np.cumsum([len(r) for r in blocks])]).astype(np.int32), (H, 1)),
                      np.tile(np.pad(blk, (0, nb * (nb + 1) // 2 - len(blk)), constant_values=-1), (H, 1)))
    Q, K, V = gen.random_qkv(H, 1, N, 128, seed=3)
    K[0, key, 17] = 0x7FC0 if value == "nan" else 0x7F80
    ses = make_session(H, 1, N, b, 64, orc.Budgets(1, 1, len(cols), len(offs), nb * (nb + 1) // 2))
    upload_index(ses, index)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    O = torch.full_like(Qd, 7.0)
    ses.prefill(Qd, Kd, Vd, O)
    torch.cuda.synchronize()
    q, k, v = (f64(x).numpy() for x in (Q, K, V))
    mask = numpy_mask(N, b, index, 0)
    with np.errstate(invalid="ignore"):
        s = np.where(mask[None], q @ k[0].T / np.sqrt(128.0), -np.inf)
        p = np.exp(s - s.max(-1, keepdims=True))
        want = (p / p.sum(-1, keepdims=True)) @ v[0]
    bad = np.isnan(want)
    # a NaN reaches every query that keeps the key, an infinity those whose score it makes +inf
    takes = np.tile(mask[:, key], (H, 1)) & ((q[:, :, 17] > 0) | (value == "nan"))
    assert (bad == takes[..., None]).all() and takes.any()
    got = host_f64(O)
    assert (np.isnan(got) == bad).all()
    check_attention(got[~takes], want[~takes], f"{by} {value}")


@pytest.mark.parametrize("H", [2, 72])
@pytest.mark.parametrize("N", [448, 64])
def test_query_rows(H, N):
    # a query with a NaN, one that keeps keys through its block, columns and diagonals and one in the first block
    print(f"case non-finite queries heads {H} N={N}", flush=True)
    b, row = 64, N - 3
    nb = N // b
    blk = np.arange(nb, dtype=np.int32)
    index = orc.Index(np.full(H, 1, np.int32), np.full(H, 2, np.int32), np.tile(np.array([5, 50], np.int32), (H, 1)),
                      np.full(H, 2, np.int32), np.tile(np.array([0, 60], np.int32), (H, 1)), np.tile(np.arange(nb + 1, dtype=np.int32), (H, 1)),
                      np.tile(np.pad(blk, (0, nb * (nb + 1) // 2 - nb), constant_values=-1), (H, 1)))
    Q, K, V = gen.random_qkv(H, 1, N, 128, seed=4)
    clean = orc.masked_rows(Q, K, V, b, index)[0]
    Q[H - 1, [9, row], 100] = 0x7FC0
    ses = make_session(H, 1, N, b, 64, orc.Budgets(1, 1, 2, 2, nb * (nb + 1) // 2))
    upload_index(ses, index)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    O = torch.full_like(Qd, 7.0)
    ses.prefill(Qd, Kd, Vd, O)
    torch.cuda.synchronize()
    bad = np.zeros((H, N), bool)
    bad[H - 1, [9, row]] = True
    got = host_f64(O)
    assert (np.isnan(got) == bad[..., None]).all()
    check_attention(got[~bad], clean[~bad], f"queries {N}")
