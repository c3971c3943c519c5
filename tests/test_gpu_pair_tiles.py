"""Key tiles that one of an item's two row blocks keeps alone (64-row blocks): as many for either block, more for one of
them, none for one, a last row block without a partner; with selected columns and diagonals inside such tiles.  Against
the oracle, with items whole (many heads) and shared by two groups of waves (few)."""
import numpy as np
import pytest
import torch

from harness import gen
from oracle import oracle as orc
from gpu_util import check_attention, dev_bf16, host_f64, make_session, random_index, upload_index

pytestmark = pytest.mark.gpu


def _kept(rng, kind, R):
    """The key blocks of row block R: those of an item's two row blocks are chosen without overlap, by parity."""
    mine = np.arange(R % 2, R + 1, 2)  # even key blocks for the upper row block, odd ones for the lower
    if kind == 0:
        return mine
    if kind == 1:  # more for the upper row block, with some that both keep
        return mine if R % 2 == 0 else np.union1d(mine[:1], rng.choice(R + 1, (R + 1) // 4, replace=False))
    if kind == 2:  # more for the lower
        return mine if R % 2 else mine[-1:]
    if kind == 3:  # none for the upper
        return mine if R % 2 else mine[:0]
    if kind == 4:  # none for the lower
        return mine[:0] if R % 2 else mine
    return np.sort(rng.choice(R + 1, rng.integers(0, R + 2), replace=False))


# items of 128 rows: 64 heads and 12 heads of 4224 tokens have more than the 256 compute units and stay whole, the others are shared, down to
# lists of no, one or two tiles for a group; full: a quarter more of the keys as columns
@pytest.mark.parametrize("Hq,Hkv,N,full", [(64, 8, 576, 0), (64, 8, 640, 0), (64, 8, 576, 1), (6, 2, 64, 1), (6, 2, 128, 0), (6, 2, 192, 0),
                                           (6, 2, 192, 1), (6, 2, 320, 0), (6, 2, 448, 1), (12, 4, 1344, 0), (12, 4, 4224, 0), (12, 4, 4224, 1)])
def test_tiles_of_one_row_block(Hq, Hkv, N, full):
    print(f"case tiles of one row block {Hq}/{Hkv} heads N={N} full {full}", flush=True)
    b, nb, k_v, k_s = 64, N // 64, min(N, 70 + full * N // 4), 5
    rng = np.random.default_rng(N + Hq)
    ses = make_session(Hq, Hkv, N, b, min(64, N), orc.Budgets(1, 1, k_v, k_s, nb * (nb + 1) // 2))
    cap = ses.index_tensors()[6].shape[1]
    index = random_index(rng, Hq, N, b, k_v, k_s, max(cap, nb * (nb + 1)))
    index.blkcols = np.full((Hq, cap), -1, np.int32)
    for h in range(Hq):
        if h % 4 == 0:
            index.n_cols[h] = 0
        if h % 4 < 2:
            index.n_offs[h] = 0
        rows = [_kept(rng, h % 6, R) for R in range(nb)]
        index.rowptr[h] = np.concatenate([[0], np.cumsum([len(r) for r in rows])])
        flat = np.concatenate(rows)
        index.blkcols[h, :len(flat)] = flat
    upload_index(ses, index)
    Q, K, V = gen.random_qkv(Hq, Hkv, N, 128, seed=N)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    O, counted = torch.full_like(Qd, 7.0), torch.full_like(Qd, 7.0)
    for _ in range(2):  # the second call meets what the first left in the workspace
        ses.prefill(Qd, Kd, Vd, O)
    _, kept = ses.prefill_counted(Qd, Kd, Vd, counted)
    torch.cuda.synchronize()
    check_attention(host_f64(O), orc.masked_rows(Q, K, V, b, index)[0], f"tiles of one row block {N}")
    assert torch.equal(O, counted)
    assert kept == sum(orc.mask_count(N, b, h, index) for h in range(Hq))
