"""Selected diagonals in batches: offset counts around the batch of 28 and the 64 that a wave looks at together, with
offsets that no query takes (keys in kept blocks, keys that are selected columns, diagonals below the row block) in
between, at the first row blocks, where most offsets reach before the sequence."""
import numpy as np
import pytest
import torch

from harness import gen
from oracle import oracle as orc
from gpu_util import check_attention, dev_bf16, host_f64, make_session, upload_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_offs", [1, 2, 27, 28, 29, 56, 57, 63, 64, 65, 130, 448])
def test_offset_counts(n_offs):
    print(f"case diagonals {n_offs}", flush=True)
    H, N, b = 2, 448, 64
    nb = N // b
    rng = np.random.default_rng(n_offs)
    k_v, cap = 96, nb * (nb + 1) // 2
    ix = dict(pattern=np.full(H, 1, np.int32), n_cols=np.zeros(H, np.int32), cols=np.full((H, k_v), -1, np.int32),
              n_offs=np.full(H, n_offs, np.int32), offs=np.full((H, n_offs), -1, np.int32),
              rowptr=np.zeros((H, nb + 1), np.int32), blkcols=np.full((H, cap), -1, np.int32))
    for h in range(H):
        # head 0: runs of columns, so that whole stretches of a diagonal are columns; head 1: none
        nc = k_v if h == 0 else 0
        start = rng.integers(0, N - k_v)
        ix["n_cols"][h] = nc
        ix["cols"][h, :nc] = start + np.arange(nc)
        ix["offs"][h] = np.sort(rng.choice(N, n_offs, replace=False))
        at = 0
        for R in range(nb):  # the diagonal block of most rows and one or two others
            keep = np.unique(np.concatenate([rng.integers(0, R + 1, 2), [R] if R % 3 else []])).astype(np.int32)
            ix["rowptr"][h, R] = at
            ix["blkcols"][h, at:at + len(keep)] = keep
            at += len(keep)
        ix["rowptr"][h, nb] = at
    index = orc.Index(**ix)
    ses = make_session(H, 1, N, b, 64, orc.Budgets(1, 1, k_v, n_offs, cap))
    upload_index(ses, index)
    Q, K, V = gen.random_qkv(H, 1, N, 128, seed=n_offs)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    O = torch.full_like(Qd, 7.0)
    ses.prefill(Qd, Kd, Vd, O)
    torch.cuda.synchronize()
    # same tolerance as every attention check: bf16 weights and outputs against fp64
    check_attention(host_f64(O), orc.masked_rows(Q, K, V, b, index)[0], f"diagonals {n_offs}")
