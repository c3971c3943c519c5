"""How many workgroups a decode step launches follows the budgets, the keys follow the index: lists at the length up to
which one workgroup per compute unit is launched and one key beyond, and lists far longer than the budgets suggest,
against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2412_06198_amd as sa
from harness import gen
from oracle import decode as dec
from gpu_util import dev_bf16, host_f64, random_index, upload_index

pytestmark = pytest.mark.gpu


# 8 heads: 32 workgroups each cover 2048 keys, here 512 columns, 2 diagonals, a block and the generated keys; 64 heads: 4,
# 256 keys; 128 heads of 64 keys: few to one; every block of the last row kept, with budgets that expect 5 or 9 of them
@pytest.mark.parametrize("Hq,Hkv,N,b,k_v,own,every", [(8, 2, 1024, 64, 512, 1470, False), (8, 2, 1024, 64, 512, 1471, False),
                                                      (64, 8, 256, 64, 100, 90, False), (64, 8, 256, 64, 100, 91, False),
                                                      (128, 8, 128, 64, 1, 1, False), (8, 2, 4096, 64, 64, 1, True),
                                                      (24, 3, 2048, 128, 64, 3, True), (1, 1, 4096, 64, 64, 1, True)])
def test_lists_at_the_edges_and_beyond(Hq, Hkv, N, b, k_v, own, every):
    print(f"case decode grid Hq={Hq} N={N} b={b} k_v={k_v} own={own} every block {every}", flush=True)
    rng = np.random.default_rng(N + own)
    nb = N // b
    Q, K, V = gen.random_qkv(Hq, Hkv, N + own, 128, seed=own + Hq)
    ses = sa.Session(Hq, Hkv, N, b, min(64, N), sink_blocks=1, local_blocks=1, k_vertical=k_v, k_slash=2, k_blocks=nb,
                     kv_head_stride=(N + own) * 128)
    ix = random_index(rng, Hq, N, b, k_v, 2, max(ses.cap_b, nb * (nb + 1)))
    ix.blkcols = np.full((Hq, ses.cap_b), -1, np.int32)
    ix.rowptr[:] = 0
    kept = np.arange(nb) if every else np.array([nb - 1])
    ix.rowptr[:, nb] = len(kept)
    ix.blkcols[:, :len(kept)] = kept
    if not every:
        ix.n_cols[:] = k_v
        ix.cols[:] = np.sort(np.stack([rng.permutation(N)[:k_v] for _ in range(Hq)]), axis=1)
    upload_index(ses, ix)
    Kd, Vd = dev_bf16(K), dev_bf16(V)
    pos = N + own - 1
    q = dev_bf16(Q[:, pos])
    ref, _ = dec.decode_step(Q[:, pos], K, V, b, ix, N, pos)
    for step in (ses.decode, ses.decode, ses.decode_static):
        o = torch.full_like(q, 7.0)
        step(q, Kd, Vd, pos, o)
        err = np.abs(host_f64(o) - ref)
        assert err.max() <= 2e-2 and err.mean() <= 2e-3, float(err.max())
