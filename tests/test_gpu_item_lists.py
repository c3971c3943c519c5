"""The work items and key-tile lists that are laid out before the attention kernel starts: groups of
more than 64 query heads (two words of the kind mask), sequences whose tile count leaves a remainder in
the bitmap words, row blocks that end in the middle, rows without any block."""
import numpy as np
import pytest
import torch

from harness import gen
from oracle import oracle as orc
from gpu_util import check_attention, dev_bf16, host_f64, make_session, random_index, upload_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,N,b", [(70, 1, 576, 64), (128, 1, 256, 128), (66, 2, 320, 64),
                                        (3, 1, 2112, 64), (2, 2, 4160, 64), (4, 2, 4224, 128)])
def test_items_and_tile_lists(Hq, Hkv, N, b):
    print(f"case items Hq={Hq} Hkv={Hkv} N={N} b={b}", flush=True)
    nb = N // b
    rng = np.random.default_rng(N + Hq)
    k_v, k_s, cap = 70, 5, nb * (nb + 1) // 2 + nb
    ix = random_index(rng, Hq, N, b, k_v, k_s, cap)
    ses = make_session(Hq, Hkv, N, b, min(64, N), orc.Budgets(1, 1, k_v, k_s, cap))
    upload_index(ses, ix)
    Q, K, V = gen.random_qkv(Hq, Hkv, N, 128, seed=N)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    O = torch.full_like(Qd, 7.0)
    ses.prefill(Qd, Kd, Vd, O)
    torch.cuda.synchronize()
    # same tolerance as every attention check: bf16 weights and outputs against fp64
    check_attention(host_f64(O), orc.masked_rows(Q, K, V, b, ix)[0], f"items {Hq}/{Hkv} {N} {b}")
