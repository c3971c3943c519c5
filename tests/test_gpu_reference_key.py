"""The weights of a row are rounded to bf16 relative to a reference, the largest score of the first key tile (64 keys) that
the row meets: where its largest score is in that tile, wherever inside, that key's weight is 1 and not rounded."""
import numpy as np
import pytest
import torch

from harness import gen
from helpers import f64
from oracle import oracle as orc
from gpu_util import dev_bf16, host_f64, make_session, upload_index

pytestmark = pytest.mark.gpu


# 2 heads: two groups of waves share an item; 64 heads of five items: more items than compute units
@pytest.mark.parametrize("H", [2, 64])
@pytest.mark.parametrize("at", [8, 40])  # the place of the largest key in the tile
def test_largest_key_of_the_first_tile(H, at):
    print(f"case largest key at {at}, heads {H}", flush=True)
    N, b = 576, 64
    nb = N // b
    rng = np.random.default_rng(at)
    q, k, v = (rng.standard_normal((n, N, 128)).astype(np.float32) for n in (H, 1, 1))
    k[..., 96:] = q[..., 96:] = 0
    v[:] = -1
    big = np.arange(at, N, b)  # one key in each block: as much weight as all the others of its block together, and V = 1
    k[:, big, :96] = 0
    k[:, big, 100] = 8
    v[:, big] = 1
    R = np.arange(N) // b
    mask = (R[:, None] == R[None]) & np.tri(N, dtype=bool)
    others = mask.copy()
    others[:, big] = False
    K, V, kd = gen.f32_to_bf16_bits(k), gen.f32_to_bf16_bits(v), f64(gen.f32_to_bf16_bits(k)).numpy()
    s = f64(gen.f32_to_bf16_bits(q)).numpy() @ kd[0].T / np.sqrt(128.0)
    q[..., 100] = np.log(np.where(others[None], np.exp(s), 0).sum(-1) + 1e-9) * np.sqrt(128.0) / 8
    Q = gen.f32_to_bf16_bits(q)
    s = np.where(mask[None], f64(Q).numpy() @ kd[0].T / np.sqrt(128.0), -np.inf)
    p = np.exp(s - s.max(-1, keepdims=True))
    want = ((p / p.sum(-1, keepdims=True)) @ f64(V).numpy()[0])[..., 0]
    blocks = np.pad(np.arange(nb, dtype=np.int32), (0, nb * (nb + 1) // 2 - nb), constant_values=-1)
    index = orc.Index(np.full(H, 1, np.int32), np.zeros(H, np.int32), np.zeros((H, 1), np.int32), np.zeros(H, np.int32),
                      np.zeros((H, 1), np.int32), np.tile(np.arange(nb + 1, dtype=np.int32), (H, 1)), np.tile(blocks, (H, 1)))
    ses = make_session(H, 1, N, b, 64, orc.Budgets(1, 1, 1, 1, nb * (nb + 1) // 2))
    upload_index(ses, index)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    O = torch.full_like(Qd, 7.0)
    ses.prefill(Qd, Kd, Vd, O)
    torch.cuda.synchronize()
    rows = np.arange(N) % b >= 48
    assert (s[:, rows].argmax(-1) == big[R[rows]]).all() and np.abs(want[:, rows]).max() < 0.05
    err = (host_f64(O)[..., 0] - want)[:, rows]
    # An output is 2 w - 1 with w = 1/2, so it moves by half of what the ratio of the two halves moves.  A rounding to bf16 is
    # 2^-8 at most and 0.4 of that in the mean square: 1.6e-3 on the largest key's weight would be 8e-4 on the output.  The
    # 48 and more others' weights are worth some 25 equal ones, whose errors average to 1.6e-3 / sqrt(25), 1.6e-4 on the output.
    assert np.sqrt((err ** 2).mean()) < 4e-4, float(np.sqrt((err ** 2).mean()))
