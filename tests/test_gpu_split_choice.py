"""Between one and two items per compute unit under a band that covers the sequence, the budgets say whether two groups of
waves share an item: with few columns they must not (the outputs are then those of a context without such a band,
bit by bit); either way against the oracle."""
import pytest
import torch

import paper_2412_06198_amd as sa
from harness import gen
from oracle import oracle as orc
from gpu_util import check_attention, dev_bf16, host_f64

pytestmark = pytest.mark.gpu


# (heads, keep: 1.0 = what the library takes for it, patterns, whether the items stay whole); None: the run-time rule
@pytest.mark.parametrize("H,keep,pattern,whole", [(40, 0.1, [1], True), (64, 0.1, None, True), (33, 0.6, [1, 0, 2], True),
                                                  (40, 1.0, [0], False), (64, 1.0, None, False), (33, 1.0, [1, 0, 2], False)])
@pytest.mark.parametrize("N,b", [(1024, 64), (960, 64), (1024, 128)])
def test_choice(H, keep, pattern, whole, N, b):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    nb, items = N // b, -(-N // 128) * H
    if not n_cu < items <= 2 * n_cu:
        pytest.skip("not between one and two items per compute unit")
    print(f"case split choice heads={H} keep={keep} pattern={pattern} b={b} N={N}", flush=True)
    Q, K, V = gen.random_qkv(H, 1, N, 128, seed=H)
    Qd, Kd, Vd = dev_bf16(Q), dev_bf16(K), dev_bf16(V)
    full = nb * (nb + 1) // 2
    ses = [sa.Session(H, 1, N, b, 64, keep=keep, local_blocks=local, k_blocks=full) for local in (nb, nb - 1)]
    ses[0].estimate(Qd, Kd)
    ses[0].build_index(None if pattern is None else [pattern[h % len(pattern)] for h in range(H)])
    index = orc.Index(*[t.cpu().numpy() for t in ses[0].index_tensors()])
    for t, u in zip(ses[1].index_tensors(), ses[0].index_tensors()):
        t.copy_(u)
    O = [torch.full_like(Qd, 7.0) for _ in range(3)]
    for s, o in zip(ses, O):
        for _ in range(2):  # the second call meets what the first left in the workspace
            s.prefill(Qd, Kd, Vd, o)
    _, kept = ses[0].prefill_counted(Qd, Kd, Vd, O[2])
    torch.cuda.synchronize()
    assert torch.equal(O[0], O[2])
    assert kept == sum(orc.mask_count(N, b, h, index) for h in range(H))
    assert torch.equal(O[0], O[1]) == whole
    check_attention(host_f64(O[0]), orc.masked_rows(Q, K, V, b, index)[0], f"choice {H}")
