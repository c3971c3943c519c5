"""The decode step's split of a head's key list over workgroups, its merge by the workgroup that arrives last,
and the arrival counters in memory that may hold anything, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2412_06198_amd as sa
from harness import gen
from oracle import decode as dec
from gpu_util import dev_bf16, host_f64, random_index, upload_index

pytestmark = pytest.mark.gpu


# one workgroup per head (63 and 64 keys), two (65), a wave with nothing to do, many keys that count
# twice, the most workgroups per head (one head) and the fewest (128 heads)
@pytest.mark.parametrize("Hq,Hkv,N,b,k_v,extra", [(2, 1, 64, 64, 1, 63), (2, 2, 64, 64, 1, 64), (3, 1, 64, 64, 1, 65),
                                                  (4, 2, 512, 128, 500, 17), (1, 1, 4096, 64, 4096, 3),
                                                  (128, 8, 1024, 64, 300, 130)])
def test_decode_splits_and_dirty_counters(Hq, Hkv, N, b, k_v, extra):
    print(f"case decode splits Hq={Hq} Hkv={Hkv} N={N} b={b} k_v={k_v} extra={extra}", flush=True)
    rng = np.random.default_rng(N + extra)
    nb = N // b
    Q, K, V = gen.random_qkv(Hq, Hkv, N + extra, 128, seed=extra)
    ses = sa.Session(Hq, Hkv, N, b, min(64, N), sink_blocks=1, local_blocks=1, k_vertical=k_v, k_slash=8,
                     k_blocks=nb * (nb + 1) // 2 + nb, kv_head_stride=(N + extra) * 128)
    ix = random_index(rng, Hq, N, b, k_v, 8, ses.cap_b)
    if nb == 1:  # generated keys alone: the number of keys is extra
        ix.n_cols[:], ix.n_offs[:], ix.rowptr[:] = 0, 0, 0
    else:
        ix.n_cols[:] = k_v
        ix.cols[:] = np.sort(np.stack([rng.permutation(N)[:k_v] for _ in range(Hq)]), axis=1)
    upload_index(ses, ix)
    Kd, Vd = dev_bf16(K), dev_bf16(V)
    pos = N + extra - 1
    q = dev_bf16(Q[:, pos])
    ref, cnt = dec.decode_step(Q[:, pos], K, V, b, ix, N, pos)
    o = torch.empty_like(q)
    first = None
    for dirt in (0, 1, 0xFF, 0x3F, None, None):  # None: what the step before left
        if dirt is not None:
            ses.ws.fill_(dirt)
        o.fill_(7.0)
        ses.decode(q, Kd, Vd, pos, o)
        err = np.abs(host_f64(o) - ref)
        assert err.max() <= 2e-2 and err.mean() <= 2e-3, (dirt, float(err.max()))
        first = o.clone() if first is None else first
        assert torch.equal(o, first)
    for _ in range(3):
        o.fill_(7.0)
        ses.decode_static(q, Kd, Vd, pos, o)
        assert torch.equal(o, first)


def test_decode_graph_replays():
    # a recorded step leaves the counters as it found them: other lists, eager steps in between
    print("case decode graph", flush=True)
    Hq, Hkv, N, b, extra = 8, 2, 2048, 64, 40
    Q, K, V = gen.random_qkv(Hq, Hkv, N + extra, 128, seed=3)
    ses = sa.Session(Hq, Hkv, N, b, 64, sink_blocks=1, local_blocks=1, k_vertical=400, k_slash=24,
                     k_blocks=1000, kv_head_stride=(N + extra) * 128)
    lists = [random_index(np.random.default_rng(s), Hq, N, b, 400, 24, ses.cap_b) for s in range(3)]
    Kd, Vd, pos = dev_bf16(K), dev_bf16(V), N + extra - 1
    q = dev_bf16(Q[:, pos])
    o = torch.empty_like(q)
    want = []
    for ix in lists:
        upload_index(ses, ix)
        ses.decode(q, Kd, Vd, pos, o)
        want.append(o.clone())
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        for _ in range(3):
            ses.decode(q, Kd, Vd, pos, o)
    for rep in range(2):
        for ix, w in zip(lists, want):
            upload_index(ses, ix)
            o.fill_(7.0)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(o, w)
            o.fill_(7.0)
            ses.decode(q, Kd, Vd, pos, o)
            torch.cuda.synchronize()
            assert torch.equal(o, w)
