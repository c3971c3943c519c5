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


def _decode_case(Hq, Hkv, N, b, extra, seed):
    Q, K, V = gen.random_qkv(Hq, Hkv, N + extra, 128, seed=seed)
    ses = sa.Session(Hq, Hkv, N, b, min(64, N), sink_blocks=1, local_blocks=1, k_vertical=200, k_slash=16,
                     k_blocks=(N // b) * (N // b + 3) // 2, kv_head_stride=(N + extra) * 128)
    ix = random_index(np.random.default_rng(seed), Hq, N, b, 200, 16, ses.cap_b)
    upload_index(ses, ix)
    return Q, K, V, ses, ix


def _add_to_words(ws, k):
    """Every 8-byte word of the workspace k higher: what a step that was cut short after k arrivals, or two steps
    that overlapped on it, can leave in an arrival counter, wherever the counters are."""
    off = (-ws.data_ptr()) % 8
    ws[off: off + (ws.numel() - off) // 8 * 8].view(torch.int64).add_(k)


@pytest.mark.parametrize("Hq,extra", [(4, 500), (1, 40)])
def test_decode_after_a_leftover_arrival_count(Hq, extra):
    # the next step gives the same bytes, eager and replayed, whatever count it finds
    print(f"case decode leftover count Hq={Hq} extra={extra}", flush=True)
    N = 1024
    Q, K, V, ses, _ = _decode_case(Hq, 1, N, 64, extra, seed=Hq + extra)
    Kd, Vd, pos = dev_bf16(K), dev_bf16(V), N + extra - 1
    q, q2 = dev_bf16(Q[:, pos]), dev_bf16(Q[:, 0])
    o, want = torch.empty_like(q), torch.empty_like(q)
    ses.ws.zero_()
    ses.decode(q, Kd, Vd, pos, want)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        ses.decode(q, Kd, Vd, pos, o)
    for k in list(range(1, 12)) + [63, 64, 255, 256, 65535, 65536, -1, -2]:
        for step in (lambda: ses.decode(q, Kd, Vd, pos, o), graph.replay):
            ses.decode(q2, Kd, Vd, pos, o)  # partials of another query, in case the step takes them for its own
            _add_to_words(ses.ws, k)
            step()
            torch.cuda.synchronize()
            assert torch.equal(o, want), k


@pytest.mark.parametrize("extra", [1, 15, 16, 33, 130, 700])
def test_decode_with_infinite_values(extra):
    # an infinite entry of V makes its own output infinite and nothing else NaN: in the last key of the list (the
    # query's own), in a key behind which a step has free places, and in a prompt key of any part of the list
    print(f"case decode infinite values extra={extra}", flush=True)
    N = 1024
    Q, K, V, ses, ix = _decode_case(3, 1, N, 64, extra, seed=extra)
    pos = N + extra - 1
    V = V.copy()
    V[0, pos, 5] = V[0, (N + pos) // 2, 70] = V[0, int(ix.cols[0, 0]) if ix.n_cols[0] > 0 else 3, 99] = 0x7F80
    q = dev_bf16(Q[:, pos])
    o = torch.empty_like(q)
    ses.decode(q, dev_bf16(K), dev_bf16(V), pos, o)
    with np.errstate(invalid="ignore"):
        ref, _ = dec.decode_step(Q[:, pos], K, V, 64, ix, N, pos)
    got, fin = host_f64(o), np.isfinite(ref)
    assert (got[~fin] == ref[~fin]).all() and (~fin).sum() >= 3
    err = np.abs(got[fin] - ref[fin])
    assert err.max() <= 2e-2 and err.mean() <= 2e-3, float(err.max())
