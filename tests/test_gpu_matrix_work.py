"""The counted variant's sub-tiles, and the matrix work the benchmark makes of them: diagonals alone, one per wave of 32 rows
and offset, and beside key tiles."""
import numpy as np
import pytest
import torch

import bench
from gpu_util import dev_bf16, make_session, upload_index
from harness import gen
from oracle import oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks", [False, True])
def test_diagonals_are_an_eighth(blocks):
    print(f"case matrix work of diagonals, blocks {blocks}", flush=True)
    N, b, H, offs = 320, 64, 2, [0, 31, 32, 130, 319]
    nb = N // b
    if blocks:
        offs = offs[2:]  # not inside the tiles that are kept, as a wave's rows are of one row block
        offs[0] = 64
    index = orc.Index(np.full(H, 1, np.int32), np.zeros(H, np.int32), np.zeros((H, 1), np.int32), np.full(H, len(offs), np.int32),
                      np.tile(np.array(offs, np.int32), (H, 1)), np.tile(np.arange(nb + 1, dtype=np.int32) * blocks, (H, 1)),
                      np.tile(np.pad(np.arange(nb, dtype=np.int32), (0, nb * (nb + 1) // 2 - nb), constant_values=-1), (H, 1)))
    ses = make_session(H, 1, N, b, 64, orc.Budgets(1, 1, 1, len(offs), nb * (nb + 1) // 2))
    upload_index(ses, index)
    Q, K, V = (dev_bf16(x) for x in gen.random_qkv(H, 1, N, 128, seed=1))
    O = torch.empty_like(Q)
    tiles, _ = ses.prefill_counted(Q, K, V, O)
    ses.n_offs.zero_()
    key_tiles, _ = ses.prefill_counted(Q, K, V, O)
    diagonals = H * sum(r0 + 31 >= o for r0 in range(0, N, 32) for o in offs)
    assert key_tiles == H * blocks * (N // 32) * 2 and tiles - key_tiles == diagonals
    # a diagonal is 16 products for its scores and 16 for V of 16 blocks of 4 x 4 x 4
    assert bench.matrix_flop(tiles, diagonals, 128) == key_tiles * 4 * 128 * 32 * 32 + diagonals * 32 * (16 * 2 * 4 * 4 * 4)


def test_the_benchmark_counts_so():
    print("case matrix work of the benchmark", flush=True)
    name = "cfg1"
    wl = gen.WORKLOADS[name]
    got = bench.run_workload(name, 1, 1, 1, False, 0, prewarm_s=0, force_pattern=1)
    diagonals = got["attention_phases"]["diagonals"]["bytes"] / (32 * 2 * wl.head_dim * 2)
    assert diagonals > 0
    assert got["flop"]["tiles"] == got["attention_phases"]["tile_loop"]["flop_on_tiles"] + diagonals * 4 * wl.head_dim * 32 * 32 / 8
