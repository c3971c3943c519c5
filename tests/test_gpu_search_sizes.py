"""Refined sizes and pair counts of the offline search around the length up to which one workgroup ranks a head's
columns and diagonals (8192), at lengths that are no power of two, with scores that tie: whole numbers, equal to the
oracle's bisection over its own indexes."""
import numpy as np
import pytest
import torch

import paper_2412_06198_amd as sa
from harness import gen
from oracle import oracle as orc
from oracle import search as srch
from gpu_util import dev_bf16, upload_scores

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,b", [(64, 64), (128, 128), (1088, 64), (4096, 128), (5056, 64), (8128, 64), (8192, 64),
                                 (8192, 128), (8256, 64), (12416, 128)])
def test_sizes_and_pairs(N, b):
    print(f"case search sizes N={N} b={b}", flush=True)
    H, w, nb = 3, 64, N // b
    rng = np.random.default_rng(N + b)
    v, s = np.exp(rng.normal(-7, 2, (2, H, N))).astype(np.float32)
    v[1], s[1] = rng.integers(0, 4, (2, N)) * np.float32(2.0 ** -11)     # ties, zeros among them
    v[2], s[2] = 0, np.float32(2.0 ** -10)                              # nothing but ties
    blk = np.tril(np.exp(rng.normal(-7, 2, (H, nb, nb)))).astype(np.float32)
    ses = sa.Session(H, 1, N, b, w, keep=0.3)
    upload_scores(ses, v, s, blk)
    Q, K, V = (dev_bf16(x) for x in gen.random_qkv(H, 1, N, 128, seed=N))
    lo, hi = srch.candidate_range(orc.INTERVAL_SLASH, N, b)
    seen = [{} for _ in range(H)]

    def pairs(h, x):
        if x not in seen[h]:
            bud = srch.candidate_budgets(orc.INTERVAL_SLASH, x, N, b, ses.cfg.sink_blocks)
            ix = orc.build_index(v[h:h + 1], s[h:h + 1], blk[h:h + 1], N, b, w, bud, override=[orc.INTERVAL_SLASH])
            seen[h][x] = orc.mask_count(N, b, 0, ix)
        return seen[h][x]

    for frac, eps in ((0.0, 0), (0.03, 0), (0.2, N), (0.5, 0), (0.8, 5), (1.0, 0)):
        target = int(frac * N * (N + 1) / 2)
        for h, got in enumerate(ses.search_patterns(Q, K, V, target, eps)):
            want = srch.refine(lambda x: pairs(h, x), lo, hi, target, eps)
            assert (got["param"][1], got["pairs"][1]) == want, (frac, eps, h, got, want)
