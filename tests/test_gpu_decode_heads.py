"""The bf16 decode at the edges of how it merges and folds: query heads per KV head around the 4, 8 and 16 that its threads are dealt by
(17 and 40: several head groups), splits around the 4, 8 and 16 partials of a chunk of the fold, r around the blocks of R_r, sequences that fill
all, some or none of their splits.  Against the oracle; the folded merge repeats its bits, an empty sequence gives zeros."""
import numpy as np
import pytest
import torch

import paper_2605_19218_amd as rk

from gpu_util import Pipeline, to_dev, to_host
from test_gpu_parity import check_out, layer, oracle_decode, run_prefill

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = rk.rk_create(0)
    yield c
    rk.rk_destroy(c)


@pytest.mark.parametrize("G,splits,r", [
    (1, 4, 16), (2, 5, 37), (4, 8, 64), (5, 9, 17), (8, 16, 80), (9, 17, 128), (12, 1, 48), (15, 3, 112), (16, 2, 96), (17, 6, 1), (40, 4, 33),
])
def test_heads_and_splits(ctx, G, splits, r):
    Hkv, L = 3, 2200
    lengths = [L, 900, 0, 1]
    B = len(lengths)
    data = layer(B, G * Hkv, Hkv, L, "bf16", 90 + G, lengths=lengths, mean_shift=1.5)
    p = run_prefill(ctx, data, B, G * Hkv, Hkv, L, r, "bf16", lengths=lengths)
    q = to_dev(data["q"], "bf16")
    results = []
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        for fuse in (1, 1, 0):
            rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, fuse)
            p.out.fill_(float("nan"))
            results.append(p.decode(q))
        want = oracle_decode(p, data["q"], lengths)
        for got in results:
            check_out(got, want, "bf16")
            assert not got[2].any()
        assert np.array_equal(results[0], results[1])
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, 1)
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)
