"""The bf16 decode at the edges of how it merges and folds: query heads per KV head around the 4, 8 and 16 that its threads are dealt by
(17 and 40: several head groups), splits around the 4, 8 and 16 partials of a chunk of the fold, r around the blocks of R_r, sequences that fill
all, some or none of their splits.  Against the oracle; the folded merge repeats its bits, an empty sequence gives zeros."""
import numpy as np
import pytest
import torch

import paper_2605_19218_amd as rk

from gpu_util import Pipeline, to_dev, to_host
from test_gpu_f32 import launches
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


# Whether the merge rides in the split launch: as many rounds on every XCD as on the device (also by many bytes more: 4 x 12000, 44 x 8000), a
# second round on some of them, and a second one of short splits.  Both forms against the plain kernels.
@pytest.mark.parametrize("units,L,splits,kernels", [
    (8, 12000, 0, 1), (4, 12000, 0, 1), (44, 8000, 0, 1), (12, 6000, 0, 1), (258, 600, 0, 1), (84, 700, 0, 1),
    (12, 12000, 0, 2), (28, 6000, 0, 2), (7, 24000, 0, 2), (84, 2000, 0, 2), (9, 2200, 17, 1), (9, 6600, 17, 2),
])
def test_where_the_merge_rides_along(ctx, units, L, splits, kernels):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the table is for 256 compute units")
    r, cap = 32, (L + 31) // 32 * 32
    lens = torch.full((units,), L, device="cuda", dtype=torch.int32)
    lay = rk.Layout(units, 1, 1, r, rk.RK_BF16, cap, L, seq_len=lens)
    kb, vb = rk.rk_cache_bytes(lay)
    g = torch.Generator("cuda").manual_seed(1)
    K, V = (torch.randn(n // 2, device="cuda", generator=g).bfloat16() for n in (kb, vb))
    q, Rr = torch.randn(units, 1, 128, device="cuda", generator=g).bfloat16(), torch.randn(units, 1, 128, r, device="cuda", generator=g) / 11.3
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        ws = torch.empty(rk.rk_decode_workspace_size(ctx, lay), device="cuda", dtype=torch.uint8)
        outs = []
        for fuse, plain in ((1, 0), (0, 0), (0, 1)):
            rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, fuse)
            rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, plain)
            out = torch.full((units, 1, 128), float("nan"), device="cuda", dtype=torch.bfloat16)
            n = launches(lambda s: rk.rk_decode_attn(ctx, lay, q, K, V, Rr, None, 0.0, out, ws, stream=s))
            assert plain or n == (kernels if fuse else 2)
            rk.rk_decode_attn(ctx, lay, q, K, V, Rr, None, 0.0, out, ws)
            outs.append(out.float())
        for got in outs[:2]:                                  # bf16 roundings of one result
            assert float((got - outs[2]).abs().max()) <= 2.0 ** -7 * float(outs[2].abs().max())
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, 0)
        rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, 1)
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)
