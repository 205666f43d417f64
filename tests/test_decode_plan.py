"""The split count of a decode and the workspace that it asks for, on the host: a workspace for one max_seq_len serves every shorter one, no shape
leaves the built-in scratch for the finer splits of idle compute units, and a plan is never coarser than one split of 512 tokens (256 in fp32)
or a quarter of a short cache per compute unit."""
import pytest

import paper_2605_19218_amd as rk

LENGTHS = [0, 1, 100, 128, 129, 257, 385, 500, 513, 700, 1025, 1500, 2000, 2049, 2944, 4000, 5000, 6000, 9000, 12000, 16384, 33000, 66000]


def coarse(units, tiles, per, n_cu=256):
    """The plan without the finer splits: one work-group a compute unit, `per` tiles a split (or four splits of a short cache)."""
    S = n_cu // units
    if S < 1:
        S, best = 1, 1e30
        for c in range(1, 5):
            cost = -(-units * c // n_cu) / c
            if cost < best - 1e-9:
                S, best = c, cost
    return max(1, min(S, 64, max(tiles // per, min(tiles // 2, 4)), tiles))


def scratch(rows, slots):
    return -(-rows * (slots * 130 + 1) * 4 // 256) * 256


@pytest.mark.parametrize("dtype", [rk.RK_F32, rk.RK_BF16])
def test_plan_and_workspace(dtype):
    ctx = rk.rk_create(rk.RK_DEVICE_NONE)
    finer = 0
    try:
        for B in (1, 2, 3, 7, 12, 20, 26, 28, 40, 64, 128, 129, 300):
            for Hq, Hkv in ((1, 1), (8, 8), (32, 32), (32, 8), (28, 4), (64, 4), (16, 1), (40, 1), (112, 7)):
                before, units = 0, B * Hkv * -(-(Hq // Hkv) // 16)
                for L in LENGTHS:
                    lay = rk.Layout(B, Hq, Hkv, 64, dtype, (L + 63) // 32 * 32, L, seq_len=1 << 20)
                    size, (S, per) = rk.rk_decode_workspace_size(ctx, lay), rk.rk_decode_plan(ctx, lay)
                    tiles = max(1, -(-L // 128))
                    least = coarse(units, tiles, 4 if dtype == rk.RK_BF16 else 2)
                    assert size >= before and size >= scratch(B * Hq, S)
                    assert 1 <= S <= tiles and per * S >= L and per == 128 * -(-tiles // S)
                    if dtype == rk.RK_BF16:
                        assert least <= S <= max(least, min(256 // units, 64)) and size >= scratch(B * Hq, S + 8)
                        if scratch(B * Hq, least + 8) <= rk.RK_STATIC_SCRATCH_BYTES:
                            assert size <= rk.RK_STATIC_SCRATCH_BYTES
                    finer += S > least
                    before = size
        assert finer > 100
    finally:
        rk.rk_destroy(ctx)
