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


def coarse_size(dtype, B, Hq, Hkv, L):
    """What the plan without the finer splits asks for."""
    rows, units, tiles = B * Hq, B * Hkv * -(-(Hq // Hkv) // 16), max(1, -(-L // 128))
    if dtype == rk.RK_BF16:
        return scratch(rows, coarse(units, tiles, 4) + 8)
    slots, S = coarse(rows, tiles, 4) + 8, coarse(units, tiles, 2)
    while S > slots and scratch(rows, S) > rk.RK_STATIC_SCRATCH_BYTES:
        S -= 1
    return scratch(rows, max(slots, S))


@pytest.mark.parametrize("dtype", [rk.RK_F32, rk.RK_BF16])
def test_a_workspace_serves_what_the_coarse_plan_lets_it(dtype):
    """A program that sizes its workspace once, for some length, batch and heads, may come with others: a call is refused for its workspace only
    where the coarse plan, whose size hardly moves on short caches, refuses it too."""
    ctx, P, shapes = rk.rk_create(rk.RK_DEVICE_NONE), 4096, []

    def layout(B, Hq, Hkv, L):
        return rk.Layout(B, Hq, Hkv, 64, dtype, (L + 63) // 32 * 32, L, seq_len=P)

    def refused(size, *shape):
        statuses = []
        for call in (lambda: rk.rk_decode_attn(ctx, layout(*shape), P, P, P, P, P, 0.0, P, P, workspace_bytes=size),
                     lambda: rk.rk_append_decode_attn(ctx, layout(*shape[:3], shape[3] - 1), P, P, P, P, P, P, P, P, 0.0, P, P, workspace_bytes=size)):
            with pytest.raises(rk.RotateKError) as e:
                call()
            statuses.append(e.value.status)
        assert statuses[0] == statuses[1] and statuses[0] in (rk.RK_ERR_NO_DEVICE, rk.RK_ERR_WORKSPACE)
        return statuses[0] == rk.RK_ERR_WORKSPACE

    try:
        size = rk.rk_decode_workspace_size(ctx, layout(1, 32, 8, 1000))
        assert not any(refused(size, 1, 32, 8, L) for L in (1025, 1030, 1200, 2000, 2400))
        for B in (1, 2, 3, 5, 8, 20, 21, 22, 40, 128, 300):
            for Hq, Hkv in ((1, 1), (8, 8), (32, 8), (28, 4), (64, 4), (40, 1)):
                for L in LENGTHS[1:]:
                    shapes.append((coarse_size(dtype, B, Hq, Hkv, L), rk.rk_decode_workspace_size(ctx, layout(B, Hq, Hkv, L)), (B, Hq, Hkv, L)))
        shapes.sort()
        most = 0                                        # of the sizes asked for so far: the coarse plan's grow along the list
        for few, size, shape in shapes:
            assert size >= most and few <= size <= max(few, min(4 * few, rk.RK_STATIC_SCRATCH_BYTES)), shape
            most = size
        for (few, size, a), (_, _, b) in zip(shapes[7::11], shapes[0::11]):
            assert not refused(size, *b), (a, b)
    finally:
        rk.rk_destroy(ctx)
