"""Values of rk_compress: lengths around the blocks of 32 tokens and the work-groups of 32 (fp32) and 128 (bf16), equal and on the device, and
a Value cache that lies over the Keys.  The layout holds copies: bit for bit, and zeros up to the end of the last block."""
import pytest
import torch

import paper_2605_19218_amd as rk

from gpu_util import DEV

pytestmark = pytest.mark.gpu


def run(dtype, B, Hkv, L, r, K, V, n_dev=None, over_keys=False):
    ctx = rk.rk_create(0)
    cap = (L + 63) // 64 * 64
    lay = rk.Layout(B, Hkv, Hkv, r, rk.RK_BF16 if dtype == "bf16" else rk.RK_F32, cap, L)
    Rr = torch.linalg.qr(torch.randn(B, Hkv, 128, r, generator=torch.Generator().manual_seed(1)))[0].to(DEV).contiguous()
    kb, vb = rk.rk_cache_bytes(lay)
    Kp = torch.zeros(kb, dtype=torch.uint8, device=DEV)
    Vc = K.view(-1).view(torch.uint8) if over_keys else torch.full((vb,), 0x3f, dtype=torch.uint8, device=DEV)
    assert Vc.numel() >= vb
    rk.rk_compress(ctx, lay, rk.Rows(K, L, n_tokens_dev=n_dev), Rr, Kp, rk.Rows(V, L, n_tokens_dev=n_dev), Vc)
    rows = torch.empty(B, Hkv, cap, 128, dtype=K.dtype, device=DEV)
    rk.rk_unpack_cache(ctx, lay, Kp, Vc, None, rows)
    torch.cuda.synchronize()
    rk.rk_destroy(ctx)
    return Kp, rows


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("L,r,lengths", [(576, 64, [0, 1, 31, 32, 33, 127, 128, 129, 513, 576]), (97, 16, None), (640, 128, None), (1, 32, None)])
def test_value_blocks(dtype, L, r, lengths):
    B, Hkv = len(lengths or [0] * 3), 3
    g = torch.Generator().manual_seed(5)
    K, V = (torch.randn(B, Hkv, L, 128, generator=g).to(DEV, torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2))
    n = torch.tensor(lengths, dtype=torch.int32, device=DEV) if lengths else None
    _, rows = run(dtype, B, Hkv, L, r, K, V, n)
    for b, m in enumerate(lengths or [L] * B):
        assert torch.equal(rows[b, :, :m], V[b, :, :m])
        assert not rows[b, :, m:(m + 31) // 32 * 32].any()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_value_cache_over_the_keys(dtype):
    B, Hkv, L, r = 4, 16, 1088, 48
    g = torch.Generator().manual_seed(6)
    K, V = (torch.randn(B, Hkv, L, 128, generator=g).to(DEV, torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2))
    want = run(dtype, B, Hkv, L, r, K, V)
    got = run(dtype, B, Hkv, L, r, K.clone(), V, over_keys=True)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(got[1], V)


def test_a_short_batch_is_fast():
    """128 sequences of 2000 tokens at most, with 100 in each: 16 work-groups of Values a sequence, one of them with rows, which have to spread over
    all XCDs.  Measured 0.20 of the full batch's time, 0.45 with all of them on one XCD."""
    B, L, r, ctx = 128, 2000, 64, rk.rk_create(0)
    lay = rk.Layout(B, 1, 1, r, rk.RK_BF16, (L + 31) // 32 * 32, L)
    n = torch.empty(B, dtype=torch.int32, device=DEV)
    K, V = (torch.randn(B, 1, L, 128, device=DEV).bfloat16() for _ in range(2))
    Rr, (kb, vb), times = torch.randn(B, 1, 128, r, device=DEV), rk.rk_cache_bytes(lay), []
    Kp, Vc = torch.zeros(kb, dtype=torch.uint8, device=DEV), torch.zeros(vb, dtype=torch.uint8, device=DEV)
    for tokens in (L, 100):
        n.fill_(tokens)
        best = float("inf")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda._sleep(1000000)                        # the calls queue up behind it
            a.record()
            for _ in range(30):
                rk.rk_compress(ctx, lay, rk.Rows(K, L, n_tokens_dev=n), Rr, Kp, rk.Rows(V, L, n_tokens_dev=n), Vc)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    rk.rk_destroy(ctx)
    assert times[1] <= 0.32 * times[0], times
