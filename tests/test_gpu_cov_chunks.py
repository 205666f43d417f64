"""The bf16 covariance takes chunks of 512, 1024 or 2048 tokens by what fills the device; lengths around the chunk and
wave edges of each, with and without a token list, against the oracle (fp32 results: 1e-4 of the largest)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_19218_amd as rk

from gpu_util import D, DEV, Pipeline, to_dev, to_host
from test_gpu_parity import layer, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,L,lengths", [
    (4, 1, 1537, [1537, 512, 513, 127]),                     # 512-token chunks
    (4, 32, 1030, [1030, 1024, 300, 1]),                     # 128 heads: 1024-token chunks
    (4, 32, 2100, [2100, 2048, 1023, 0]),                    # 128 heads, longer: 2048-token chunks
])
@pytest.mark.parametrize("lists", [False, True])
def test_chunk_lengths(B, Hkv, L, lengths, lists):
    ctx = rk.rk_create(0)
    data = layer(B, Hkv, Hkv, L, "bf16", 71, lengths=lengths, mean_shift=2.0)
    p = Pipeline(ctx, B, Hkv, Hkv, 16, "bf16", L)
    if lists:
        rows = [np.arange(n - 1, -1, -1) for n in lengths]   # every row, last first
        idx = np.concatenate(rows).astype(np.int32)
        off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
        p.fit(to_dev(data["K"], "bf16"), L, tok_idx=torch.from_numpy(idx).to(DEV), tok_off=torch.from_numpy(off).to(DEV))
    else:
        p.fit(to_dev(data["K"], "bf16"), L, n_dev=torch.tensor(lengths, device=DEV, dtype=torch.int32))
    cov, mu = to_host(p.cov), to_host(p.mu)
    rk.rk_destroy(ctx)
    for b in range(B):
        n = lengths[b]
        for h in range(0, Hkv, 37):
            if n == 0:
                assert not cov[b, h].any() and not mu[b, h].any()
                continue
            mu_o, C_o = oracle.mean_scatter(data["K"][b, h, :n])
            scale = max(np.abs(C_o).max(), 1e-2 * np.abs(data["K"][b, h, :n]).max() ** 2 * n)
            assert np.abs(cov[b, h] - C_o).max() <= 1e-4 * scale
            assert rel_max(mu[b, h], mu_o) <= 1e-4


def test_many_units_fp32():
    """With 128 heads the reduction goes by rows, four chunks at a time: five of 512 tokens here, in the fp32 kernel's channel order
    (the bf16 one above has two).  Against the oracle; the bits are held below."""
    B, Hkv, L, lengths = 4, 32, 2100, [2100, 2048, 513, 0]
    ctx = rk.rk_create(0)
    data = layer(B, Hkv, Hkv, L, "f32", 73, lengths=lengths, mean_shift=2.0)
    p = Pipeline(ctx, B, Hkv, Hkv, 16, "f32", L)
    p.cov.fill_(float("nan"))
    for center in (True, False):
        p.fit(to_dev(data["K"], "f32"), L, center=center, n_dev=torch.tensor(lengths, device=DEV, dtype=torch.int32))
        cov, mu = to_host(p.cov), to_host(p.mu)
        for b in range(B):
            n = lengths[b]
            for h in (0, 9, 31):
                assert np.array_equal(cov[b, h], cov[b, h].T)
                if n == 0:
                    assert not cov[b, h].any() and not mu[b, h].any()
                    continue
                mu_o, C_o = oracle.mean_scatter(data["K"][b, h, :n], center=center)
                assert np.abs(cov[b, h] - C_o).max() <= 1e-4 * np.abs(C_o).max()
                assert rel_max(mu[b, h], mu_o) <= 1e-4
    rk.rk_destroy(ctx)


@pytest.mark.parametrize("dtype,B,L", [("f32", 4, 2100), ("bf16", 4, 24576), ("bf16", 4, 26000), ("bf16", 12, 26000)])
def test_reduction_by_rows_keeps_the_bits(dtype, B, L):
    """128 heads with 5 (fp32) and 12 chunks, and 384 with 13, are reduced by rows, 128 with 13 by positions, as are the calls of 64
    heads that they are compared with: the same partials added in the same order, so the same bits."""
    Hkv, ctx = 32, rk.rk_create(0)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    base = torch.randn(L + 8 * B * Hkv, D, device=DEV, generator=torch.Generator(DEV).manual_seed(4)).add_(1.0).to(td)
    K = base.as_strided((B, Hkv, L, D), (8 * Hkv * D, 8 * D, D, 1))                  # unit u: the L rows from 8 u on
    lens = torch.tensor([L, L - 511, 2049, 0] * (B // 4), device=DEV, dtype=torch.int32)
    for center in (True, False):
        got = []
        for n in (B, 2):
            for b in range(0, B, n):
                p = Pipeline(ctx, n, Hkv, Hkv, 16, dtype, 32)
                p.cov.fill_(float("nan"))
                p.fit(K[b:b + n], L, center=center, n_dev=lens[b:b + n].clone())
                got.append((p.cov, p.mu))
        assert torch.equal(got[0][0], torch.cat([c for c, _ in got[1:]]))
        assert torch.equal(got[0][1], torch.cat([m for _, m in got[1:]]))
    rk.rk_destroy(ctx)


@pytest.mark.parametrize("dtype,Hkv", [("bf16", 1), ("bf16", 8), ("f32", 1)])      # chunks of 512 and of 2048 tokens; fp32: of 128
@pytest.mark.parametrize("lists", [False, True])
def test_shares_of_the_waves(dtype, Hkv, lists):
    """Lengths that leave the last wave of a sequence whole turns of its ring, one to three k-steps more, a part of one, or nothing."""
    lengths = [2064, 2080, 2096, 2095, 1553, 1568, 1040, 1056, 528, 544, 560, 576, 144, 160, 192, 255, 257, 64, 63, 65, 16, 15, 17, 1]
    B, L, ctx = len(lengths), max(lengths), rk.rk_create(0)
    data = layer(B, Hkv, Hkv, L, dtype, 75, lengths=lengths, mean_shift=2.0)
    p = Pipeline(ctx, B, Hkv, Hkv, 16, dtype, L)
    p.cov.fill_(float("nan"))
    if lists:
        idx = np.concatenate([np.arange(n - 1, -1, -1) for n in lengths]).astype(np.int32)          # every row, last first
        off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
        p.fit(to_dev(data["K"], dtype), L, tok_idx=torch.from_numpy(idx).to(DEV), tok_off=torch.from_numpy(off).to(DEV))
    else:
        p.fit(to_dev(data["K"], dtype), L, n_dev=torch.tensor(lengths, device=DEV, dtype=torch.int32))
    cov, mu = to_host(p.cov), to_host(p.mu)
    rk.rk_destroy(ctx)
    for b, n in enumerate(lengths):
        for h in range(0, Hkv, 5):
            mu_o, C_o = oracle.mean_scatter(data["K"][b, h, :n])
            # (what few rows leave behind their mean is the rounding of the products, against their own size)
            scale = max(np.abs(C_o).max(), 1e-2 * np.abs(data["K"][b, h, :n]).max() ** 2 * n)
            assert np.abs(cov[b, h] - C_o).max() <= 1e-4 * scale
            assert rel_max(mu[b, h], mu_o) <= 1e-4
