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
