"""bf16 compress in blocks of 512 tokens: lengths around the passes (128 tokens) and blocks, equal, on the device or by token lists;
block counts of either parity, with the last one full or partly filled, and more work-groups than compute units (a partly filled last
block's then start behind the others) or fewer.  Against the oracle: one bf16 unit plus the accumulation bound, as everywhere in this suite."""
import numpy as np
import pytest
import torch

import paper_2605_19218_amd as rk

from gpu_util import DEV, Pipeline, to_dev, to_host
from test_gpu_parity import check_packed, layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["lengths", "lists", "equal"])
@pytest.mark.parametrize("r,Hkv,L", [
    (37, 16, 1100), (128, 16, 1100), (64, 12, 520), (64, 12, 1024), (128, 6, 1536), (16, 6, 1600), (64, 6, 2100), (96, 3, 520), (48, 3, 1100)])
def test_blocks(r, Hkv, L, form):
    lengths = [L, 1025, 1024, 513, 512, 511, 129, 1, 0] + [640] * 7 if form != "equal" else [L] * 16
    lengths = [min(n, L) for n in lengths]
    B = len(lengths)
    ctx = rk.rk_create(0)
    data = layer(B, Hkv, Hkv, L, "bf16", 72, lengths=lengths)
    p = Pipeline(ctx, B, Hkv, Hkv, r, "bf16", L)
    p.Rr.copy_(torch.linalg.qr(torch.randn(B, Hkv, 128, r, generator=torch.Generator().manual_seed(1)))[0])
    p.Kp.zero_()
    kw, rows = {}, [np.arange(n) for n in lengths]
    if form == "lists":
        rows = [x[::-1].copy() for x in rows]
        kw = dict(tok_idx=torch.from_numpy(np.concatenate(rows).astype(np.int32)).to(DEV),
                  tok_off=torch.from_numpy(np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)).to(DEV))
    elif form == "lengths":
        kw = dict(n_dev=torch.tensor(lengths, device=DEV, dtype=torch.int32))
    p.compress(to_dev(data["K"], "bf16"), L, V_dev=to_dev(data["V"], "bf16"), **kw)
    Kt, Vc = p.unpacked()
    Rr, seq = to_host(p.Rr), p.seq_len.cpu().tolist()
    rk.rk_destroy(ctx)
    assert seq == lengths
    for b in range(B):
        for h in (0, Hkv - 1):
            check_packed(Kt[b, h, :lengths[b]], data["K"][b, h][rows[b]].astype(np.float64), Rr[b, h], "bf16")
            assert np.array_equal(Vc[b, h, :lengths[b]], data["V"][b, h][rows[b]])
            assert not Kt[b, h, lengths[b]:].any()
