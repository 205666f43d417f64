"""bf16 compress in blocks of 512 tokens, with lengths on the device and enough heads to fill it; lengths around the passes (128
tokens) and blocks; and with equal lengths, where r = 128 takes one 2048-token block a head.  Against the oracle: one bf16 unit
plus the accumulation bound, as everywhere in this suite."""
import numpy as np
import pytest
import torch

import paper_2605_19218_amd as rk

from gpu_util import DEV, Pipeline, to_dev, to_host
from test_gpu_parity import check_packed, layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["lengths", "lists", "equal"])
@pytest.mark.parametrize("r", [37, 128])
def test_blocks(r, form):
    lengths = [1100, 1025, 1024, 513, 512, 511, 129, 1, 0] + [640] * 7 if form != "equal" else [1100] * 16
    B, Hkv, L = len(lengths), 16, max(lengths)               # 256 heads
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
        for h in (0, 15):
            check_packed(Kt[b, h, :lengths[b]], data["K"][b, h][rows[b]].astype(np.float64), Rr[b, h], "bf16")
            assert np.array_equal(Vc[b, h, :lengths[b]], data["V"][b, h][rows[b]])
            assert not Kt[b, h, lengths[b]:].any()
