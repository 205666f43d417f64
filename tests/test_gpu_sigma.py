"""rk_query_sigma over windows whose rows are not on 16-byte boundaries (the entry point takes any base and strides) and
over row counts around the kernel's passes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_19218_amd as rk

from gpu_util import D, DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,Hq,Hkv,W,offset,pad", [
    (2, 14, 2, 32, 0, 0), (1, 4, 2, 33, 1, 0), (1, 6, 2, 7, 0, 3), (1, 1, 1, 1, 5, 1), (1, 8, 1, 100, 0, 0), (1, 2, 1, 257, 3, 5),
    (16, 32, 32, 33, 0, 0), (16, 64, 32, 40, 1, 0), (17, 96, 32, 31, 0, 8),            # 512 units on: smaller work-groups
])
def test_sigma(dtype, B, Hq, Hkv, W, offset, pad):
    ctx = rk.rk_create(0)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    sw = D + pad
    sh, sb = W * sw + pad, Hq * (W * sw + pad) + 2 * pad
    flat = torch.randn(B * sb + offset + 64, device=DEV, generator=torch.Generator(DEV).manual_seed(5)).to(td)
    win = flat[offset:].as_strided((B, Hq, W, D), (sb, sh, sw, 1))
    sigma = torch.zeros(B, Hkv, D, device=DEV)
    rk.rk_query_sigma(ctx, rk.Layout(B, Hq, Hkv, 32, rk.RK_BF16 if dtype == "bf16" else rk.RK_F32, 32, 0),
                      flat.data_ptr() + offset * flat.element_size(), W, sigma, strides=(sb, sh, sw))
    torch.cuda.synchronize()
    rk.rk_destroy(ctx)
    Q, G = win.double().cpu().numpy(), Hq // Hkv
    for b in range(B):
        for h in range(Hkv):
            want = oracle.sigma_window(Q[b, h * G:(h + 1) * G])
            # fp32 sums of W G squares: a relative W G 2^-24 / 2 at the very most
            assert np.abs(sigma[b, h].double().cpu().numpy() - want).max() <= want.max() * (W * G + 4) * 2.0 ** -24
