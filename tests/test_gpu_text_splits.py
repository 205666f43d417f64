"""The text attention inside the splits of the bf16 dual decode: text lengths around the 32-row tiles and the shares of
the splits, long text beside a short or an empty cache (more splits than the cache alone would take), one split that
writes the output itself, several head groups, and the appended row taken from the inputs.  Against the oracle, bf16
outputs within 2e-2 as everywhere in this suite; rows behind the end hold NaN patterns."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2605_19218_amd as rk

from gpu_util import D, DEV, Pipeline, to_dev, to_host
from test_gpu_f32 import launches
from test_gpu_parity import check_out, layer, run_prefill

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = rk.rk_create(0)
    yield c
    rk.rk_destroy(c)


CASES = [
    # B, Hq, Hkv, L, lengths, r, text capacity, text lengths, splits
    (5, 14, 2, 700, [700, 300, 128, 1, 0], 64, 200, [33, 32, 31, 1, 0], 0),
    (2, 8, 2, 300, [300, 0], 32, 1500, [1500, 1029], 0),            # long text, short and empty cache
    (1, 4, 4, 4096, None, 128, 300, [257], 2),                      # the widest kernel, steady loop
    (2, 20, 1, 500, [500, 129], 96, 140, [129, 65], 3),             # two head groups
    (2, 2, 1, 200, [200, 64], 16, 700, [700, 97], 1),               # a lone split
    (9, 16, 2, 900, [900] * 8 + [5], 48, 64, [64, 63, 0, 1, 2, 40, 50, 60, 33], 0),
    (32, 8, 2, 2048, None, 32, 127, [(37 * i) % 128 for i in range(32)], 0),      # a full device, one split more
    (16, 8, 8, 1024, None, 16, 300, [300 - 17 * i for i in range(16)], 0),        # a full device, two splits more
    (8, 4, 4, 3700, None, 32, 1500, [1500, 1499, 0, 1, 1400, 33, 700, 65], 0),     # one unit in seven left, eight splits
    (40, 8, 8, 600, [600 - 13 * i for i in range(40)], 16, 300, [7 * i for i in range(40)], 0),    # several rounds, two splits
    (40, 8, 8, 600, None, 16, 600, [600 - 15 * i for i in range(40)], 0),         # several rounds, shared
]


def with_text(p, data, cid, cap, lens, extra=0):
    B, Hkv = p.B, p.Hkv
    t = layer(B, p.Hq, Hkv, max(cap, 1), "bf16", cid)
    kt, vt = to_dev(t["K"], "bf16"), to_dev(t["V"], "bf16")
    dk = torch.full((B, Hkv, cap + extra, D), float("nan"), device=DEV, dtype=torch.bfloat16)
    dv = dk.clone()
    for b in range(B):
        dk[b, :, :lens[b]], dv[b, :, :lens[b]] = kt[b, :, :lens[b]], vt[b, :, :lens[b]]
    return t, dk, dv, torch.tensor(lens, device=DEV, dtype=torch.int32)


def want_dual(p, q, lens, t, tlens, extra=None):
    Kt, V = p.unpacked()
    pad = np.zeros((p.B, p.Hkv, 1, D))
    kt, vt = np.concatenate([t["K"], pad], 2), np.concatenate([t["V"], pad], 2)
    n = np.asarray(tlens, np.int32)
    if extra is not None:
        for b in range(p.B):
            kt[b, :, n[b]], vt[b, :, n[b]] = extra[0][b], extra[1][b]
        n = n + 1
    return oracle.decode_dual_batch(q.astype(np.float64), Kt, V, kt, vt, to_host(p.Rr), to_host(p.dmu),
                                    lens=np.asarray(lens, np.int32), lens_t=n.astype(np.int32))


@pytest.mark.parametrize("case", CASES)
def test_text_in_splits(ctx, case):
    B, Hq, Hkv, L, lengths, r, cap, tlens, splits = case
    data = layer(B, Hq, Hkv, L, "bf16", 81, lengths=lengths, mean_shift=1.5)
    p = run_prefill(ctx, data, B, Hq, Hkv, L, r, "bf16", lengths=lengths)
    lens = lengths or [L] * B
    t, dk, dv, dlen = with_text(p, data, 82, cap, tlens, extra=1)
    q = to_dev(data["q"], "bf16")
    new = layer(B, Hq, Hkv, 1, "bf16", 83)
    kn, vn = to_dev(new["k_new"], "bf16"), to_dev(new["v_new"], "bf16")
    results = []
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        for fuse in (1, 1, 0):
            rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, fuse)
            ws = torch.empty(rk.rk_decode_workspace_size(ctx, p.layout()), device=DEV, dtype=torch.uint8)
            rk.rk_decode_attn_dual(ctx, p.layout(), q, p.Kp, p.Vc, p.Rr, p.dmu, rk.Text(dk, dv, cap, len=dlen), 0.0, p.out, ws)
            torch.cuda.synchronize()
            results.append(to_host(p.out))
        want = want_dual(p, data["q"], lens, t, tlens)
        for got in results:
            check_out(got, want, "bf16")
        assert np.array_equal(results[0], results[1])
        for b in range(B):
            if lens[b] == 0 and tlens[b] == 0:
                assert not results[0][b].any()
        for fuse in (1, 0):                                   # the appended row joins this step's softmax
            rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, fuse)
            k2, v2, l2 = dk.clone(), dv.clone(), dlen.clone()
            ws = torch.empty(rk.rk_decode_workspace_size(ctx, p.layout()), device=DEV, dtype=torch.uint8)
            rk.rk_append_text_decode_attn_dual(ctx, p.layout(), kn, vn, q, p.Kp, p.Vc, p.Rr, p.dmu,
                                               rk.Text(k2, v2, cap, len=l2), 0.0, p.out, ws)
            torch.cuda.synchronize()
            check_out(to_host(p.out), want_dual(p, data["q"], lens, t, tlens, (new["k_new"], new["v_new"])), "bf16")
            assert l2.cpu().tolist() == [n + 1 for n in tlens]
            for b in range(B):
                assert torch.equal(k2[b, :, tlens[b]], kn[b]) and torch.equal(v2[b, :, tlens[b]], vn[b])
                assert torch.equal(k2[b, :, :tlens[b]], dk[b, :, :tlens[b]])
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, 1)
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)


# Rows whose score is minus infinity weigh nothing, also where they fill a whole tile, a wave's first one, or the text.
@pytest.mark.parametrize("L,n,masked,splits", [
    (700, 33, [32], 0), (700, 33, [32], 3), (200, 200, range(32), 1), (300, 200, range(32), 2), (300, 200, range(150), 0),
    (300, 5, range(5), 0), (300, 5, range(5), 1), (0, 5, range(5), 1), (0, 40, range(40), 0),
])
def test_infinite_text_scores(ctx, L, n, masked, splits):
    B, Hq, Hkv, r, cap = 1, 4, 2, 32, 256
    data = layer(B, Hq, Hkv, max(L, 32), "bf16", 84, mean_shift=1.5)
    p = run_prefill(ctx, data, B, Hq, Hkv, max(L, 32), r, "bf16", lengths=[L])
    t, dk, dv, dlen = with_text(p, data, 85, cap, [n])
    data["q"][..., 0] = 1.0
    q = to_dev(data["q"], "bf16")
    dk[:, :, list(masked), 0] = float("-inf")
    left = [i for i in range(n) if i not in masked]
    kept = {k: np.concatenate([t[k][:, :, left], t[k]], 2)[:, :, :max(len(left), 1)] for k in ("K", "V")}
    want = want_dual(p, data["q"], [L], kept, [len(left)])
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        for fuse in (1, 0):
            rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, fuse)
            ws = torch.empty(rk.rk_decode_workspace_size(ctx, p.layout()), device=DEV, dtype=torch.uint8)
            rk.rk_decode_attn_dual(ctx, p.layout(), q, p.Kp, p.Vc, p.Rr, p.dmu, rk.Text(dk, dv, cap, len=dlen), 0.0, p.out, ws)
            torch.cuda.synchronize()
            got = to_host(p.out)
            assert np.isfinite(got).all()
            if L == 0 and not left:
                assert not got.any()
            else:
                check_out(got, want, "bf16")
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, 1)
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)


def cancelling_rows():
    """Scores and Values of a text whose output all but cancels, so that an error of the softmax weights shows: rows with the
    largest remainders of a weight against a sum of two bf16 numbers, signs along them, and two rows that balance the sum."""
    def bf16(x):
        return float(torch.tensor(x, dtype=torch.float32).to(torch.bfloat16))

    rows = []
    for j in range(1, 256):                               # scores -j / 256
        p = float(np.float32(np.exp(np.float64(-j / 256))))
        rest = p - bf16(p)
        rows.append(((rest - bf16(rest)) / p, -j / 256))
    rows.sort()
    pick = [(-1.0, s) for _, s in rows[:3]] + [(1.0, s) for _, s in rows[-3:]]
    total = sum(v * math.exp(s) for v, s in pick)
    for s in (0.0, -0.5):                                 # exp(0) has no remainder; the last Value is 2^-9 of the others
        v = bf16(-total / math.exp(s))
        pick.append((v, s))
        total += v * math.exp(s)
    v, s = np.array([x[0] for x in pick]), np.array([x[1] for x in pick])
    p = np.exp(s)
    return s, v, (p * v).sum() / p.sum(), (p * np.abs(v)).sum() / p.sum()


@pytest.mark.parametrize("splits", [0, 1])
def test_text_weights_keep_fp32(ctx, splits):
    """Eight rows: a weight in fp32 is off by 2^-22 of itself at most (exp2 one place, the scaled score half a place of 1),
    the sum by 8 2^-24, so 2^-20.4 of sum(p |v|) in all; 17-bit weights would be off by 2^-17.3 of it here."""
    s, v, want, size = cancelling_rows()
    p = Pipeline(ctx, 1, 1, 1, 16, "bf16", 32)
    k, val = torch.zeros(1, 1, 8, D), torch.zeros(1, 1, 8, D)
    k[0, 0, :, 0], val[0, 0] = torch.from_numpy(s), torch.from_numpy(v)[:, None].expand(8, D)
    q = torch.zeros(1, 1, D)
    q[..., 0] = 1.0
    bf = dict(device=DEV, dtype=torch.bfloat16)
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        ws = torch.empty(rk.rk_decode_workspace_size(ctx, p.layout()), device=DEV, dtype=torch.uint8)
        rk.rk_decode_attn_dual(ctx, p.layout(), q.to(**bf), p.Kp, p.Vc, p.Rr, None, rk.Text(k.to(**bf), val.to(**bf), 8), 1.0,
                               p.out, ws)
        torch.cuda.synchronize()
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)
    err = np.abs(to_host(p.out) - want).max()
    assert err <= 2.0 ** -20.4 * size + 2.0 ** -9 * abs(want), (err / size, want / size)


@pytest.mark.parametrize("splits", [1, 2])
def test_large_bias_beside_text(ctx, splits):
    """A bias of 2^20 (log2 domain) leaves the cache's own softmax alone: with a text that weighs nothing the result is the
    plain decode's, bit for bit."""
    B, Hq, Hkv, L, r = 1, 4, 2, 600, 32
    data = layer(B, Hq, Hkv, L, "bf16", 86)
    p = run_prefill(ctx, data, B, Hq, Hkv, L, r, "bf16")
    data["q"][..., 0] = 1.0
    q = to_dev(data["q"], "bf16")
    p.dmu.zero_()
    p.dmu[..., 0] = 2.0 ** 20 / math.log2(math.e) * math.sqrt(D)
    t, dk, dv, dlen = with_text(p, data, 87, 40, [40])
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        plain = p.decode(q).copy()
        ws = torch.empty(rk.rk_decode_workspace_size(ctx, p.layout()), device=DEV, dtype=torch.uint8)
        rk.rk_decode_attn_dual(ctx, p.layout(), q, p.Kp, p.Vc, p.Rr, p.dmu, rk.Text(dk, dv, 40, len=dlen), 0.0, p.out, ws)
        torch.cuda.synchronize()
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)
    assert np.array_equal(to_host(p.out), plain)


# Whether the merge rides in the split launch where some splits are text's: more work-groups than a round of the compute units, but splits of text
# beside those of the cache (the first three), and an XCD with too many bytes of the cache (the last two).  Against the plain kernels.
@pytest.mark.parametrize("units,L,rows,kernels", [(100, 6000, 500, 1), (84, 8000, 200, 1), (44, 16384, 1200, 1), (28, 16384, 1200, 2), (36, 16384, 1200, 2)])
def test_where_the_merge_rides_along_with_text(ctx, units, L, rows, kernels):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the table is for 256 compute units")
    r = 64
    lay = rk.Layout(units, 1, 1, r, rk.RK_BF16, (L + 31) // 32 * 32, L, seq_len=torch.full((units,), L, device=DEV, dtype=torch.int32))
    kb, vb = rk.rk_cache_bytes(lay)
    g = torch.Generator(DEV).manual_seed(2)
    K, V, q = (torch.randn(n, device=DEV, generator=g).bfloat16() for n in (kb // 2, vb // 2, units * D))
    q, Rr = q.view(units, 1, D), torch.randn(units, 1, D, r, device=DEV, generator=g) / 11.3
    kt, vt = (torch.randn(units, 1, rows, D, device=DEV, generator=g).bfloat16() for _ in range(2))
    ws, outs = torch.empty(rk.rk_decode_workspace_size(ctx, lay), device=DEV, dtype=torch.uint8), []
    try:
        for plain in (0, 1):
            out = torch.full((units, 1, D), float("nan"), device=DEV, dtype=torch.bfloat16)

            def call(stream=None):
                rk.rk_decode_attn_dual(ctx, lay, q, K, V, Rr, None, rk.Text(kt, vt, rows), 0.0, out, ws, stream=stream)

            if not plain:
                assert launches(call) == kernels
            rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, plain)
            call()
            torch.cuda.synchronize()
            outs.append(to_host(out))
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, 0)
    check_out(outs[0], outs[1], "bf16")
