"""fp32 storage on the matrix-core kernels (covariance, compress, decode) at the edges of their tiles, against the
oracle and against the plain kernels.  fp32 results: max|x - y| / max|y| <= 1e-4, as everywhere in this suite."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import paper_2605_19218_amd as rk

from gpu_util import D, DEV, Pipeline, to_dev, to_host
from test_gpu_parity import check_out, check_packed, layer, oracle_decode, rel_max, run_prefill

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = rk.rk_create(0)
    yield c
    rk.rk_destroy(c)


# lengths around the two-token steps, the 32-token quarters and 128-token chunks, the 512-token chunks of a call with
# more than 512 short ones, and chunks of 256 (two matrices) and 512 (one) where the reduction of short ones costs more
@pytest.mark.parametrize("B,Hkv,L,lengths,center", [
    (5, 1, 129, [129, 128, 127, 1, 0], True), (3, 2, 97, [97, 33, 2], False), (1, 1, 2000, None, True),
    (2, 40, 1100, [1100, 513], True), (2, 1, 16001, [16001, 257], True), (1, 1, 66000, None, True),
])
def test_covariance(ctx, B, Hkv, L, lengths, center):
    data = layer(B, Hkv, Hkv, L, "f32", 61, lengths=lengths, mean_shift=3.0)
    p = Pipeline(ctx, B, Hkv, Hkv, 16, "f32", L)
    n_dev = None if lengths is None else torch.tensor(lengths, device=DEV, dtype=torch.int32)
    p.fit(to_dev(data["K"], "f32"), L, center=center, n_dev=n_dev)
    cov, mu = to_host(p.cov), to_host(p.mu)
    for b in range(B):
        n = L if lengths is None else lengths[b]
        for h in range(0, Hkv, 13):
            if n == 0:
                assert not cov[b, h].any() and not mu[b, h].any()
                continue
            mu_o, C_o = oracle.mean_scatter(data["K"][b, h, :n], center=center)
            # centring one row leaves the rounding of the fp32 products, against their own size
            scale = max(np.abs(C_o).max(), 1e-6 * np.abs(data["K"][b, h, :n]).max() ** 2 * n / 1e-4)
            assert np.abs(cov[b, h] - C_o).max() <= 1e-4 * scale
            assert rel_max(mu[b, h], mu_o) <= 1e-4
            assert np.array_equal(cov[b, h], cov[b, h].T)


@pytest.mark.parametrize("r", [1, 16, 37, 64, 100, 128])
def test_compress_and_token_list(ctx, r):
    B, Hkv, L = 3, 2, 300
    lengths = [300, 129, 15]
    data = layer(B, Hkv, Hkv, L, "f32", 62, lengths=lengths)
    p = run_prefill(ctx, data, B, Hkv, Hkv, L, r, "f32", lengths=lengths)
    (Kt, Vc), Rr = p.unpacked(), to_host(p.Rr)
    for b in range(B):
        for h in range(Hkv):
            check_packed(Kt[b, h, :lengths[b]], data["K"][b, h, :lengths[b]].astype(np.float64), Rr[b, h], "f32")
            assert not Kt[b, h, lengths[b]:].any()
    idx = np.concatenate([np.arange(0, n, 2) for n in lengths]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum([(n + 1) // 2 for n in lengths])]).astype(np.int64)
    p2 = Pipeline(ctx, B, Hkv, Hkv, r, "f32", 160)
    p2.fit(to_dev(data["K"], "f32"), 150, tok_idx=torch.from_numpy(idx).to(DEV), tok_off=torch.from_numpy(off).to(DEV))
    p2.compress(to_dev(data["K"], "f32"), 150, V_dev=to_dev(data["V"], "f32"), tok_idx=torch.from_numpy(idx).to(DEV),
                tok_off=torch.from_numpy(off).to(DEV))
    Kt, Rr, cov = p2.unpacked()[0], to_host(p2.Rr), to_host(p2.cov)
    for b in range(B):
        rows = idx[off[b]:off[b + 1]]
        check_packed(Kt[b, 1, :rows.size], data["K"][b, 1][rows].astype(np.float64), Rr[b, 1], "f32")
        assert rel_max(cov[b, 1], oracle.mean_scatter(data["K"][b, 1], tok=rows)[1]) <= 1e-4


@pytest.mark.parametrize("r", [1, 18, 37])
def test_padding_of_non_finite_keys(ctx, r):
    """The padding channels of a row are zero whatever its Key holds: as NaN they would reach every score of the row."""
    L, rp = 40, (r + 15) // 16 * 16
    p = Pipeline(ctx, 1, 1, 1, r, "f32", L)
    p.Rr.copy_(torch.eye(D, r, device=DEV).expand_as(p.Rr))
    p.Kp.fill_(0xff)
    K = np.ones((1, 1, L, D), np.float32)
    K[0, 0, 3, 0], K[0, 0, 21, 1], K[0, 0, 39, 127] = np.inf, np.nan, -np.inf
    p.compress(to_dev(K, "f32"), L, V_dev=to_dev(np.ones_like(K), "f32"))
    rows = p.Kp.view(torch.float32)[:48 * rp].view(3, rp // 8, 16, 8).permute(0, 2, 1, 3).reshape(48, rp)[:L]
    assert not rows[:, r:].any()
    rest = torch.ones(L, r, device=DEV)
    assert torch.equal(rows[[0, 20, 38], :r], rest[:3])


DECODE = [
    # B, Hq, Hkv, L, lengths, r, splits
    (6, 4, 2, 129, [129, 65, 64, 17, 16, 1], 64, 0),
    (3, 14, 2, 700, [700, 0, 513], 37, 0),          # G = 7, an empty sequence, padded channels
    (2, 16, 1, 300, [300, 31], 16, 3),              # a full block of 16 heads
    (1, 20, 1, 260, None, 100, 2),                  # two head groups
    (1, 2, 2, 4096, None, 128, 2),                  # the steady loop: 32 tiles per wave
    (2, 2, 1, 1500, [1500, 200], 1, 7),
    (1, 2, 2, 90, None, 80, 1),                     # a lone split writes the output itself
]


@pytest.mark.parametrize("case", DECODE)
def test_decode(ctx, case):
    B, Hq, Hkv, L, lengths, r, splits = case
    data = layer(B, Hq, Hkv, L, "f32", 63, lengths=lengths, mean_shift=1.5)
    p = run_prefill(ctx, data, B, Hq, Hkv, L, r, "f32", lengths=lengths)
    q = to_dev(data["q"], "f32")
    # rows behind the end hold NaN patterns, in the last token's own block and in the one behind it: they may be read, never used
    rp = (r + 15) // 16 * 16
    K = p.Kp.view(torch.float32).view(B * Hkv, -1)[:, :p.cap * rp].view(B, Hkv, p.cap // 16, rp // 8, 16, 8)
    V = p.Vc.view(torch.float32).view(B * Hkv, -1)[:, :p.cap * D].view(B, Hkv, p.cap // 32, D // 16, 4, 16, 2, 4)
    for b in range(B):
        n = (lengths or [L] * B)[b]
        for t in range(n, min(p.cap, (n // 32 + 2) * 32)):
            K[b, :, t // 16, :, t % 16] = float("nan")
            V[b, :, t // 32, :, t % 16 // 4, :, t % 32 // 16, t % 4] = float("nan")
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        got, again = p.decode(q).copy(), p.decode(q).copy()
        nobias = p.decode(q, use_bias=False).copy()
        rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, 1)
        plain = p.decode(q).copy()
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FORCE_GENERIC, 0)
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)
    lens = lengths or [L] * B
    want = oracle_decode(p, data["q"], lens)
    for x in (got, nobias, plain):
        check_out(x, want, "f32")
    assert np.array_equal(got, again)
    for b in range(B):
        if lens[b] == 0:
            assert not got[b].any()


def launches(call):
    """Kernels that call(stream) enqueues, counted in a graph that is captured and never run."""
    hip = C.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    stream, graph, n = torch.cuda.Stream(), C.c_void_p(), C.c_size_t()
    assert hip.hipStreamBeginCapture(C.c_void_p(stream.cuda_stream), 2) == 0
    try:
        call(stream)
    finally:
        assert hip.hipStreamEndCapture(C.c_void_p(stream.cuda_stream), C.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0 and hip.hipGraphDestroy(graph) == 0
    return n.value


# The merge inside the split launch against the merge launch: the same partials folded in the same order, so the same bits.  Unit
# counts around the eight XCDs, 17 and 40 splits (two and three rounds of loads), empty splits and sequences, two head groups, and a
# result that is only 4-byte aligned.
@pytest.mark.parametrize("B,Hq,Hkv,L,lengths,r,splits", [
    (2, 14, 7, 700, [700, 0], 37, 0), (1, 8, 8, 513, None, 64, 2), (3, 9, 3, 1300, [1300, 129, 1], 128, 9), (1, 40, 2, 300, None, 100, 3),
    (1, 24, 24, 2300, None, 32, 17), (1, 16, 16, 5200, None, 16, 40), (5, 32, 8, 260, [260, 0, 128, 129, 31], 112, 2),
    (1, 9, 9, 2100, None, 48, 16),
])
def test_merge_in_the_split_launch(ctx, B, Hq, Hkv, L, lengths, r, splits):
    data = layer(B, Hq, Hkv, L, "f32", 65, lengths=lengths, mean_shift=1.0)
    p = run_prefill(ctx, data, B, Hq, Hkv, L, r, "f32", lengths=lengths)
    q = to_dev(data["q"], "f32")
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    got = []
    try:
        for fuse in (1, 0, 1):
            rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, fuse)
            lay = p.layout()
            ws = torch.full((rk.rk_decode_workspace_size(ctx, lay),), 0xff, device=DEV, dtype=torch.uint8)
            out = torch.full((B * Hq * D + 1,), float("nan"), device=DEV)[1:].view(B, Hq, D)

            def call(stream=None):
                rk.rk_decode_attn(ctx, lay, q, p.Kp, p.Vc, p.Rr, p.dmu, 0.0, out, ws, stream=stream)

            assert launches(call) == 2 - fuse
            call()
            got.append(out.cpu().numpy())
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_FUSE_MERGE, 1)
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)
    check_out(got[0], oracle_decode(p, data["q"], lengths or [L] * B), "f32")
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])


# Whether the merge rides in the split launch: unit counts that load the XCDs evenly; unevenly but within one round of their compute
# units; unevenly with a second round on some (7 units of 36 splits, 9 of 17); and by more bytes than the second launch is worth.
@pytest.mark.parametrize("units,L,splits,kernels", [
    (8, 24000, 0, 1), (64, 3000, 0, 1), (12, 3000, 0, 1), (7, 6000, 0, 1), (36, 1000, 0, 1), (258, 600, 0, 1), (9, 2100, 16, 1),
    (9, 2200, 17, 2), (7, 12000, 0, 2), (7, 24000, 0, 2), (20, 3000, 0, 2), (28, 6000, 0, 2), (36, 3000, 0, 2), (60, 8000, 0, 2),
])
def test_where_the_merge_rides_along(ctx, units, L, splits, kernels):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the table is for 256 compute units")
    lay = rk.Layout(1, units, units, 64, rk.RK_F32, (L + 31) // 32 * 32, L, seq_len=torch.full((1,), L, device=DEV, dtype=torch.int32))
    kb, vb = rk.rk_cache_bytes(lay)
    K, V, q, Rr, out = (torch.zeros(n, device=DEV) for n in (kb // 4, vb // 4, units * D, units * D * 64, units * D))
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        ws = torch.empty(rk.rk_decode_workspace_size(ctx, lay), device=DEV, dtype=torch.uint8)
        assert launches(lambda s: rk.rk_decode_attn(ctx, lay, q, K, V, Rr, None, 0.0, out, ws, stream=s)) == kernels
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)


# Tokens whose score overflows to minus infinity weigh nothing, also where they fill a 16-token tile, a wave's first one,
# or the cache (its output is then zero).
@pytest.mark.parametrize("L,masked,splits", [(200, range(16), 1), (200, [199], 1), (97, [96], 2), (400, range(64), 3),
                                             (400, range(256, 272), 1), (129, [128], 0), (40, range(40), 1), (300, range(300), 2)])
def test_infinite_scores(ctx, L, masked, splits):
    B, Hq, Hkv, r = 1, 4, 2, 16
    data = layer(B, Hq, Hkv, L, "f32", 64)
    data["K"][:, :, list(masked), :] = 0.0
    data["K"][:, :, list(masked), 0] = -3e38
    data["q"][..., 0] = 64.0
    p = Pipeline(ctx, B, Hq, Hkv, r, "f32", L)
    p.Rr.copy_(torch.eye(D, r, device=DEV).expand_as(p.Rr))
    p.compress(to_dev(data["K"], "f32"), L, V_dev=to_dev(data["V"], "f32"))
    q = to_dev(data["q"], "f32")
    rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, splits)
    try:
        got = p.decode(q, use_bias=False).copy()
    finally:
        rk.rk_set_option(ctx, rk.RK_OPT_DECODE_SPLITS, 0)
    left = [i for i in range(L) if i not in masked]
    if not left:
        assert not got.any()
        return
    Kt, V = p.unpacked()
    want = oracle.decode_batch(data["q"].astype(np.float64), np.ascontiguousarray(Kt[:, :, left]),
                               np.ascontiguousarray(V[:, :, left]), to_host(p.Rr), None,
                               lens=np.asarray([len(left)], np.int32), scale=0.0)
    check_out(got, want, "f32")


def test_workspace_of_a_longer_input_serves_a_shorter_one():
    """Short inputs take shorter chunks: the workspace size must not fall as the bound on the rows grows."""
    for H in (1, 4, 32, 300, 600):
        lay = rk.Layout(1, H, H, 32, rk.RK_F32, 64, 0)
        sizes = [rk.rk_fit_workspace_size(lay, n) for n in (0, 1, 128, 129, 511, 513, 2048, 4097, 16384, 16385, 65537, 300000)]
        assert sizes == sorted(sizes)
