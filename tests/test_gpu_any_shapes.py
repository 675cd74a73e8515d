"""Clipped sums and materialised norms at the edges of the any-shape kernel
(tiles of 128 x 128, and of 64 x 192 for d_out <= 64; 16-byte row loads;
16-row groups of an example) and of the 384 x 256 tiles with padding, against the float64 oracle, and what it does with
infinities in float32 (whose three bf16 parts do not exist)."""

import math

import numpy as np
import pytest

import oracle
from paper_2609_20532_amd import workloads as wl

from parity_util import (assert_sum_close, device_layers, oracle_layers, rel_err, tile256,
                         torch_to_float64, wide_tile)

pytestmark = pytest.mark.gpu

# (dtype, B, [(T, d_in, d_out), ...])
CASES = [
    (wl.F32, 3, [(1, 128, 128), (17, 129, 127), (64, 127, 129)]),
    (wl.F32, 2, [(31, 191, 63), (33, 192, 64), (16, 193, 65)]),
    (wl.F32, 5, [(40, 3, 200), (40, 200, 3), (7, 2, 2), (2, 5, 1)]),       # rows below 16 bytes
    (wl.F32, 2, [(1024, 27, 16), (300, 577, 40)]),                        # one tile, long K
    (wl.BF16, 3, [(64, 128, 120), (72, 129, 127), (100, 127, 129)]),     # weight on the accumulator
    (wl.BF16, 2, [(57, 191, 63), (183, 192, 64), (128, 193, 65)]),
    (wl.BF16, 4, [(1, 130, 67), (17, 192, 9), (50, 129, 200)]),          # weight on the operand
    (wl.BF16, 3, [(65, 7, 300), (65, 300, 7), (20, 2, 300), (3, 1, 1)]),    # rows below 16 bytes
    (wl.BF16, 1, [(512, 72, 24)]),
    # the 384 x 256 tiles with padding (last row, column and K slice partly filled; T
    # one row past a slice and one row short of one, one partial 16-row group)
    (wl.BF16, 3, [(1025, 1608, 2000), (1000, 512, 392)]),
    (wl.BF16, 7, [(191, 2040, 3000), (257, 776, 1544), (130, 256, 4104)]),
]
PADDED_TILES = (9, 10)   # of CASES


def _takes_padded_tiles(B, dims):
    """The library's rule for the 384 x 256 tiles with padding, for a bf16 call:
    every layer eligible (widths that are multiples of 8, weights on the
    accumulator, not much more tile area than the any-shape kernel's, no other
    large tile), together at least 20 GFLOP and nine tiles."""
    tiles = 0
    for T, di, do in dims:
        n = -(-do // 384) * -(-di // 256)
        flat = not ((-T) % 64 * 8 <= T or (T >= 64 and (-T) % 16 * 8 <= T))
        small = (-(-do // 64) * -(-di // 192) * 64 * 192 if do <= 64
                 else -(-do // 128) * -(-di // 128) * 128 * 128)
        if (di % 8 or do % 8 or flat or n * 384 * 256 * 0.62 > small or wide_tile(T, di, do)
                or tile256(T, di, do)):
            return False
        tiles += n
    return tiles >= 9 and sum(2.0 * B * T * di * do for T, di, do in dims) >= 2e10


def _host_layer(B, T, d_in, d_out, dtype, seed, tensor_id):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((B, T, d_in)).astype(np.float32)
    G = (rng.standard_normal((B, T, d_out)) * 0.05).astype(np.float32)
    store = wl.bf16_bits_from_f32 if dtype == wl.BF16 else (lambda x: x)
    return wl.HostLayer(A=store(A), G=store(G), d_in=d_in, d_out=d_out, tensor_id=tensor_id,
                        dtype=dtype)


def _bound(dtype, T, d_in, d_out):
    # float32 and float32 weights: a few thousand float32 additions at most.
    # bf16 with the weight on the operand: one rounding (2^-9) per term.
    if dtype == wl.F32 or d_in * d_out <= 512:
        return 2e-6
    pad16, pad64 = (-T) % 16, (-T) % 64
    return 2e-6 if pad64 * 8 <= T or (T >= 64 and pad16 * 8 <= T) else 5e-3


@pytest.mark.parametrize("case", range(len(CASES)))
def test_sums_and_materialised_norms(dp, case):
    import torch
    dtype, B, dims = CASES[case]
    if case in PADDED_TILES:
        assert _takes_padded_tiles(B, dims)
    hs = [_host_layer(B, T, di, do, dtype, 900 + 10 * case + k, k)
          for k, (T, di, do) in enumerate(dims)]
    dev = device_layers(hs)
    Ls = [d[0] for d in dev]
    ol = oracle_layers(hs)
    nsq_ref = oracle.per_example_norms_sq(ol)
    mode = dp.DPSGD_NORM_MATERIALIZE
    buf = dp.alloc_step(Ls, mode)
    dp.dpsgd_per_example_norms_multi(Ls, mode, buf.norms_sq, workspace=buf.norms_ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(buf.norms_sq.cpu().numpy().astype(np.float64), nsq_ref, rtol=3e-6)
    C = float(np.median(np.sqrt(nsq_ref))) * 0.9
    c = np.minimum(1.0, C / np.sqrt(nsq_ref))
    for accumulate in (False, True):
        for g in buf.grads:
            g.fill_(0.25)
        dp.dpsgd_clip_accumulate_multi(Ls, buf.norms_sq, C, buf.grads, accumulate=accumulate,
                                       workspace=buf.clip_ws)
        torch.cuda.synchronize()
        for k, (T, di, do) in enumerate(dims):
            S = sum(c[i] * ol[k].G[i].T @ ol[k].A[i] for i in range(B))
            got = torch_to_float64(buf.grads[k]) - (0.25 if accumulate else 0.0)
            bound = _bound(dtype, T, di, do)
            if accumulate:   # the sum is rounded next to the 0.25 that was there
                bound += 2.0 ** -24 * (0.25 + np.abs(S).max()) / np.sqrt(np.mean(S * S))
            assert rel_err(got, S) <= bound, (dims[k], accumulate, rel_err(got, S))


@pytest.mark.parametrize("T,d_in,d_out", [(32, 130, 70), (40, 200, 24), (5, 64, 64)])
def test_float32_infinities(dp, T, d_in, d_out):
    """An infinity in one row of A: that example's norm is infinite and its
    factor 0. With clipping off (C = inf) the sum holds the infinities that
    float32 arithmetic gives and every other entry is unharmed."""
    import torch
    B, bad, col = 3, 1, 7
    h = _host_layer(B, T, d_in, d_out, wl.F32, 77, 0)
    h.A[bad] = np.round(h.A[bad] * 4) / 4    # few bits: their lower bf16 parts are 0
    h.G[bad] = np.where(h.G[bad] < 0, -0.5, 0.5)
    h.A[bad, 2, col] = np.inf
    (L, A, G), = device_layers([h])
    for mode in (dp.DPSGD_NORM_MATERIALIZE, dp.DPSGD_NORM_GHOST):
        nsq = torch.empty(B, device="cuda")
        ws = torch.empty(dp.dpsgd_norms_workspace_bytes([L], mode), dtype=torch.uint8, device="cuda")
        dp.dpsgd_per_example_norms_multi([L], mode, nsq, workspace=ws)
        torch.cuda.synchronize()
        got = nsq.cpu().numpy()
        if mode == dp.DPSGD_NORM_MATERIALIZE:
            assert math.isinf(got[bad])
        assert np.isfinite(np.delete(got, bad)).all()
    nsq = torch.ones(B, device="cuda")
    grad = torch.empty(d_out, d_in, device="cuda")
    ws = torch.empty(dp.dpsgd_clip_workspace_bytes([L]), dtype=torch.uint8, device="cuda")
    dp.dpsgd_clip_accumulate(L, nsq, math.inf, grad, workspace=ws)
    torch.cuda.synchronize()
    S = grad.cpu().numpy().astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = sum(h.G[i].astype(np.float64).T @ h.A[i].astype(np.float64) for i in range(B))
    assert np.isinf(ref[:, col]).all()
    np.testing.assert_array_equal(S[:, col], ref[:, col])
    keep = np.delete(np.arange(d_in), col)
    assert_sum_close(S[:, keep], ref[:, keep], 2e-6, "finite entries")


@pytest.mark.parametrize("T,d_in,d_out", [(64, 16, 16), (300, 27, 16), (100, 130, 70), (80, 9, 200)])
def test_bf16_infinities(dp, T, d_in, d_out):
    """bf16 tiles that are partly padding: an infinity in one example gives that
    example an infinite norm and factor 0, and the sum of the others is what it
    is without the example (padded entries are 0 x inf and do not count)."""
    import torch
    B, bad = 3, 1
    h = _host_layer(B, T, d_in, d_out, wl.BF16, 78, 0)
    half = wl.bf16_bits_from_f32(np.float32([-0.5, 0.5]))
    h.G[bad] = np.where(h.G[bad] >= 0x8000, half[0], half[1])   # no zeros: no NaN inside the matrix
    h.A[bad, 2, 7] = wl.bf16_bits_from_f32(np.float32([np.inf]))[0]
    dev = device_layers([h])
    L = dev[0][0]
    assert dp.dpsgd_select_norm_mode(L) == dp.DPSGD_NORM_MATERIALIZE
    ol, = oracle_layers([h])
    keep = [0, 2]
    ref = oracle.per_example_norms_sq([oracle.OracleLayer(ol.A[keep], ol.G[keep], 0)])
    C = float(np.sqrt(ref.min())) * 0.9
    for mode in (dp.DPSGD_NORM_MATERIALIZE, dp.DPSGD_NORM_AUTO):
        buf = dp.alloc_step([L], mode)
        dp.run_clipped_sum([L], buf, C, mode)
        torch.cuda.synchronize()
        nsq = buf.norms_sq.cpu().numpy().astype(np.float64)
        assert math.isinf(nsq[bad])
        np.testing.assert_allclose(nsq[keep], ref, rtol=3e-6)
        assert buf.factors[bad].item() == 0.0 and buf.mask.cpu().tolist() == [1, 1, 1]
        S = sum(C / np.sqrt(n) * ol.G[i].T @ ol.A[i] for i, n in zip(keep, ref))
        assert_sum_close(torch_to_float64(buf.grads[0]), S, _bound(wl.BF16, T, d_in, d_out), "sum")


@pytest.mark.parametrize("exp_a,exp_g", [(-122, 100), (100, -122), (-60, -30), (30, 40), (60, 40)])
@pytest.mark.parametrize("T,d_in,d_out", [(64, 128, 128), (33, 130, 70), (20, 200, 24)])
def test_float32_magnitudes(dp, T, d_in, d_out, exp_a, exp_g):
    """float32 operands near the ends of the float32 range (their lower bf16
    parts would leave it) keep the accuracy of ordinary ones, in the sums and,
    where the squares are in range, in the materialised norms."""
    import torch
    B = 3
    h = _host_layer(B, T, d_in, d_out, wl.F32, 79, 0)
    h.A[:] = np.ldexp(h.A, exp_a)
    h.G[:] = np.ldexp(h.G, exp_g)
    (L, A, G), = device_layers([h])
    ol, = oracle_layers([h])
    if abs(exp_a + exp_g) < 40:
        nsq = torch.empty(B, device="cuda")
        mode = dp.DPSGD_NORM_MATERIALIZE
        ws = torch.empty(dp.dpsgd_norms_workspace_bytes([L], mode), dtype=torch.uint8, device="cuda")
        dp.dpsgd_per_example_norms_multi([L], mode, nsq, workspace=ws)
        torch.cuda.synchronize()
        np.testing.assert_allclose(nsq.cpu().numpy().astype(np.float64),
                                   oracle.per_example_norms_sq([ol]), rtol=3e-6)
    factors = np.float32([0.25, 1.0, 0.01])
    nsq = torch.from_numpy((1.0 / factors.astype(np.float64) ** 2).astype(np.float32)).cuda()
    c = np.minimum(1.0, 1.0 / np.sqrt(nsq.cpu().numpy().astype(np.float64)))
    grad = torch.empty(d_out, d_in, device="cuda")
    ws = torch.empty(dp.dpsgd_clip_workspace_bytes([L]), dtype=torch.uint8, device="cuda")
    dp.dpsgd_clip_accumulate(L, nsq, 1.0, grad, workspace=ws)
    torch.cuda.synchronize()
    S = sum(c[i] * ol.G[i].T @ ol.A[i] for i in range(B))
    assert rel_err(torch_to_float64(grad), S) <= 2e-6


@pytest.mark.parametrize("accumulate", [False, True])
def test_padded_tiles_leave_out_examples_of_factor_0(dp, accumulate):
    """384 x 256 tiles with padding: an example in the middle and the last one have
    an infinite norm and rows of NaN and infinities; the sum is that of the others."""
    import torch
    B, T, d_in, d_out = 4, 1025, 1608, 2104
    assert _takes_padded_tiles(B, [(T, d_in, d_out)])
    h = _host_layer(B, T, d_in, d_out, wl.BF16, 80, 0)
    for i, value in ((1, np.nan), (3, np.inf)):
        bits = wl.bf16_bits_from_f32(np.float32([value]))[0]
        h.A[i, ::3], h.G[i, 1::5] = bits, bits
    (L, A, G), = device_layers([h])
    ol, = oracle_layers([h])
    keep = [0, 2]
    nsq = torch.tensor([4.0, math.inf, 0.25, math.inf], device="cuda")
    grad = torch.full((d_out, d_in), 0.25, device="cuda")
    ws = torch.empty(dp.dpsgd_clip_workspace_bytes([L]), dtype=torch.uint8, device="cuda")
    dp.dpsgd_clip_accumulate(L, nsq, 1.0, grad, accumulate=accumulate, workspace=ws)
    torch.cuda.synchronize()
    S = sum(c * ol.G[i].T @ ol.A[i] for i, c in zip(keep, (0.5, 1.0)))
    assert_sum_close(torch_to_float64(grad), S + (0.25 if accumulate else 0.0), 2e-6, "sum")
