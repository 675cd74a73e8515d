"""Results of the kernels that small calls and narrow layers are dealt to, on both
sides of each dispatch line, against the float64 oracle."""

import numpy as np
import pytest

import oracle
from paper_2609_20532_amd import dpsgd, workloads as wl

from parity_util import device_layers, oracle_layers, rel_err, torch_to_float64


def _layers(dtype, B, dims, seed):
    rng = np.random.default_rng(seed)
    store = wl.bf16_bits_from_f32 if dtype == wl.BF16 else (lambda x: x)
    hs = [wl.HostLayer(A=store(rng.standard_normal((B, T, di)).astype(np.float32)),
                       G=store((rng.standard_normal((B, T, do)) * 0.05).astype(np.float32)),
                       d_in=di, d_out=do, tensor_id=k, dtype=dtype)
          for k, (T, di, do) in enumerate(dims)]
    return device_layers(hs), oracle_layers(hs)


def _norms(Ls, mode, B):
    import torch
    nsq = torch.empty(B, device="cuda")
    ws = torch.empty(dpsgd.dpsgd_norms_workspace_bytes(Ls, mode), dtype=torch.uint8, device="cuda")
    dpsgd.dpsgd_per_example_norms_multi(Ls, mode, nsq, workspace=ws)
    torch.cuda.synchronize()
    return nsq.cpu().numpy().astype(np.float64)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("widths", [(1, 3), (255, 1020), (1027, 2049), (4096, 771), (4099, 6),
                                    (12289, 5), (8200, 4097)])
def test_t1_norms_at_the_edges_of_their_loads(dp, dtype, widths):
    """Four loads of a kilobyte a wave, single loads, and the last elements; one
    wave an example, and four from 48 KB on."""
    B = 5
    dev, ol = _layers(dtype, B, [(1,) + widths, (1,) + widths[::-1]], 3)
    got = _norms([d[0] for d in dev], dp.DPSGD_NORM_AUTO, B)
    np.testing.assert_allclose(got, oracle.per_example_norms_sq(ol), rtol=2e-6)


# (B, [(T, d_in, d_out), ...]): few columns, many, widths that are no multiple of
# 16 bytes, widths below them; then the same with the columns of each tile split.
GRAM = [(5, [(130, 64, 64), (130, 520, 64), (130, 65, 40), (130, 5, 3), (17, 1, 9)]),
        (5, [(2, 3, 300), (128, 384, 8), (128, 8, 392), (129, 2, 1)]),
        (1, [(100, 2000, 3), (100, 64, 64), (64, 999, 1500), (64, 2048, 16)])]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("case", range(len(GRAM)))
def test_gram_norms_of_every_kind_of_load(dp, dtype, case):
    """Each layer alone and all in one call (one launch). A tile's elements are
    added in at most 64 steps a lane, then over the lanes and tiles: up to about 80
    roundings relative to the sum of the products' absolute values."""
    B, dims = GRAM[case]
    dev, ol = _layers(dtype, B, dims, 5)

    def check(ks):
        got = _norms([dev[k][0] for k in ks], dp.DPSGD_NORM_GHOST, B)
        ref = oracle.per_example_norms_sq([ol[k] for k in ks])
        size = sum((np.abs(ol[k].A @ ol[k].A.transpose(0, 2, 1)) *
                    np.abs(ol[k].G @ ol[k].G.transpose(0, 2, 1))).sum((1, 2)) for k in ks)
        assert (np.abs(got - ref) <= 80 * 2.0 ** -24 * size).all(), [dims[k] for k in ks]

    for k in range(len(dims)):
        check([k])
    check(list(range(len(dims))))


def _partial_bytes(B, T, d_in, d_out, dtype):
    dpsgd.load()
    L = dpsgd.shape_layer(B, T, d_in, d_out, dtype, 0)
    return dpsgd.dpsgd_clip_workspace_bytes([L]) - -(-4 * B // 256) * 256


@pytest.mark.parametrize("dims,dtype,valu", [
    ((256, 256, 2, 2), dpsgd.DPSGD_F32, True),        # 28 us, 38 on an MFMA tile
    ((256, 256, 3, 16), dpsgd.DPSGD_F32, True),
    ((256, 1024, 64, 3), dpsgd.DPSGD_F32, True),
    ((256, 256, 27, 16), dpsgd.DPSGD_F32, False),
    ((16, 1024, 16, 16), dpsgd.DPSGD_F32, False),
    ((512, 16, 16, 16), dpsgd.DPSGD_F32, False),
    ((32, 100, 3, 64), dpsgd.DPSGD_BF16, True),       # 18 us, 23
    ((256, 256, 2, 2), dpsgd.DPSGD_BF16, True),
    ((512, 16, 16, 16), dpsgd.DPSGD_BF16, True),      # the weight would be rounded
    ((256, 300, 3, 64), dpsgd.DPSGD_BF16, False),
    ((32, 100, 16, 16), dpsgd.DPSGD_BF16, False),
])
def test_kernel_of_tiny_sums(dims, dtype, valu):
    """The VALU kernel keeps one partial sum per job of examples (min(B, 512) of
    them here), the MFMA kernel one per K range."""
    B, T, d_in, d_out = dims
    jobs = -(-min(B, 512) * 4 * d_in * d_out // 256) * 256
    assert (_partial_bytes(*dims, dtype) == jobs) == valu


# (dtype, B, [(T, d_in, d_out), ...]): VALU and MFMA kernels, tiny layers that join
# another's launch, partial sums of entries that are no multiple of 4.
TINY = [
    (wl.F32, 256, [(128, 2, 2), (128, 3, 24)]),
    (wl.F32, 16, [(300, 16, 16), (300, 27, 16), (100, 7, 70)]),
    (wl.F32, 8, [(31, 22, 22), (32, 22, 22), (128, 4, 7), (128, 7, 200)]),
    (wl.F32, 3, [(20, 1, 500), (40, 257, 1), (33, 7, 35)]),
    (wl.BF16, 4, [(100, 3, 64), (100, 64, 3)]),
    (wl.BF16, 4, [(300, 2, 2), (301, 2, 2), (64, 10, 10), (64, 10, 7), (65, 33, 100)]),
    (wl.BF16, 8, [(5, 10, 24), (15, 16, 16), (16, 16, 16), (17, 65, 10)]),
    (wl.BF16, 3, [(256, 16, 16), (192, 3, 20), (1024, 7, 70)]),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(TINY)))
def test_tiny_layers(dp, case):
    import torch
    dtype, B, dims = TINY[case]
    dev, ol = _layers(dtype, B, dims, 11 + case)
    Ls = [d[0] for d in dev]
    ref = oracle.per_example_norms_sq(ol)
    for mode in (dp.DPSGD_NORM_MATERIALIZE, dp.DPSGD_NORM_AUTO):
        np.testing.assert_allclose(_norms(Ls, mode, B), ref, rtol=2e-5)
    nsq = torch.from_numpy(ref.astype(np.float32)).cuda()
    C = float(np.median(np.sqrt(ref))) * 0.9
    c = np.minimum(1.0, C / np.sqrt(nsq.cpu().numpy().astype(np.float64)))
    grads = [torch.full((do, di), 0.25, device="cuda") for _, di, do in dims]
    ws = torch.empty(dp.dpsgd_clip_workspace_bytes(Ls), dtype=torch.uint8, device="cuda")
    for accumulate in (False, True):
        dp.dpsgd_clip_accumulate_multi(Ls, nsq, C, grads, accumulate=accumulate, workspace=ws)
    torch.cuda.synchronize()
    for k, (T, di, do) in enumerate(dims):
        S = 2.0 * np.einsum("i,itm,itn->mn", c, ol[k].G, ol[k].A, optimize=True)
        # float32 sums; bf16 with short T and more than 512 entries rounds c G.
        flat = dtype == wl.BF16 and di * do > 512 and not ((-T) % 64 * 8 <= T or
                                                           (T >= 64 and (-T) % 16 * 8 <= T))
        assert rel_err(torch_to_float64(grads[k]), S) <= (5e-3 if flat else 4e-6), dims[k]


@pytest.mark.parametrize("dims,dtype,form", [
    # Gram and materialised, us: 757 and 1270, 141 and 253, 11 and 21; 283 and 119,
    # 74 and 23, 766 and 657 (a short second round of Gram tiles); 19 and 25, 29 and 24.
    ((512, 256, 768, 1152), dpsgd.DPSGD_F32, dpsgd.DPSGD_NORM_GHOST),
    ((512, 128, 576, 512), dpsgd.DPSGD_F32, dpsgd.DPSGD_NORM_GHOST),
    ((64, 256, 12, 32), dpsgd.DPSGD_F32, dpsgd.DPSGD_NORM_GHOST),
    ((8, 512, 768, 3072), dpsgd.DPSGD_F32, dpsgd.DPSGD_NORM_MATERIALIZE),
    ((64, 100, 768, 256), dpsgd.DPSGD_F32, dpsgd.DPSGD_NORM_MATERIALIZE),
    ((16, 1000, 1536, 2304), dpsgd.DPSGD_F32, dpsgd.DPSGD_NORM_MATERIALIZE),
    ((2048, 65, 16, 48), dpsgd.DPSGD_BF16, dpsgd.DPSGD_NORM_GHOST),
    ((2048, 65, 144, 12), dpsgd.DPSGD_BF16, dpsgd.DPSGD_NORM_MATERIALIZE),
])
def test_auto_takes_the_faster_norm_form(dims, dtype, form):
    dpsgd.load()
    assert dpsgd.dpsgd_select_norm_mode(dpsgd.shape_layer(*dims, dtype, 0)) == form


@pytest.mark.parametrize("dims,wide", [
    ((107, 1000, 256, 200), False),     # one 384 x 256 tile: 212 us there, 40 on 128 x 128
    ((439, 183, 392, 768), False),      # four
    ((1024, 64, 192, 1000), False),     # three
    ((163, 183, 776, 776), True),       # twelve: 88 us and 98
])
def test_padded_tiles_need_several_tiles(dims, wide):
    """Partial sums are 384 x 256 tiles on the padded large tiles, whole sums on
    the any-shape kernel."""
    part = _partial_bytes(*dims, dpsgd.DPSGD_BF16)
    assert (part % (4 * 384 * 256) == 0) == wide
    assert (part % (4 * dims[2] * dims[3]) == 0) != wide


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["norms", "factors", "mask"])
def test_norms_or_outputs_inside_a_gradient(dp, where):
    """The squared norms of a small call may lie in the buffer of a gradient that
    it writes (they are read before), and an output there is overwritten by it."""
    import torch
    B, T, d_in, d_out = 512, 1, 96, 40
    dev, ol = _layers(wl.F32, B, [(T, d_in, d_out)], 23)
    L = dev[0][0]
    n = np.sqrt(oracle.per_example_norms_sq(ol))
    C = float(np.median(n))
    grad = torch.empty(d_out, d_in, device="cuda")
    inside = grad.view(-1)[64:64 + B]
    nsq = inside if where == "norms" else torch.empty(B, device="cuda")
    factors = inside if where == "factors" else torch.empty(B, device="cuda")
    mask = inside.view(torch.uint8)[:B] if where == "mask" else torch.empty(B, dtype=torch.uint8,
                                                                           device="cuda")
    nsq.copy_(torch.from_numpy((n * n).astype(np.float32)))
    ws = torch.empty(dp.dpsgd_clip_workspace_bytes([L]), dtype=torch.uint8, device="cuda")
    dp.dpsgd_clip_accumulate(L, nsq, C, grad, factors_out=factors, mask_out=mask, workspace=ws)
    torch.cuda.synchronize()
    c = np.minimum(1.0, C / n)
    S = np.einsum("i,itm,itn->mn", c, ol[0].G, ol[0].A)
    assert rel_err(torch_to_float64(grad), S) <= 2e-6
    if where != "factors":
        np.testing.assert_allclose(factors.cpu().numpy(), c, rtol=1e-6)


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(40, 130, 70), (300, 24, 16), (1, 200, 33), (1, 1000, 900)])
def test_float32_sums_with_a_nan_factor(dp, dims):
    """A NaN norm makes the example's factor NaN and with it every entry."""
    import torch
    B = 70
    dev, ol = _layers(wl.F32, B, [dims], 29)
    L = dev[0][0]
    nsq = torch.from_numpy(oracle.per_example_norms_sq(ol).astype(np.float32)).cuda()
    nsq[B - 2] = float("nan")
    grad = torch.zeros(dims[2], dims[1], device="cuda")
    factors = torch.empty(B, device="cuda")
    ws = torch.empty(dp.dpsgd_clip_workspace_bytes([L]), dtype=torch.uint8, device="cuda")
    dp.dpsgd_clip_accumulate(L, nsq, 1.0, grad, factors_out=factors, workspace=ws)
    torch.cuda.synchronize()
    assert torch.isnan(grad).all()
    assert torch.isnan(factors[B - 2]) and torch.isfinite(factors).sum().item() == B - 1
