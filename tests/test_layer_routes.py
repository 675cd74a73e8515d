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
@pytest.mark.parametrize("widths", [(1, 3), (255, 1020), (1027, 2049), (4096, 771), (4099, 6)])
def test_t1_norms_at_the_edges_of_their_loads(dp, dtype, widths):
    """Four loads of a kilobyte a wave, single loads, and the last elements."""
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
