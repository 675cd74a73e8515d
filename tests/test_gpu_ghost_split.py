"""Gram-form norms of calls with few tiles, whose columns are split over
several workgroups, against the float64 oracle, against the unsplit tiles and
against the allocation-free call, which splits the same way.

A batch with many copies of the examples has too many tiles to be split, so
its first examples give the unsplit result.
The cases sit at the edges of the split: one example, one and several row
blocks, T at and around a multiple of 128, widths that are a multiple of the
column slice, of 16 bytes, and odd, a last slice of one column, and one of the
two sides far wider than the other; both element types.
"""

import numpy as np
import pytest

import oracle
from paper_2609_20532_amd import workloads as wl

from parity_util import device_layers, oracle_layers

pytestmark = pytest.mark.gpu

# (dtype, B, [(T, d_in, d_out), ...])
CASES = [
    (wl.BF16, 1, [(128, 1024, 4096)]),
    (wl.BF16, 4, [(128, 768, 5025)]),               # odd width, one row block
    (wl.BF16, 2, [(129, 1031, 1000)]),              # second row block of one row
    (wl.BF16, 3, [(200, 2048, 64)]),               # G takes a single slice
    (wl.BF16, 2, [(300, 1000, 1608)]),              # three row blocks, multiples of 8
    (wl.BF16, 2, [(17, 4097, 3)]),                  # last slices of one and three columns
    (wl.BF16, 2, [(64, 2048, 2048), (100, 999, 2000), (1, 64, 48)]),   # several layers, one T = 1
    (wl.F32, 2, [(128, 1000, 1500)]),
    (wl.F32, 1, [(130, 2049, 513)]),                # odd widths
    (wl.F32, 3, [(65, 1027, 1028), (257, 516, 800)]),
]


def _host_layer(B, T, d_in, d_out, dtype, seed, tensor_id):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((B, T, d_in)).astype(np.float32)
    G = (rng.standard_normal((B, T, d_out)) * 0.05).astype(np.float32)
    store = wl.bf16_bits_from_f32 if dtype == wl.BF16 else (lambda x: x)
    return wl.HostLayer(A=store(A), G=store(G), d_in=d_in, d_out=d_out, tensor_id=tensor_id,
                        dtype=dtype)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_split_tiles_match_oracle_and_whole_tiles(dp, case):
    import torch
    dtype, B, dims = CASES[case]
    hs = [_host_layer(B, T, di, do, dtype, 500 + 10 * case + k, k)
          for k, (T, di, do) in enumerate(dims)]
    dev = device_layers(hs)
    Ls = [d[0] for d in dev]
    # The split needs room for the partial 128 x 128 tiles (64 KB each).
    need = dp.dpsgd_norms_workspace_bytes(Ls, dp.DPSGD_NORM_GHOST)
    assert need >= 2 * 65536, "the case does not take the split route"
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    got = torch.full((B,), 0.25, dtype=torch.float32, device="cuda")
    dp.dpsgd_per_example_norms_multi(Ls, dp.DPSGD_NORM_GHOST, got, accumulate=True, workspace=ws)
    again = torch.empty_like(got)
    dp.dpsgd_per_example_norms_multi(Ls, dp.DPSGD_NORM_GHOST, again, workspace=ws)
    noalloc = torch.empty_like(got)
    dp.dpsgd_per_example_norms_multi_noalloc(Ls, dp.DPSGD_NORM_GHOST, noalloc)
    # 60 examples or more: over 112 / 3 tiles.
    rep = -(-60 // B)
    copies = [(A.repeat(rep, 1, 1), G.repeat(rep, 1, 1)) for _, A, G in dev]
    many = [dp.make_layer(A, G, k) for k, (A, G) in enumerate(copies)]
    whole = torch.empty(rep * B, dtype=torch.float32, device="cuda")
    ws2 = torch.empty(dp.dpsgd_norms_workspace_bytes(many, dp.DPSGD_NORM_GHOST), dtype=torch.uint8,
                      device="cuda")
    dp.dpsgd_per_example_norms_multi(many, dp.DPSGD_NORM_GHOST, whole, workspace=ws2)
    torch.cuda.synchronize()
    ref = oracle.per_example_norms_sq(oracle_layers(hs))
    g = again.cpu().numpy().astype(np.float64)
    # Sums of float32 products over at most 128 x 128 Gram entries: rounding
    # errors of about 1e-7 relative to the sum of squares that dominates it.
    np.testing.assert_allclose(g, ref, rtol=5e-6)
    np.testing.assert_allclose(g, whole[:B].cpu().numpy().astype(np.float64), rtol=5e-6)
    assert torch.equal(noalloc, again)
    np.testing.assert_allclose(got.cpu().numpy().astype(np.float64) - 0.25, ref, rtol=1e-5,
                               atol=1e-6)
