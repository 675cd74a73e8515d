"""float32 layers that AUTO moves from the Gram form to the materialised one:
where the line lies, that calls whose partials would outgrow the
allocation-free call's scratch keep the Gram form, and the results against the
float64 oracle, the explicit Gram form and the allocation-free call."""

import numpy as np
import pytest

import oracle
from paper_2609_20532_amd import dpsgd, workloads as wl

from parity_util import device_layers, oracle_layers


def _shape(B, T, d_in, d_out, dtype):
    return dpsgd.shape_layer(B, T, d_in, d_out, dtype, 0)


@pytest.mark.parametrize("dims,form", [
    ((8, 512, 768, 3072), dpsgd.DPSGD_NORM_MATERIALIZE),
    ((123, 128, 512, 1536), dpsgd.DPSGD_NORM_GHOST),
    ((64, 8, 770, 3072), dpsgd.DPSGD_NORM_MATERIALIZE),
    ((256, 64, 1152, 256), dpsgd.DPSGD_NORM_GHOST),          # the T <= 64 Gram kernel
    ((1700, 450, 384, 50257), dpsgd.DPSGD_NORM_MATERIALIZE),  # 1179 partials an example: 8.0 MB
    ((1800, 450, 384, 50257), dpsgd.DPSGD_NORM_GHOST),        # 8.5 MB of partials
])
def test_auto_form_of_float32_layers(dims, form):
    dpsgd.load()
    L = _shape(*dims, dpsgd.DPSGD_F32)
    assert dpsgd.dpsgd_select_norm_mode(L) == form
    partials = 4 * dims[0] * (-(-dims[2] // 128)) * (-(-dims[3] // 128))
    ws = dpsgd.dpsgd_norms_workspace_bytes([L], dpsgd.DPSGD_NORM_AUTO)
    if form == dpsgd.DPSGD_NORM_MATERIALIZE:
        assert partials <= ws <= 8 << 20
    else:
        assert ws == dpsgd.dpsgd_norms_workspace_bytes([L], dpsgd.DPSGD_NORM_GHOST)


def test_bf16_forms_do_not_move():
    dpsgd.load()
    for dims in [(8, 512, 770, 3072), (64, 200, 770, 768), (64, 100, 384, 1500)]:
        assert dpsgd.dpsgd_select_norm_mode(_shape(*dims, dpsgd.DPSGD_BF16)) == dpsgd.DPSGD_NORM_GHOST


@pytest.mark.gpu
@pytest.mark.parametrize("B,dims", [
    (3, [(512, 256, 520)]),
    (5, [(8, 257, 1031)]),                                 # odd widths, short rows
    (2, [(513, 129, 900)]),                                # one row past the row blocks
    (4, [(65, 96, 700), (65, 300, 40), (64, 64, 128), (1, 33, 7)]),   # both forms in one call
])
def test_auto_matches_oracle_and_gram_form(B, dims):
    import torch
    dpsgd.load()
    rng = np.random.default_rng(7)
    hs = [wl.HostLayer(A=rng.standard_normal((B, T, di)).astype(np.float32),
                       G=(rng.standard_normal((B, T, do)) * 0.05).astype(np.float32),
                       d_in=di, d_out=do, tensor_id=k, dtype=wl.F32)
          for k, (T, di, do) in enumerate(dims)]
    dev = device_layers(hs)
    Ls = [d[0] for d in dev]
    assert dpsgd.dpsgd_select_norm_mode(Ls[0]) == dpsgd.DPSGD_NORM_MATERIALIZE
    out = {}
    for mode in (dpsgd.DPSGD_NORM_AUTO, dpsgd.DPSGD_NORM_GHOST):
        ws = torch.empty(dpsgd.dpsgd_norms_workspace_bytes(Ls, mode), dtype=torch.uint8, device="cuda")
        out[mode] = torch.empty(B, device="cuda")
        dpsgd.dpsgd_per_example_norms_multi(Ls, mode, out[mode], workspace=ws)
    noalloc = torch.empty(B, device="cuda")
    dpsgd.dpsgd_per_example_norms_multi_noalloc(Ls, dpsgd.DPSGD_NORM_AUTO, noalloc)
    torch.cuda.synchronize()
    assert torch.equal(noalloc, out[dpsgd.DPSGD_NORM_AUTO])
    ref = oracle.per_example_norms_sq(oracle_layers(hs))
    for v in out.values():
        # Every entry is a float32 dot product over T or d rows: rounding errors
        # of about 1e-7 relative to the sum of squares that dominates the norm.
        np.testing.assert_allclose(v.cpu().numpy().astype(np.float64), ref, rtol=5e-6)
