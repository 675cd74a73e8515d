"""Stored per-example gradients at the edges of their kernels' loads: the last
rows and columns of the tensors, every way the narrow block is read (ranks that
are multiples of 4, and others), a wide side of one 16-byte chunk, partly filled
row blocks, and float32 layers with and without shared activations."""

import numpy as np
import pytest

import oracle
from paper_2609_20532_amd import workloads as wl

from parity_util import device_layers, oracle_layers, rel_err, torch_to_float64

pytestmark = pytest.mark.gpu

# (dtype, B, [(T, d_in, d_out), ...], share the first layer's A)
CASES = [
    (wl.BF16, 1, [(33, 136, 4), (33, 4, 136)], False),
    (wl.BF16, 3, [(65, 8, 8), (97, 128, 8), (64, 8, 264)], False),
    (wl.BF16, 2, [(115, 128, 16), (127, 16, 136), (101, 12, 128)], False),
    (wl.BF16, 2, [(31, 128, 1), (40, 5, 136), (90, 136, 7), (120, 15, 256)], False),
    (wl.F32, 2, [(33, 260, 4), (17, 3, 256)], False),
    (wl.F32, 3, [(70, 768, 4), (70, 768, 8)], True),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_stored_gradients_match_oracle(dp, case):
    import torch
    dtype, B, dims, share = CASES[case]
    rng = np.random.default_rng(40 + case)
    store = wl.bf16_bits_from_f32 if dtype == wl.BF16 else (lambda x: x)
    hs = []
    for k, (T, di, do) in enumerate(dims):
        A = hs[0].A if share and k else store(rng.standard_normal((B, T, di)).astype(np.float32))
        G = store((rng.standard_normal((B, T, do)) * 0.05).astype(np.float32))
        hs.append(wl.HostLayer(A=A, G=G, d_in=di, d_out=do, tensor_id=k, dtype=dtype))
        esz = 2 if dtype == wl.BF16 else 4
        assert min(di, do) <= 16 and 16 * di * do <= T * (di + do) * esz, "not a stored layer"
    dev = device_layers(hs)
    Ls = [d[0] for d in dev]
    ol = oracle_layers(hs)
    nsq = oracle.per_example_norms_sq(ol)
    C = float(np.median(np.sqrt(nsq))) * 0.95
    buf = dp.alloc_step(Ls, fused=True)
    dp.run_clipped_sum(Ls, buf, C, fused=True)
    torch.cuda.synchronize()
    # float32 sums of at most a few hundred terms.
    np.testing.assert_allclose(buf.norms_sq.cpu().numpy().astype(np.float64), nsq, rtol=2e-6)
    c = np.minimum(1.0, C / np.sqrt(nsq))
    for k in range(len(dims)):
        S = sum(c[i] * ol[k].G[i].T @ ol[k].A[i] for i in range(B))
        assert rel_err(torch_to_float64(buf.grads[k]), S) <= 2e-6, dims[k]
