"""Pseudo-inverse at the edges of the tridiagonalisation's panels (16), of its
workgroups' rows (4, 32) and of the back-transformation's blocks (64)."""
import numpy as np
import pytest
import torch

from oracle import minsr as ominsr
from tests.gpu_common import gpu, need_gpu, to_dev
from tests import inputs

pytestmark = gpu


@pytest.fixture(scope="module")
def pmodel():
    need_gpu()
    import paper_2608_18065_amd as pm
    return pm.Model(16, hidden=16, dtype="f64", seed=1, max_Ns=1100, pinv=True)


# forward error of a backward-stable eigensolver, ~ n u lambda_max / lambda_min,
# on both sides: 4 n u cond <= 1e-9 at cond = 1e3 and these n
@pytest.mark.parametrize("n", [2, 8, 9, 15, 16, 17, 18, 63, 66, 127, 128, 129, 1024, 1025, 1026])
def test_pinv_at_block_edges(pmodel, n):
    rng = np.random.default_rng(n)
    T, _ = inputs.psd_matrix(inputs.spectrum_loguniform(n, 1e3, rng), seed=n)
    # identity rows: reflectors that are the identity, at the end and across a
    # panel boundary
    if n > 17:
        for k in (16, n - 1):
            T[k, :] = 0.0
            T[:, k] = 0.0
            T[k, k] = 0.5
    b = inputs.rhs(n, seed=n)
    x, st = pmodel.solve(to_dev(T), to_dev(b), lam=0.0, pinv_cutoff=1e-8)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    ref = ominsr.solve(T, b, 0.0, 1e-8)
    assert np.linalg.norm(x.cpu().numpy() - ref) < 1e-9 * np.linalg.norm(ref)
