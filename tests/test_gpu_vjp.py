"""The vector-Jacobian product against the product of the library's own rows:
one row, ragged chunks of 32 rows, widths beside a multiple of 64 columns."""
import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Ns,cplx,dtype", [(8, 1, True, "f64"), (16, 33, False, "f32"),
                                             (32, 95, True, "f32"), (64, 290, False, "f64")])
def test_vjp_is_the_weighted_row_sum(H, Ns, cplx, dtype):
    m = pm.Model(7, hidden=H, complex_head=cplx, dtype=dtype, seed=Ns, max_Ns=Ns)
    sig, _ = m.sample(Ns, key=4)
    g = torch.randn((Ns, 2), dtype=torch.float64, generator=torch.Generator().manual_seed(H)).cuda()
    got = m.logpsi_vjp(sig, torch.view_as_complex(g))
    O = m.jacobian(sig)[0].double() * Ns ** 0.5
    w = torch.cat([g[:, 0], g[:, 1]]) if cplx else g[:, 0]
    # FP64 sums of the same rows in another order
    tol = 4 * O.shape[0] * 2.0 ** -53 * (O.abs().T @ w.abs())
    assert ((got - O.T @ w).abs() <= tol + 1e-300).all()
    m.close()
