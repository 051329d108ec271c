"""The parameter-space metric of few rows, whose tiles write it directly:
parameter counts beside a multiple of 64 columns, one row to a K step and
more, against torch's product of the same centred rows, each entry within
4 K u sqrt(S_ii S_jj) (K rows, u = 2^-53, twice the bound of either order) and
1e-13 of the largest diagonal entry for the centring's rounding; FP32 rows to
1e-5.  Exactly symmetric, and no entry outside the metric written."""
import ctypes

import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Ns,max_Ns,cplx,dtype", [(8, 1, 1, False, "f64"), (8, 7, 400, True, "f64"),
                                                    (16, 17, 17, False, "f64"), (16, 33, 33, True, "f32"),
                                                    (64, 3, 3, False, "f64"), (32, 40, 40, True, "f64")])
def test_metric_of_few_rows(H, Ns, max_Ns, cplx, dtype):
    m = pm.Model(3, 4, 2, hidden=H, complex_head=cplx, dtype=dtype, seed=H + Ns, max_Ns=max_Ns)
    sig, _ = m.sample(Ns, key=Ns)
    R = torch.cat([o - o.mean(dim=0, keepdim=True) for o in m.jacobian(sig)[0].double().split(Ns)])
    n = m.Np
    buf = torch.full((n + 2, n), 7.0, dtype=torch.float64, device="cuda")
    p = ctypes.c_void_p
    assert pm.lib().minsr_param_gram(m.handle, Ns, p(sig.data_ptr()), p(buf[1].data_ptr()),
                                     p(torch.cuda.current_stream().cuda_stream)) == 0
    torch.cuda.synchronize()
    S, ref = buf[1:-1], R.T.contiguous() @ R
    assert (buf[0] == 7.0).all() and (buf[-1] == 7.0).all()
    assert torch.equal(S, S.T)
    if dtype == "f64":
        d = torch.sqrt(torch.diagonal(ref))
        tol = 4 * R.shape[0] * 2.0 ** -53 * torch.outer(d, d) + 1e-13 * d.max() ** 2 + 1e-300
        assert ((S - ref).abs() <= tol).all()
    else:
        assert (S - ref).abs().max() <= 1e-5 * S.abs().max()
    m.close()
