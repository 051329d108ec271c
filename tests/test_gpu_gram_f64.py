"""FP64 Gram and parameter-space metric tiles at their edges: one row, one
tile and a row more, ragged last tiles, K ranges of one block and several, a
metric with more rows than parameters and the reverse.

Both are sums of n products in FP64: against torch's product of the same
centred rows each entry is held to 4 K u sqrt(T_ii T_jj), u = 2^-53, twice the
bound of either summation order.
"""
import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu


def centred(m, sig):
    O = m.jacobian(sig)[0]
    Ns = sig.shape[0]
    return torch.cat([o - o.mean(dim=0, keepdim=True) for o in O.split(Ns)])


def check(T, R):
    ref = R @ R.T.contiguous()
    d = torch.sqrt(torch.diagonal(ref))
    tol = 4 * R.shape[1] * 2.0 ** -53 * torch.outer(d, d) + 1e-300
    # the centring's own rounding (u |row mean|) enters both operands
    assert ((T - ref).abs() <= tol + 1e-13 * d.max() ** 2).all()
    assert torch.equal(T, T.T)


@pytest.mark.parametrize("H,Ns,cplx,split", [(8, 1, False, 0), (8, 64, False, 0), (16, 65, False, 0),
                                             (16, 130, True, 3), (32, 37, True, 64), (64, 200, False, 1)])
def test_gram_f64_tiles(H, Ns, cplx, split):
    m = pm.Model(9, hidden=H, complex_head=cplx, dtype="f64", seed=H + Ns, max_Ns=Ns)
    m.set_tunable("gram_split", split)
    sig, _ = m.sample(Ns, key=Ns)
    check(m.gram(sig), centred(m, sig))
    m.close()


@pytest.mark.parametrize("H,Ns,cplx,dtype", [(8, 1, True, "f64"), (8, 700, True, "f64"), (16, 33, False, "f64"),
                                             (16, 65, True, "f32"), (32, 16, False, "f64")])
def test_param_gram_tiles(H, Ns, cplx, dtype):
    m = pm.Model(3, 4, 2, hidden=H, complex_head=cplx, dtype=dtype, seed=H + Ns, max_Ns=Ns)
    sig, _ = m.sample(Ns, key=Ns)
    R = centred(m, sig).double()
    S = m.param_gram(sig)
    if dtype == "f64":
        check(S, R.T.contiguous())
    else:   # FP32 rows centred in FP32: their rounding
        assert (S - R.T @ R).abs().max() <= 1e-5 * S.abs().max()
    m.close()
