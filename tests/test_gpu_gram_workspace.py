"""FP64 Grams of fewer rows than a model's workspace is sized for: the split
over columns that suits the call has more partial tiles than the workspace.
Against torch's product of the same centred rows, each entry within
4 K u sqrt(T_ii T_jj), u = 2^-53, twice the bound of either summation order,
and 1e-13 of the largest diagonal entry for the centring's own rounding."""
import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu


# (largest Ns, Ns, split asked for): 484 columns, two rows a sample
@pytest.mark.parametrize("max_Ns,Ns,split", [(1280, 1248, 0), (1280, 1248, 64), (1088, 1024, 8), (33, 20, 64)])
def test_gram_f64_below_the_largest_size(max_Ns, Ns, split):
    m = pm.Model(3, 3, 2, hidden=8, complex_head=True, marshall=True, dtype="f64", seed=Ns, max_Ns=max_Ns)
    m.set_tunable("gram_split", split)
    sig, _ = m.sample(Ns, key=Ns)
    T = m.gram(sig)
    R = torch.cat([o - o.mean(dim=0, keepdim=True) for o in m.jacobian(sig)[0].split(Ns)])
    ref = R @ R.T.contiguous()
    d = torch.sqrt(torch.diagonal(ref))
    tol = 4 * R.shape[1] * 2.0 ** -53 * torch.outer(d, d) + 1e-13 * d.max() ** 2
    assert ((T - ref).abs() <= tol).all()
    assert torch.equal(T, T.T)
    m.close()
