"""The gate tape of 2D models, which the matrix-core Jacobian reads, as every
form of the vector recurrence writes it (one and four sequences a thread, in
evaluation and in sampling) against the matrix-core recurrence's: rows and
steps equal bit for bit.  FP64 models of 8 units to 1e-12 (order of sums)."""
import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,Lx,Ly,Ns", [("f32", 32, 3, 4, 17), ("f32", 64, 5, 2, 33), ("f32", 128, 4, 3, 770),
                                              ("f64", 8, 3, 3, 33), ("f64", 16, 2, 5, 18), ("f64", 32, 4, 3, 9),
                                              ("f64", 64, 3, 3, 5)])
def test_tape_of_every_form(dtype, H, Lx, Ly, Ns):
    m = pm.Model(Lx, Ly, 2, hidden=H, complex_head=True, marshall=True, dtype=dtype, seed=H, max_Ns=Ns)
    sig, _ = m.sample(Ns, key=2)
    ham = pm.hamiltonian("j1j2", J=1.0, J2=0.5)
    form = pm.FORM_FP64_REF if dtype == "f64" else pm.FORM_BF16_FP64
    got = []
    for r in (0, 1, 4):
        m.set_tunable("sample_r", r)
        mom = torch.zeros(m.Np, dtype=torch.float64, device="cuda")
        rows = m.jacobian(sig)[0].clone()
        m.step(ham, Ns, 0.01, 1e-2, 0.0, mom, 3, 0, form=form, apply_update=False)
        got.append((rows, m.intermediates(form)["Oprime"].clone()))
        torch.cuda.synchronize()
    for a in got[1:]:
        for x, y in zip(a, got[0]):
            if H == 8:
                assert (x.double() - y.double()).abs().max() <= 1e-12 * y.double().abs().max()
            else:
                assert torch.equal(x, y)
    m.close()
