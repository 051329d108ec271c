"""The matrix-core recurrence against the vector recurrence, bit for bit, at the
ends of what it serves: evaluations of narrow chains, which it takes from twice
the samples on (N_s d_h = 196608, FP64 131072) and whose conditionals it forms
four sites at a time; the widest lattices whose state window fits shared memory
(Lx = 13 at d_h = 128, FP64 64; 14 is the vector kernel's); models of eight
units, whose tiles are half filled."""
import numpy as np
import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu

# (dim, dtype, H, Lx, Ly, Ns, cplx, zero_mag)
CASES = [
    (1, "f32", 16, 5, 1, 12289, False, False),
    (1, "f32", 16, 8, 1, 12303, True, True),
    (1, "f32", 32, 9, 1, 6145, True, False),
    (1, "f32", 32, 2, 1, 6144, False, False),
    (1, "f64", 16, 6, 1, 8195, True, True),
    (1, "f64", 16, 7, 1, 8192, False, False),
    (1, "f64", 8, 19, 1, 16385, True, False),
    (1, "f64", 8, 4, 1, 16384, False, True),
    (2, "f32", 128, 13, 2, 769, True, False),
    (2, "f32", 128, 14, 2, 769, True, False),
    (2, "f64", 64, 13, 2, 18, True, True),
    (2, "f64", 64, 14, 2, 18, False, False),
    (2, "f64", 8, 2, 2, 1, True, False),
    (2, "f64", 8, 16, 3, 17, False, True),
    (2, "f64", 8, 3, 7, 33, True, False),
]


@pytest.mark.parametrize("dim,dtype,H,Lx,Ly,Ns,cplx,zm", CASES)
def test_ends_of_the_matrix_core_recurrence(dim, dtype, H, Lx, Ly, Ns, cplx, zm):
    m = pm.Model(Lx, Ly, dim, hidden=H, complex_head=cplx, marshall=dim == 2, zero_mag=zm,
                 dtype=dtype, seed=3 * H + Lx, max_Ns=Ns)
    th = m.get_params()
    rng = np.random.default_rng(H + Lx)
    m.set_params(th + torch.from_numpy(0.2 * rng.normal(size=th.numel())).cuda())
    got = []
    for r in (0, 1):
        m.set_tunable("sample_r", r)
        out = list(m.sample(Ns, key=3, counter=7))
        out.append(m.logpsi(out[0]))
        out.append(m.jacobian(out[0], ckpt_every=1)[0])   # from the evaluation's states and tape
        torch.cuda.synchronize()
        got.append([t.clone() for t in out])
    m.close()
    assert torch.isfinite(torch.view_as_real(got[0][2])).all()
    for a, b in zip(*got):
        assert torch.equal(a, b)


# complex models whose tapes are larger than the workspace: the second seed's
# adjoints of a later chunk of samples
@pytest.mark.parametrize("dtype,H,parts,Ns", [("f32", 32, 1, 2190), ("f64", 16, 1, 2170)])
def test_chunked_jacobian_of_a_complex_model(dtype, H, parts, Ns):
    m = pm.Model(16, 64, 2, hidden=H, complex_head=True, marshall=True, dtype=dtype, seed=H, max_Ns=Ns)
    sig, _ = m.sample(Ns, key=1, counter=2)
    O = m.jacobian(sig)[0].clone()
    m.set_tunable("jac_parts", parts)
    ref = m.jacobian(sig)[0]
    torch.cuda.synchronize()
    assert torch.isfinite(ref).all() and ref[Ns:].abs().max() > 0
    if dtype == "f32":
        assert torch.equal(O, ref)
    else:
        assert (O - ref).abs().max() <= 1e-12 * ref.abs().max()
    m.close()
