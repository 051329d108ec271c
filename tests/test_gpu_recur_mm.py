"""The matrix-core recurrence against the vector recurrence, bit for bit.

Both evaluate the same fused multiply-add chains, cell and head expressions,
so samples, log-amplitudes and the stored states (through the Jacobian's
rows) must be equal, not merely close.  Sizes sit where the built-in choice
takes the matrix cores, at ragged last workgroups, and around the largest
lattice whose state window fits shared memory.
"""
import numpy as np
import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu

# (dim, dtype, H, Lx, Ly, Ns, cplx, zero_mag)
CASES = [
    (1, "f32", 16, 5, 1, 6145, False, False),
    (1, "f32", 32, 9, 1, 3073, True, False),
    (1, "f32", 64, 34, 1, 1537, False, True),
    (1, "f32", 128, 12, 1, 770, True, False),
    (1, "f64", 16, 6, 1, 4099, True, True),
    (1, "f64", 32, 19, 1, 7, False, False),
    (1, "f64", 64, 2, 1, 17, True, False),
    (2, "f32", 16, 3, 2, 1, True, False),
    (2, "f32", 32, 16, 2, 15, False, True),
    (2, "f32", 64, 4, 5, 33, True, False),
    (2, "f32", 128, 5, 4, 769, False, True),
    (2, "f32", 128, 16, 2, 769, True, False),    # window too large: vector either way
    (2, "f64", 16, 2, 7, 31, False, False),
    (2, "f64", 32, 7, 3, 16, True, False),
    (2, "f64", 64, 16, 2, 18, True, True),
]


@pytest.mark.parametrize("dim,dtype,H,Lx,Ly,Ns,cplx,zm", CASES)
def test_matrix_core_recurrence_equals_vector(dim, dtype, H, Lx, Ly, Ns, cplx, zm):
    m = pm.Model(Lx, Ly, dim, hidden=H, complex_head=cplx, marshall=True, zero_mag=zm,
                 dtype=dtype, seed=11 * H + Lx, max_Ns=Ns)
    th = m.get_params()
    rng = np.random.default_rng(H + Lx)
    m.set_params(th + torch.from_numpy(0.2 * rng.normal(size=th.numel())).cuda())
    u = torch.from_numpy(rng.random((Ns, Lx * Ly)))
    got = []
    for r in (0, 1):
        m.set_tunable("sample_r", r)
        out = list(m.sample(Ns, key=3, counter=7)) + list(m.sample(Ns, uniforms=u))
        out.append(m.logpsi(out[2]))
        out += [m.jacobian(out[2], ckpt_every=C)[0] for C in ((1, 3) if dim == 1 else (1,))]
        torch.cuda.synchronize()
        got.append([t.clone() for t in out])
    m.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert torch.isfinite(torch.view_as_real(got[0][4])).all()
