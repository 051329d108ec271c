"""2D local energies with the state window in shared memory: FP32 models
against an FP64 model of the same parameters, 2e-4 relative (the bound of the
FP32 local energies; 144 sites of FP32 rounding in an exponent), at one sample,
ragged groups of 16, two columns, the widest lattices that fit and the first
that does not, with the mask, with J2 = 0, and FP64 against the oracle."""
import numpy as np
import pytest
import torch

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Lx,Ly,Ns,cplx,zm,J2", [
    (16, 2, 2, 1, True, False, 0.5), (16, 9, 4, 33, False, True, 0.5), (16, 16, 2, 17, True, False, 0.0),
    (32, 5, 4, 16, True, False, 0.5), (32, 16, 3, 47, False, True, 0.0), (64, 3, 6, 31, True, True, 0.5),
    (128, 4, 4, 15, False, False, 0.5), (128, 13, 2, 20, True, False, 0.5), (128, 14, 2, 20, True, False, 0.5),
])
def test_eloc_2d_against_fp64(H, Lx, Ly, Ns, cplx, zm, J2):
    ms = [pm.Model(Lx, Ly, 2, hidden=H, complex_head=cplx, marshall=True, zero_mag=zm, dtype=d,
                   seed=H + Lx, max_Ns=Ns) for d in ("f32", "f64")]
    rng = np.random.default_rng(Lx * Ly)
    th = ms[1].get_params()
    th = th + torch.from_numpy(0.1 * rng.normal(size=th.numel())).cuda()
    for m in ms:
        m.set_params(th)
    sig, _ = ms[1].sample(Ns, key=2)
    ham = pm.hamiltonian("j1j2", J=1.0, J2=J2)
    e = [m.local_energy(ham, sig, m.logpsi(sig))[0] for m in ms]
    assert (e[0] - e[1]).abs().max() <= 2e-4 * e[1].abs().max()
    for m in ms:
        m.close()


@pytest.mark.parametrize("dim,H,Lx,Ly,Ns", [(1, 16, 10, 1, 5), (1, 64, 6, 1, 19), (2, 32, 4, 3, 18)])
def test_eloc_fp64_against_oracle(dim, H, Lx, Ly, Ns):
    from oracle import hamiltonian, model
    spec = model.Spec(Lx=Lx, Ly=Ly, dim=dim, H=H, complex_head=True)
    m = pm.Model(Lx, Ly, dim, hidden=H, complex_head=True, dtype="f64", seed=9, max_Ns=Ns)
    sig, lp = m.sample(Ns, key=6)
    kind = "cluster" if dim == 1 else "j1j2"
    e = m.local_energy(pm.hamiltonian(kind, J2=0.5, pbc=True), sig, lp)[0].cpu().numpy()
    th = m.get_params().cpu().numpy()
    ref = hamiltonian.local_energy(spec, th, hamiltonian.Ham(kind, J2=0.5, pbc=True),
                                   sig.cpu().numpy().astype(np.int64))
    assert np.max(np.abs(e - ref)) <= 1e-10 * np.max(np.abs(ref))
    m.close()
