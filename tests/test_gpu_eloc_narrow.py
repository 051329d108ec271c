"""Local energies of FP32 chains of 16 units, which the matrix-core recurrence
serves: against an FP64 model of the same parameters."""
import pytest

import paper_2608_18065_amd as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Lx,Ns", [(3, 1), (10, 17), (33, 31)])
def test_narrow_chain_eloc_fp32_against_fp64(Lx, Ns):
    # chains of 16 units in FP32, 2e-4 relative: the bound of FP32 local energies
    ms = [pm.Model(Lx, 1, 1, hidden=16, complex_head=True, dtype=d, seed=Lx, max_Ns=Ns)
          for d in ("f32", "f64")]
    sig, _ = ms[1].sample(Ns, key=2)
    for kind in ("cluster", "tfim"):
        ham = pm.hamiltonian(kind, J=1.0, h=0.7, pbc=False)
        ms[0].set_params(ms[1].get_params())
        e = [m.local_energy(ham, sig, m.logpsi(sig))[0] for m in ms]
        assert (e[0] - e[1]).abs().max() <= 2e-4 * e[1].abs().max()
    for m in ms:
        m.close()
