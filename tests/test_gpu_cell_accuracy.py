"""The FP64 nonlinearities against 80-bit values, each seen through a model
whose other parts are exact: with zero weights the first site's state is
u tanh(b_in), u the logistic function of b_u, and the phase's derivative by
U_phi[0] is pi times it (one rounding); with two equal spins log Psi is
-log(1 + e^-d), d the difference of the output biases.

Bounds in 2^-52 of the value: the functions' largest errors in units in the
last place as cell.hpp states them (tanh 0.86, logistic 2.38, log1p 0.71 with
its argument's 0.64), and the product's half: 1.4, 2.9, 1.4.  Both kernels of
the recurrence."""
import numpy as np
import pytest
import torch

import paper_2608_18065_amd as pm
from oracle import model as omodel

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(np.finfo(np.longdouble).nmant < 63, reason="no 80-bit long double")]
H = 64


@pytest.fixture(params=[0, 1], ids=["matrix", "vector"])
def model(request):
    m = pm.Model(2, hidden=H, complex_head=True, dtype="f64", seed=1, max_Ns=1)
    m.set_tunable("sample_r", request.param)
    m.set_tunable("jac_parts", request.param)
    yield m
    m.close()


def _blocks():
    at, out = 0, {}
    for name, shape in omodel.layout(omodel.Spec(Lx=2, H=H, complex_head=True)):
        n = int(np.prod(shape))
        out[name] = slice(at, at + n)
        at += n
    return out, at


def _states(m, b_u, b_in):
    """pi times the first site's state, units with the given biases"""
    blk, n = _blocks()
    got = []
    for i in range(0, len(b_u), H):
        th = np.zeros(n)
        th[blk["bu"]], th[blk["bin"]] = b_u[i:i + H], b_in[i:i + H]
        m.set_params(torch.from_numpy(th).cuda())
        O = m.jacobian(torch.tensor([[0, 1]], dtype=torch.uint8, device="cuda"))[0]
        got.append(O[1].cpu().numpy()[blk["Uphi"]][:H])
    return np.concatenate(got)


def _close(got, ref, bound):
    err = np.abs(got.astype(np.longdouble) - ref) / np.abs(ref)
    assert float(err.max()) <= bound * 2.0 ** -52, float(err.max()) * 2.0 ** 52


PI = np.longdouble(np.pi)


def test_tanh(model):
    rng = np.random.default_rng(1)
    x = np.concatenate([rng.uniform(-20, 20, 8 * H), rng.normal(size=8 * H),
                        10.0 ** rng.uniform(-290, 0, 4 * H) * rng.choice((-1, 1), 4 * H)])
    _close(_states(model, np.full(len(x), 60.0), x), PI * np.tanh(x.astype(np.longdouble)), 1.4)


def test_logistic(model):
    rng = np.random.default_rng(2)
    x = np.concatenate([rng.uniform(-700, 40, 8 * H), rng.uniform(-8, 8, 8 * H)])
    x[:6] = -689.9, -690.0, -690.1, -700.0, 745.0, np.inf
    ref = PI / (1 + np.exp(-x.astype(np.longdouble)))
    _close(_states(model, x, np.full(len(x), 50.0)), ref, 2.9)
    # below the normal numbers: e^x to a unit and a half of the smallest, times pi
    x = np.resize([-710.0, -720.0, -744.0, -746.0, -800.0, -1e300, -np.inf], H)
    got = _states(model, x, np.full(H, 50.0))
    assert (np.abs(got - PI * np.exp(x.astype(np.longdouble))) <= 6 * 2.0 ** -1074).all()
    assert (got[x <= -746.0] == 0.0).all()


def test_log1p(model):
    rng = np.random.default_rng(3)
    blk, n = _blocks()
    d = np.concatenate([rng.uniform(0, 36, 150), rng.uniform(0, 2, 150), [0.0, 1e-9, 700.0]])
    sig = torch.ones((1, 2), dtype=torch.uint8, device="cuda")
    got = []
    for v in d:
        th = np.zeros(n)
        th[blk["c"]] = -v, 0.0
        model.set_params(torch.from_numpy(th).cuda())
        got.append(float(model.logpsi(sig).real.item()))
    _close(np.array(got), -np.log1p(np.exp(-d.astype(np.longdouble))), 1.4)
