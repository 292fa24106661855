"""The adjoint of a uniform flow in every launch shape over neighbour lists, and over
the row windows of plumes whose lists do not fit, against the FP64 oracle's discrete
adjoint.  Tolerances as in test_gpu_adjoint.py: 1e-10 relative in FP64, 1e-4 in FP32
(observations are half the plume's values, so that J is no cancellation)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2108_09488_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 1), (4, 1), (1, 2), (4, 2)]


def _problem(dim, rb, integrator, x_of):
    """dt v is a whole number of fixed-point units, as in test_gpu_adjoint.py."""
    if dim == 2:
        spec = I.config("cfg5", n_side=45, steps=11, dt=2.0 ** -12, real_bytes=rb, v=(0.75, 0.5, 0.0), alpha_L=1e-2,
                        alpha_T=5e-3)
        lo, hi = [0.05, 0.05], [0.45, 0.45]
    else:
        spec = I.config("cfg3", n_side=13, h_over_dp=1.7, steps=7, dt=2.0 ** -9, real_bytes=rb, v=(0.75, 0.5, 0.25),
                        alpha_L=1e-2, alpha_T=5e-3)
        lo, hi = [0.1, 0.1, 0.1], [0.4, 0.4, 0.4]
    x = x_of(spec)
    C0 = 0.2 + spec.concentration(x)
    xs = I.sensors(70, lo, hi)
    if rb == 4:
        C0 = C0.astype(np.float32).astype(np.float64)
    m = O.model_from_spec(spec)
    kw = dict(mass=spec.mass, rho=spec.rho0, integrator=integrator)
    _, obs = O.misfit(m, x, C0, spec.velocity(), spec.dt, spec.steps, xs, None, **kw)
    obs = 0.5 * obs
    if rb == 4:
        obs = obs.astype(np.float32).astype(np.float64)
    ref = O.adjoint(m, x, C0, spec.velocity(), spec.dt, spec.steps, xs, obs, **kw)
    return spec, x, C0, xs, obs, ref


def _check(spec, x, C0, xs, obs, ref, rb, integrator, lists):
    from paper_2108_09488_amd.context import Context, params_from_spec
    Jo, go, Co = ref
    tol = 1e-10 if rb == 8 else 1e-4
    c = Context([params_from_spec(spec, integrator=integrator)], [x.shape[1]])
    for lanes, targets in SHAPES:
        if (lanes, targets, rb) == (4, 2, 8):
            continue
        c.set_tuning(block=64, lanes=lanes, targets=targets)
        for K in (spec.steps, 3):
            print(f"[case] adjoint dim={spec.dim} rb={rb} integrator={integrator} shape=({lanes},{targets}) K={K}",
                  flush=True)
            c.init(torch.from_numpy(x), torch.from_numpy(C0)).build()
            J, g = c.adjoint(spec.steps, K, torch.from_numpy(xs), torch.from_numpy(obs))
            assert c.lists() == {"built": lists, "read": lists}, (lanes, targets)
            assert J == pytest.approx(Jo, rel=tol), (lanes, targets, K)
            assert np.allclose(g, go, rtol=tol, atol=tol * np.abs(go).max()), (lanes, targets, K)
            Cg = c.read_C().double().cpu().numpy()
            assert np.linalg.norm(Cg - Co) < (1e-12 if rb == 8 else 1e-5) * np.linalg.norm(Co)
    c.close()


@pytest.mark.parametrize("dim,rb,integrator", [(2, 4, 1), (2, 4, 2), (2, 8, 1), (2, 8, 2), (3, 4, 1), (3, 4, 2),
                                               (3, 8, 1), (3, 8, 2)])
def test_over_lists(dim, rb, integrator):
    """Ragged plumes: 2022 particles (2D), 2195 (3D)."""
    p = _problem(dim, rb, integrator, lambda s: np.ascontiguousarray(s.positions()[:, :s.n - 3 + (s.dim == 3)]))
    _check(*p, rb, integrator, 1)


@pytest.mark.parametrize("dim,rb,integrator", [(2, 4, 1), (2, 8, 2), (3, 4, 2), (3, 8, 1)])
def test_over_windows(dim, rb, integrator):
    """A plume squeezed into a corner of its box, whose lists do not fit."""
    p = _problem(dim, rb, integrator, lambda s: I.quantize(0.5 * s.positions(), s.L))
    _check(*p, rb, integrator, 0)
