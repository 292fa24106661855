"""Sensor interpolation on both sides of the number of sensors from which a lane
takes the place of a sensor's wavefront."""
import numpy as np
import pytest
import torch

from paper_2108_09488_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,rb,n_side,last", [(2, 4, 40, 20480), (2, 8, 40, 10240), (3, 4, 14, 20480), (3, 8, 12, 10240)])
def test_many_sensors_as_few(dim, rb, n_side, last):
    """The sums of a sensor are the same bits however many sensors the call has, at
    the last size that takes wavefronts, the first that takes lanes and a ragged
    larger one, in a plume that has moved."""
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, h_over_dp=1.5, jitter=0.1,
                    v=(0.7, -0.4, 0.3))
    print(f"[case] sensors dim={dim} rb={rb} n={spec.n} bound={last}", flush=True)
    c = Context([params_from_spec(spec)], [spec.n])
    c.init(torch.from_numpy(spec.positions()), torch.from_numpy(spec.concentration(spec.positions()))).build().step(3)
    xs = torch.from_numpy(I.sensors(last + 777, [0.0] * dim, [0.999] * dim)).cuda()
    parts = torch.cat([c.sensor_interp(xs[:, k:k + 1000]) for k in range(0, xs.shape[1], 1000)]).cpu().numpy()
    assert np.isfinite(parts).all() and (parts > 0).any()
    for n in (last, last + 1, last + 777):
        assert np.array_equal(c.sensor_interp(xs[:, :n]).cpu().numpy(), parts[:n]), n
    c.close()


def test_adjoint_of_many_sensors():
    """J of an adjoint whose sensors take lanes, from the values of few at a time:
    FP64, sums of 10300 squares in another order, 1e-12 relative."""
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = I.config("cfg2_h20_r10", n_side=32, real_bytes=8, h_over_dp=1.5, jitter=0.1)
    x, C = torch.from_numpy(spec.positions()), torch.from_numpy(spec.concentration(spec.positions()))
    xs = torch.from_numpy(I.sensors(10300, [0.1, 0.1], [0.9, 0.9])).cuda()
    obs = torch.full((10300,), 0.1, dtype=torch.float64, device="cuda")
    c = Context([params_from_spec(spec)], [spec.n])
    J, g = c.init(x, C).build().adjoint(5, 2, xs, obs)
    Cs = torch.cat([c.sensor_interp(xs[:, k:k + 100].contiguous()) for k in range(0, 10300, 100)])
    ref = float(((Cs - obs) ** 2).sum())
    assert abs(J - ref) <= 1e-12 * ref and np.isfinite(g).all()
    c.close()
