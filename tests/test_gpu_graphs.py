"""The graphs of ade_step_graph, which hold 16 steps and serve runs of 512 steps
of a uniform flow and more (a velocity field: of 16), and callers' captures of
the call."""
import numpy as np
import pytest
import torch

from paper_2108_09488_amd import inputs as I

pytestmark = pytest.mark.gpu


def _uniform(stream, dim=2, n_side=24, rb=8, integrator=1, **over):
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, h_over_dp=1.5, jitter=0.1,
                    v=(0.7, -0.4, 0.3), dt=1e-4, **over)
    x = spec.positions()
    C = spec.concentration(x)
    if rb == 4:
        C = C.astype(np.float32).astype(np.float64)
    c = Context([params_from_spec(spec, integrator=integrator)], [spec.n], stream=stream)
    return spec, c, x, C


def test_a_captured_call_takes_nothing_from_the_contexts_graph():
    """A caller captures a run that the context holds a graph of its own for, and
    replays it after the particles, and with them the lists of that graph, were
    replaced.  The captured steps walk the row windows: FP64 sums in another order,
    2^-53 relative to the terms of about 30 neighbours in each of 515 steps that
    change C by less than itself: 515 * 30 * 1.1e-16 = 2e-12."""
    stream = torch.cuda.Stream()
    spec, c, x, C = _uniform(stream)
    c.init(torch.from_numpy(x), torch.from_numpy(C)).build().step_graph(515)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        c.step_graph(515)
    for k in range(3):
        print(f"[case] captured step_graph, particles {k}", flush=True)
        y = I.quantize(np.mod(x[:, ::-1] + 0.217 * k, spec.L), spec.L)
        c.init(torch.from_numpy(y), torch.from_numpy(C)).build().step_graph(515)
        eager, xe = c.read_C().cpu().numpy(), c.read_x().cpu().numpy()
        c.init(torch.from_numpy(y), torch.from_numpy(C)).build().rhs()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            g.replay()
        torch.cuda.synchronize()
        assert c.info()["step"] == 515
        assert np.array_equal(c.read_x().cpu().numpy(), xe)
        assert np.linalg.norm(c.read_C().cpu().numpy() - eager) <= 2e-12 * np.linalg.norm(eager)
    c.close()


def test_read_outs_captured_on_another_stream():
    """A caller's capture on a stream that is not the context's takes the context's
    read-outs in, and they follow the context's state from replay to replay: the
    bits of the eager calls."""
    spec, c, x, C = _uniform(torch.cuda.Stream(), rb=4)
    c.init(torch.from_numpy(x), torch.from_numpy(C)).build().step(2)
    xs = torch.from_numpy(I.sensors(30, [0.1, 0.1], [0.9, 0.9])).cuda()

    def read():
        return [c.rhs(), c.read_C(), c.read_x(), c.mass(), c.conc_range(), c.sensor_interp(xs)]

    read()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = read()
    for k in range(3):
        print(f"[case] captured read-outs, replay {k}", flush=True)
        c.step(k + 1)
        if k == 1:
            c.init(torch.from_numpy(np.ascontiguousarray(x[:, ::-1])), torch.from_numpy(C)).build()
        eager = [t.cpu().numpy() for t in read()]
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(outs, eager):
            assert np.array_equal(a.cpu().numpy(), b)
    c.close()


@pytest.mark.parametrize("dim,rb,integrator", [(2, 4, 1), (2, 4, 2), (2, 8, 2), (3, 4, 1), (3, 8, 2)])
def test_uniform_runs_past_the_threshold(dim, rb, integrator):
    """515 and 512 steps, both over the graph and the first with a rest, against
    eager ones: the same bits."""
    stream = torch.cuda.Stream()
    outs = []
    for graph in (False, True):
        print(f"[case] graph dim={dim} rb={rb} integrator={integrator} graph={graph}", flush=True)
        spec, c, x, C = _uniform(stream, dim, 20 if dim == 2 else 10, rb, integrator)
        c.init(torch.from_numpy(x), torch.from_numpy(C)).build()
        for n in (515, 3, 512):
            if graph:
                c.step_graph(n)
            else:
                for k in (n // 2, n - n // 2):  # each part below the threshold of the graph
                    c.step(k)
            torch.cuda.synchronize()
            assert c.lists() == {"built": 1, "read": 1}
        assert c.info()["step"] == 1030
        outs.append((c.read_C().cpu().numpy(), c.read_x().cpu().numpy()))
        c.close()
    assert np.isfinite(outs[0][0]).all()
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


def _field(stream, dim, n_side, rb, integrator, flags=0):
    from paper_2108_09488_amd import _lib
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, h_over_dp=1.5, dt=1e-4)
    x = spec.positions()
    c = Context([params_from_spec(spec, integrator=integrator, flags=_lib.ADE_VELOCITY_FIELD | flags)], [spec.n],
                stream=stream)
    c.init(torch.from_numpy(x), torch.from_numpy(spec.concentration(x)))
    v = np.stack([1.0 + 0.3 * np.sin(2.0 * np.pi * x[1]), 0.3 * np.cos(2.0 * np.pi * x[0])] + [0.2 * x[0]] * (dim - 2))
    c.set_velocities(torch.from_numpy(v)).build()
    return spec, c


@pytest.mark.parametrize("dim,rb,integrator", [(2, 4, 1), (2, 4, 2), (2, 8, 1), (3, 4, 2), (3, 8, 1)])
def test_velocity_field_runs_past_the_threshold(dim, rb, integrator):
    """19, 32 and 5 steps, the first two over the graph: the bits of 56 eager ones."""
    stream = torch.cuda.Stream()
    outs = []
    for graph in (False, True):
        print(f"[case] field graph dim={dim} rb={rb} integrator={integrator} graph={graph}", flush=True)
        spec, c = _field(stream, dim, 24 if dim == 2 else 10, rb, integrator)
        for n in (19, 32, 5):
            (c.step_graph if graph else c.step)(n)
            torch.cuda.synchronize()
        assert c.info()["step"] == 56
        outs.append((c.read_C().cpu().numpy(), c.read_x().cpu().numpy()))
        c.close()
    assert np.isfinite(outs[0][0]).all()
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


def test_finite_check_after_the_graph():
    """ADE_CHECK_FINITE behind replays: silent on finite runs, and an infinite
    concentration is reported, in both kinds of flow."""
    from paper_2108_09488_amd import _lib
    from paper_2108_09488_amd.context import Context, params_from_spec
    stream = torch.cuda.Stream()
    spec = I.config("cfg2_h20_r10", n_side=20, h_over_dp=1.5, dt=1e-4)
    x, C = torch.from_numpy(spec.positions()), torch.from_numpy(spec.concentration(spec.positions()))
    bad = C.clone()
    bad[7] = float("inf")
    u = Context([params_from_spec(spec, flags=_lib.ADE_CHECK_FINITE)], [spec.n], stream=stream)
    f = Context([params_from_spec(spec, flags=_lib.ADE_CHECK_FINITE | _lib.ADE_VELOCITY_FIELD)], [spec.n], stream=stream)
    v = torch.ones(2, spec.n, dtype=torch.float64)
    for c, n in ((u, 515), (f, 19)):
        for state in (C, bad, C):
            c.init(x, state)
            if c is f:
                c.set_velocities(v)
            c.build()
            if state is bad:
                with pytest.raises(_lib.AdeError) as e:
                    c.step_graph(n)
                assert e.value.code == _lib.ADE_ENONFINITE
            else:
                c.step_graph(n)
                assert torch.isfinite(c.read_C()).all()
        c.close()
