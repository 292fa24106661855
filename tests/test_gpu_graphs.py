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
