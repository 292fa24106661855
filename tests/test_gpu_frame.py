"""A uniform flow in the plume's frame: no step moves or sorts the particles,
so calls of any number of steps, graphs of them and states saved at any step
have to agree.

Tolerances: the runs compared do the same sums in the same order, so C and x
are equal bit for bit; FP64 against the oracle as in test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2108_09488_amd import _lib
from paper_2108_09488_amd import inputs as I

pytestmark = pytest.mark.gpu


def _plume(dim=2, n_side=24, rb=4, integrator=1, stream=None, **over):
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, jitter=0.1,
                    v=(0.7, -0.4, 0.3), dt=1e-4, **over)
    print(f"[case] frame dim={dim} n_side={n_side} rb={rb} integrator={integrator}", flush=True)
    x = spec.positions()
    C = spec.concentration(x)
    if rb == 4:
        C = C.astype(np.float32).astype(np.float64)

    def fresh():
        c = Context([params_from_spec(spec, integrator=integrator)], [spec.n], stream=stream)
        return c.init(torch.from_numpy(x), torch.from_numpy(C)).build()

    return spec, x, C, fresh


@pytest.mark.parametrize("dim,rb,integrator", [(2, 4, 1), (2, 8, 1), (2, 4, 2), (3, 4, 1), (3, 8, 2)])
def test_calls_of_any_number_of_steps_agree(dim, rb, integrator):
    """37 steps in one call, one by one, in odd and even parts, and replayed
    from graphs (the captured block and a rest): the same bits, at the
    positions of 37 exact displacements."""
    spec, x, C, fresh = _plume(dim, 24 if dim == 2 else 14, rb, integrator, torch.cuda.Stream())
    outs = []
    for parts in ([37], [1] * 37, [2, 3, 16, 1, 15], "graph", "both"):
        c = fresh()
        if parts == "graph":
            c.step_graph(37)
        elif parts == "both":
            c.step(3).step_graph(17).step_graph(16).step(1)
        else:
            for p in parts:
                c.step(p)
        assert c.info()["step"] == 37
        outs.append((c.read_C().cpu().numpy(), c.read_x().cpu().numpy()))
        c.close()
    for Cg, xg in outs[1:]:
        assert np.array_equal(Cg, outs[0][0]) and np.array_equal(xg, outs[0][1])
    u0 = np.rint(x / spec.L * 2.0 ** 32)
    for k in range(dim):
        s = np.rint(37 * (spec.dt * spec.v[k] / spec.L * 2.0 ** 32))
        assert np.array_equal(outs[0][1][k], np.mod(u0[k] + s, 2.0 ** 32) * (spec.L / 2.0 ** 32))
    if rb == 8:
        _, Co, _ = O.run(O.model_from_spec(spec), x, C, spec.dt, 37, v_uniform=spec.velocity(), mass=spec.mass,
                         rho=spec.rho0, integrator=integrator)
        assert np.linalg.norm(outs[0][0] - Co) < 1e-10 * np.linalg.norm(Co)


def test_a_callers_graph_holds_between_other_calls():
    """A caller's own capture of three steps, replayed with eager steps and
    reads between the replays: every replay continues from the context's
    state."""
    stream = torch.cuda.Stream()
    spec, x, C, fresh = _plume(stream=stream)
    ref, c = fresh(), fresh()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        c.step(3)
    for k in range(4):
        with torch.cuda.stream(stream):
            g.replay()
        c.step(k)
        ref.step(3).step(k)
        torch.cuda.synchronize()
        assert np.array_equal(c.read_x().cpu().numpy(), ref.read_x().cpu().numpy())
        a, b = c.read_C().double().cpu().numpy(), ref.read_C().double().cpu().numpy()
        assert np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b)
    assert c.info()["step"] == ref.info()["step"]


def test_states_of_the_first_form_are_read():
    """A saved state whose positions and cells are those of its own step (the
    form without the frame's origin) continues from there."""
    spec, x, C, fresh = _plume()
    a = fresh().step(5)
    b = fresh()
    b.init(a.read_x(), a.read_C()).build()  # order and cells of step 5
    buf = b.save_state()
    head = buf[:56].view(np.uint64).copy()  # magic, dim..integrator, N, cells, bytes, layout
    assert head[0] == 0x3254415453454441
    head[0] = 0x3154415453454441
    words = buf.size - 8
    assert head[5] == buf.size
    head[5] = words
    old = np.concatenate([head.view(np.uint8), buf[56:words]])
    old[-8:] = np.array([5], dtype=np.int64).view(np.uint8)
    d = fresh().load_state(old)
    assert d.info()["step"] == 5
    d.step(4)
    a.step(4)
    b.step(4)
    assert np.array_equal(d.read_x().cpu().numpy(), a.read_x().cpu().numpy())
    assert np.array_equal(d.read_C().cpu().numpy(), b.read_C().cpu().numpy())
    with pytest.raises(_lib.AdeError):
        d.load_state(old[:-8])


@pytest.mark.parametrize("rb,integrator", [(4, 1), (4, 2), (8, 1)])
def test_adjoint_with_and_without_recompute(rb, integrator):
    """600 steps of a small plume: with a checkpoint every 24 steps the states
    do not all fit the workspace and the segments are recomputed, with every
    600 nothing is; J, the gradient and the final state are the same bits."""
    spec, x, C, fresh = _plume(n_side=20, rb=rb, integrator=integrator)
    xs = torch.from_numpy(I.sensors(40, [0.1, 0.3], [0.6, 0.8])).cuda()
    obs = torch.full((40,), 0.1, dtype=torch.float32 if rb == 4 else torch.float64, device="cuda")
    outs = []
    for K in (24, 600, 25, 1):
        c = fresh()
        J, g = c.adjoint(600, K, xs, obs)
        outs.append((J, g, c.read_C().cpu().numpy(), c.read_x().cpu().numpy()))
        assert c.info()["step"] == 600
        c.close()
    fwd = fresh().step(600)
    for J, g, Cg, xg in outs:
        assert J == outs[0][0] and g == outs[0][1] and np.isfinite(J)
        assert np.array_equal(Cg, fwd.read_C().cpu().numpy()) and np.array_equal(xg, fwd.read_x().cpu().numpy())
