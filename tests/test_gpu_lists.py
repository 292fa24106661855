"""Neighbour lists of a uniform flow where they can go wrong: every launch shape
at sizes around a wavefront's and a tile's targets, plumes of more than 65536
particles (entries count from a base, across the periodic seam), particles that
do not fit their lists, such plumes beside others, and captured calls, which walk
the row windows.

Tolerances: FP32 right-hand sides within 1e-5 relative L2 of the FP64 oracle
(the forward bound of test_gpu_parity.py), FP64 within 1e-12; runs over the same
lists are equal bit for bit; the lists against the row windows differ by the
order of FP32 sums only, 1e-6 relative L2 over a few steps."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2108_09488_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 1), (4, 1), (1, 2), (4, 2)]


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def _oracle(spec, x, C):
    return O.rhs(O.model_from_spec(spec), x, C, v_uniform=spec.velocity(), mass=spec.mass, rho=spec.rho0)


def _context(specs, xs, stream=None):
    from paper_2108_09488_amd.context import Context, params_from_spec
    c = Context([params_from_spec(s) for s in specs], [x.shape[1] for x in xs], stream=stream)
    x = np.concatenate(xs, axis=1)
    C = np.concatenate([s.concentration(v) for s, v in zip(specs, xs)])
    if specs[0].real_bytes == 4:
        C = C.astype(np.float32).astype(np.float64)
    c.init(torch.from_numpy(x), torch.from_numpy(C)).build()
    return c, C


@pytest.mark.parametrize("dim,rb,n_side,drop,hod", [
    (2, 4, 23, 0, 1.3), (2, 4, 16, 1, 2.0), (2, 8, 16, 0, 1.5), (2, 8, 33, 3, 2.5), (2, 4, 300, 0, 1.5),
    (2, 8, 257, 5, 1.3), (3, 4, 13, 2, 1.7), (3, 4, 8, 0, 1.3), (3, 8, 9, 1, 1.5)])
def test_rhs_of_every_shape(dim, rb, n_side, drop, hod):
    """Ragged last tiles (drop: particles left out at the end), whole tiles,
    and plumes past 65536 particles: the right-hand side of a call, over the
    row windows, and that of a step, over the lists, from one of a dt so long
    that it outweighs C a hundred times."""
    spec = I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, h_over_dp=hod,
                    v=(0.6, 0.8, 0.0))
    x = spec.positions()[:, :spec.n - drop]
    C0 = spec.concentration(x)
    spec.dt = float(100.0 * np.linalg.norm(C0) / np.linalg.norm(_oracle(spec, x, C0)))
    c, C = _context([spec], [x])
    ref = _oracle(spec, x, C)
    tol = 1e-5 if rb == 4 else 1e-12
    for lanes, targets in SHAPES:
        if targets == 2 and lanes == 4 and rb == 8:
            continue
        try:
            c.set_tuning(block=64, lanes=lanes, targets=targets)
        except Exception:
            continue  # its candidate lists do not fit in LDS
        print(f"[case] lists dim={dim} rb={rb} n={x.shape[1]} shape=({lanes},{targets})", flush=True)
        assert _rel(c.rhs().double().cpu().numpy(), ref) < tol, (lanes, targets)
        c.step(1)
        assert _rel((c.read_C().double().cpu().numpy() - C) / spec.dt, ref) < tol, (lanes, targets)
        c.init(torch.from_numpy(x), torch.from_numpy(C)).build()
    c.close()


def test_particles_that_do_not_fit():
    """Sites of 12 particles (nine times the expected neighbours at a site): the
    plume walks the row windows, beside a plume that keeps its lists and as it
    does alone."""
    a = I.config("cfg2_h20_r10", n_side=40)
    b = I.config("cfg2_h20_r10", n_side=48)
    xb = I.clustered(8, 2, 36, 0.02, b.L)
    xa = a.positions()
    for lanes, targets in [(4, 1), (1, 2)]:
        c, C = _context([a, b], [xa, xb])
        c.set_tuning(block=64, lanes=lanes, targets=targets)
        both = c.rhs().double().cpu().numpy()
        c.step(3)
        Cs = c.read_C().cpu().numpy()
        c.close()
        off = 0
        for s, x in ((a, xa), (b, xb)):
            n = x.shape[1]
            assert _rel(both[off:off + n], _oracle(s, x, C[off:off + n])) < 1e-5
            one, _ = _context([s], [x])
            one.set_tuning(block=64, lanes=lanes, targets=targets)
            assert np.array_equal(one.rhs().double().cpu().numpy(), both[off:off + n])
            one.step(3)
            assert np.array_equal(one.read_C().cpu().numpy(), Cs[off:off + n])
            one.close()
            off += n


@pytest.mark.parametrize("dim,n_side", [(2, 40), (3, 13)])
def test_captured_calls_walk_the_windows(dim, n_side):
    """Three captured steps of every shape against three eager ones, replayed
    after new particles and another launch shape."""
    stream = torch.cuda.Stream()
    spec = I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=n_side, h_over_dp=1.5)
    x = spec.positions()
    c, C = _context([spec], [x], stream)
    for lanes, targets in SHAPES:
        try:
            c.set_tuning(block=64, lanes=lanes, targets=targets)
        except Exception:
            continue
        print(f"[case] captured windows dim={dim} shape=({lanes},{targets})", flush=True)
        c.rhs()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            c.step(3)
        for k in range(2):
            y = np.ascontiguousarray(np.mod(x + 0.013 * k, spec.L))
            y = I.quantize(y, spec.L)
            c.init(torch.from_numpy(y), torch.from_numpy(C)).build().step(3)
            eager = c.read_C().double().cpu().numpy()
            c.set_tuning(block=64, lanes=2, targets=1)
            c.init(torch.from_numpy(y), torch.from_numpy(C)).build().rhs()
            torch.cuda.synchronize()
            with torch.cuda.stream(stream):
                g.replay()
            torch.cuda.synchronize()
            assert _rel(c.read_C().double().cpu().numpy(), eager) < 1e-6, (lanes, targets, k)
            c.set_tuning(block=64, lanes=lanes, targets=targets)
    c.close()


def test_steps_of_the_graph_follow_the_lists():
    """The captured steps of a context whose second plume now fits its lists and
    now does not, each time as a fresh context runs them (a run long enough for the
    graph)."""
    stream = torch.cuda.Stream()
    a = I.config("cfg2_h20_r10", n_side=40)
    b = I.config("cfg2_h20_r10", n_side=48)
    xs = {"lattice": b.positions(), "clustered": I.clustered(8, 2, 36, 0.02, b.L)[:, :b.n]}
    assert xs["clustered"].shape == xs["lattice"].shape
    ctx = None
    for name in ("lattice", "clustered", "lattice", "lattice", "clustered", "clustered"):
        print(f"[case] graph over {name}", flush=True)
        if ctx is None:
            ctx, C = _context([a, b], [a.positions(), xs[name]], stream)
        else:
            x = np.concatenate([a.positions(), xs[name]], axis=1)
            C = np.concatenate([a.concentration(a.positions()), b.concentration(xs[name])])
            ctx.init(torch.from_numpy(x), torch.from_numpy(C.astype(np.float32).astype(np.float64))).build()
        fresh, _ = _context([a, b], [a.positions(), xs[name]], stream)
        ctx.step_graph(515)
        fresh.step(515)
        assert np.array_equal(ctx.read_C().cpu().numpy(), fresh.read_C().cpu().numpy())
        fresh.close()
    ctx.close()
