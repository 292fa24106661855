"""The workspace with and without room for neighbour lists: sizes on the CPU, contexts
made with either on the GPU."""
import ctypes as ct

import numpy as np
import pytest
import torch

from paper_2108_09488_amd import _lib
from paper_2108_09488_amd import inputs as I
from paper_2108_09488_amd.context import params_from_spec, workspace_bytes


@pytest.mark.parametrize("name,n_side,rb,hod,least", [
    # what a context takes that keeps no lists, a quarter more at most: state, hashed
    # buffer, cell tables (40 bytes a cell), second C
    ("cfg3", 64, 4, 2.0, 41e6), ("cfg3", 47, 8, 1.6, 15.5e6), ("cfg3", 128, 4, 2.0, 330e6),
    ("cfg2_h20_r10", 512, 4, 2.0, 32e6)])
def test_workspace_without_lists(name, n_side, rb, hod, least):
    s = I.config(name, n_side=n_side, real_bytes=rb, h_over_dp=hod)
    p = [params_from_spec(s)]
    small, full = workspace_bytes(p, [s.n], lists=False), workspace_bytes(p, [s.n])
    assert 0.75 * least <= small <= 1.25 * least and small < full


def test_nothing_to_leave_out():
    """Velocity fields and dense plumes keep no lists."""
    s = I.config("cfg2_h20_r10", n_side=64)
    d = I.config("cfg2_h20_r10", n_side=90, h_over_dp=14.0)
    for p, n in ((params_from_spec(s, flags=_lib.ADE_VELOCITY_FIELD), s.n), (params_from_spec(d), d.n)):
        assert workspace_bytes([p], [n], lists=False) == workspace_bytes([p], [n])
    bad = params_from_spec(s)
    bad.dim = 5
    nb = ct.c_size_t(0)
    n = (ct.c_int64 * 1)(s.n)
    assert _lib.lib().ade_workspace_bytes_min((_lib.AdeParams * 1)(bad), n, 1, ct.byref(nb)) == _lib.ADE_EINVAL
    assert _lib.lib().ade_workspace_bytes_min((_lib.AdeParams * 1)(bad), n, 1, None) == _lib.ADE_EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("dim,rb,integrator", [(2, 4, 1), (3, 4, 2), (3, 8, 1)])
def test_a_context_without_lists(dim, rb, integrator):
    """Steps, adjoint and states of a context without lists against one with them: the
    order of the sums differs (1e-6 relative L2, FP64 1e-14); workspaces between the
    two sizes are taken, smaller ones refused."""
    from paper_2108_09488_amd.context import Context
    spec = I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=40 if dim == 2 else 13, real_bytes=rb, h_over_dp=1.5)
    print(f"[case] without lists dim={dim} rb={rb} integrator={integrator}", flush=True)
    p = [params_from_spec(spec, integrator=integrator)]
    x, C = torch.from_numpy(spec.positions()), torch.from_numpy(spec.concentration(spec.positions()))
    xs, obs = torch.full((dim, 3), 0.4, dtype=torch.float64), torch.zeros(3)
    out = []
    for lists in (True, False):
        c = Context(p, [spec.n], lists=lists)
        assert c.ws_bytes == workspace_bytes(p, [spec.n], lists=lists)
        c.init(x, C).build().step(4)
        assert c.lists() == {"built": int(lists), "read": int(lists)}
        one = c.read_C().double().cpu().numpy()
        state = c.save_state()
        J, g = c.adjoint(3, 2, xs, obs)
        out.append((one, c.read_C().double().cpu().numpy(), J, np.array(g), state))
        c.close()
    tol = 1e-6 if rb == 4 else 1e-14
    for k in (0, 1):
        assert np.linalg.norm(out[0][k] - out[1][k]) <= tol * np.linalg.norm(out[0][k])
    assert abs(out[0][2] - out[1][2]) <= 4 * tol * out[0][2]
    c = Context(p, [spec.n]).load_state(out[1][4])
    assert np.array_equal(c.read_C().double().cpu().numpy(), out[1][0])
    c.close()

    L = _lib.lib()
    arr, n, h = (_lib.AdeParams * 1)(*p), (ct.c_int64 * 1)(spec.n), ct.c_void_p()
    small, full = workspace_bytes(p, [spec.n], lists=False), workspace_bytes(p, [spec.n])
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for size, rc in ((small - 1, _lib.ADE_EWORKSPACE), (small, 0), (full - 1, 0), (full, 0)):
        assert L.ade_create(arr, n, 1, ct.c_void_p(ws.data_ptr()), size, None, ct.byref(h)) == rc, size
        if rc == 0:
            L.ade_destroy(h)
