"""The launch shapes a new context starts with, on both sides of each bound of
their rule, and the bound on the bytes of 2D neighbour lists.  Steps at the
default shape against those at four lanes a target differ by the order of FP32
sums: 1e-6 relative L2 (FP64: 1e-14) over two steps."""
import numpy as np
import pytest
import torch

from paper_2108_09488_amd import inputs as I


def _spec(dim, rb, n_side, hod):
    return I.config("cfg2_h20_r10" if dim == 2 else "cfg3", n_side=n_side, real_bytes=rb, h_over_dp=hod)


@pytest.mark.parametrize("rb,last,first", [(4, 1330, 1340), (8, 1880, 1895)])
def test_large_2d_contexts_keep_no_lists(rb, last, first):
    """113 neighbours: 2 bytes each pass 96 MiB per byte of the working precision
    between 1334^2 and 1335^2 (FP32), 1886^2 and 1888^2 (FP64) particles; the
    workspace of the larger context, without lists, is the smaller one."""
    from paper_2108_09488_amd.context import params_from_spec, workspace_bytes
    a, b = _spec(2, rb, last, 3.0), _spec(2, rb, first, 3.0)
    wa = workspace_bytes([params_from_spec(a)], [a.n])
    wb = workspace_bytes([params_from_spec(b)], [b.n])
    assert wb < wa


@pytest.mark.gpu
@pytest.mark.parametrize("dim,rb,n_side,hod,shape", [
    (2, 4, 361, 3.0, (256, 4, 1)), (2, 4, 363, 2.0, (256, 2, 1)), (2, 4, 363, 3.0, (64, 4, 2)),
    (2, 4, 513, 1.3, (256, 1, 1)), (2, 4, 513, 2.0, (128, 1, 2)), (2, 4, 723, 3.0, (64, 4, 2)),
    (2, 4, 726, 3.0, (128, 1, 2)), (2, 8, 726, 2.0, (256, 1, 1)), (2, 4, 90, 14.0, (256, 4, 1)),
    (2, 4, 444, 14.0, (256, 4, 2)), (3, 4, 50, 1.3, (256, 4, 1)), (3, 4, 51, 1.3, (64, 4, 2)),
    (3, 4, 81, 1.3, (128, 4, 2)), (3, 8, 31, 1.5, (64, 4, 1))])
def test_default_shape(dim, rb, n_side, hod, shape):
    from paper_2108_09488_amd.context import Context, params_from_spec
    spec = _spec(dim, rb, n_side, hod)
    x = torch.from_numpy(spec.positions())
    C = torch.from_numpy(spec.concentration(spec.positions()))
    out = []
    for default in (True, False):
        c = Context([params_from_spec(spec)], [spec.n])
        t = c.get_tuning()
        print(f"[case] default shape dim={dim} rb={rb} n={spec.n} {t}", flush=True)
        assert (t["block"], t["lanes"], t["targets"]) == shape
        if not default:
            c.set_tuning(block=64, lanes=4, targets=1)
        c.init(x, C).build().step(2)
        out.append(c.read_C().double().cpu().numpy())
        c.close()
    assert np.linalg.norm(out[0] - out[1]) <= (1e-6 if rb == 4 else 1e-14) * np.linalg.norm(out[1])
