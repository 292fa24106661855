"""The autotuner of a context in which some plumes walk row windows beside others'
lists."""
import numpy as np
import pytest
import torch

from paper_2108_09488_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_plumes_without_lists_are_timed_too():
    """A large plume of few neighbours, over lists fastest with one lane a target, and a
    squeezed one without lists, which one lane a target makes several times slower than
    four: the tuned step is at most half again as long as four lanes'."""
    from paper_2108_09488_amd.context import Context, params_from_spec
    a = I.config("cfg2_h20_r10", n_side=600, h_over_dp=1.2)
    b = I.config("cfg2_h20_r10", n_side=160, h_over_dp=3.0)
    xb = I.quantize(0.5 * b.positions(), b.L)
    x = torch.from_numpy(np.concatenate([a.positions(), xb], axis=1))
    C = torch.from_numpy(np.concatenate([a.concentration(a.positions()), b.concentration(xb)]))
    c = Context([params_from_spec(a), params_from_spec(b)], [a.n, b.n], stream=torch.cuda.Stream())

    def step_us():
        c.init(x, C).build().step(3)
        assert c.lists() == {"built": 1, "read": 1}
        times = []
        for _ in range(5):
            c.timing_start()
            c.step(10)
            times.append(c.timing_stop()[0] * 100.0)
        return min(times)

    c.set_tuning(block=256, lanes=4, targets=1)
    four = step_us()
    tuned = c.autotune(reps=3)
    us = step_us()
    print(f"[case] tuner: four lanes {four:.1f} us, tuned {tuned} {us:.1f} us", flush=True)
    assert us <= 1.5 * four
    c.close()


def test_timing_of_more_launches_than_events():
    """Two timed launches a step, past the 2048 launches that the event pool holds."""
    from paper_2108_09488_amd.context import Context, params_from_spec
    a = I.config("cfg2_h20_r10", n_side=16)
    b = I.config("cfg2_h20_r10", n_side=24)
    xb = I.quantize(0.5 * b.positions(), b.L)
    x = torch.from_numpy(np.concatenate([a.positions(), xb], axis=1))
    c = Context([params_from_spec(a), params_from_spec(b)], [a.n, b.n])
    c.init(x, torch.ones(x.shape[1])).build().step(3)
    assert c.lists() == {"built": 1, "read": 1}
    c.timing_start()
    c.rhs()  # one launch, so that a step's pair straddles the end of the pool
    c.step(1500)
    ms, n = c.timing_stop()
    assert n == 3001 and ms > 0.0
    c.close()


def test_a_tuned_context_has_its_lists():
    """The lists of the shape that the autotuner chose stand when it returns."""
    from paper_2108_09488_amd.context import Context, params_from_spec
    a = I.config("cfg2_h20_r10", n_side=200)
    x = a.positions()
    c = Context([params_from_spec(a)], [a.n])
    c.init(torch.from_numpy(x), torch.from_numpy(a.concentration(x))).build()
    c.autotune(reps=1)
    assert c.lists()["built"] == 1
    c.step(1)
    assert c.lists() == {"built": 1, "read": 0}  # the first two steps of a large context walk the windows
    c.step(2)
    assert c.lists() == {"built": 1, "read": 1}
    c.close()
