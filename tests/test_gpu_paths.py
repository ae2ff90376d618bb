"""GPU tests of single kernels and dispatch branches at the sizes where they change, against
the FP64 oracle (gates of conftest: 1e-9 relative plus 1e-12 of the summed magnitudes)."""
import numpy as np
import pytest
import torch

from conftest import FLOOR, REL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    assert torch.cuda.is_available(), "needs a GPU"
    from paper_1801_10277_amd import binding
    return binding


def say(*a):
    print("[case]", *a, flush=True)


def device(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("steps", [0, 1, 4])
@pytest.mark.parametrize("hess_mode,rows", [(0, 16), (0, 4), (1, 16)])
def test_newton_elbo_out_is_the_elbo_of_the_returned_point(B, O, synth, steps, hess_mode, rows):
    """celeste_newton's elbo_out is that of the last accepted point (both Hessian modes: the
    pixel-level gradient pass and the full one; 0 steps: the entry point)."""
    f = synth.tiny(S=3, n_bands=2, size=45, side=35, seed=311)
    plan = B.Plan(f)
    plan.set_launch(strip_rows=rows)
    plan.set_hessian_mode(hess_mode)
    for s in range(3):
        say("newton elbo_out steps", steps, "mode", hess_mode, "rows", rows, "source", s)
        th = device(f.theta)
        e, _ = plan.newton(th, [s], steps)
        th = th.cpu().numpy()
        others = [t for t in range(3) if t != s]
        np.testing.assert_array_equal(th[others], f.theta[others])
        assert (steps == 0) == bool(np.array_equal(th[s], f.theta[s]))
        val, _, _ = O.source_grad(O.Problem(f, th), s)
        ref = val[0] + val[1]
        assert abs(float(e[s]) - ref) <= REL * abs(ref) + FLOOR * abs(val[2]), (s, float(e[s]), ref)
