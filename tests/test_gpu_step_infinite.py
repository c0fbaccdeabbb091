"""FE-BE step with an infinite coefficient in A, on columns of one degree (their step is a scalar function): the infinity stays
in its coefficient and its part, on 2D and 3D plans; all other coefficients stay finite."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nz", [1, 4])
def test_infinite_source_stays_infinite(nz):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    print("infinite source", nz, flush=True)
    plan = Plan(4, 8, nz, 1.0, 4.0)          # orders 0 .. 3: the last row is order 3's only degree
    plan.step_setup(0.02, 1e-5, 4, 0.02)
    rng = np.random.default_rng(3)
    s, a = (rng.standard_normal((plan.tau, nz)) + 1j * rng.standard_normal((plan.tau, nz)) for _ in range(2))
    a[-1, 0] = complex(-np.inf, 1.0)
    out = plan.empty_spec()
    plan.step_febe(0, torch.from_numpy(s).cuda(), torch.from_numpy(a).cuda(), out)
    got = out.cpu().numpy()
    assert got[-1, 0].real == -np.inf and np.isfinite(got[-1, 0].imag)
    got[-1, 0] = 0
    assert np.isfinite(got.view(np.float64)).all()
