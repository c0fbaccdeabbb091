"""Rounding error of the two-pass axial transform (csrc/fft_mix.hip) on lines of white noise.

A state of the one row m = 0, n = 0 makes the backward transform its axial transform times the constant Pbar_0^0, so
the output is compared with the sums in extended precision.  Bound, root mean square over 600 lines: the two passes with every
twiddle factor rounded once and every product and sum rounded (no fused operations) leave 1.275e-16, 1.462e-16 and
1.613e-16 of the output at 12, 24 and 48 points (computed on the CPU), and the product with the constant at most
2^-53 / sqrt(3).  Factors formed as products of other factors leave more."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PASSES = {12: 1.275e-16, 24: 1.462e-16, 48: 1.613e-16}
LD = np.longdouble


@pytest.mark.parametrize("n", sorted(PASSES))
def test_axial_rounding(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    print("axial rounding", n, flush=True)
    plan = Plan(2, 4, n, 1.0, 8.0)
    spec, phys = plan.empty_spec(), plan.empty_phys()
    j = np.arange(n)
    keep = np.minimum(j, n - j) < n // 2
    pi = LD("3.14159265358979323846264338327950288")
    arg = 2 * pi * (np.outer(j, j) % n).astype(LD) / n
    C, D, p0 = np.cos(arg), np.sin(arg), LD(np.sqrt(0.5))
    rng = np.random.default_rng(n)
    err = tot = 0.0
    for _ in range(600):
        z = (rng.standard_normal(n) + 1j * rng.standard_normal(n)) * keep
        spec.zero_()
        spec[0] = torch.from_numpy(z).cuda()
        plan.backward(spec, phys)
        ref = (C @ z.real.astype(LD) - D @ z.imag.astype(LD)) * p0
        err += float(((phys[:, 0, 0].cpu().numpy().astype(LD) - ref) ** 2).sum())
        tot += float((ref ** 2).sum())
    rms, bound = (err / tot) ** 0.5, (PASSES[n] ** 2 + 2.0 ** -106 / 3) ** 0.5
    print("  rms", rms, "bound", bound, flush=True)
    assert rms < bound
