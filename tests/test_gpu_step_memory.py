"""Device memory of mlg_step_setup: the operator tables and the scratch of one field.  The second potential of mlg_tp_advance
uses the caller's workspace.  The grid makes the scratch (34 MB) the larger part."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_step_setup_holds_the_scratch_of_one_field():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import Plan
    print("step setup memory", flush=True)
    nr, nphi, nz = 64, 128, 1024
    warm = Plan(8, 8, 8, 1.0, 4.0)
    warm.step_setup(1e-2, 1e-8, 8, 1e-2)
    plan = Plan(nr, nphi, nz, 1.0, 4.0)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    plan.step_setup(1e-2, 1e-8, 8, 1e-2)
    held = before - torch.cuda.mem_get_info()[0]
    scratch = (plan.tau + plan.layout.nrc - 1) * nz * 16
    tables = sum(2 * 8 * (nr - m) ** 2 for m in range(plan.layout.M))
    print("  held", held, "scratch of one field", scratch, "tables", tables, flush=True)
    assert held < tables + scratch + 12 * 2 ** 20     # allocations in pages of 2 MB
