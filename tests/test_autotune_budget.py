"""The autotuner's register budgets where the sample runs four cells to a
wavefront: those kernels have one build, so a budget timed there says nothing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2501_00011_amd import mcchem, synth  # noqa: E402


@pytest.mark.gpu
@pytest.mark.parametrize("n,tail,cells", [(20, 0, 9), (72, 32, 2600)])
def test_one_budget_where_one_build_serves_all(n, tail, cells):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = synth.make_mechanism(n, 2 * n)
    few = synth.make_cells(m, 8, seed=61)
    of = np.arange(cells) % 8
    sample = synth.Cells(T=few.T[of], P=few.P[of], jscale=few.jscale[of], y0=few.y0[:, of])
    kw = dict(candidates=(tail,), schedules=("identity",), reps=1)
    own = mcchem.Mechanism(m, dense_tail=tail).schedule_info()["waves_per_simd"]
    h, times, choice = mcchem.autotune_solver(m, sample, 1.0, **kw)
    assert h.solver_dispatch(cells)["cells_per_wavefront"] == 4
    assert list(times) == [f"{tail}/{own}/identity"] and choice == (tail, own, "identity")
    assert h.schedule_info()["waves_per_simd"] == own
    # a budget asked for alone is the caller's choice
    h, times, choice = mcchem.autotune_solver(m, sample, 1.0, waves=(1,), **kw)
    assert list(times) == [f"{tail}/1/identity"] and h.schedule_info()["waves_per_simd"] == 1
    # one cell a wavefront: two builds, both timed
    one = synth.Cells(T=few.T, P=few.P, jscale=few.jscale, y0=few.y0)
    if tail:
        _, times, _ = mcchem.autotune_solver(m, one, 1.0, **kw)
        assert set(times) == {f"{tail}/{own}/identity", f"{tail}/1/identity"}
