"""Which kernel a batch gets (host logic, no GPU)."""
import numpy as np
import pytest

from paper_2501_00011_amd import mcchem, synth


def _cells_per_wavefront(h, n_cells, n_cu=256):
    return h.solver_dispatch(n_cells, n_cu)["cells_per_wavefront"]


@pytest.mark.parametrize("n,halves", [(33, 20), (36, 20), (37, 17), (48, 17), (49, 17), (72, 17)])
@pytest.mark.parametrize("n_cu", [256, 64])
def test_four_cells_with_a_front_only_beyond_what_the_one_cell_kernels_hold(n, halves, n_cu):
    """`halves` half cells per compute unit: below that line the four-cells
    kernels are the slower ones (2,049 cells of 33 to 40 species by 7 to 27 per
    cent)."""
    h = mcchem.Mechanism(synth.make_mechanism(n, 2 * n), device=-1, dense_tail=32)
    line = halves * n_cu // 2
    for cells in (1, 8 * n_cu, 8 * n_cu + 1, line):
        assert _cells_per_wavefront(h, cells, n_cu) == 1, cells
    for cells in (line + 1, 12 * n_cu, 100 * n_cu):
        assert _cells_per_wavefront(h, cells, n_cu) == 4, cells


def test_shapes_of_one_solver():
    """Without a front (and without a tail) four cells a wavefront at any size;
    shapes those kernels do not take, one cell."""
    h = mcchem.Mechanism(synth.make_mechanism(20, 40), device=-1, dense_tail=0)
    assert _cells_per_wavefront(h, 1) == _cells_per_wavefront(h, 100000) == 4
    for n, r, tail in ((72, 144, 48), (72, 144, 0), (20, 129, 0), (96, 201, 32), (150, 350, 64)):
        h = mcchem.Mechanism(synth.make_mechanism(n, r), device=-1, dense_tail=tail)
        assert _cells_per_wavefront(h, 1) == _cells_per_wavefront(h, 100000) == 1


@pytest.mark.parametrize("n,tail,cells,doubles", [
    (72, 32, 10000, 7 * 5 * 16 + 16),   # four cells a wavefront: 7 differences in 3 + 2 blocks of 16 rows
    (72, 32, 1000, 8 * 2 * 64 + 15),    # one cell a wavefront: 8 differences in two slots of 64
    (20, 0, 10, 7 * 2 * 16 + 16),
    (150, 64, 10, 8 * 3 * 64 + 15),
])
def test_state_of_the_per_launch_form(n, tail, cells, doubles):
    """What the benchmark counts as moved between launches is what the kernel
    that takes the batch reads and writes: a cell of s steps in launches of K
    writes its state ceil(s / K) - 1 times, and it is read as often."""
    import bench
    h = mcchem.Mechanism(synth.make_mechanism(n, 2 * n), device=-1, dense_tail=tail)
    d = h.solver_dispatch(cells, 256)
    assert d["state_moved"] == doubles <= d["state_doubles"]
    sn = np.zeros(cells, dtype=mcchem.STATS_DTYPE)
    sn["steps"] = 10
    sn["steps"][0] = 11
    got = bench.per_launch_state(sn, 5, h, 256)
    assert got == {"state_bytes_per_cell": 8 * doubles, "launches_max": 3,
                   "bytes_per_outer_step": 2.0 * 8 * doubles * (cells + 1)}
    assert bench.per_launch_state(sn, 0, h, 256) is None


def test_dispatch_arguments():
    h = mcchem.Mechanism(synth.make_mechanism(20, 40), device=-1)
    with pytest.raises(mcchem.MccError, match="status 5"):
        h.solver_dispatch(10)
    for cells, n_cu in ((-1, 256), (1 << 31, 256), (10, -1)):
        with pytest.raises(mcchem.MccError, match="status 1"):
            h.solver_dispatch(cells, n_cu)


def _lanes(h, kind, n_cells, ld=None):
    g = h.generated_launch(kind, n_cells, ld)
    assert g["workgroups"] * g["lanes"] * g["cells_per_lane"] >= n_cells
    return g["lanes"], g["group"]


@pytest.mark.parametrize("n,r", [(72, 156), (150, 350)])
def test_generated_launches(n, r):
    """One cell a lane up to 512 cells.  256-lane workgroups: odd leading
    dimensions of 64 such tiles or more, for the VJP kernel only where its inputs
    exceed the memory-side cache (50,001 cells of 150 species: 72.5 us with them,
    64.8 with 64 lanes); even ones beyond that cache, grouped where J is written
    (f alone, 100,000 cells of 150 species: 149 us grouped, 126 not); not for the
    VJP kernel."""
    h = mcchem.Mechanism(synth.make_mechanism(n, r), device=-1)
    for kind in ("f", "jac", "fj", "vjp"):
        assert h.generated_launch(kind, 512)["cells_per_lane"] == 1
        assert h.generated_launch(kind, 513)["cells_per_lane"] == 2
        rows = r + (2 * n if kind == "vjp" else n)
        fits = (256 << 20) // (8 * rows)  # cells whose inputs the cache holds
        odd = fits | 1
        first_wide = 2 * 63 * 256 + 1
        assert first_wide < fits
        assert _lanes(h, kind, first_wide - 2, first_wide - 2 | 1) == (64, 1)
        assert _lanes(h, kind, first_wide, first_wide) == ((64, 1) if kind == "vjp" else (256, 1))
        assert _lanes(h, kind, odd - 2) == ((64, 1) if kind == "vjp" else (256, 1))
        assert _lanes(h, kind, odd + 2) == (256, 1)
        even = fits // 2 * 2
        assert _lanes(h, kind, even) == (64, 1)
        wide = {"f": (256, 1), "jac": (256, 4), "fj": (256, 4), "vjp": (64, 1)}[kind]
        assert _lanes(h, kind, even + 2) == wide and _lanes(h, kind, 400000) == wide
    for args in ((0, -1, 5), (0, 6, 5), (0, 1 << 31, 1 << 31)):
        with pytest.raises(mcchem.MccError, match="status 1"):
            h.generated_launch(("f",)[args[0]], args[1], args[2])
