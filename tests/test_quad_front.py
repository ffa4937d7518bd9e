"""The four-cells-per-wavefront solver with a sparse front (33 to 96 species, a
32-row tail), on the smallest batches that it takes, where the cells of a
wavefront fare differently: healthy cells keep their bits beside cells that
fail, in any order and in every launch form, and what fails, fails as in the
oracle.  The batches are copies of six cells, so that each of them comes to lie
in different places of a wavefront and beside different neighbours; the last
wavefront holds one cell."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2501_00011_amd import mcchem, synth  # noqa: E402

import tape_format  # noqa: E402

DT = 60.0
KINDS = 6


class Copies:
    """A batch just beyond the line where the four-cells kernels begin, the
    last wavefront with one cell."""

    def __init__(self, n, oracle):
        self.dev = torch.device("cuda:0")
        self.m = synth.make_mechanism(n, 2 * n if n <= 72 else 3 * n // 2)
        self.h = mcchem.Mechanism(self.m, dense_tail=32)
        lo, hi = 1, 1 << 20
        while lo < hi:  # the smallest batch they take
            mid = (lo + hi) // 2
            lo, hi = (lo, mid) if self.h.solver_dispatch(mid)["cells_per_wavefront"] == 4 else (mid + 1, hi)
        self.first = lo
        self.cells = lo + (1 - lo) % 4
        assert self.h.solver_dispatch(lo - 1)["cells_per_wavefront"] == 1 and self.cells % 4 == 1
        self.six = synth.make_cells(self.m, KINDS, seed=1800 + n)
        self.of = np.arange(self.cells) % KINDS
        self.o = oracle.Oracle(self.m)
        self.k = self.o.rate_constants(self.six.T, self.six.jscale)
        self.b = self.batch(self.cells)
        self.y0 = self.up(self.six.y0[:, self.of])
        self.y, self.status, self.stats = self.step()
        torch.cuda.synchronize()

    def up(self, a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(self.dev)

    def batch(self, cells):
        b = mcchem.Cells(self.h, cells)
        of = np.arange(cells) % KINDS
        b.bind(self.up(self.six.T[of]), self.up(self.six.P[of]), self.up(self.six.jscale[of]))
        return b

    def step(self, y0=None, stats=None, **opts):
        y = (self.y0 if y0 is None else y0).clone()
        st, stats = self.b.step(y, DT, mcchem.default_opts(**opts), stats=stats)
        return y, st, stats

    def same_in_copies(self, y, of=None):
        """Every cell's column has the bits of the first cell of its kind."""
        of = self.of if of is None else of
        kinds, first = np.unique(of, return_index=True)
        at = np.zeros(kinds.max() + 1, dtype=np.int64)
        at[kinds] = first
        y = y.cpu().numpy()
        return np.array_equal(y, y[:, at[of]], equal_nan=True)


def within(y, ref):
    """The library's bar for one outer step."""
    return bool(np.all(np.abs(y - ref) <= 1e-6 * np.abs(ref) + 1e2))


# one to four blocks of front positions: the last one full, nearly empty, in between
@pytest.fixture(scope="module", params=[33, 36, 48, 49, 64, 65, 72, 80, 81, 88])
def copies(request, oracle_mod):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"four cells a wavefront behind a front: {request.param} species", flush=True)
    return Copies(request.param, oracle_mod)


def test_oracle_and_one_cell_kernels(copies):
    """The six cells against the oracle, every copy with the same bits, from
    the first batch size on; one size below, the one-cell kernels agree within
    the bar of the step sequence's rounding."""
    c = copies
    yo, so, _ = c.o.solve(c.k, c.six.y0, DT)
    assert np.all(so == 0) and int(c.status.abs().max()) == 0
    assert within(c.y.cpu().numpy()[:, :KINDS], yo) and c.same_in_copies(c.y)
    for cells in (c.first, c.first - 1):
        b = c.batch(cells)
        y = c.y0[:, :cells].clone()
        st, _ = b.step(y, DT)
        torch.cuda.synchronize()
        assert int(st.abs().max()) == 0 and c.same_in_copies(y, c.of[:cells])
        if cells == c.first:
            assert torch.equal(y, c.y[:, :cells])
        else:
            assert within(y.cpu().numpy()[:, :KINDS], yo)
        b.close()


def test_any_order_and_launch_form(copies):
    """A permuted schedule and the per-launch form: the same bits and counters."""
    c = copies
    c.b.set_schedule(np.random.default_rng(3).permutation(c.cells).astype(np.int32))
    y, st, stats = c.step()
    yk, stk, statsk = c.step(steps_per_launch=100)
    c.b.set_schedule(None)
    torch.cuda.synchronize()
    for got in ((y, st, stats), (yk, stk, statsk)):
        assert all(torch.equal(a, b) for a, b in zip(got, (c.y, c.status, c.stats)))


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("steps_per_launch", [0, 100])
def test_non_finite_cells_beside_healthy_ones(copies, value, steps_per_launch):
    """One cell of every wavefront, each place in turn, starts non-finite: it
    says so and keeps its state, its neighbours keep their bits."""
    c = copies
    sick = np.arange(c.cells) % 4 == np.arange(c.cells) // 4 % 4
    y0 = c.y0.clone()
    y0[np.random.default_rng(5).integers(0, c.m.n_species), c.up(np.flatnonzero(sick))] = value
    y, st, stats = c.step(y0, steps_per_launch=steps_per_launch)
    torch.cuda.synchronize()
    assert np.array_equal(st.cpu().numpy(), np.where(sick, 4, 0))
    well = c.up(np.flatnonzero(~sick))
    assert torch.equal(y[:, well], c.y[:, well]) and torch.equal(stats[well], c.stats[well])
    assert np.array_equal(y.cpu().numpy()[:, sick], y0.cpu().numpy()[:, sick], equal_nan=True)


def test_work_limit(copies):
    """A limit on step attempts between those of the six cells: the cells within
    it keep their bits, the others stop at it, where the oracle stands; a limit
    of one attempt stops all."""
    import oracle
    c = copies
    sn = mcchem.stats_numpy(c.stats)
    attempts = (sn["steps"] + sn["rejects"] + sn["newton_fails"])[:KINDS]
    limit = int(np.sort(attempts)[KINDS // 2 - 1])
    y, st, stats = c.step(max_steps=limit)
    torch.cuda.synchronize()
    over = attempts[c.of] > limit
    assert 0 < over.sum() < c.cells
    assert np.array_equal(st.cpu().numpy(), np.where(over, 1, 0))
    well = c.up(np.flatnonzero(~over))
    assert torch.equal(y[:, well], c.y[:, well]) and torch.equal(stats[well], c.stats[well])
    assert c.same_in_copies(y)
    s2 = mcchem.stats_numpy(stats)
    assert np.all((s2["steps"] + s2["rejects"] + s2["newton_fails"])[over] == limit)
    _, so, _ = c.o.solve(c.k, c.six.y0, DT, oracle.default_opts(max_steps=1))
    _, st, _ = c.step(max_steps=1)
    assert np.all(so == 1) and np.all(st.cpu().numpy() == 1)
    # forty attempts from the start: the same steps as the oracle's, so its state
    yo, so, sto = c.o.solve(c.k, c.six.y0, DT, oracle.default_opts(max_steps=40))
    y, st, stats = c.step(max_steps=40)
    s2 = mcchem.stats_numpy(stats)
    assert np.all(so == 1) and np.all(st.cpu().numpy() == 1)
    for i in range(KINDS):
        if s2["steps"][i] == sto["steps"][i] and s2["rejects"][i] == sto["rejects"][i]:
            assert within(y.cpu().numpy()[:, i:i + 1], yo[:, i:i + 1])


def test_newton_failures(copies):
    """One Newton iteration never converges a step, so every cell gives up at
    the least step size, after as many failures as in the oracle."""
    import oracle
    c = copies
    kw = dict(max_newton=1, h_min_rel=1e-12)
    yo, so, sto = c.o.solve(c.k, c.six.y0, DT, oracle.default_opts(**kw))
    y, st, stats = c.step(**kw)
    torch.cuda.synchronize()
    sn = mcchem.stats_numpy(stats)
    assert np.all(so == 2) and np.all(st.cpu().numpy() == 2)
    assert np.array_equal(sn["newton_fails"], sto["newton_fails"][c.of]) and np.all(sn["steps"] == 0)
    assert torch.equal(y, c.y0)  # no step was accepted


def test_warm_start(copies):
    """First step sizes from the stats records, against the oracle given the
    same; records without a usable one start as a cold step does, bit for bit,
    beside cells that do not."""
    import oracle
    c = copies
    hw = 10.0 ** np.random.default_rng(31).uniform(-4.0, 1.0, KINDS)

    def records(h):
        st = np.zeros(c.cells, dtype=mcchem.STATS_DTYPE)
        st["h_next"] = h
        return c.up(st.view(np.uint8).reshape(c.cells, -1).copy())

    y, st, stats = c.step(stats=records(hw[c.of]), warm_start=1)
    torch.cuda.synchronize()
    yo, so, _ = c.o.solve(c.k, c.six.y0, DT, oracle.default_opts(warm_start=1), h_warm=hw)
    assert np.all(so == 0) and int(st.abs().max()) == 0
    assert within(y.cpu().numpy()[:, :KINDS], yo) and c.same_in_copies(y)
    cold = np.arange(c.cells) % 3 == 0
    bad = np.array([0.0, -1.0, np.nan, np.inf])[np.arange(c.cells) % 4]
    y2, st2, stats2 = c.step(stats=records(np.where(cold, bad, hw[c.of])), warm_start=1)
    torch.cuda.synchronize()
    assert int(st2.abs().max()) == 0
    for sel, ref in ((cold, (c.y, c.stats)), (~cold, (y, stats))):
        at = c.up(np.flatnonzero(sel))
        assert torch.equal(y2[:, at], ref[0][:, at]) and torch.equal(stats2[at], ref[1][at])


def test_tapes(copies):
    """The taping form (another build, with other registers) gives the plain
    one's bits and counters.  Tapes with room for some of the cells: those are
    whole beside the others, which are marked; the reverse mode of the whole
    ones is the oracle's adjoint of the same tapes (1e-8 of each element and
    1e-13 of the largest), and it refuses the marked ones."""
    import oracle
    c = copies
    N = c.m.n_species
    sn = mcchem.stats_numpy(c.stats)
    bound = 4 + 8 * (sn["steps"] + sn["rejects"] + sn["newton_fails"]).astype(np.int64) + N * sn["steps"].astype(np.int64)
    full = None
    for stride in (int(bound.max()), int(np.sort(bound[:KINDS])[2])):
        tape = torch.full((c.cells, stride), -7.0, dtype=torch.float64, device=c.dev)
        tl = torch.empty(c.cells, dtype=torch.int64, device=c.dev)
        y = c.y0.clone()
        stats = torch.empty_like(c.stats)
        st, _ = c.b.step_taped(y, DT, tape, tl, stats=stats)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in ((y, c.y), (st, c.status), (stats, c.stats)))
        lens = tl.cpu().numpy()
        if full is None:
            full = lens
            assert np.all(lens > 0)
        fits = full <= stride
        assert np.array_equal(lens, np.where(fits, full, -1))
        lam = np.random.default_rng(6).normal(size=(N, KINDS)) / np.maximum(np.abs(c.y.cpu().numpy()[:, :KINDS]), 1.0)
        lam_d = c.up(lam[:, c.of])
        g, ast = c.b.adjoint_step(c.y0, tape, tl, lam_d)
        torch.cuda.synchronize()
        assert np.array_equal(ast.cpu().numpy(), np.where(fits, mcchem.CELL_OK, mcchem.CELL_BAD_TAPE))
        assert c.same_in_copies(lam_d) and c.same_in_copies(g)
    # the short tapes: those that fit, against the oracle
    assert 0 < fits.sum() < c.cells
    for i in range(KINDS):
        if not fits[i]:
            continue
        ov = tape_format.to_oracle(tape[i, :int(full[i])].cpu().numpy(), N)
        assert tape_format.count_steps(ov, N) == sn["steps"][i]
        lr, gr = c.o.adjoint(c.k[:, i], c.six.y0[:, i], oracle.Tape.from_values(c.o.lib, ov), lam[:, i])
        for got, ref in ((lam_d, lr), (g, gr)):
            got = got[:, i].cpu().numpy()
            assert np.all(np.abs(got - ref) <= 1e-8 * np.abs(ref) + 1e-13 * np.abs(ref).max())


def test_every_cell_of_a_full_batch_against_the_one_cell_kernels(oracle_mod):
    """10,000 different cells of the 72-species workload in one launch, and the
    same cells in batches that the one-cell kernels take: the same within the
    difference of two accurate step sequences, each cell (the bar of one step
    against the oracle)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    m, c, dt = synth.workload("medium10k")
    h = mcchem.Mechanism(m, dense_tail=32)

    def solve(sel):
        b = mcchem.Cells(h, len(sel))
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
        b.bind(up(c.T[sel]), up(c.P[sel]), up(c.jscale[sel]))
        y = up(c.y0[:, sel])
        st, _ = b.step(y, dt)
        torch.cuda.synchronize()
        assert int(st.abs().max()) == 0
        b.close()
        return y.cpu().numpy(), h.solver_dispatch(len(sel))["cells_per_wavefront"]

    yq, four = solve(np.arange(c.n_cells))
    assert four == 4
    for s in range(0, c.n_cells, 2000):
        yo, one = solve(np.arange(s, s + 2000))
        assert one == 1 and within(yq[:, s:s + 2000], yo)
