"""The four-cells-per-wavefront solver: its host-compiled tables run on the
CPU (mcc_debug_emulate_quad) against the oracle's f and a dense solve, and the
kernels on the GPU against the oracle, at the sizes where its shapes begin and
end (blocks of 16 rows, 16 / 24 / 32 dense columns, one to four blocks of
front positions, the last block full, nearly empty) and at batch sizes that
leave rows of the last wavefront empty."""
import numpy as np
import pytest

from paper_2501_00011_amd import mcchem, synth

# species, dense tail: dense in registers up to 32 species; a 32-row tail behind 1 .. 64 front positions
SHAPES = [(5, 0), (16, 0), (17, 0), (24, 0), (25, 0), (32, 0),
          (33, 32), (36, 32), (48, 32), (49, 32), (64, 32), (65, 32), (72, 32), (80, 32), (81, 32), (88, 32)]


def _mechanism(n):
    """Twice as many reactions as species; fewer above 72, where three
    wavefronts' cells would not fit a compute unit's local memory otherwise."""
    return synth.make_mechanism(n, 2 * n if n <= 72 else 3 * n // 2)


@pytest.mark.parametrize("n,tail", SHAPES)
def test_tables_against_oracle_and_dense_solve(n, tail):
    """f within 1e-12 of its scale (the bound of the library's other f
    checks); x = (I - c J)^-1 b within 1e-9 relative (norm) of LAPACK's
    solve: the matrices' condition times 2^-53 leaves three digits to spare;
    no index out of range, no constant cell written, nothing read before it
    is written."""
    oracle = pytest.importorskip("oracle")
    m = _mechanism(n)
    h = mcchem.Mechanism(m, device=-1, dense_tail=tail)
    o = oracle.Oracle(m)
    c = synth.make_cells(m, 1, seed=700 + n)
    k = o.rate_constants(c.T, c.jscale)
    fr, fs = o.deriv(k, c.y0)
    J = o.jac(k, c.y0)[0]
    J = np.asarray(J).reshape(n, n) if np.asarray(J).size == n * n else np.asarray(J)[..., 0]
    rng = np.random.default_rng(n)
    for step in (1e-6, 1e-3, 1.0):
        b = rng.normal(size=n) * c.y0[:, 0]
        f, x, bad = h.emulate_cell(k[:, 0], c.y0[:, 0], step, b, quad=True)
        assert bad == 0
        assert np.all(np.abs(f - fr[:, 0]) <= 1e-12 * fs[:, 0])
        ref = np.linalg.solve(np.eye(n) - step * J, b)
        assert np.linalg.norm(x - ref) <= 1e-9 * np.linalg.norm(ref)


def test_shapes_it_does_not_take():
    for n, tail in ((40, 0), (72, 48), (96, 32), (97, 32), (150, 64)):
        h = mcchem.Mechanism(synth.make_mechanism(n, 2 * n), device=-1, dense_tail=tail)
        with pytest.raises(mcchem.MccError, match="four-cells"):
            h.emulate_cell(np.ones(h.n_reactions), np.ones(n), 1.0, np.ones(n), quad=True)
    # more reactions than the kernels hold rate constants for
    h = mcchem.Mechanism(synth.make_mechanism(20, 129), device=-1)
    with pytest.raises(mcchem.MccError, match="four-cells"):
        h.emulate_cell(np.ones(129), np.ones(20), 1.0, np.ones(20), quad=True)


@pytest.mark.gpu
@pytest.mark.parametrize("n,tail", SHAPES)
def test_solve_parity_and_forms(n, tail):
    """y(dt) within the library's bar of the oracle (1e-6 |y| + 1e2 atol), for
    batches whose last wavefront holds one to four cells: a few cells without
    a front, where these kernels take every batch, and otherwise copies of six
    cells just beyond eight for each compute unit, where they begin to.  Every
    copy has the same bits, and so have the per-launch and the taping form; the
    batch at that limit (the one-cell kernels) meets the same bar."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle = pytest.importorskip("oracle")
    dev = torch.device("cuda:0")
    m = _mechanism(n)
    h = mcchem.Mechanism(m, dense_tail=tail)
    c = synth.make_cells(m, 6, seed=800 + n)
    o = oracle.Oracle(m)
    k = o.rate_constants(c.T, c.jscale)
    yo, so, _ = o.solve(k, c.y0, 60.0)
    base = 8 * torch.cuda.get_device_properties(0).multi_processor_count if tail else 0
    ref = None
    for cells in (base + 6, base + 5, base + 1, base):
        if cells == 0:
            continue
        print(f"quad solver: {n} species, {cells} cells", flush=True)
        of = np.arange(cells) % 6
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a[..., of])).to(dev)  # noqa: E731
        b = mcchem.Cells(h, cells, cells + 1)
        b.bind(up(c.T), up(c.P), up(c.jscale))
        y0 = torch.zeros((n, cells + 1), dtype=torch.float64, device=dev)
        y0[:, :cells] = up(c.y0)
        y = y0.clone()
        st, stats = b.step(y, 60.0)
        torch.cuda.synchronize()
        yg = y.cpu().numpy()
        assert np.array_equal(st.cpu().numpy(), so[of]) and np.all(so == 0)
        assert np.all(yg[:, cells] == 0.0)  # nothing written beyond the cells
        yg = yg[:, :cells]
        assert np.all(np.abs(yg[:, :6] - yo[:, of[:6]]) <= 1e-6 * np.abs(yo[:, of[:6]]) + 1e2)
        assert np.array_equal(yg, yg[:, of])
        if cells > base:
            ref = yg[:, :6] if ref is None else ref
            assert np.array_equal(yg[:, :6], ref[:, of[:6]])
        if cells == base + 5:
            y2 = y0.clone()
            st2, stats2 = b.step(y2, 60.0, mcchem.default_opts(steps_per_launch=150 if tail else 7))
            assert torch.equal(y2, y) and torch.equal(st2, st) and torch.equal(stats2, stats)
            tape = torch.empty((cells, 4 + 2000 * (n + 12)), dtype=torch.float64, device=dev)
            tlen = torch.empty(cells, dtype=torch.int64, device=dev)
            y3 = y0.clone()
            b.step_taped(y3, 60.0, tape, tlen)
            assert torch.equal(y3, y) and int(tlen.min()) > 0
            y4, _ = b.replay_step(y0, tape, tlen)
            torch.cuda.synchronize()
            # the replay solves each step to convergence: within the Newton tolerance of the solve
            y4 = y4.cpu().numpy()[:, :cells]
            assert np.all(np.abs(y4 - yg) <= 1e-7 * np.abs(yg) + 1e1)
        b.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,cells", [(5, 1), (16, 3), (16, 257), (17, 4), (24, 130), (32, 65), (40, 257)])
def test_multicell(n, cells):
    """One system over all cells, at batch sizes around a full wavefront (four
    cells) and around what a wavefront's lanes read of the others' sums at a
    time (16 wavefronts of four values, 256 of the one-cell kernels, which take
    40 species): the oracle's shared step sequence and y(dt) within the
    library's bar, every call with the same bits, and one cell with those of
    its own solve."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle = pytest.importorskip("oracle")
    dev = torch.device("cuda:0")
    m = synth.make_mechanism(n, 2 * n)
    h = mcchem.Mechanism(m, dense_tail=0)
    c = synth.make_cells(m, cells, seed=900 + n)
    o = oracle.Oracle(m)
    k = o.rate_constants(c.T, c.jscale)
    yo, so, sto = o.solve_multicell(k, c.y0, 20.0)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    print(f"Multi-cells: {n} species, {cells} cells", flush=True)
    b = mcchem.Cells(h, cells)
    b.bind(up(c.T), up(c.P), up(c.jscale))
    y0 = up(c.y0)
    out = []
    for call in (dict(), dict(), dict(noalloc=True)):
        y = y0.clone()
        st, stats = b.step_multicell(y, 20.0, **call)
        torch.cuda.synchronize()
        assert so == 0 and int(st.abs().max()) == 0
        out.append((y, stats))
    assert all(torch.equal(out[0][0], y) and torch.equal(out[0][1], s) for y, s in out[1:])
    yg, sn = out[0][0].cpu().numpy(), mcchem.stats_numpy(out[0][1])
    assert np.all(np.abs(yg - yo) <= 1e-6 * np.abs(yo) + 1e2)
    assert np.all(sn["steps"] == sn["steps"][0])
    assert abs(int(sn["steps"][0]) - int(sto["steps"])) <= 0.05 * int(sto["steps"]) + 2
    if cells == 1:
        y = y0.clone()
        st, stats = b.step(y, 20.0)
        assert torch.equal(y, out[0][0]) and torch.equal(stats, out[0][1])
    b.close()


@pytest.mark.gpu
def test_error_weights_beyond_the_range():
    """rtol |y| beyond the largest double: a weight of zero, as in the oracle
    and the one-cell kernels, and no NaN (tolerances this loose accept every
    step, so both take the same ones)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle = pytest.importorskip("oracle")
    dev = torch.device("cuda:0")
    m = synth.make_mechanism(20, 40)
    c = synth.make_cells(m, 5, seed=77)
    y0 = np.maximum(c.y0, 1e9)
    o = oracle.Oracle(m)
    yo, so, sto = o.solve(o.rate_constants(c.T, c.jscale), y0, 60.0, oracle.default_opts(rtol=1e300))
    assert np.all(so == 0)
    h = mcchem.Mechanism(m, dense_tail=0)
    b = mcchem.Cells(h, 5)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    b.bind(up(c.T), up(c.P), up(c.jscale))
    y = up(y0)
    st, stats = b.step(y, 60.0, mcchem.default_opts(rtol=1e300))
    torch.cuda.synchronize()
    assert np.array_equal(st.cpu().numpy(), so)
    assert np.array_equal(mcchem.stats_numpy(stats)["steps"], sto["steps"])
    assert np.all(np.abs(y.cpu().numpy() - yo) <= 1e-6 * np.abs(yo) + 1e2)
    b.close()


def test_tables_cost_little_to_build():
    """Compiling a mechanism with these tables takes about as long as without
    them (a tail of 48 rows): measured 1.5 times; 5.5 times while every split of
    the front that was tried laid out all entries."""
    import time
    m = synth.make_mechanism(94, 150)
    best = {}
    for tail in 5 * (32, 48):
        t = time.process_time()
        mcchem.Mechanism(m, device=-1, dense_tail=tail).close()
        best[tail] = min(best.get(tail, 9.0), time.process_time() - t)
    assert best[32] <= 3.0 * best[48], best


@pytest.mark.gpu
@pytest.mark.parametrize("n,tail,cells", [(20, 0, 9), (32, 0, 4), (40, 0, 9), (72, 48, 9)])
def test_multicell_failures(n, tail, cells):
    """What stops the one system stops every cell, where the oracle's stops: a
    work limit, a Newton iteration that cannot converge, a non-finite state in
    one cell (nothing is written then).  A call after that is as the first."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle = pytest.importorskip("oracle")
    dev = torch.device("cuda:0")
    m = synth.make_mechanism(n, 2 * n)
    h = mcchem.Mechanism(m, dense_tail=tail)
    c = synth.make_cells(m, cells, seed=950 + n)
    o = oracle.Oracle(m)
    k = o.rate_constants(c.T, c.jscale)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    b = mcchem.Cells(h, cells)
    b.bind(up(c.T), up(c.P), up(c.jscale))

    def step(y0, **kw):
        y = up(y0)
        st, stats = b.step_multicell(y, 5.0, mcchem.default_opts(**kw))
        torch.cuda.synchronize()
        return y.cpu().numpy(), st.cpu().numpy(), mcchem.stats_numpy(stats)

    first = step(c.y0)
    for kw, status in ((dict(max_steps=1), 1), (dict(max_steps=30), 1), (dict(max_newton=1, h_min_rel=1e-12), 2)):
        print(f"Multi-cells: {n} species, {cells} cells, {kw}", flush=True)
        yo, so, sto = o.solve_multicell(k, c.y0, 5.0, oracle.default_opts(**kw))
        y, st, sn = step(c.y0, **kw)
        assert so == status and np.all(st == status)
        assert np.all(sn["newton_fails"] == sto["newton_fails"]) and np.all(sn["steps"] == sto["steps"])
        assert np.all(np.abs(y - yo) <= 1e-6 * np.abs(yo) + 1e2)
    sick = c.y0.copy()
    sick[n // 2, cells - 1] = np.nan
    y, st, _ = step(sick)
    assert np.all(st == 4) and np.array_equal(y, sick, equal_nan=True)
    again = step(c.y0)
    assert all(np.array_equal(p, q) for p, q in zip(first, again))
    b.close()
