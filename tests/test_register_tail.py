"""The dense tail held in registers: its tables on the CPU (mcc_debug_emulate_cell)
against a dense solve, and the solver and its reverse mode on the GPU against
the oracle, where the front is empty, smaller than one k-step of the Schur
product, a whole number of k-steps or one more, and where it takes a third
register slot."""
import numpy as np
import pytest

import tape_format
from paper_2501_00011_amd import mcchem, synth

SHAPES = [(32, 32), (33, 32), (36, 32), (49, 32), (96, 32), (48, 48), (49, 48), (64, 48), (65, 48), (112, 48),
          (64, 64), (65, 64), (68, 64), (69, 64), (80, 64), (81, 64), (129, 64)]


@pytest.mark.parametrize("n,tail", SHAPES)
def test_tables(n, tail):
    """x = (I - c J)^-1 b within 1e-9 relative (norm) of LAPACK's solve: the
    matrices' condition times 2^-53 leaves three digits to spare; no index out
    of range, every stored entry set exactly once."""
    oracle = pytest.importorskip("oracle")
    m = synth.make_mechanism(n, 2 * n)
    h = mcchem.Mechanism(m, device=-1, dense_tail=tail)
    o = oracle.Oracle(m)
    c = synth.make_cells(m, 1, seed=300 + n)
    k = o.rate_constants(c.T, c.jscale)
    J = np.asarray(o.jac(k, c.y0)[0]).reshape(n, n)
    b = np.random.default_rng(n).normal(size=n) * c.y0[:, 0]
    for step in (1e-6, 1e-3, 1.0):
        _, x, bad = h.emulate_cell(k[:, 0], c.y0[:, 0], step, b)
        assert bad == 0
        ref = np.linalg.solve(np.eye(n) - step * J, b)
        assert np.linalg.norm(x - ref) <= 1e-9 * np.linalg.norm(ref)


@pytest.mark.gpu
@pytest.mark.parametrize("n,tail", SHAPES)
def test_solve_and_reverse_parity(n, tail):
    """y(dt) within the library's bar of the oracle (1e-6 |y| + 1e2 atol), and
    the reverse mode of the taped steps within its bar of the oracle's
    (1e-8 |ref| + 1e-13 max |ref|), both walking the oracle's replayed tapes."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle = pytest.importorskip("oracle")
    dev = torch.device("cuda:0")
    cells = 3
    m = synth.make_mechanism(n, 2 * n)
    h = mcchem.Mechanism(m, dense_tail=tail)
    c = synth.make_cells(m, cells, seed=400 + n)
    o = oracle.Oracle(m)
    k = o.rate_constants(c.T, c.jscale)
    print(f"register tail: {n} species, tail {tail}", flush=True)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    b = mcchem.Cells(h, cells)
    b.bind(up(c.T), up(c.P), up(c.jscale))
    y0 = up(c.y0)
    y = y0.clone()
    st, _ = b.step(y, 60.0)
    tape = torch.empty((cells, 4 + 2000 * (n + 12)), dtype=torch.float64, device=dev)
    tlen = torch.empty(cells, dtype=torch.int64, device=dev)
    y2 = y0.clone()
    b.step_taped(y2, 60.0, tape, tlen)
    assert torch.equal(y, y2) and int(st.abs().max()) == 0 and int(tlen.min()) > 0
    yr, _ = b.replay_step(y0, tape, tlen)
    torch.cuda.synchronize()
    yo, so, _ = o.solve(k, c.y0, 60.0)
    yg = y.cpu().numpy()
    assert np.all(so == 0) and np.all(np.abs(yg - yo) <= 1e-6 * np.abs(yo) + 1e2)
    assert np.all(np.abs(yr.cpu().numpy() - yg) <= 1e-7 * np.abs(yg) + 1e1)
    lam_ref, g_ref = np.zeros_like(c.y0), np.zeros((m.n_reactions, cells))
    W, tapes = np.zeros_like(c.y0), []
    rng = np.random.default_rng(n)
    for i in range(cells):
        yt, s, _, tp = o.solve_taped(k[:, i], c.y0[:, i], 60.0)
        _, rt = o.replay(k[:, i], c.y0[:, i], tp)
        W[:, i] = rng.normal(size=n) / np.maximum(np.abs(yt), 1.0)
        lam_ref[:, i], g_ref[:, i] = o.adjoint(k[:, i], c.y0[:, i], rt, W[:, i])
        tapes.append(tape_format.to_device(rt.values(), n))
    buf, lens = tape_format.pack(tapes)
    lam = up(W)
    glnk, st = b.adjoint_step(y0, up(buf), up(lens), lam)
    torch.cuda.synchronize()
    assert int(st.abs().max()) == 0
    for got, ref in ((lam.cpu().numpy(), lam_ref), (glnk.cpu().numpy(), g_ref)):
        assert np.all(np.abs(got - ref) <= 1e-8 * np.abs(ref) + 1e-13 * np.abs(ref).max(axis=0))
    b.close()
