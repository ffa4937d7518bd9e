"""How much tape autograd.solve_step allocates and keeps (host logic: the
library's calls replaced by ones that only say whether a tape fits, and an
allocator with a limit)."""
import types
import weakref

import pytest

torch = pytest.importorskip("torch")

from paper_2501_00011_amd import autograd, mcchem  # noqa: E402

N, C = 4, 8
LEAST = 4 + 256 * (N + 16)


def doubled(width, need):
    while width < need:
        width *= 2
    return width


class Cells:
    """A batch whose tapes need `need` doubles each."""

    def __init__(self, need, n_cells=C):
        self.n_cells, self.need = n_cells, need
        self.mech = types.SimpleNamespace(n_species=N)
        self.widths, self.kept = [], None

    def set_rate_constants(self, k):
        pass

    def step_taped(self, y, dt, tape, tape_len, opts=None):
        self.widths.append(tape.shape[1])
        tape_len.fill_(self.need if self.need <= tape.shape[1] else -1)
        tape[:, :min(self.need, tape.shape[1])] = 3.0
        y += 1.0
        return torch.zeros(self.n_cells, dtype=torch.int32), None

    def adjoint_step(self, y0, tape, tape_len, lam):
        assert tape.is_contiguous() and bool((tape[:, :self.need] == 3.0).all())
        self.kept = tape.shape[1]
        return torch.zeros(2, self.n_cells, dtype=torch.float64), torch.zeros(self.n_cells, dtype=torch.int32)


def run(cells, stride=None):
    y0 = torch.ones(N, cells.n_cells, dtype=torch.float64, requires_grad=True)
    lnk = torch.zeros(2, cells.n_cells, dtype=torch.float64, requires_grad=True)
    y = autograd.solve_step(cells, y0, lnk, 1.0, tape_stride=stride)
    assert torch.equal(y.detach(), torch.full_like(y, 2.0))
    y.sum().backward()


@pytest.fixture
def limit(monkeypatch):
    """limit(d): tapes of more than d doubles in all, at one time, are refused."""
    real, live = torch.empty, []

    def set_limit(doubles):
        def empty(*shape, **kw):
            n = 1
            for x in (shape[0] if isinstance(shape[0], tuple) else shape):
                n *= x
            if kw.get("dtype") == torch.float64:
                held = sum(t().numel() for t in live if t() is not None)
                if held + n > doubles:
                    raise torch.cuda.OutOfMemoryError("no room")
            t = real(*shape, **kw)
            if kw.get("dtype") == torch.float64:
                live.append(weakref.ref(t))
            return t
        monkeypatch.setattr(torch, "empty", empty)
    return set_limit


@pytest.mark.parametrize("steps", [1, 255, 256, 257, 700, 1024, 2000, 4000])
def test_kept_tape_is_no_wider_than_doublings(steps):
    need = 4 + steps * (N + 16)
    c = Cells(need)
    run(c)
    assert len(c.widths) == 1  # the first attempt has room
    assert need <= c.kept <= doubled(LEAST, need)


def test_large_batches_double_and_keep_no_more(monkeypatch):
    """A first tape that is no doubling of the least (305 steps of room)."""
    monkeypatch.setattr(autograd, "_first_steps", lambda n_cells, n_species: 305)
    for steps in (300, 306, 1326, 2100):
        c = Cells(4 + steps * (N + 16))
        run(c)
        assert c.need <= c.kept <= doubled(LEAST, c.need)


@pytest.mark.parametrize("steps", [100, 300, 1326, 3000])
def test_short_memory(limit, steps):
    """Memory for one tape of the least room's doublings is enough: neither the
    larger first tape nor the copy that cuts it needs more."""
    need = 4 + steps * (N + 16)
    enough = doubled(LEAST, need)
    limit(C * enough)
    c = Cells(need)
    run(c)
    assert need <= c.kept <= enough
    limit(C * enough - 1 if enough == LEAST else C * (enough // 2))
    with pytest.raises(torch.cuda.OutOfMemoryError):
        run(Cells(need))


def test_no_room_for_the_copy(limit):
    """The first tape fits, the copy beside it does not: the step is taken again
    with the doubling that holds it."""
    first = 4 + 4096 * (N + 16)
    need = 4 + 1326 * (N + 16)
    limit(C * first)
    c = Cells(need)
    run(c)
    assert c.widths == [first, doubled(LEAST, need)] and c.kept == c.widths[1]


def test_given_stride_is_doubled():
    c = Cells(1000)
    run(c, stride=300)
    assert c.widths == [300, 600, 1200] and c.kept == 1200


def test_empty_batch():
    c = Cells(0, n_cells=0)
    run(c)
    assert c.kept is not None
    assert mcchem.CELL_OK == 0
