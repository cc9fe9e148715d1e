"""Graph replay of the iteration against one-by-one launches (bitwise), with
the program's own eager work and synchronisations between replays."""
import numpy as np
import pytest

from paper_1601_08201_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    import torch
    assert torch.cuda.is_available()
    from paper_1601_08201_amd import sgtv
    sgtv.lib()
    return sgtv


@pytest.mark.parametrize("n", [10, 7])
def test_graph_replays_match_eager(sg, n):
    prob = datagen.make_problem("small", 3)
    eager = sg.Reconstructor().set_graphs(False).set_problem(prob)
    graph = sg.Reconstructor().set_problem(prob)
    for rep in range(4):
        eager.iterate(n)
        graph.iterate(n)
        # eager work between replays: an objective (launches + sync) and copies
        r1, r2 = eager.objective(), graph.objective()
        assert r1 == r2
        for a, b in zip(eager.state()[:3], graph.state()[:3]):
            np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(eager.image(), graph.image())


def test_graphs_dropped_when_data_changes(sg):
    prob = datagen.make_problem("small", 4)
    R = sg.Reconstructor().set_problem(prob)
    R.iterate(6)
    a = R.image()
    R.set_data(prob.y, prob.r, prob.beta * 2, prob.rho, 1)
    R.iterate(6)
    E = sg.Reconstructor().set_graphs(False).set_problem(prob)
    E.set_data(prob.y, prob.r, prob.beta * 2, prob.rho, 1)
    E.iterate(6)
    np.testing.assert_array_equal(R.image(), E.image())
    assert not np.array_equal(a, R.image())


@pytest.mark.parametrize("first", [0, 3])
def test_prepare_captures_without_running(sg, first):
    """prepare(n) leaves the state as it is and the iterate(n) after it equals
    the run without prepare bitwise, from either buffer parity."""
    prob = datagen.make_problem("small", 5)
    plain = sg.Reconstructor().set_problem(prob)
    prep = sg.Reconstructor().set_problem(prob)
    plain.iterate(first)
    prep.iterate(first)
    before = prep.state()
    prep.prepare(12)
    prep.prepare(12)   # already cached: nothing to do
    for a, b in zip(before, prep.state()):
        np.testing.assert_array_equal(a, b)
    assert prep.objective()["iter"] == first
    for rep in range(3):
        plain.iterate(12)
        prep.iterate(12)
        assert plain.objective() == prep.objective()
        np.testing.assert_array_equal(plain.image(), prep.image())
    assert prep.objective()["iter"] == first + 36


def test_prepare_arguments(sg):
    prob = datagen.make_problem("small", 6)
    R = sg.Reconstructor()
    with pytest.raises(sg.SgtvError):
        R.prepare(5)   # no system yet
    R.set_problem(prob)
    with pytest.raises(sg.SgtvError):
        R.prepare(-1)
    R.prepare(0)
    R.prepare(1)
    R.set_graphs(False).prepare(8)   # graphs off: nothing to capture
    R.set_graphs(True)
    R.prepare(8)
    R.set_data(prob.y, prob.r, prob.beta, prob.rho, 1)   # drops the graph; the next call captures again
    R.iterate(8)
    E = sg.Reconstructor().set_graphs(False).set_problem(prob)
    E.iterate(8)
    np.testing.assert_array_equal(R.image(), E.image())
    R.close()
    E.close()


def test_pieces_and_kept_graphs(sg):
    """Past 80, iterations run in graph pieces of 40 and a rest, and graphs outlive
    set_data with the same parameters: bit for bit the eager run, from host and
    device arrays, after refused data, and past the graphs that are kept."""
    import torch
    prob = datagen.make_problem("small", 6)
    other = datagen.make_problem("small", 7)
    E = sg.Reconstructor().set_graphs(False).set_problem(prob)
    G = sg.Reconstructor().set_problem(prob)
    y2 = other.y * np.float32(1.5)
    dev = [torch.from_numpy(a).cuda() for a in (y2, prob.r)]
    bad = prob.y.copy()
    bad[[7, 90]] = np.nan, -1.0
    bad_r = prob.r.copy()
    bad_r[5] = 0.0
    for n in (39, 80, 81, 123, 2, 3, 4, 5, 6, 7, 8, 9, 120):
        for R in (E, G):
            R.set_data(prob.y, prob.r, prob.beta, prob.rho, 1)
            R.iterate(n)
            a = R.state()
            with pytest.raises(sg.SgtvError, match="y has a negative or non-finite value at 7"):
                R.set_data(bad, prob.r, prob.beta, prob.rho, 1)
            with pytest.raises(sg.SgtvError, match="index 5"):
                R.set_data(bad, bad_r, prob.beta, prob.rho, 1)
            for u, v in zip(a[:3], R.state()[:3]):
                np.testing.assert_array_equal(u, v)
        np.testing.assert_array_equal(E.image(), G.image())
        E.set_data(y2, prob.r, prob.beta, prob.rho, 1).iterate(n)
        G.set_data(dev[0], dev[1], prob.beta, prob.rho, 1).iterate(n)
        np.testing.assert_array_equal(E.image(), G.image())
        assert E.objective() == G.objective()


@pytest.mark.parametrize("case", ["first data", "data again", "sliced ELL"])
def test_set_data_waits_for_the_default_stream(sg, case):
    """Device arrays that the default stream is still writing when set_data is called, from a context on a
    stream of its own: the values that the default stream leaves there are the ones that are used."""
    import torch
    prob = datagen.make_problem("small", 6)
    y, r = torch.from_numpy(prob.y).cuda(), torch.from_numpy(prob.r).cuda()
    side = torch.cuda.Stream()
    R, E = sg.Reconstructor(stream=side.cuda_stream), sg.Reconstructor()
    for X in (R, E):
        if case == "sliced ELL":
            X.set_schedule(format=1)
        X.set_system(prob.I, prob.ny, prob.nx, prob.Q, prob.rowptr, prob.col, prob.val)
    if case == "data again":
        R.set_data(torch.ones_like(y), r, prob.beta, prob.rho, 1).iterate(3)
    late = torch.zeros_like(y)
    a = torch.rand((8192, 8192), device="cuda")
    torch.cuda.synchronize()
    for _ in range(8):               # some milliseconds of work before y is there
        a = (a @ a) * 1e-4
    late.copy_(y)
    R.set_data(late, r, prob.beta, prob.rho, 1).iterate(4)
    E.set_data(y, r, prob.beta, prob.rho, 1).iterate(4)
    np.testing.assert_array_equal(R.image(), E.image())
