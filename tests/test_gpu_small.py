"""Small scans: the automatic schedule iterates on a second, sliced-ELL copy in
two launches; the same schedule given field by field keeps to the tiles.  Both
add in the same order, so images, splits, objectives and checkpoints agree bit
for bit, whatever the weights, grouping, value type, sweeps and slabs, with
unsorted and duplicate columns, empty rows and columns, and lines at and past
the longest that the copy takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sg():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1601_08201_amd import sgtv
    return sgtv


def csr(I, J, per_col, seed, kind):
    rng = np.random.default_rng(seed)
    rows = rng.integers(0, I, J * per_col)
    cols = np.repeat(np.arange(J), per_col)
    if kind == "long":       # a row of 192 entries, the longest that is taken, and one past it
        rows[rows == 3] = 4
        rows[:192] = 3
    if kind == "too long":
        rows[rows == 3] = 4
        rows[:193] = 3
    if kind == "gaps":
        rows, cols = rows // 3 * 3, cols // 2 * 2
    order = np.lexsort((rng.random(rows.size), rows)) if kind == "unsorted" else np.lexsort((cols, rows))
    rowptr = np.zeros(I + 1, np.int64)
    rowptr[1:] = np.bincount(rows, minlength=I).cumsum()
    return rowptr, cols[order].astype(np.int32), (rng.random(rows.size) + 0.01).astype(np.float32)


CASES = [
    # I, ny, nx, Q, per_col, kind, storage, weights, grouping, sweeps
    (4096, 16, 16, 32, 16, "even", "f32", None, 0, 1),
    (8192, 9, 41, 54, 24, "even", "f32", 4, 0, 1),
    (8192, 9, 41, 54, 24, "even", "f32", "full", 1, 2),
    (24001, 23, 29, 61, 21, "even", "bf16", None, 0, 1),      # several slabs both ways
    (40000, 17, 31, 77, 20, "unsorted", "f32", 4, 1, 1),
    (30011, 13, 37, 40, 9, "gaps", "f16", "full", 0, 3),
    (3000, 5, 7, 129, 6, "long", "f32", None, 0, 1),
    (3000, 5, 7, 129, 6, "too long", "f32", None, 0, 1),
    (65, 1, 3, 1, 2, "even", "f32", None, 1, 1),
    (1, 1, 1, 1, 1, "even", "bf16", None, 0, 1),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_small_equals_tiled(sg, case):
    I, ny, nx, Q, per_col, kind, storage, weights, grouping, sweeps = CASES[case]
    J = ny * nx * Q
    rowptr, col, val = csr(I, J, per_col, case, kind)
    rng = np.random.default_rng(50 + case)
    w = None if weights is None else (rng.random(4 if weights == 4 else 4 * J) + 0.3).astype(np.float32)
    y, r = rng.poisson(6.0, I).astype(np.float32), np.full(I, 0.1, np.float32)

    def run(**sched):
        R = sg.Reconstructor()
        if sched:
            R.set_schedule(**sched)
        R.set_system(I, ny, nx, Q, rowptr, col, val, storage=storage, w=w)
        R.set_grouping(grouping)
        return R.set_data(y, r, 0.2, 1.0, sweeps)

    S = run()
    T = run(**S.schedule())
    assert S.schedule() == T.schedule()
    for n in (1, 2, 5, 90):
        S.iterate(n)
        T.iterate(n)
        for a, b in zip(S.state()[:3], T.state()[:3]):
            np.testing.assert_array_equal(a, b)
        assert S.objective() == T.objective()
    S.set_graphs(False).iterate(7)
    T.iterate(7)
    state = T.state()
    for a, b in zip(S.state()[:3], state[:3]):
        np.testing.assert_array_equal(a, b)
    S.set_graphs(True)
    S.set_state(*state).iterate(3)   # resume from the other's checkpoint
    S.set_epilogues(True).iterate(2)
    S.set_epilogues(False).iterate(2)
    T.iterate(7)
    np.testing.assert_array_equal(S.image(), T.image())


def test_an_infinite_ratio_stays_in_its_row(sg):
    """Row 0 is empty and its ratio overflows: no voxel sees it."""
    rowptr, col, val = csr(2999, 5 * 7 * 9, 6, 4, "even")
    rowptr = np.concatenate([[0], rowptr])
    y, r = np.random.default_rng(3).poisson(6.0, 3000).astype(np.float32), np.full(3000, 0.1, np.float32)
    y[0], r[0] = 1e5, 1e-37
    S = sg.Reconstructor().set_system(3000, 5, 7, 9, rowptr, col, val).set_data(y, r, 0.2, 1.0)
    T = sg.Reconstructor().set_schedule(**S.schedule()).set_system(3000, 5, 7, 9, rowptr, col, val)
    T.set_data(y, r, 0.2, 1.0)
    image = S.iterate(20).image()
    assert np.isfinite(image).all()
    np.testing.assert_array_equal(image, T.iterate(20).image())


def test_small_scan_from_a_file_and_a_workspace(sg, tmp_path):
    import torch
    rowptr, col, val = csr(8192, 19926, 24, 1, "even")
    y, r = np.random.default_rng(3).poisson(6.0, 8192).astype(np.float32), np.full(8192, 0.1, np.float32)
    args = (8192, 9, 41, 54, rowptr, col, val)
    A = sg.Reconstructor().set_system(*args)
    A.save_system(str(tmp_path / "s"))
    B = sg.Reconstructor().load_system(str(tmp_path / "s"))
    C = sg.Reconstructor()
    ws = torch.empty(C.plan_system(*args), dtype=torch.uint8, device="cuda")
    C.commit_system(ws)
    images = [R.set_data(y, r, 0.2, 1.0).iterate(25).image() for R in (A, B, C)]
    np.testing.assert_array_equal(images[0], images[1])
    np.testing.assert_array_equal(images[0], images[2])
    assert C.device_bytes() == 0


@pytest.mark.parametrize("I,ny,nx,Q,weights,grouping,sweeps,storage", [
    (4096, 16, 16, 32, None, 0, 1, "f32"),    # four rows of the ratio per thread
    (4097, 9, 41, 54, 4, 0, 2, "f32"),        # one row per thread
    (3002, 5, 7, 129, "full", 1, 1, "bf16"),  # more spectral bins than a segment has lanes
    (30001, 1, 3, 1, None, 0, 3, "f32"),      # fewer bins than a block of the split update
])
def test_split_beside_ratio_equals_apart(sg, I, ny, nx, Q, weights, grouping, sweeps, storage):
    """With kernel timing on, every step of an iteration has its own launch."""
    J = ny * nx * Q
    rowptr, col, val = csr(I, J, 6, 2, "even")
    rng = np.random.default_rng(5)
    w = None if weights is None else (rng.random(4 if weights == 4 else 4 * J) + 0.3).astype(np.float32)
    y, r = rng.poisson(6.0, I).astype(np.float32), np.full(I, 0.1, np.float32)
    A, B = sg.Reconstructor(), sg.Reconstructor()
    for R in (A, B):
        R.set_schedule(variant=1).set_system(I, ny, nx, Q, rowptr, col, val, storage=storage, w=w)
        R.set_grouping(grouping)
        R.set_data(y, r, 0.2, 1.0, sweeps)
    B.set_profiling(True)
    for n in (1, 2, 13):
        A.iterate(n)
        B.iterate(n)
        for a, b in zip(A.state()[:3], B.state()[:3]):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("deep,taken", [(40, True), (150, False)])
def test_padding_of_uneven_columns_is_bounded(sg, deep, taken):
    """Every 64th voxel with many entries, two in the others: slices of 64 columns are as deep as the longest. The copy
    is left out where it is mostly padding; the images do not depend on it."""
    I, ny, nx, Q = 131072, 64, 64, 64
    J = ny * nx * Q
    rng = np.random.default_rng(8)
    cols = np.repeat(np.arange(J), np.where(np.arange(J) % 64 == 0, deep, 2))
    rows = rng.integers(0, I, cols.size)
    order = np.lexsort((cols, rows))
    rowptr = np.zeros(I + 1, np.int64)
    rowptr[1:] = np.bincount(rows, minlength=I).cumsum()
    args = (I, ny, nx, Q, rowptr, cols[order].astype(np.int32), (rng.random(cols.size) + 0.01).astype(np.float32))
    y, r = rng.poisson(6.0, I).astype(np.float32), np.full(I, 0.1, np.float32)
    A = sg.Reconstructor().set_system(*args).set_data(y, r, 0.2, 1.0)
    T = sg.Reconstructor().set_schedule(**A.schedule()).set_system(*args).set_data(y, r, 0.2, 1.0)
    copy = A.device_bytes() - T.device_bytes()
    assert (copy > 0) == taken and copy <= 3 * T.device_bytes()
    np.testing.assert_array_equal(A.iterate(5).image(), T.iterate(5).image())
