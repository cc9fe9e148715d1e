"""Streamed lists of the tiled products against the FP64 oracle (image relative
L2 <= 1e-5, the bound of the FP32 path; 16-bit values: the oracle on the
dequantised matrix), and run twice bit for bit.  That every row sum is the one
of the CSR rows, bit for bit, is checked on the host
(tests/test_host_stream.py).

Sizes sit at the edges: one row, row blocks and column blocks with remainders,
blocks at the limits of 13 and 14 column bits, few waves, empty lists and
streams, runs of one row longer than a chunk, steps wider than a delta."""
from types import SimpleNamespace

import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


def problem(I, ny, nx, Q, per_col, seed, kind="even"):
    rng = np.random.default_rng(seed)
    J = ny * nx * Q
    if kind == "runs":      # a few rows hold most entries
        rows = np.where(rng.random((J, per_col)) < 0.6, rng.integers(0, 5, (J, per_col)),
                        rng.integers(0, I, (J, per_col)))
    elif kind == "gaps":    # entries in every 40th row and a band of columns only
        rows = rng.integers(0, max(1, I // 40), (J, per_col)) * 40
    else:
        rows = rng.integers(0, I, (J, per_col))
    cols = np.repeat(np.arange(J), per_col)
    if kind == "gaps":
        cols = cols % max(1, J // 7)
    A = sp.csr_matrix((rng.random(J * per_col).astype(np.float32) + 0.01, (rows.ravel(), cols)), shape=(I, J))
    y = rng.poisson(5.0, I).astype(np.float32)
    return A, y, np.full(I, 0.1, np.float32)


CASES = {
    # name: (I, ny, nx, Q, per_col, kind, schedule)
    "13 bits, full block": (30000, 9, 41, 54, 24, "even", dict(fwd_rows_per_wave=64, fwd_block_cols=4092,
                                                              back_rows_per_wave=64, back_block_cols=8188,
                                                              fwd_slabs=1, back_slabs=1)),
    "14 bits, widest block": (50000, 11, 23, 140, 24, "even", dict(fwd_rows_per_wave=128, fwd_block_cols=12000,
                                                                  back_rows_per_wave=100, back_block_cols=16380,
                                                                  fwd_slabs=1, back_slabs=1)),
    "all of the LDS": (60000, 16, 32, 64, 24, "even", dict(fwd_rows_per_wave=2048, fwd_block_cols=8188,
                                                         back_rows_per_wave=1560, back_block_cols=15976,
                                                         fwd_slabs=1, back_slabs=1)),
    "narrow blocks, slabs": (3001, 7, 13, 33, 16, "even", dict(waves=4, fwd_rows_per_wave=65, fwd_block_cols=256,
                                                             fwd_slabs=3, back_rows_per_wave=70,
                                                             back_block_cols=128, back_slabs=5)),
    "one wave": (700, 5, 6, 31, 9, "even", dict(waves=1, fwd_rows_per_wave=64, fwd_block_cols=512,
                                              back_rows_per_wave=300, back_block_cols=100)),
    "long runs": (2500, 6, 9, 40, 30, "runs", dict(waves=8, fwd_rows_per_wave=64, fwd_block_cols=1024,
                                                 back_rows_per_wave=64, back_block_cols=2048)),
    "wide steps": (9000, 6, 9, 40, 20, "gaps", dict(waves=8, fwd_rows_per_wave=1000, fwd_block_cols=4096,
                                                  back_rows_per_wave=64, back_block_cols=4096)),
    "one row": (1, 4, 4, 16, 1, "even", dict()),
    "automatic": (131072, 16, 16, 64, 20, "even", dict()),
}


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("name", list(CASES))
def test_streamed_matches_oracle(name, storage):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"   # before the library is loaded
    import oracle
    from paper_1601_08201_amd import sgtv
    I, ny, nx, Q, per_col, kind, sched = CASES[name]
    A, y, r = problem(I, ny, nx, Q, per_col, 3, kind)
    rowptr = A.indptr.astype(np.int64)
    out = []
    for _ in range(2):
        R = sgtv.Reconstructor(device=0)
        if sched:
            R.set_schedule(**sched)
        R.set_system(I, ny, nx, Q, rowptr, A.indices, A.data, storage=storage)
        R.set_data(y, r, 0.1, 1.0)
        R.iterate(3)
        out.append((R.image(),) + R.split())
        R.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    p = SimpleNamespace(ny=ny, nx=nx, Q=Q, I=I, J=ny * nx * Q, rowptr=rowptr, col=A.indices, val=A.data, y=y, r=r,
                        beta=0.1, rho=1.0, sweeps=1)
    if storage != "f32":
        p.val = oracle.quantise(p.col, p.val, p.J, storage)[2]
    f = oracle.admm(p, 3, report=False)[0]
    err = np.linalg.norm(out[0][0] - f) / np.linalg.norm(f)
    print(name, storage, "rel_l2", err, flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_slabs_too_short_to_stream(storage):
    """Slabs of one or two column blocks, tiles too tall and wide for 24-bit indices: both products read 32-bit
    lists (tests/test_host_choices.py walks such lists)."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import oracle
    from paper_1601_08201_amd import sgtv
    I, ny, nx, Q = 250000, 20, 20, 100
    A, y, r = problem(I, ny, nx, Q, 1, 5)
    rowptr = A.indptr.astype(np.int64)
    R = sgtv.Reconstructor(device=0)
    R.set_schedule(fwd_rows_per_wave=1500, fwd_block_cols=15000, fwd_slabs=2, back_rows_per_wave=1500,
                   back_block_cols=15000, back_slabs=9)
    R.set_system(I, ny, nx, Q, rowptr, A.indices, A.data, storage=storage).set_data(y, r, 0.1, 1.0)
    image = R.iterate(3).image()
    R.close()
    val = A.data if storage == "f32" else oracle.quantise(A.indices, A.data, ny * nx * Q, storage)[2]
    p = SimpleNamespace(ny=ny, nx=nx, Q=Q, I=I, J=ny * nx * Q, rowptr=rowptr, col=A.indices, val=val, y=y, r=r,
                        beta=0.1, rho=1.0, sweeps=1)
    f = oracle.admm(p, 3, report=False)[0]
    assert np.linalg.norm(image - f) <= 1e-5 * np.linalg.norm(f)


@pytest.mark.parametrize("name,I,ny,nx,Q,per_col", [
    ("sparse", 524288, 128, 128, 64, 4),    # more than 1024 rows per wave beside more than 8188 columns
    ("band", 400000, 80, 100, 100, 6),      # every voxel in a tenth of the detector: low tiles
])
def test_automatic_schedule_matches_oracle(name, I, ny, nx, Q, per_col):
    """Past the small scans, with the schedule that the model takes."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import oracle
    from paper_1601_08201_amd import sgtv
    J = ny * nx * Q
    rng = np.random.default_rng(9)
    rows = rng.integers(0, I, (J, per_col))
    if name == "band":
        rows = rows // 10 + (np.arange(J) * (I - I // 10) // J)[:, None]
    A = sp.csr_matrix((rng.random(J * per_col).astype(np.float32) + 0.01,
                       (rows.ravel(), np.repeat(np.arange(J), per_col))), shape=(I, J))
    y, r = rng.poisson(5.0, I).astype(np.float32), np.full(I, 0.1, np.float32)
    rowptr = A.indptr.astype(np.int64)
    R = sgtv.Reconstructor(device=0)
    R.set_system(I, ny, nx, Q, rowptr, A.indices, A.data).set_data(y, r, 0.1, 1.0)
    image, sched = R.iterate(3).image(), R.schedule()
    R.close()
    assert sched["fwd_rows_per_wave"] > 1024 if name == "sparse" else sched["fwd_rows_per_wave"] <= 512
    p = SimpleNamespace(ny=ny, nx=nx, Q=Q, I=I, J=J, rowptr=rowptr, col=A.indices, val=A.data, y=y, r=r, beta=0.1,
                        rho=1.0, sweeps=1)
    f = oracle.admm(p, 3, report=False)[0]
    assert np.linalg.norm(image - f) <= 1e-5 * np.linalg.norm(f)


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_one_row_in_three_blocks(storage):
    """One measurement that sees every voxel once: the forward list streams as one run a column block
    (tests/test_host_choices.py asserts the format)."""
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import oracle
    from paper_1601_08201_amd import sgtv
    J = 768
    val = np.random.default_rng(2).random(J).astype(np.float32) + np.float32(0.01)
    p = SimpleNamespace(ny=4, nx=4, Q=48, I=1, J=J, rowptr=np.array([0, J], np.int64), col=np.arange(J, dtype=np.int32),
                        val=val, y=np.array([40.0], np.float32), r=np.array([0.1], np.float32), beta=0.1, rho=1.0, sweeps=1)
    R = sgtv.Reconstructor(device=0)
    R.set_schedule(fwd_rows_per_wave=64, fwd_block_cols=256, fwd_slabs=1, back_rows_per_wave=64, back_block_cols=4)
    R.set_system(1, 4, 4, 48, p.rowptr, p.col, p.val, storage=storage).set_data(p.y, p.r, 0.1, 1.0)
    image = R.iterate(3).image()
    R.close()
    if storage != "f32":
        p.val = oracle.quantise(p.col, p.val, J, storage)[2]
    f = oracle.admm(p, 3, report=False)[0]
    assert np.linalg.norm(image - f) <= 1e-5 * np.linalg.norm(f)
