"""GPU parity of CSR SpMV where its pipelined slices can go wrong: slices of
no, one, three and four nonzeros, row counts that end inside a slice or an
item, and slices of few and of many nonzeros side by side (a worker's next
slice is requested while the previous one is added up). Rows are added in the
stored order, so every result equals the oracle bit for bit."""
import numpy as np
import pytest

from tests.gpu_helpers import dev, host, scalars

pytestmark = pytest.mark.gpu


def _lens(kind, n):
    rng = np.random.default_rng(n)
    if kind == "empty":
        return np.zeros(n, dtype=np.int64)
    if kind == "few":        # 0..4 nonzeros in a whole 32-row slice
        lens = np.zeros(n, dtype=np.int64)
        for a in range(0, n, 32):
            lens[a + int(rng.integers(0, min(32, n - a)))] = rng.integers(0, 5)
        return lens
    if kind == "short":
        return rng.integers(0, 4, n)
    return np.where(rng.integers(0, 3, n) == 0, 0, rng.integers(0, 90, n))   # "mixed": LDS and row loop


@pytest.mark.parametrize("kind", ["empty", "few", "short", "mixed"])
@pytest.mark.parametrize("n,num_wg", [(1, 0), (31, 0), (33, 0), (129, 1), (1000, 2), (4096, 3)])
def test_spmv_uneven_slices(gfx, oracle_lib, kind, n, num_wg):
    import paper_2306_11686_amd as gf
    lens = _lens(kind, n)
    rng = np.random.default_rng(7 * n)
    rowptr = np.zeros(n + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(lens)
    nnz = int(rowptr[-1])
    col = rng.integers(0, n, max(nnz, 1)).astype(np.int32)
    val = rng.standard_normal(max(nnz, 1))
    x = rng.standard_normal(n)
    ref = oracle_lib.spmv(rowptr, col, val, x)
    prog = gf.Program.make([gf.Step.make(gf.GF_R_SPMV, arr=(0, 1, 2, 3, 4), np=0)], [], 0)
    for mode in (gf.GF_EXEC_PERSISTENT, gf.GF_EXEC_PER_REGION):
        ty = dev(np.full(n, np.nan))
        inst = gf.Instance.make({0: dev(rowptr), 1: dev(col), 2: dev(val), 3: dev(x), 4: ty}, scalars(), ip=(n,))
        gfx.run(prog, inst, mode=mode, launch=gf.Launch.make(num_wg=num_wg) if num_wg else None)
        gfx.sync()
        assert np.array_equal(host(ty), ref), mode


# Work items of 128 rows as multiples of the resident workgroups, and the items of a workgroup where some start
# late rather than that a few take an item more (0: as many workgroups as are resident).
@pytest.mark.parametrize("items,each", [(1, 1), (17 / 16, 1), (3 / 2, 1), (33 / 32, 0), (13 / 8, 0), (2, 0),
                                        (35 / 16, 2), (8 / 3, 2), (11 / 4, 0), (13 / 4, 0)])
def test_spmv_grid_past_the_resident_workgroups(gfx, oracle_lib, items, each):
    import paper_2306_11686_amd as gf
    prog = gf.Program.make([], [gf.Step.make(gf.GF_R_SPMV, arr=(0, 1, 2, 3, 4), np=0),
                                gf.Step.make(gf.GF_S_SET, sc=(2,), c=1.0)], 2)

    def run(n, mode):
        rng = np.random.default_rng(n)
        rowptr = np.arange(n + 1, dtype=np.int32)
        col = rng.integers(0, n, n).astype(np.int32)
        val, x = rng.standard_normal(n), rng.standard_normal(n)
        ty = dev(np.full(n, np.nan))
        inst = gf.Instance.make({0: dev(rowptr), 1: dev(col), 2: dev(val), 3: dev(x), 4: ty}, scalars(), ip=(n,))
        st = gfx.run(prog, inst, mode=mode, launch=gf.Launch.make(wg_size=256))
        gfx.sync()
        assert np.array_equal(host(ty), oracle_lib.spmv(rowptr, col, val, x))
        return st["num_wg"]

    resident = run(128 * 16384, gf.GF_EXEC_PER_REGION)
    count = int(items * resident)
    want = -(-count // each) if each else resident
    for mode in (gf.GF_EXEC_PER_REGION, gf.GF_EXEC_PER_REGION_GRAPH):
        assert run(128 * count - 5, mode) == want
