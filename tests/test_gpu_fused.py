"""Several sweeps per pass (launch shape left to the library) against one
sweep per pass (a given tile) of the same program on the same data: both
grids bit for bit, also where the outer layers of the two buffers differ, and
every sweep's residual (a 2D residual is a sum taken in another order: within
1e-12 of it, all terms being >= 0; a 3D one is a max and must be equal)."""
import math

import numpy as np
import pytest

import gf_inputs as gi
from tests.gpu_helpers import dev, host, scalars

pytestmark = pytest.mark.gpu


def _run(ctx, prog, u0, w0, sweeps, launch, mode=None, record=None):
    import torch
    import paper_2306_11686_amd as gf
    u, w = dev(u0), dev(w0)
    res = torch.zeros(max(1, sweeps), dtype=torch.float64, device="cuda") if record is None else record(u, w)
    sc = scalars({5: 3.0})
    inst = gf.Instance.make({0: u, 1: w, 2: res}, sc, ip=(u0.shape[0],))
    st = ctx.run(prog, inst, mode=gf.GF_EXEC_PERSISTENT, launch=launch)
    ctx.sync()
    return host(u), host(w), host(res).copy(), host(sc), st


def _outer_differs(u0, seed):
    """A second buffer with its own outer layer and interior."""
    return gi.um11(seed, 33, np.arange(u0.size, dtype=np.uint64)).reshape(u0.shape)


# sides: one and several 128-column items, odd and even, ends of a segment;
# sweeps: every remainder of the pass lengths seven, three and one
@pytest.mark.parametrize("n,sweeps", [(3, 4), (16, 5), (17, 8), (64, 7), (128, 11), (129, 9), (241, 15), (256, 22),
                                      (345, 8), (513, 10), (1000, 9), (1023, 8)])
def test_fused_2d_equals_sweep_by_sweep(gfx, n, sweeps):
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    print(f"fused 2d n={n} sweeps={sweeps}", flush=True)
    u0 = gi.um11(3, 32, np.arange(n * n, dtype=np.uint64)).reshape(n, n)
    w0 = _outer_differs(u0, 4)
    prog = programs.jacobi2d(sweeps)
    a = _run(gfx, prog, u0, w0, sweeps, None)
    b = _run(gfx, prog, u0, w0, sweeps, gf.Launch.make(wg_size=256, tile_y=16))
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert np.all(np.abs(a[2] - b[2]) <= 1e-12 * b[2])
    assert b[4]["barriers"] == sweeps and (n < 16 or a[4]["barriers"] < sweeps)


def test_fused_2d_grid_sizes_and_xcd_remap(gfx):
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    n, sweeps = 300, 10
    u0 = gi.grid2d(n, seed=6)
    prog = programs.jacobi2d(sweeps)
    b = _run(gfx, prog, u0, u0, sweeps, gf.Launch.make(wg_size=256, tile_y=16))
    for nwg in (1, 2, 7, 100, 300):
        a = _run(gfx, prog, u0, u0, sweeps, gf.Launch.make(num_wg=nwg, xcd_remap=nwg % 2))
        assert a[4]["num_wg"] == nwg
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert np.all(np.abs(a[2] - b[2]) <= 1e-12 * b[2])


def _steps_around(gf, kind, red_op, n_sweeps, swap_first=False):
    """A body with scalar steps before, between and after the region: a
    running sum of the residuals, a quotient and a copy."""
    S = gf.Step
    swap = S.make(gf.GF_S_SWAP, arr=(1, 0))
    region = S.make(kind, arr=(0, 1), sc=(0,), red_op=red_op, np=0)
    body = [S.make(gf.GF_S_SET, sc=(0,), c=0.0), region, S.make(gf.GF_S_DIV, sc=(1, 0, 5)), swap,
            S.make(gf.GF_S_SQRT, sc=(2, 1)), S.make(gf.GF_S_COPY, sc=(3, 2)),
            S.make(gf.GF_S_RECORD, arr=(2,), sc=(3,))]
    if swap_first:
        body.remove(swap)
        body.insert(0, swap)
    return gf.Program.make([S.make(gf.GF_S_COPY, sc=(6, 5))], body, n_sweeps)


@pytest.mark.parametrize("swap_first", [False, True])
@pytest.mark.parametrize("red", [True, False])
def test_fused_serial_steps_and_forms(gfx, red, swap_first):
    """Scalar steps around the region see every sweep in order; a body whose
    SWAP comes first, and one without a reduction, give the same grids."""
    import paper_2306_11686_amd as gf
    n, sweeps = 150, 13
    u0 = gi.grid2d(n, seed=7)
    w0 = _outer_differs(u0, 8)
    prog = _steps_around(gf, gf.GF_R_JACOBI2D, gf.GF_OP_SUM if red else gf.GF_OP_NONE, sweeps, swap_first)
    a = _run(gfx, prog, u0, w0, sweeps, None)
    b = _run(gfx, prog, u0, w0, sweeps, gf.Launch.make(wg_size=256, tile_y=16))
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    assert np.all(np.abs(a[2] - b[2]) <= 1e-12 * b[2])
    assert np.all(np.abs(a[3] - b[3]) <= 1e-12 * np.abs(b[3]))


def test_fused_records_that_share_memory_with_a_grid(gfx):
    """A body that records into the grid's own memory is run sweep by sweep:
    the recorded value is what the next sweep reads (one workgroup: with more,
    nothing orders the record before the other workgroups' reads)."""
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    n, sweeps = 64, 6
    u0 = gi.grid2d(n, seed=9)
    prog = programs.jacobi2d(sweeps)
    out = [_run(gfx, prog, u0, u0, sweeps, l, record=lambda u, w: u.view(-1)[n * 20:n * 20 + sweeps])
           for l in (gf.Launch.make(num_wg=1), gf.Launch.make(num_wg=1, wg_size=256, tile_y=16))]
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    assert out[0][4]["barriers"] == sweeps


def test_fused_2d_batch_in_groups_on_one_xcd_and_in_order(gfx, monkeypatch):
    """Uneven instances in one launch, groups kept to one XCD (group barrier
    without write-back) and laid out in order, against each one sweep by
    sweep; the last instance has fewer rows than a pass has sweeps."""
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    sides, sweeps = [400, 65, 128, 700, 33, 3], 16
    grids = [gi.batched_grid(i, n, 11) for i, n in enumerate(sides)]
    prog = programs.jacobi2d(sweeps)
    ref = [_run(gfx, prog, g, g, sweeps, gf.Launch.make(wg_size=256, tile_y=16)) for g in grids]
    for align in ("1", "0"):
        monkeypatch.setenv("GF_BATCH_ALIGN", align)
        with gf.Context(0) as ctx:
            us, ws = [dev(g) for g in grids], [dev(g) for g in grids]
            rs = [torch.zeros(sweeps, dtype=torch.float64, device="cuda") for _ in sides]
            insts = [gf.Instance.make({0: u, 1: w, 2: r}, scalars(), ip=(n,))
                     for u, w, r, n in zip(us, ws, rs, sides)]
            ctx.run(prog, insts, mode=gf.GF_EXEC_PERSISTENT)
            ctx.sync()
            for i in range(len(sides)):
                assert np.array_equal(host(us[i]), ref[i][0]), (align, i)
                assert np.array_equal(host(ws[i]), ref[i][1]), (align, i)
                assert np.all(np.abs(host(rs[i]) - ref[i][2]) <= 1e-12 * ref[i][2]), (align, i)


# sides: one and several 128-column items, odd and even, rows and planes that
# do not fill the last tile or segment; sweeps: every remainder of the pass
# lengths three and one
@pytest.mark.parametrize("n,sweeps", [(3, 4), (4, 5), (13, 7), (14, 6), (15, 8), (32, 4), (65, 9), (128, 5), (129, 10),
                                      (137, 7), (250, 5), (257, 6)])
def test_fused_3d_equals_sweep_by_sweep(gfx, n, sweeps):
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    print(f"fused 3d n={n} sweeps={sweeps}", flush=True)
    u0 = gi.um11(13, 32, np.arange(n ** 3, dtype=np.uint64)).reshape(n, n, n)
    prog = programs.jacobi3d(sweeps)
    given = gf.Launch.make(wg_size=256, tile_y=4, tile_z=32)
    for w0 in (u0, _outer_differs(u0, 14)):   # the second: outer layers differ, one sweep per pass
        a = _run(gfx, prog, u0, w0, sweeps, None)
        b = _run(gfx, prog, u0, w0, sweeps, given)
        for k in range(3):
            assert np.array_equal(a[k], b[k]), k
        assert a[3][0] == b[3][0]


@pytest.mark.parametrize("face", range(6))
def test_fused_3d_notices_one_differing_outer_value(gfx, face):
    """One value of one face differs between the two buffers (by its sign
    bit alone): the run has to take the sweep-by-sweep course."""
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    n, sweeps = 40, 7
    u0 = gi.um11(15, 32, np.arange(n ** 3, dtype=np.uint64)).reshape(n, n, n)
    w0 = u0.copy()
    at = [17, 23, 29]
    at[face // 2] = 0 if face % 2 == 0 else n - 1
    w0[tuple(at)] = -w0[tuple(at)]
    prog = programs.jacobi3d(sweeps)
    a = _run(gfx, prog, u0, w0, sweeps, None)
    b = _run(gfx, prog, u0, w0, sweeps, gf.Launch.make(wg_size=256, tile_y=4, tile_z=32))
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])


def test_fused_3d_grid_sizes_no_reduction_and_batch(gfx):
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    n, sweeps = 70, 8
    u0 = gi.grid3d(n, seed=16)
    given = gf.Launch.make(wg_size=256, tile_y=4, tile_z=32)
    prog = programs.jacobi3d(sweeps)
    b = _run(gfx, prog, u0, u0, sweeps, given)
    for nwg in (1, 3, 130, 255):
        a = _run(gfx, prog, u0, u0, sweeps, gf.Launch.make(num_wg=nwg, xcd_remap=nwg % 2))
        assert a[4]["num_wg"] == nwg
        assert all(np.array_equal(a[k], b[k]) for k in range(3))
    plain = programs.jacobi3d(sweeps, reduce=False)
    a = _run(gfx, plain, u0, u0, sweeps, None)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    sides = [33, 70, 8, 131]
    grids = [gi.grid3d(m, seed=17 + i) for i, m in enumerate(sides)]
    ref = [_run(gfx, prog, g, g, sweeps, given) for g in grids]
    us, ws = [dev(g) for g in grids], [dev(g) for g in grids]
    rs = [torch.zeros(sweeps, dtype=torch.float64, device="cuda") for _ in sides]
    gfx.run(prog, [gf.Instance.make({0: u, 1: w, 2: r}, scalars(), ip=(m,))
                   for u, w, r, m in zip(us, ws, rs, sides)], mode=gf.GF_EXEC_PERSISTENT)
    gfx.sync()
    for i in range(len(sides)):
        assert np.array_equal(host(us[i]), ref[i][0]) and np.array_equal(host(ws[i]), ref[i][1])
        assert np.array_equal(host(rs[i]), ref[i][2])


@pytest.mark.parametrize("n", [27, 28, 29, 31, 33, 34, 54, 55, 124, 125])
@pytest.mark.parametrize("num_wg", [0, 5])
def test_fused_3d_tile_edges(gfx, n, num_wg):
    """Sides where a workgroup's tile of 32 rows (26 of them written in a full
    pass, 30 in a pass of one sweep) just fits or spills over, and where the
    last tile is moved up to end at the last row; few workgroups give several
    tiles to each."""
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    u0 = gi.grid3d(n, seed=n)
    prog, w0 = programs.jacobi3d(8), u0.copy()
    a = _run(gfx, prog, u0, w0, 8, gf.Launch.make(num_wg=num_wg) if num_wg else None)
    b = _run(gfx, prog, u0, w0, 8, gf.Launch.make(tile_y=4, tile_z=8))
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)


def test_capacity_does_not_follow_the_grid_side(gfx):
    """A grid of workgroups past gf_persistent_capacity is refused whatever
    tile the library would choose for the grid's side, and so are more
    instances than that."""
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    prog, n = programs.jacobi3d(4), 8
    cap = gfx.capacity(prog)
    u = torch.zeros((n, n, n), dtype=torch.float64, device="cuda")
    def instance():
        return gf.Instance.make({0: u.clone(), 1: u.clone(), 2: torch.zeros(4, dtype=torch.float64, device="cuda")},
                                scalars(), ip=(n,))
    with pytest.raises(gf.GfError):
        gfx.run(prog, instance(), mode=gf.GF_EXEC_PERSISTENT, launch=gf.Launch.make(num_wg=cap + 1))
    with pytest.raises(gf.GfError):
        gfx.run(prog, [instance() for _ in range(cap + 1)], mode=gf.GF_EXEC_PERSISTENT)
    gfx.run(prog, instance(), mode=gf.GF_EXEC_PERSISTENT, launch=gf.Launch.make(num_wg=cap))
    gfx.sync()


def _passes(kind, sweeps):
    """Fused passes of a run: full ones, then three sweeps, the last alone."""
    full, n = (7 if kind == 2 else 3), 0
    while sweeps > 0:
        sweeps -= full if sweeps > full else (3 if sweeps > 3 else 1)
        n += 1
    return n


@pytest.mark.parametrize("n,num_wg", [(29, 0), (40, 3), (64, 0), (131, 0), (258, 100)])
def test_fused_3d_runs_the_passes_it_reports(gfx, n, num_wg):
    """A 3D run whose tile is left to the library takes the fused kernel
    (512 threads, one barrier per pass and one after the comparison of the
    outer layers), with few long segments and many short ones, and gives what
    a sweep at a time gives, also where the two buffers' outer layers differ."""
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    u0 = gi.um11(21, 32, np.arange(n ** 3, dtype=np.uint64)).reshape(n, n, n)
    given = gf.Launch.make(wg_size=256, tile_y=4, tile_z=32)
    own = gf.Launch.make(num_wg=num_wg) if num_wg else None
    for sweeps in (4, 9, 11):
        prog = programs.jacobi3d(sweeps)
        for w0 in (u0, _outer_differs(u0, 22)):
            a = _run(gfx, prog, u0, w0, sweeps, own)
            b = _run(gfx, prog, u0, w0, sweeps, given)
            assert all(np.array_equal(a[k], b[k]) for k in range(3))
            assert a[4]["wg_size"] == 512 and a[4]["barriers"] == _passes(3, sweeps) + 1
            assert b[4]["barriers"] == sweeps


def test_fused_batches_take_the_fused_kernels(gfx):
    """Batches of instances run fused too: 128 threads in 2D, 512 in 3D, and
    the barriers of the longest instance."""
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    sweeps = 16
    for kind, sides, grid, prog in ((2, [400, 65, 3], gi.grid2d, programs.jacobi2d(sweeps)),
                                    (3, [33, 70, 8], gi.grid3d, programs.jacobi3d(sweeps))):
        insts = []
        for n in sides:
            u = dev(grid(n, seed=n))
            insts.append(gf.Instance.make({0: u, 1: u.clone(), 2: torch.zeros(sweeps, dtype=torch.float64,
                                                                              device="cuda")}, scalars(), ip=(n,)))
        st = gfx.run(prog, insts, mode=gf.GF_EXEC_PERSISTENT)
        gfx.sync()
        assert st["wg_size"] == (128 if kind == 2 else 512)
        # the 2D grid of side 3 takes a sweep per pass
        assert st["barriers"] == (sweeps if kind == 2 else _passes(3, sweeps) + 1)


def test_fused_3d_batches_of_large_grids(gfx):
    """The scratch that a batch reserves for its partials is what its passes
    can write: two grids of 256 or one of 400 fit it many times over."""
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    sweeps = 7
    prog = programs.jacobi3d(sweeps)
    for sides in ((256, 256), (400, 40)):
        grids = [gi.grid3d(n, seed=60 + i) for i, n in enumerate(sides)]
        us, ws = [dev(g) for g in grids], [dev(g) for g in grids]
        rs = [torch.zeros(sweeps, dtype=torch.float64, device="cuda") for _ in sides]
        st = gfx.run(prog, [gf.Instance.make({0: u, 1: w, 2: r}, scalars(), ip=(n,))
                            for u, w, r, n in zip(us, ws, rs, sides)], mode=gf.GF_EXEC_PERSISTENT)
        gfx.sync()
        assert st["wg_size"] == 512 and st["barriers"] == _passes(3, sweeps) + 1
        for i, g in enumerate(grids):
            b = _run(gfx, prog, g, g, sweeps, gf.Launch.make(wg_size=256, tile_y=4, tile_z=32))
            assert np.array_equal(host(us[i]), b[0]) and np.array_equal(host(ws[i]), b[1])
            assert np.array_equal(host(rs[i]), b[2])
