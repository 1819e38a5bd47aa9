"""Tiles and launch rules that follow the grid's side, against the oracle."""
import numpy as np
import pytest

import gf_inputs as gi
from tests.gpu_helpers import run_jacobi3d

pytestmark = pytest.mark.gpu


# items of one column per thread: 8; 3 * 127 * 2 = 762 and 3 * 64 * 2 = 384 (limit
# 512, per region in small workgroups 1,024); 189 * 3 = 567 and 189 * 2 = 378;
# 96 * 3 = 288 and 96 * 2 = 192 (limit 256); 3 * 80 * 3 = 720; 2 * 38 * 3 = 228
# and 2 * 38 * 5 = 380; none from side 300 on
@pytest.mark.parametrize("n,wg,ty,tz", [(65, 256, 8, 64), (129, 64, 1, 64), (129, 64, 2, 64), (191, 256, 1, 64),
                                        (191, 256, 1, 95), (193, 256, 2, 95), (193, 256, 2, 96), (299, 256, 8, 100),
                                        (161, 64, 2, 64), (299, 256, 8, 64), (301, 256, 16, 64), (3, 64, 1, 1), (5, 64, 16, 2)])
def test_odd_sides_with_one_and_two_columns_per_thread(gfx, oracle_lib, n, wg, ty, tz):
    import paper_2306_11686_amd as gf
    print(f"odd side n={n} wg={wg} tile {ty}x{tz}", flush=True)
    u0 = gi.grid3d(n, seed=31)
    g_ref, r_ref = oracle_lib.jacobi3d(u0, 2)
    for mode in (gf.GF_EXEC_PERSISTENT, gf.GF_EXEC_PER_REGION):
        g, r, _ = run_jacobi3d(gfx, u0, 2, mode, launch=gf.Launch.make(wg_size=wg, tile_y=ty, tile_z=tz))
        assert np.array_equal(g, g_ref) and np.array_equal(r, r_ref)


@pytest.mark.parametrize("mode", ["persistent", "per_region"])
def test_rows_per_tile_of_3d_instances_whatever_the_side(gfx, oracle_lib, mode):
    """Instances that give their rows per tile and leave the rest of the
    launch out run with the fixed default tile: eight rows are taken, others
    refused, also on small grids, whose own default is another."""
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    from tests.gpu_helpers import dev, host, scalars
    m = gf.GF_EXEC_PERSISTENT if mode == "persistent" else gf.GF_EXEC_PER_REGION
    sides, sweeps = [33, 20], 4
    grids = [gi.grid3d(n, seed=40 + n) for n in sides]
    prog = programs.jacobi3d(sweeps)

    def instances():
        us = [dev(g) for g in grids]
        rs = [torch.zeros(sweeps, dtype=torch.float64, device="cuda") for _ in sides]
        return us, [gf.Instance.make({0: u, 1: u.clone(), 2: r}, scalars(), ip=(n,))
                    for u, r, n in zip(us, rs, sides)]

    for rows in ((8, 8), (8, 0), (0, 0)):
        us, insts = instances()
        gfx.run_batched(prog, insts, [gf.Launch.make(tile_y=r) for r in rows], mode=m)
        gfx.sync()
        for u, g in zip(us, grids):
            assert np.array_equal(host(u), oracle_lib.jacobi3d(g, sweeps)[0]), rows
    for rows in ((2, 2), (4, 8), (0, 2)):
        with pytest.raises(gf.GfError):
            gfx.run_batched(prog, instances()[1], [gf.Launch.make(tile_y=r) for r in rows], mode=m)


@pytest.mark.parametrize("mode", ["persistent", "per_region"])
def test_prefetch_names_the_fixed_tile(gfx, oracle_lib, mode):
    """prefetch = 2 alone: a 3D launch keeps the fixed default tile, and a 2D
    one, whose fixed tile has 16 rows, is refused at every side."""
    import paper_2306_11686_amd as gf
    from tests.gpu_helpers import run_jacobi2d
    m = gf.GF_EXEC_PERSISTENT if mode == "persistent" else gf.GF_EXEC_PER_REGION
    l = gf.Launch.make(prefetch=2)
    for n in (33, 64):
        u0 = gi.grid3d(n, seed=50 + n)
        g, r, st = run_jacobi3d(gfx, u0, 5, m, launch=l)
        g_ref, r_ref = oracle_lib.jacobi3d(u0, 5)
        assert np.array_equal(g, g_ref) and np.array_equal(r, r_ref)
        assert st["wg_size"] == 256
    for n in (64, 512, 2048):
        with pytest.raises(gf.GfError):
            run_jacobi2d(gfx, gi.grid2d(n, seed=3), 2, m, launch=l)


def test_reduction_capacity_does_not_follow_the_grid_side():
    """The largest 2D grids have more reduction tiles of the fixed 16 rows
    than the scratch holds, and are refused also where the default tile has
    32 rows; a side below the limit is accepted."""
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    from tests.gpu_helpers import scalars
    n = 92700                                   # ceil(n / 512) * ceil((n - 2) / 16) = 182 * 5794 > 2^20
    if torch.cuda.mem_get_info()[0] < (20 << 30) + 16 * n * n:
        pytest.skip("two grids of this side do not fit the card")
    u = torch.empty(n * n, dtype=torch.float64, device="cuda")
    w = torch.empty(n * n, dtype=torch.float64, device="cuda")
    r = torch.zeros(1, dtype=torch.float64, device="cuda")
    inst = gf.Instance.make({0: u, 1: w, 2: r}, scalars(), ip=(n,))
    ctx = gf.Context(0)                         # without a predictor
    for mode in (gf.GF_EXEC_PER_REGION, gf.GF_EXEC_PERSISTENT):
        with pytest.raises(gf.GfError):
            ctx.run(programs.jacobi2d(1), inst, mode=mode)
    ok = gf.Instance.make({0: u, 1: w, 2: r}, scalars(), ip=(92000,))   # 180 * 5750 < 2^20
    ctx.run(programs.jacobi2d(1), ok, mode=gf.GF_EXEC_PER_REGION)
    ctx.sync()
    ctx.close()
    del u, w, inst, ok
    torch.cuda.empty_cache()


# the sides at which a rule changes, in both orders of a list of instances
@pytest.mark.parametrize("mode", ["persistent", "per_region", "per_region_graph"])
@pytest.mark.parametrize("sides", [(33, 129, 20), (20, 255, 64), (257, 3, 96)])
def test_default_tiles_of_3d_instances(gfx, oracle_lib, mode, sides):
    """Each instance of a list against the oracle, in a second run of the
    same list too (a replay in graph mode); with a given number of workgroups
    the tile is another one. Three sweeps: no fused passes."""
    import torch
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    from tests.gpu_helpers import dev, host, scalars
    m = {"persistent": gf.GF_EXEC_PERSISTENT, "per_region": gf.GF_EXEC_PER_REGION,
         "per_region_graph": gf.GF_EXEC_PER_REGION_GRAPH}[mode]
    sweeps, grids = 3, [gi.grid3d(n, seed=70 + n) for n in sides]
    us, ws = [dev(g) for g in grids], [dev(g) for g in grids]
    rs = [torch.zeros(sweeps, dtype=torch.float64, device="cuda") for _ in sides]
    insts = [gf.Instance.make({0: u, 1: w, 2: r}, scalars(), ip=(n,)) for u, w, r, n in zip(us, ws, rs, sides)]
    refs = [oracle_lib.jacobi3d(g, sweeps) for g in grids]
    for launch in (None, None, gf.Launch.make(num_wg=16), gf.Launch.make(num_wg=100)):
        for u, w, g in zip(us, ws, grids):
            u.copy_(dev(g))
            w.copy_(u)
        gfx.run(programs.jacobi3d(sweeps), insts, mode=m, launch=launch)
        gfx.sync()
        for i, (g_ref, r_ref) in enumerate(refs):
            assert np.array_equal(host(ws[i]), g_ref) and np.array_equal(host(rs[i]), r_ref), (i, launch)


@pytest.mark.parametrize("mode", ["persistent", "per_region"])
@pytest.mark.parametrize("n", [255, 256, 511, 513, 1025])
@pytest.mark.parametrize("num_wg", [0, 7, 200])
def test_default_tiles_2d(gfx, oracle_lib, n, num_wg, mode):
    import paper_2306_11686_amd as gf
    from tests.gpu_helpers import run_jacobi2d
    m = gf.GF_EXEC_PERSISTENT if mode == "persistent" else gf.GF_EXEC_PER_REGION
    u0 = gi.grid2d(n, seed=80)
    g, r, _ = run_jacobi2d(gfx, u0, 3, m, launch=gf.Launch.make(num_wg=num_wg) if num_wg else None)
    g_ref, _, r_comp, _ = oracle_lib.jacobi2d(u0, 3)
    assert np.array_equal(g, g_ref) and np.all(np.abs(r - r_comp) <= 1e-12 * r_comp)


def test_instances_of_a_per_region_run_follow_their_own_side():
    """A small grid beside a large one runs the launch it gets alone: the
    workgroups of the largest launch are those of its own tile."""
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    import torch
    from tests.gpu_helpers import scalars

    def inst(n):
        u = torch.zeros((n, n, n), dtype=torch.float64, device="cuda")
        return gf.Instance.make({0: u, 1: u.clone(), 2: scalars()}, scalars(), ip=(n,))

    a, b = inst(64), inst(300)
    prog = programs.jacobi3d(1)
    with gf.Context(0) as ctx:                  # without a predictor
        for mode in (gf.GF_EXEC_PER_REGION, gf.GF_EXEC_PER_REGION_GRAPH):
            alone = [ctx.run(prog, i, mode=mode)["num_wg"] for i in (a, b)]
            assert ctx.run(prog, [a, b], mode=mode)["num_wg"] == max(alone)
            assert ctx.run(prog, [a, a], mode=mode)["num_wg"] == alone[0]
        ctx.sync()


# rows per segment in launches per sweep, and the workgroups (512 columns each) that they give
@pytest.mark.parametrize("n,rows,columns", [(1599, 8, 4), (1600, 16, 4), (4500, 32, 9), (4608, 16, 9), (5631, 16, 11),
                                            (5700, 32, 12)])
def test_default_rows_of_2d_launches_per_sweep(gfx, oracle_lib, n, rows, columns):
    import paper_2306_11686_amd as gf
    from tests.gpu_helpers import run_jacobi2d
    u0 = gi.grid2d(n, seed=81)
    g, r, st = run_jacobi2d(gfx, u0, 2, gf.GF_EXEC_PER_REGION, launch=gf.Launch.make())
    assert st["num_wg"] == columns * -(-(n - 2) // rows)
    g_ref, _, r_comp, _ = oracle_lib.jacobi2d(u0, 2)
    assert np.array_equal(g, g_ref) and np.all(np.abs(r - r_comp) <= 1e-12 * r_comp)
