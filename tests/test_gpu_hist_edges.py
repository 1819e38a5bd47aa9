"""GPU parity of the histogram where its counters can go wrong: every number
of copies of a bin (eight up to 8,192 bins, one from 65,536), skewed and constant
keys that fill the 16-bit counters between and after scans, key counts around
a chunk, and more workgroups than chunks. Counts are whole numbers, so every
result equals the oracle."""
import numpy as np
import pytest

from tests.gpu_helpers import dev, host, scalars

pytestmark = pytest.mark.gpu


def _keys(kind, n):
    rng = np.random.default_rng(n)
    if kind == "constant":
        return np.full(n, 0x7FF3A5C1, dtype=np.uint32)
    if kind == "two":       # both halves of one counter word
        return (0xA5A5A5A4 + rng.integers(0, 2, n)).astype(np.uint32)
    k = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    return np.where(rng.random(n) < 0.4, np.uint32(0xFFFFFFFF), k) if kind == "skewed" else k


@pytest.mark.parametrize("mode", ["persistent", "per_region"])
@pytest.mark.parametrize("kind", ["uniform", "skewed", "constant", "two"])
@pytest.mark.parametrize("nbins", [1, 2, 8, 1024, 2048, 32768, 65536, 1 << 18])
@pytest.mark.parametrize("n,num_wg,items", [(4095, 0, 0), (16385, 64, 4), ((1 << 21) + 5, 4, 4), ((1 << 19) + 1, 4, 8)])
def test_hist_counters(gfx, oracle_lib, mode, kind, nbins, n, num_wg, items):
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    keys = _keys(kind, n)
    init = (np.arange(nbins) % 7).astype(np.uint32)
    bins = dev(init.copy())
    inst = gf.Instance.make({0: dev(keys), 1: bins}, scalars(), ip=(n,))
    gfx.run(programs.histogram(nbins), inst,
            mode=gf.GF_EXEC_PERSISTENT if mode == "persistent" else gf.GF_EXEC_PER_REGION,
            launch=gf.Launch.make(num_wg=num_wg, items=items) if num_wg else None)
    gfx.sync()
    assert np.array_equal(host(bins), oracle_lib.hist_u32(keys, nbins, bins=init.copy()))


# rows of a part: 1, 3, 4, 31, 32 and 64 (where the merge's slices change); four
# parts, 69 chunks of 1,024 keys each
@pytest.mark.parametrize("mode", ["per_region", "persistent"])
@pytest.mark.parametrize("part_rows", [1, 3, 4, 31, 32, 64])
def test_merge_of_few_and_many_rows_per_part(gfx, oracle_lib, part_rows, mode):
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    n, nbins = 70001, 1 << 18
    keys = _keys("skewed", n)
    bins = dev(np.zeros(nbins, dtype=np.uint32))
    inst = gf.Instance.make({0: dev(keys), 1: bins}, scalars(), ip=(n,))
    gfx.run(programs.histogram(nbins), inst,
            mode=gf.GF_EXEC_PER_REGION if mode == "per_region" else gf.GF_EXEC_PERSISTENT,
            launch=gf.Launch.make(wg_size=256, items=1, num_wg=4 * part_rows))
    gfx.sync()
    assert np.array_equal(host(bins), oracle_lib.hist_u32(keys, nbins))


@pytest.mark.parametrize("mode", ["per_region", "persistent"])
@pytest.mark.parametrize("nbins", [2, 256, 16384, 1 << 17, 1 << 20])
@pytest.mark.parametrize("n", [3, 5000, 300001, 2500000])
def test_default_chunks(gfx, oracle_lib, n, nbins, mode):
    import paper_2306_11686_amd as gf
    from paper_2306_11686_amd import programs
    keys = _keys("uniform", n)
    bins = dev(np.zeros(nbins, dtype=np.uint32))
    inst = gf.Instance.make({0: dev(keys), 1: bins}, scalars(), ip=(n,))
    gfx.run(programs.histogram(nbins), inst,
            mode=gf.GF_EXEC_PER_REGION if mode == "per_region" else gf.GF_EXEC_PERSISTENT)
    gfx.sync()
    assert np.array_equal(host(bins), oracle_lib.hist_u32(keys, nbins))
