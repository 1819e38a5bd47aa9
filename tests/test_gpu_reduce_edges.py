"""gf_reduce and gf_reduce_noalloc at the edges of their work split: one
workgroup up to 8,192 elements and several above, whole trips of eight
16-byte loads per thread and ragged ends, inputs aligned to no more than one
element. Integers and maxima are exact; a sum of n doubles is held to
1e-12 of sum |a_i| around the oracle's compensated value."""
import numpy as np
import pytest

import gf_inputs as gi
from tests.gpu_helpers import host

pytestmark = pytest.mark.gpu

# one vector, one trip (4,096 doubles, 8,192 u32), the one-workgroup limit,
# two and three workgroups, the largest grid (1,024) and one element more
SIZES = [1, 2, 5, 4095, 4096, 4097, 8191, 8192, 8193, 12289, (1 << 22), (1 << 22) + 1, (1 << 23) + 4093]


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n", SIZES)
def test_reduce_edges(gfx, oracle_lib, n, offset):
    import torch
    import paper_2306_11686_amd as gf
    print(f"reduce edges n={n} offset={offset}", flush=True)
    h = gi.hash_u64(5, 31, np.arange(n, dtype=np.uint64))
    f64 = gi.um11(5, 32, np.arange(n, dtype=np.uint64))
    u32 = (h >> np.uint64(32)).astype(np.uint32)
    for dt, a in ((gf.GF_F64, f64), (gf.GF_U32, u32), (gf.GF_U64, h), (gf.GF_I64, h.view(np.int64))):
        bits = a.view(np.int32) if a.dtype.itemsize == 4 else a.view(np.int64)
        buf = torch.zeros(n + 8, dtype=torch.int32 if a.dtype.itemsize == 4 else torch.int64, device="cuda")
        x = buf[offset:offset + n]
        x.copy_(torch.from_numpy(bits))
        for op, name in ((gf.GF_OP_SUM, "sum"), (gf.GF_OP_MAX, "max")):
            got = []
            for call in (gfx.reduce, gfx.reduce_noalloc):
                out = torch.full((1,), -1, dtype=torch.int64, device="cuda")
                call(op, dt, x, n, out)
                got.append(host(out)[0])
            assert got[0] == got[1]
            if dt == gf.GF_F64:
                v = np.int64(got[0]).view(np.float64)
                if name == "max":
                    assert v == oracle_lib.reduce("max", a)
                else:
                    ref = oracle_lib.reduce("sum", a, compensated=True)
                    assert abs(v - ref) <= 1e-12 * float(np.sum(np.abs(a)))
            else:
                v = int(got[0]) if dt == gf.GF_I64 else int(np.uint64(np.int64(got[0])))
                assert v == oracle_lib.reduce(name, a)
