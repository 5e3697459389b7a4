"""GPU parity of the prolongation on a lattice of 131072 sites, from which on one
field in FP32 or FP64 and two in FP64 take the kernel with a thread per site, and
of 32768, where groups of right-hand sides of every size share a thread; a field
has the same bits whichever kernel it goes through."""
import numpy as np
import pytest

import latgen
from gpu_common import TOL32, TOL64, rel, say
from oracle import solvers
from test_gpu_coarse import to_dev_coarse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,agg", [((16, 16, 16, 32), (4, 2, 8, 4)), ((16, 16, 8, 16), (4, 4, 4, 4))])
def test_prolong(dims, agg):
    from paper_1202_2462_amd.mgdd import F16, F32, F64, Lattice
    N, small = 5, (4, 4, 4, 4)
    U = latgen.gauge_field(small, 0.5, 81).reshape(*small, 4, 3, 3)
    U = np.tile(U, tuple(d // 4 for d in dims[::-1]) + (1, 1, 1)).reshape(-1, 4, 3, 3)
    lat = Lattice(dims, (4, 4, 4, 4))
    lat.set_gauge(U, 0.1, 1.0)
    tv = latgen.gaussian_fields(dims, N, 82)
    lat.build_P(agg, lat.pack(tv, F64))
    tl = solvers.TwoLevel(solvers.Operator(dims, U, 0.1, 1.0), agg, tv, (4, 4, 4, 4))
    c = latgen.gaussian_vector(13 * lat.Vc * 2 * N, 83).reshape(13, lat.Vc, 2, N)
    want = [tl.prolong(v) for v in c[:3]]
    # half storage: P and the output are rounded to 11 bits
    for prec, tol in ((F64, TOL64), (F32, TOL32), (F16, 2.0 ** -9)):
        dev = to_dev_coarse(lat, c, F64 if prec == F64 else F32)
        alone = [lat.prolong(dev[i:i + 1].contiguous(), lat.field(prec, 1))[0] for i in range(13)]
        for i in range(3):
            assert rel(lat.unpack(alone[i][None])[0], want[i]) < tol, (prec, i)
        for nrhs in (2, 3, 4, 5, 7, 12, 13):
            say("prolong", dims, "prec", prec, "right-hand sides", nrhs)
            got = lat.prolong(dev[:nrhs].contiguous(), lat.field(prec, nrhs))
            for i in range(nrhs):
                assert bool((got[i] == alone[i]).all()), (prec, nrhs, i)
    lat.close()
