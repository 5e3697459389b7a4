"""GPU parity of the coarse operator's build at the edges of its tiles: vector
counts around 16 and 32 (row tiles), aggregates whose site or face count is
not a multiple of 4, with extents of 1, larger than 256 sites and as large as
the lattice, on both sides of the 64 sites from which another kernel is used."""
import numpy as np
import pytest

import latgen
from gpu_common import TOL32, TOL64, lattice, problem, rel, say
from oracle import solvers
from test_gpu_coarse import to_dev_coarse, to_np_coarse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block,agg,N", [
    ((12, 4, 4, 4), (2, 4, 4, 4), (3, 1, 2, 1), 16),
    ((12, 4, 4, 4), (2, 4, 4, 4), (3, 2, 1, 1), 17),
    ((4, 4, 4, 8), (4, 4, 4, 4), (2, 2, 2, 2), 32),
    ((4, 4, 4, 4), (4, 4, 4, 4), (1, 1, 1, 1), 1),
    ((8, 8, 4, 8), (4, 4, 4, 4), (4, 8, 4, 4), 21),
    ((8, 4, 4, 4), (4, 4, 4, 4), (8, 4, 4, 4), 9),
    ((12, 12, 4, 4), (2, 2, 4, 4), (3, 3, 4, 2), 25),
    ((20, 4, 4, 4), (2, 4, 4, 4), (5, 4, 4, 1), 8),
    ((8, 4, 4, 4), (4, 4, 4, 4), (4, 4, 4, 1), 32),
    ((8, 4, 4, 4), (4, 4, 4, 4), (4, 4, 2, 2), 1),
    ((12, 12, 4, 4), (2, 2, 4, 4), (6, 3, 2, 4), 24),
    ((12, 4, 4, 4), (2, 4, 4, 4), (3, 4, 4, 1), 20),
])
def test_coarse_operator_tile_edges(dims, block, agg, N):
    from paper_1202_2462_amd.mgdd import F32, F64
    say("coarse operator tile edges", dims, agg, N)
    op = problem(dims, seed=11, m0=0.1)
    lat = lattice(op, block)
    tv = latgen.gaussian_fields(dims, N, 12)
    lat.build_P(agg, lat.pack(tv, F64))
    tl = solvers.TwoLevel(op, agg, tv, block, mr_iters=4)
    x = latgen.gaussian_vector(2 * lat.Vc * 2 * N, 13).reshape(2, lat.Vc, 2, N)
    want = np.stack([tl.coarse_apply(v) for v in x])
    for prec, tol in ((F64, TOL64), (F32, TOL32)):
        got = to_np_coarse(lat.coarse_apply(to_dev_coarse(lat, x, prec)))
        assert rel(got, want) < tol, (prec, rel(got, want))
    lat.close()
