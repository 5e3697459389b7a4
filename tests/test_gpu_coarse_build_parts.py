"""GPU parity of the coarse operator's build on both sides of the 512 aggregates
up to which an aggregate's self term is divided over up to four workgroups: the
site counts at which these are 4 and 3, and the whole list in one."""
import numpy as np
import pytest

import latgen
from gpu_common import TOL32, TOL64, lattice, problem, rel, say
from oracle import solvers
from test_gpu_coarse import to_dev_coarse, to_np_coarse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block,agg,N", [
    ((16, 16, 16, 8), (4, 4, 4, 4), (2, 2, 4, 4), 5),      # 512 aggregates of 64 sites, 4 parts
    ((12, 12, 4, 8), (2, 2, 4, 4), (3, 3, 4, 4), 18),      # of 144 sites, 3 parts
    ((16, 16, 16, 16), (4, 4, 4, 4), (2, 2, 4, 4), 5),     # 1024 aggregates, one part
])
def test_coarse_operator_parts(dims, block, agg, N):
    from paper_1202_2462_amd.mgdd import F32, F64
    say("coarse operator parts", dims, agg, N)
    op = problem(dims, seed=15, m0=0.1)
    lat = lattice(op, block)
    tv = latgen.gaussian_fields(dims, N, 16)
    lat.build_P(agg, lat.pack(tv, F64))
    tl = solvers.TwoLevel(op, agg, tv, block, mr_iters=4)
    x = latgen.gaussian_vector(lat.Vc * 2 * N, 17).reshape(1, lat.Vc, 2, N)
    want = tl.coarse_apply(x[0])
    for prec, tol in ((F64, TOL64), (F32, TOL32)):
        got = to_np_coarse(lat.coarse_apply(to_dev_coarse(lat, x, prec)))
        assert rel(got[0], want) < tol, (prec, rel(got[0], want))
    lat.close()
