"""GPU parity of restriction and prolongation with several right-hand sides:
every count the kernels hold per thread and one more, aggregates smaller than a
wave, not a multiple of one, and larger than a workgroup, in every precision."""
import numpy as np
import pytest

import latgen
from gpu_common import TOL32, TOL64, lattice, problem, rel, say
from oracle import solvers
from test_gpu_coarse import to_dev_coarse, to_np_coarse

pytestmark = pytest.mark.gpu

SHAPES = [
    ((12, 4, 4, 8), (2, 4, 4, 4), (3, 2, 4, 2), 5),
    ((12, 4, 8, 8), (2, 4, 4, 4), (6, 4, 4, 4), 11),
    ((16, 4, 4, 8), (4, 4, 4, 4), (8, 4, 4, 4), 6),
]


@pytest.mark.parametrize("dims,block,agg,N", SHAPES)
def test_transfer_right_hand_sides(dims, block, agg, N):
    from paper_1202_2462_amd.mgdd import F16, F32, F64
    op = problem(dims, seed=51, m0=0.1)
    lat = lattice(op, block)
    tv = latgen.gaussian_fields(dims, N, 52)
    lat.build_P(agg, lat.pack(tv, F64))
    tl = solvers.TwoLevel(op, agg, tv, block)
    f = latgen.gaussian_fields(dims, 13, 53)
    c = latgen.gaussian_vector(13 * lat.Vc * 2 * N, 54).reshape(13, lat.Vc, 2, N)
    want_r = np.stack([tl.restrict(v) for v in f])
    want_p = np.stack([tl.prolong(v) for v in c])
    for nrhs in (1, 2, 3, 4, 6, 7, 8, 9, 12, 13):
        # half storage: P, the fine field and the output are rounded to 11 bits
        for prec, tol in ((F64, TOL64), (F32, TOL32), (F16, 2.0 ** -9)):
            say("transfer", dims, agg, "nrhs", nrhs, "prec", prec)
            got = to_np_coarse(lat.restrict(lat.pack(f[:nrhs], prec)))
            out = lat.field(prec, nrhs + 1)
            out[nrhs] = 7.0   # the field after the last one is left alone
            lat.prolong(to_dev_coarse(lat, c[:nrhs], F64 if prec == F64 else F32), out[:nrhs])
            assert float((out[nrhs] - 7.0).abs().max()) == 0
            back = lat.unpack(out[:nrhs])
            for i in range(nrhs):
                assert rel(got[i], want_r[i]) < tol, (nrhs, prec, i)
                assert rel(back[i], want_p[i]) < tol, (nrhs, prec, i)
    lat.close()
