"""GPU parity of the FP32 coarse GMRES on the compact D_c at the edges of its
kernels: block sizes 2N around multiples of 4 and 16, one and several
right-hand sides (a full tile of 16 and one more), coarse extents of 1, 2 and
more, step counts at which the passes take another register count, and the
fixed scratch array with too little room for the vectors of these steps."""
import numpy as np
import pytest

import latgen
from gpu_common import lattice, problem, rel, say
from oracle import solvers
from test_gpu_coarse import to_dev_coarse, to_np_coarse

pytestmark = pytest.mark.gpu

# as the FP32 coarse GMRES elsewhere: an FP32 Krylov basis
TOL = 1e-4


@pytest.mark.parametrize("dims,block,agg,N,nrhs,iters", [
    ((8, 4, 4, 8), (4, 4, 4, 4), (2, 2, 2, 2), 1, 1, 1),
    ((8, 4, 4, 8), (4, 4, 4, 4), (2, 2, 2, 4), 7, 1, 5),
    ((8, 4, 4, 8), (4, 4, 4, 4), (4, 2, 4, 2), 9, 2, 4),
    ((8, 8, 4, 4), (4, 4, 4, 4), (2, 2, 4, 4), 16, 16, 8),
    ((8, 8, 4, 4), (4, 4, 4, 4), (2, 4, 4, 2), 17, 17, 9),
    ((8, 8, 4, 4), (4, 4, 4, 4), (2, 4, 4, 2), 25, 3, 15),
    ((8, 8, 8, 8), (4, 4, 4, 4), (2, 4, 2, 4), 32, 1, 15),
    ((8, 8, 8, 8), (4, 4, 4, 4), (1, 2, 2, 1), 3, 1, 12),
])
def test_compact_coarse_steps(dims, block, agg, N, nrhs, iters):
    from paper_1202_2462_amd.mgdd import F32, F64, mgdd_coarse_solve_noalloc
    say("compact coarse steps", dims, agg, N, nrhs, iters)
    op = problem(dims, seed=41, m0=0.2)
    lat = lattice(op, block)
    tv = latgen.gaussian_fields(dims, N, 42)
    lat.build_P(agg, lat.pack(tv, F64))
    tl = solvers.TwoLevel(op, agg, tv, block)
    b = latgen.gaussian_vector(nrhs * lat.Vc * 2 * N, 43).reshape(nrhs, lat.Vc, 2, N)
    if nrhs > 2:
        b[1] = 0   # a zero right-hand side beside others
    dev = to_dev_coarse(lat, b, F32)
    got = to_np_coarse(lat.coarse_solve(dev, iters))
    x = lat.torch.full_like(dev, 7.0)
    mgdd_coarse_solve_noalloc(lat.ctx, F32, nrhs, iters, dev, x)
    for i in range(nrhs):
        want = solvers.gmres_fixed(tl.coarse_apply, b[i], iters) if np.any(b[i]) else np.zeros_like(b[i])
        for r in (got[i], to_np_coarse(x)[i]):
            assert np.linalg.norm(r - want) <= TOL * np.linalg.norm(want), (i, np.linalg.norm(r - want))
    # NaN is reported, whichever right-hand side holds it
    from paper_1202_2462_amd.mgdd import ENAN, MgddError
    dev[-1, 0, 0, 0, 1] = float("nan")
    with pytest.raises(MgddError) as e:
        lat.coarse_solve(dev, iters)
    assert e.value.code == ENAN
    lat.close()


def test_scratch_array_without_room_for_the_compact_steps():
    """4096 coarse sites, N = 8, 12 steps: the solve needs 8.4 MiB a right-hand
    side at least and 9.6 MiB with the vectors of the compact steps, so that 7
    right-hand sides run in the 64 MiB without these and 6 with them."""
    from paper_1202_2462_amd.mgdd import F32, F64, mgdd_coarse_solve_noalloc
    dims, block, agg, N, m = (16, 16, 16, 16), (4, 4, 4, 4), (2, 2, 2, 2), 8, 12
    op = problem(dims, seed=44, m0=0.2)
    lat = lattice(op, block)
    lat.build_P(agg, lat.pack(latgen.gaussian_fields(dims, N, 45), F64))
    for nrhs in (4, 5, 6, 7):
        say("noalloc with", nrhs, "right-hand sides")
        g = lat.torch.Generator(device="cuda").manual_seed(nrhs)
        b = lat.torch.randn((nrhs, lat.Vc, 2, N, 2), dtype=lat.torch.float32, device="cuda", generator=g)
        want = lat.coarse_solve(b, m)
        x = lat.torch.zeros_like(b)
        mgdd_coarse_solve_noalloc(lat.ctx, F32, nrhs, m, b, x)
        assert float((x - want).norm() / want.norm()) < TOL
    lat.close()
