"""FP32 coarse GMRES with more steps than the coarse space has dimensions: from
the last dimension on a basis vector is what rounding leaves (its squared norm, a
difference of two sums, is noise of either sign), and the solution stays that of
the linear system, for one right-hand side and for several."""
import numpy as np
import pytest

import latgen
from gpu_common import lattice, problem, say
from test_gpu_coarse import to_dev_coarse, to_np_coarse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,N", [((4, 4, 4, 4), 1), ((4, 4, 4, 4), 3), ((4, 4, 4, 4), 6), ((8, 4, 4, 4), 2),
                                    ((8, 4, 4, 8), 1)])
def test_more_steps_than_dimensions(dims, N):
    from paper_1202_2462_amd.mgdd import F32, F64
    for seed in range(4):
        op = problem(dims, seed=41 + seed, m0=0.2)
        lat = lattice(op, (4, 4, 4, 4))
        lat.build_P((4, 4, 4, 4), lat.pack(latgen.gaussian_fields(dims, N, 42 + seed), F64))
        n = lat.Vc * 2 * N
        eye = np.eye(n, dtype=complex).reshape(n, lat.Vc, 2, N)
        D = to_np_coarse(lat.coarse_apply(to_dev_coarse(lat, eye, F64))).reshape(n, n).T
        b = to_np_coarse(to_dev_coarse(lat, latgen.gaussian_vector(3 * n, 43 + seed).reshape(3, lat.Vc, 2, N), F32))
        want = np.linalg.solve(D, b.reshape(3, n).T).T
        # D_c and the basis are rounded to FP32: an error of a few ulp in the residual
        tol = 8 * 2.0 ** -24 * np.linalg.cond(D)
        for m in sorted({n, n + 1, n + 2, 15}):
            for nrhs in (1, 3):
                got = to_np_coarse(lat.coarse_solve(to_dev_coarse(lat, b[:nrhs], F32), m)).reshape(nrhs, n)
                err = np.linalg.norm(got - want[:nrhs], axis=1) / np.linalg.norm(want[:nrhs], axis=1)
                say("dimension", n, "steps", m, "right-hand sides", nrhs, "error", err.max(), "of", tol)
                assert (err < tol).all()
        lat.close()
