"""GPU parity of the Wilson-clover apply with several right-hand sides on blocks
of 256 sites: counts that the threads' groups divide and counts that leave a
remainder, lattices on both sides of the size from which the threads hold more
than one, a direction of one block, links that are special unitary and not, in
every precision; each right-hand side equals its apply alone bit for bit. And
the solver's FP64 apply of FP32 and half fields, through a solve of several."""
import numpy as np
import pytest

import latgen
from gpu_common import TOL32, TOL64, lattice, problem, rel, say
from oracle import solvers
from test_gpu_fp16 import round16

pytestmark = pytest.mark.gpu

# 16, 64 and 128 blocks: 192 workgroups are reached by no count, from 5 and from 3 on
LATTICES = [((8, 8, 8, 8), True), ((16, 8, 16, 8), True), ((4, 32, 16, 16), True), ((16, 16, 16, 8), False)]


@pytest.mark.parametrize("dims,unitary", LATTICES)
def test_apply_right_hand_sides(dims, unitary):
    from paper_1202_2462_amd.mgdd import F16, F32, F64
    if unitary:
        op = problem(dims, seed=71, m0=0.1)
    else:
        op = solvers.Operator(dims, 1.01 * latgen.gauge_field(dims, 0.6, 71), 0.1, 1.2)
    lat = lattice(op, (4, 4, 4, 4))
    x = round16(latgen.gaussian_fields(dims, 13, 72))
    want = np.stack([op.apply(v) for v in x])
    # half storage: the result is rounded to 11 bits
    for prec, tol in ((F64, TOL64), (F32, TOL32), (F16, 2.0 ** -10)):
        b = lat.pack(x, prec)
        alone = [lat.dirac(b[i:i + 1].contiguous()) for i in range(13)]
        for nrhs in (1, 2, 3, 4, 5, 6, 7, 8, 13):
            say("apply", dims, "nrhs", nrhs, "prec", prec)
            out = lat.field(prec, nrhs + 1)
            out[nrhs] = 7.0   # the field after the last one is left alone
            lat.dirac(b[:nrhs].contiguous(), out[:nrhs])
            assert float((out[nrhs] - 7.0).abs().max()) == 0
            got = lat.unpack(out[:nrhs])
            for i in range(nrhs):
                assert bool((out[i] == alone[i][0]).all()), (prec, nrhs, i)
                assert rel(got[i], want[i]) < tol, (prec, nrhs, i, rel(got[i], want[i]))
    lat.close()


@pytest.mark.parametrize("half", [False, True])
def test_solve_right_hand_sides(half):
    from paper_1202_2462_amd.mgdd import F64, MIXED, MIXED_F16
    dims, agg, N = (16, 8, 16, 8), (4, 4, 4, 4), 8
    op = problem(dims, seed=73, m0=0.1, eps=0.5)
    lat = lattice(op, (4, 4, 4, 4))
    lat.build_P(agg, lat.pack(latgen.gaussian_fields(dims, N, 74), F64))
    b = latgen.gaussian_fields(dims, 6, 75)
    kw = dict(precision=MIXED_F16 if half else MIXED, restart=20, tol=1e-9, maxit=400)
    say("solve", dims, "half", half)
    z, stats = lat.solve(lat.pack(b, F64), **kw)
    got = lat.unpack(z)
    for i in range(6):
        assert stats[i].converged
        assert np.linalg.norm(b[i] - op.apply(got[i])) <= 1e-9 * np.linalg.norm(b[i])
    z1, _ = lat.solve(lat.pack(b[4:5], F64), **kw)
    assert rel(lat.unpack(z1)[0], got[4]) < 1e-12
    lat.close()


@pytest.mark.parametrize("dims,block,unitary", [
    ((4, 4, 4, 4), (2, 2, 2, 2), True),
    ((8, 4, 4, 8), (4, 4, 4, 4), True),
    ((4, 4, 8, 8), (2, 2, 4, 4), False),
    ((8, 8, 16, 16), (4, 4, 4, 4), True),
])
def test_few_sites(dims, block, unitary):
    """Up to 16384 sites of all right-hand sides the sites' hops are shared by
    four lanes: the same bits as from the kernel for more, and the oracle's."""
    from paper_1202_2462_amd.mgdd import F16, F32, F64, mgdd_set_kernel_options
    if unitary:
        op = problem(dims, seed=76, m0=0.1)
    else:
        op = solvers.Operator(dims, 1.01 * latgen.gauge_field(dims, 0.6, 76), 0.1, 1.2)
    lat = lattice(op, block)
    x = round16(latgen.gaussian_fields(dims, 3, 77))
    want = np.stack([op.apply(v) for v in x])
    for prec, tol in ((F64, TOL64), (F32, TOL32), (F16, 2.0 ** -10)):
        b = lat.pack(x, prec)
        for nrhs in (1, 2, 3):
            say("few sites", dims, "nrhs", nrhs, "prec", prec)
            seen = []
            for stage in (0, -1):
                mgdd_set_kernel_options(lat.ctx, dirac_stage=stage)
                out = lat.field(prec, nrhs + 1)
                out[nrhs] = 7.0
                lat.dirac(b[:nrhs].contiguous(), out[:nrhs])
                assert float((out[nrhs] - 7.0).abs().max()) == 0
                seen.append(out[:nrhs])
            assert bool((seen[0] == seen[1]).all()), (prec, nrhs)
            got = lat.unpack(seen[0])
            for i in range(nrhs):
                assert rel(got[i], want[i]) < tol, (prec, nrhs, i)
    lat.close()
