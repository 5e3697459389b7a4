"""GPU parity of the Schwarz sweep's kernels for special unitary links: the
one-lane-per-site kernel, which lattices of 262144 sites or more use, at every
block volume, with and without a shift, blocks that span a direction, both time
boundaries, in FP32 and half storage; the same lattice size in FP64; a
right-hand side alone and among others; and the sizes on both sides of the rule."""
import numpy as np
import pytest

import latgen
from gpu_common import TOL32, TOL64, rel, say
from oracle import solvers
from test_gpu_fp16 import round16

pytestmark = pytest.mark.gpu

# the last is smaller than the one-lane kernel's lattices
SHAPES = [
    ((16, 16, 32, 32), (4, 4, 4, 4), True),
    ((32, 16, 16, 32), (4, 4, 4, 2), False),
    ((64, 32, 32, 4), (2, 2, 4, 4), True),
    ((4, 32, 64, 32), (4, 4, 4, 4), True),
    ((16, 16, 24, 40), (4, 4, 4, 4), True),
]


@pytest.mark.parametrize("dims,block,anti", SHAPES)
def test_sap_sweep(dims, block, anti):
    from paper_1202_2462_amd.mgdd import F16, F32, F64, Lattice
    U = latgen.gauge_field(dims, 0.5, 61)
    Uo = U
    if not anti:   # the oracle's boundary is antiperiodic: negate the links across it
        Uo = U.reshape(dims[3], -1, 4, 3, 3).copy()
        Uo[-1, :, 3] *= -1.0
        Uo = Uo.reshape(-1, 4, 3, 3)
    op = solvers.Operator(dims, Uo, 0.1, 1.0)
    lat = Lattice(dims, block, t_antiperiodic=anti)
    lat.set_gauge(U, 0.1, 1.0)
    b = round16(latgen.gaussian_fields(dims, 2, 62))
    z0 = round16(0.3 * latgen.gaussian_fields(dims, 2, 63))
    for shift in (0.0, 0.03):
        want = np.stack([op.sap(block, b[i], z0[i], 1, 3, shift) for i in range(2)])
        # half storage: each colour step's z is rounded to 11 bits
        for prec, tol in ((F64, TOL64), (F32, TOL32), (F16, 2.0 ** -9)):
            say("sweep", dims, block, "shift", shift, "prec", prec)
            pb, z, z1 = lat.pack(b, prec), lat.pack(z0, prec), lat.pack(z0[1:], prec)
            lat.sap(pb, z, 1, 3, shift)
            got = lat.unpack(z)
            for i in range(2):
                assert rel(got[i], want[i]) < tol, (prec, shift, i, rel(got[i], want[i]))
            lat.sap(lat.pack(b[1:], prec), z1, 1, 3, shift)
            assert bool((z1[0] == z[1]).all()), (prec, shift)
    lat.close()
