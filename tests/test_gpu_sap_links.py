"""GPU parity of the FP64 Schwarz sweep for links that are special unitary to
1e-12 only: the sweep takes them as they are, to the accuracy it has for others,
and does not rebuild their third row."""
import numpy as np
import pytest

import latgen
from gpu_common import rel, say
from oracle import solvers

pytestmark = pytest.mark.gpu

# 2 colours of 4 operator applications, sums of about 100 products each: the
# rounding of 800 operations in a row adds up to 800^(1/2) 2^-53 = 3e-15 if it is
# random. A third row off by 8e-13 changes the result by more than 1e-13.
TOL = 1e-14


@pytest.mark.parametrize("off", [0.0, 8e-13])
@pytest.mark.parametrize("dims,block", [((8, 8, 8, 8), (4, 4, 4, 4)), ((8, 8, 4, 8), (4, 4, 4, 2)),
                                        ((8, 4, 8, 8), (2, 2, 4, 4))])
def test_sap_sweep(dims, block, off):
    from paper_1202_2462_amd.mgdd import F64, KERNEL_SAP, Lattice, mgdd_timing_enable, mgdd_timing_read
    say("FP64 sweep", dims, block, "third rows off by", off)
    U = latgen.gauge_field(dims, 0.5, 91).copy()
    rng = np.random.default_rng(92)
    row = U.reshape(-1, 3, 3)[:, 2]
    row += off * (rng.uniform(-1, 1, row.shape) + 1j * rng.uniform(-1, 1, row.shape))
    op = solvers.Operator(dims, U, 0.1, 1.0)
    lat = Lattice(dims, block)
    lat.set_gauge(U, 0.1, 1.0)
    b, z0 = latgen.gaussian_fields(dims, 2, 93), latgen.gaussian_fields(dims, 2, 94)
    for shift in (0.0, 0.03):
        z = lat.pack(z0, F64)
        lat.sap(lat.pack(b, F64), z, 1, 4, shift)
        got = lat.unpack(z)
        for i in range(2):
            e = rel(got[i], op.sap(block, b[i], z0[i], 1, 4, shift))
            say("  shift", shift, "field", i, "error", e)
            assert e < TOL
    # the bytes charged for the links and the clover term tell the kernels apart
    mgdd_timing_enable(lat.ctx, True)
    lat.sap(lat.pack(b[:1], F64), z[:1], 1, 4)
    ms, sites, n, nbytes = mgdd_timing_read(lat.ctx, KERNEL_SAP, F64)
    assert nbytes / sites == 576 + (1152 if off else 960)
    lat.close()
