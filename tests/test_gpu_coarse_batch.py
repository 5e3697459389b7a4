"""The FP32 coarse GMRES gives a right-hand side the same bits alone, among
others and, in the fixed scratch array, among more than fit it at once: on
thousands of coarse sites, where the smallest difference of a coefficient shows
in some rounded component."""
import numpy as np
import pytest

import latgen
from gpu_common import say

pytestmark = pytest.mark.gpu


def tiled_lattice(small, reps, block, agg, N, seed):
    """a lattice of `reps` copies of a small gauge field in every direction, P from random fields"""
    from paper_1202_2462_amd.mgdd import F64, Lattice
    U = latgen.gauge_field(small, 0.5, seed).reshape(*small[::-1], 4, 3, 3)
    lat = Lattice([r * d for r, d in zip(reps, small)], block)
    lat.set_gauge(np.tile(U, tuple(reps[::-1]) + (1, 1, 1)).reshape(-1, 4, 3, 3), 0.1, 1.0)
    tv = lat.field(F64, N)
    tv.copy_(lat.torch.randn(tv.shape, dtype=tv.dtype, device="cuda", generator=rng(lat, seed)))
    lat.build_P(agg, tv)
    return lat


def rng(lat, seed):
    return lat.torch.Generator(device="cuda").manual_seed(seed)


def coarse_rhs(lat, n, seed):
    from paper_1202_2462_amd.mgdd import F32
    b = lat.coarse_field(F32, n)
    return b.copy_(lat.torch.randn(b.shape, dtype=b.dtype, device="cuda", generator=rng(lat, seed)))


@pytest.mark.parametrize("small,reps,agg,N,iters", [
    ((4, 4, 4, 8), (2, 2, 2, 2), (4, 4, 4, 4), 20, 12),        # 32 coarse sites
    ((4, 8, 8, 8), (4, 2, 2, 4), (2, 2, 4, 4), 17, 15),        # 2048
    ((6, 6, 6, 12), (4, 4, 4, 4), (3, 4, 4, 4), 28, 12),       # 3456
    ((4, 8, 8, 8), (4, 2, 2, 4), (2, 2, 4, 4), 8, 6),
    ((4, 8, 8, 8), (4, 2, 2, 4), (2, 2, 4, 4), 31, 6),
])
def test_alone_and_among_others(small, reps, agg, N, iters):
    lat = tiled_lattice(small, reps, (4, 4, 4, 4), agg, N, 71)
    b = coarse_rhs(lat, 17, 72)
    alone = lat.torch.cat([lat.coarse_solve(b[i:i + 1].contiguous(), iters) for i in range(17)])
    for nrhs in (2, 3, 4, 7, 12, 16, 17):
        say("coarse GMRES", agg, N, "right-hand sides", nrhs)
        got = lat.coarse_solve(b[:nrhs].contiguous(), iters)
        assert bool((got == alone[:nrhs]).all()), (nrhs, int((got != alone[:nrhs]).sum()))
    lat.close()


def test_in_the_scratch_array():
    from paper_1202_2462_amd.mgdd import F32, mgdd_coarse_solve_noalloc
    lat = tiled_lattice((8, 8, 8, 8), (2, 2, 2, 2), (4, 4, 4, 4), (2, 2, 2, 2), 8, 73)   # 4096 coarse sites
    b = coarse_rhs(lat, 7, 74)
    alone = lat.torch.cat([lat.coarse_solve(b[i:i + 1].contiguous(), 12) for i in range(7)])
    for nrhs in (1, 5, 6, 7):   # the array has room for the 7 only without the vectors t of 64 bytes an entry
        say("scratch array", nrhs)
        x = lat.torch.full_like(b[:nrhs], 7.0)
        mgdd_coarse_solve_noalloc(lat.ctx, F32, nrhs, 12, b[:nrhs].contiguous(), x)
        assert bool((x == alone[:nrhs]).all()), nrhs
    lat.close()
