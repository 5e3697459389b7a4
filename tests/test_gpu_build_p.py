"""GPU parity of P where its columns are taken in panels of four: vector counts
around multiples of the panel, aggregates that fill a wave partly, and rank
deficiency within a panel and across panels."""
import numpy as np
import pytest

import latgen
from gpu_common import TOL64, lattice, problem, rel, say
from oracle import solvers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block,agg,N", [
    ((8, 4, 4, 4), (4, 4, 4, 4), (4, 4, 4, 4), 1),
    ((12, 4, 4, 4), (2, 4, 4, 4), (3, 2, 2, 2), 5),
    ((12, 4, 4, 4), (2, 4, 4, 4), (3, 4, 2, 4), 7),
    ((4, 4, 4, 8), (4, 4, 4, 4), (4, 4, 2, 4), 31),
    ((8, 4, 4, 8), (4, 4, 4, 4), (8, 4, 4, 4), 6),
])
def test_p_columns(dims, block, agg, N):
    from paper_1202_2462_amd.mgdd import F64
    say("P by panels", dims, agg, N)
    op = problem(dims, seed=21, m0=0.1)
    lat = lattice(op, block)
    tv = latgen.gaussian_fields(dims, N, 22)
    lat.build_P(agg, lat.pack(tv, F64))
    tl = solvers.TwoLevel(op, agg, tv, block, mr_iters=4)
    c = latgen.gaussian_vector(lat.Vc * 2 * N, 23).reshape(1, lat.Vc, 2, N)
    import torch
    dev = torch.tensor(np.stack([c.real, c.imag], -1), dtype=torch.float64, device="cuda")
    got = lat.unpack(lat.prolong(dev))
    assert rel(got, tl.prolong(c[0])[None]) < TOL64
    back = lat.unpack(lat.prolong(lat.restrict(lat.pack(tv, F64))))
    assert rel(back, tv) < TOL64
    lat.close()


@pytest.mark.parametrize("copy", [1, 3, 4, 5])
def test_rank_deficiency_within_and_across_panels(copy):
    from paper_1202_2462_amd.mgdd import ERANK, F64, MgddError
    dims, block, agg = (8, 4, 4, 4), (4, 4, 4, 4), (4, 4, 4, 4)
    say("rank deficiency of column", copy)
    lat = lattice(problem(dims, seed=21, m0=0.1), block)
    tv = latgen.gaussian_fields(dims, 6, 24)
    tv[copy] = 0.5j * tv[0]
    with pytest.raises(MgddError) as e:
        lat.build_P(agg, lat.pack(tv, F64))
    assert e.value.code == ERANK
    lat.close()


@pytest.mark.parametrize("agg", [(3, 4, 4, 4), (12, 4, 4, 8)])
def test_test_vectors_off_the_16_byte_grid(agg):
    """Vectors that kernels cannot read in 16-byte loads give the same P in every
    precision and the same kept copy, also in aggregates past a workgroup."""
    import torch
    from paper_1202_2462_amd.mgdd import F16, F32, F64
    dims, N = (12, 4, 4, 8), 6
    lat = lattice(problem(dims, seed=21, m0=0.1), (2, 4, 4, 4))
    tv = lat.pack(latgen.gaussian_fields(dims, N, 25), F64)
    shifted = torch.empty(tv.numel() + 1, dtype=tv.dtype, device=tv.device)[1:].view(tv.shape)
    shifted.copy_(tv)
    assert shifted.data_ptr() % 16 == 8
    c = latgen.gaussian_fields((12 // agg[0], 4 // agg[1], 4 // agg[2], 8 // agg[3]), 1, 26)   # (1, Vc, 4, 3): N = 6
    dev = torch.tensor(np.stack([c.real, c.imag], -1).reshape(1, -1, 2, N, 2), device="cuda")
    seen = []
    for vectors in (tv, shifted):
        lat.build_P(agg, vectors)
        say("kept copy and P", agg)
        assert bool((lat.test_vectors() == tv).all())
        seen.append([lat.prolong(dev.to(torch.float64 if p == F64 else torch.float32), lat.field(p, 1)) for p in (F64, F32, F16)])
    for x, y in zip(*seen):
        assert bool((x == y).all())
    lat.close()
