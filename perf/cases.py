"""The work that a user has this library do, as a list of cases that can be
timed and checked: one call (or one short chain of calls) of the public
binding each, from a latency-bound apply on 8^4 sites to the largest lattice
that fits one GPU.

  listed()            the cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) inputs and context on the GPU
  run(state)          one pass, its outputs
  work(case)          bytes and operations the pass cannot do without
  exact(case, seed)   the same outputs from plain torch in FP64

Gauge fields follow the recipe of the workloads (links exp(i 0.5 H), two APE
steps with alpha = 0.5, c_sw = 1); large lattices repeat a smaller field in
every direction, as the benchmark's does. The bare mass -0.02 keeps the
leftmost eigenvalue of that recipe near 0.03 at 16^3 x 32.
"""
import math

import numpy as np
import torch

from paper_1202_2462_amd import mgdd

PREC = {"f64": mgdd.F64, "f32": mgdd.F32, "f16": mgdd.F16}
REAL = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}
SOLVE = {"f64": mgdd.PLAIN_F64, "mixed": mgdd.MIXED, "mixed_f16": mgdd.MIXED_F16}
EPS, ALPHA, APE, MASS, CSW = 0.5, 0.5, 2, -0.02, 1.0
C128 = torch.complex128


def _case(kind, dims, block="4x4x4x4", **more):
    return dict(kind=kind, dims=dims, block=block, **more)


def listed():
    return [
        # one apply on the smallest lattice of the tests: a launch and little else
        dict(_case("dirac", "8x8x8x8", prec="f64", nrhs=1), name="dirac_f64_8x8x8x8"),
        # the outer solver's operator on the largest workload
        dict(_case("dirac", "48x48x48x96", prec="f64", nrhs=1), name="dirac_f64_48x48x48x96"),
        # twelve point sources (one propagator) through the operator in single precision
        dict(_case("dirac", "24x24x24x48", prec="f32", nrhs=12), name="dirac_f32_24x24x24x48_12rhs"),
        # the smoother as the preconditioner calls it: one sweep, four MR steps
        dict(_case("sap", "32x32x32x64", prec="f32", nrhs=1, nsweeps=1, mr=4, shift=0.0), name="sap_f32_32x32x32x64"),
        # the smoother on half-precision storage, twelve sources
        dict(_case("sap", "16x16x16x32", prec="f16", nrhs=12, nsweeps=1, mr=4, shift=0.0), name="sap_f16_16x16x16x32_12rhs"),
        # shifted sweeps of the setup in double precision, smaller blocks on an uneven lattice
        dict(_case("sap", "12x20x16x24", block="2x2x4x4", prec="f64", nrhs=3, nsweeps=3, mr=4, shift=0.05),
             name="sap_f64_12x20x16x24_3rhs_shift"),
        # the coarse solve of a preconditioner application at 32^3 x 64
        dict(_case("coarse_solve", "32x32x32x64", agg="4x4x4x4", ntv=20, prec="f32", nrhs=1, iters=12),
             name="coarse_f32_32x32x32x64_n20"),
        # one preconditioner application on the small workload: many short kernels
        dict(_case("precondition", "16x16x16x32", agg="4x4x4x4", ntv=20, prec="f32", nrhs=1, nu=1, mr=4, iters=12),
             name="precondition_f32_16x16x16x32"),
        # the same for twelve sources on a larger lattice
        dict(_case("precondition", "24x24x24x48", agg="4x4x4x4", ntv=24, prec="f32", nrhs=12, nu=1, mr=4, iters=12),
             name="precondition_f32_24x24x24x48_12rhs"),
        # P and D_c again from kept test vectors, then their first use; odd aggregate and vector count
        dict(_case("build_P", "24x24x24x48", agg="3x4x4x4", ntv=21, prec="f64", nrhs=1), name="build_P_24x24x24x48_n21"),
        # a new gauge configuration: ingest, bootstrap setup, one mixed-precision solve
        dict(_case("setup_solve", "16x16x16x32", agg="4x4x4x4", ntv=20, precision="mixed", nrhs=1), name="setup_solve_16x16x16x32"),
        # one solve with the setup in hand at 32^3 x 64
        dict(_case("solve", "32x32x32x64", agg="4x4x4x4", ntv=24, precision="mixed", nrhs=1), name="solve_mixed_32x32x32x64"),
    ]


# ------------------------------------------------------------------ drawn cases

BLOCKS = ["4x4x4x4"] * 4 + ["2x4x4x4", "4x4x4x2", "2x2x4x4", "4x2x4x8", "2x4x4x8", "8x4x4x2", "4x4x2x2"]


def _draw_dims(rng, block, lo, hi):
    """extents the block allows (their count even or one per direction), volume near a log-uniform target"""
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    best = None
    for _ in range(200):
        d = [rng.choice([b] * (b >= 4) + [2 * b * k for k in range(1, 13) if 4 <= 2 * b * k <= 48]) for b in block]
        v = math.prod(d)
        if v <= hi and (best is None or abs(math.log(v / target)) < best[0]):
            best = (abs(math.log(v / target)), d)
    return best[1]


def _draw_agg(rng, dims, ntv):
    for _ in range(300):
        agg = [rng.choice([a for a in (2, 3, 4, 5, 6) if d % a == 0]) for d in dims]
        if 6 * math.prod(agg) >= 4 * ntv and math.prod(agg) <= 256 and all(d // a >= 2 for d, a in zip(dims, agg)):
            return agg
    return None


def draw(rng):
    text = lambda v: "x".join(map(str, v))  # noqa: E731
    while True:
        kind = rng.choice(["dirac", "dirac", "sap", "sap", "sap", "coarse_solve", "precondition", "precondition", "build_P",
                           "setup_solve", "solve"])
        block = rng.choice(BLOCKS)
        bl = [int(v) for v in block.split("x")]
        nrhs = rng.choice([1, 1, 1, 2, 3, 4, 5, 7, 12])
        if kind in ("dirac", "sap"):
            dims = _draw_dims(rng, bl, 4096, 1_500_000)
            prec = rng.choice(["f64", "f32", "f32", "f16"])
            if math.prod(dims) * nrhs > 6_000_000:
                continue
            more = dict(prec=prec, nrhs=nrhs)
            if kind == "sap":
                more.update(nsweeps=rng.choice([1, 1, 2, 3]), mr=rng.choice([2, 3, 4, 4, 5, 6]), shift=rng.choice([0.0, 0.0, 0.05]))
            return _case(kind, text(dims), block, **more)
        ntv = rng.choice([8, 11, 12, 16, 17, 20, 20, 23, 24, 28, 32])
        if kind in ("setup_solve", "solve"):
            dims = _draw_dims(rng, bl, 8192, 140_000)
            nrhs, prec = rng.choice([1, 1, 2, 3]), None
            more = dict(precision=rng.choice(["mixed", "mixed", "mixed_f16", "f64"]), nrhs=nrhs)
        elif kind == "coarse_solve":
            dims = _draw_dims(rng, bl, 8192, 1_000_000)
            more = dict(prec=rng.choice(["f32", "f32", "f64"]), nrhs=nrhs, iters=rng.choice([6, 8, 12, 12, 15]))
        elif kind == "precondition":
            dims = _draw_dims(rng, bl, 8192, 400_000)
            more = dict(prec=rng.choice(["f32", "f32", "f64"]), nrhs=nrhs, nu=rng.choice([1, 1, 2]), mr=rng.choice([3, 4, 5]), iters=12)
        else:
            dims = _draw_dims(rng, bl, 8192, 500_000)
            more = dict(prec="f64", nrhs=1)
        agg = _draw_agg(rng, dims, ntv)
        if agg is None or math.prod(dims) * nrhs > 4_000_000 or math.prod(dims) * ntv > 16_000_000:
            continue
        return _case(kind, text(dims), block, agg=text(agg), ntv=ntv, **more)


# ------------------------------------------------------------------ plain torch: gauge field, operator, aggregation
# Fields are (n, 4, 3, Lt, Lz, Ly, Lx) complex128, links (4, 3, 3, Lt, Lz, Ly, Lx)
# with the antiperiodic sign on the last time slice, A (2, 6, 6, ...) the clover
# term of both chiralities.

def _ints(t):
    return [int(v) for v in t.split("x")]


def _gen(seed, tag):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 16 + tag) % (1 << 62))


def _randn(g, *shape):
    return torch.view_as_complex(torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=g))


def _base(dims):
    """the extents of the field that is repeated, and how often per direction"""
    d, r = list(dims), [1, 1, 1, 1]
    while math.prod(d) > 200_000:
        for i in sorted(range(4), key=lambda i: -d[i]):
            f = next((f for f in (3, 2) if d[i] % f == 0 and d[i] // f >= 4), None)
            if f:
                d[i] //= f
                r[i] *= f
                break
        else:
            break
    return d, r


def _dag(m):
    return m.conj().transpose(-1, -2)


def _unitary(m):
    """rows 0 and 1 by Gram-Schmidt, row 2 = conj(row 0 x row 1)"""
    r0 = m[..., 0, :] / torch.linalg.vector_norm(m[..., 0, :], dim=-1, keepdim=True)
    r1 = m[..., 1, :] - (r0.conj() * m[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    return torch.stack([r0, r1, torch.linalg.cross(r0, r1).conj()], dim=-2)


def _su3(m):
    """polar projection (Newton's iteration), then the determinant's phase taken out"""
    for _ in range(10):
        a, b, c = m[..., 0, :], m[..., 1, :], m[..., 2, :]
        cof = torch.stack([torch.linalg.cross(b, c), torch.linalg.cross(c, a), torch.linalg.cross(a, b)], dim=-2)
        det = (a * cof[..., 0, :]).sum(-1)[..., None, None]
        m = 0.5 * (m + (cof / det).conj())
    det = (m[..., 0, :] * torch.linalg.cross(m[..., 1, :], m[..., 2, :])).sum(-1)
    return _unitary(m / torch.polar(torch.ones_like(det.real), det.angle() / 3)[..., None, None])


def _links(dims, seed):
    """(Lt, Lz, Ly, Lx, 4, 3, 3), periodic"""
    x, y, z, t = dims
    w = torch.randn(t, z, y, x, 4, 8, dtype=torch.float64, device="cuda", generator=_gen(seed, 1)) * 0.5
    h = torch.zeros(t, z, y, x, 4, 3, 3, dtype=C128, device="cuda")
    for k, (i, j) in ((0, (0, 1)), (3, (0, 2)), (5, (1, 2))):
        h[..., i, j] = torch.complex(w[..., k], -w[..., k + 1])
        h[..., j, i] = h[..., i, j].conj()
    s3 = 1 / math.sqrt(3)
    h[..., 0, 0] = w[..., 2] + w[..., 7] * s3
    h[..., 1, 1] = -w[..., 2] + w[..., 7] * s3
    h[..., 2, 2] = -2 * s3 * w[..., 7]
    e = 1j * EPS * h / 16
    u = torch.eye(3, dtype=C128, device="cuda").expand_as(e).clone()
    for k in range(10, 0, -1):                                       # exp(e) by its series, squared four times
        u = torch.eye(3, dtype=C128, device="cuda") + e @ u / k
    for _ in range(4):
        u = u @ u
    u = _unitary(u)
    for _ in range(APE):
        new = []
        for mu in range(4):
            um, st = u[..., mu, :, :], 0
            for nu in range(4):
                if nu == mu:
                    continue
                un = u[..., nu, :, :]
                st = st + un @ _sh(um, nu, 1) @ _dag(_sh(un, mu, 1))
                dn = _sh(un, nu, -1)
                st = st + _dag(dn) @ _sh(um, nu, -1) @ _sh(dn, mu, 1)
            new.append(_su3((1 - ALPHA) * um + (ALPHA / 6) * st))
        u = torch.stack(new, dim=-3)
    return u


def _sh(m, mu, step):
    """the matrix field (Lt, Lz, Ly, Lx, 3, 3) at x + step mu"""
    return torch.roll(m, -step, 3 - mu)


def _gauge(case, seed):
    """canonical (V, 4, 3, 3) links of the case"""
    dims = _ints(case["dims"])
    base, r = _base(dims)
    return _links(base, seed).repeat(r[3], r[2], r[1], r[0], 1, 1, 1).contiguous()


_S = [np.array([[0, 1], [1, 0]], complex), np.array([[0, -1j], [1j, 0]]), np.diag([1, -1]).astype(complex)]
_B = [-1j * s for s in _S] + [-np.eye(2, dtype=complex)]           # gamma_mu = [[0, B], [C, 0]]
_C = [1j * s for s in _S] + [-np.eye(2, dtype=complex)]


def _two(m, p):
    """2 x 2 spin matrix with one entry per row on (n, 2, 3, ...)"""
    rows = []
    for i in range(2):
        j = int(np.argmax(np.abs(m[i])))
        rows.append(p[:, j] * complex(m[i, j]))
    return torch.stack(rows, 1)


def _colour(u, h):
    """sum_b u[a, b] h[:, :, b]"""
    return torch.stack([u[a, 0] * h[:, :, 0] + u[a, 1] * h[:, :, 1] + u[a, 2] * h[:, :, 2] for a in range(3)], 2)


class _Operator:
    """D of the canonical links (Lt, Lz, Ly, Lx, 4, 3, 3), in FP64; clover=(links, repeats): the clover term of a
    smaller field, repeated"""

    def __init__(self, u, clover=None):
        src, rep = clover or (u, (1, 1, 1, 1))
        self.A = self._clover(src).repeat(1, 1, 1, rep[3], rep[2], rep[1], rep[0])
        self.U = u.permute(4, 5, 6, 0, 1, 2, 3).contiguous()
        self.U[3, :, :, -1] *= -1

    @staticmethod
    def _clover(u):
        gam = [np.block([[np.zeros((2, 2)), b], [c, np.zeros((2, 2))]]) for b, c in zip(_B, _C)]
        A = torch.zeros((2, 2, 3, 2, 3) + tuple(u.shape[:4]), dtype=C128, device="cuda")
        for s in range(2):
            for a in range(3):
                A[:, s, a, s, a] = 4 + MASS
        for mu in range(4):
            for nu in range(mu + 1, 4):
                um, un = u[..., mu, :, :], u[..., nu, :, :]
                q = um @ _sh(un, mu, 1) @ _dag(_sh(um, nu, 1)) @ _dag(un)
                q = q + un @ _dag(_sh(_sh(um, mu, -1), nu, 1)) @ _dag(_sh(un, mu, -1)) @ _sh(um, mu, -1)
                c = _sh(_sh(um, mu, -1), nu, -1)
                q = q + _dag(_sh(um, mu, -1)) @ _dag(_sh(_sh(un, mu, -1), nu, -1)) @ c @ _sh(un, nu, -1)
                q = q + _dag(_sh(un, nu, -1)) @ _sh(um, nu, -1) @ _sh(_sh(un, nu, -1), mu, 1) @ _dag(um)
                f = ((q - _dag(q)) / 8).permute(4, 5, 0, 1, 2, 3)
                sig = 0.5j * (gam[mu] @ gam[nu] - gam[nu] @ gam[mu]) * (0.5j * CSW)
                for chi in range(2):
                    for s in range(2):
                        for t in range(2):
                            v = complex(sig[2 * chi + s, 2 * chi + t])
                            if v:
                                A[chi, s, :, t] += v * f
        return A.reshape((2, 6, 6) + tuple(u.shape[:4]))

    def blocked(self, dims, block):
        """the same with the hops that leave a block dropped"""
        o = object.__new__(_Operator)
        o.A, o.U = self.A, self.U.clone()
        for mu in range(4):
            if dims[mu] != block[mu]:
                o.U[mu].transpose(2, 5 - mu)[:, :, block[mu] - 1::block[mu]] = 0
        return o

    def __call__(self, p):
        n, sites = p.shape[0], tuple(p.shape[3:])
        v = p.reshape((n, 2, 6) + sites)
        out = torch.stack([sum(self.A[:, i, j] * v[:, :, j] for j in range(6)) for i in range(6)], 2).reshape(p.shape)
        for mu in range(4):
            ax, u = -1 - mu, self.U[mu]
            f = torch.roll(p, -1, ax)
            h = _colour(u, f[:, :2] - _two(_B[mu], f[:, 2:]))
            del f
            out[:, :2] -= 0.5 * h
            out[:, 2:] += 0.5 * _two(_C[mu], h)
            h = _colour(u.transpose(0, 1).conj(), p[:, :2] + _two(_B[mu], p[:, 2:]))
            h = torch.roll(h, 1, ax)
            out[:, :2] -= 0.5 * h
            out[:, 2:] -= 0.5 * _two(_C[mu], h)
        return out


def _operator(case, seed):
    dims = _ints(case["dims"])
    base, r = _base(dims)
    u = _links(base, seed)
    return _Operator(u.repeat(r[3], r[2], r[1], r[0], 1, 1, 1), (u, r))


def _field(c, dims):
    """canonical (n, V, 4, 3) -> (n, 4, 3, Lt, Lz, Ly, Lx)"""
    n = c.shape[0]
    return c.permute(0, 2, 3, 1).reshape(n, 4, 3, dims[3], dims[2], dims[1], dims[0])


def _site_order(dims, block):
    """canonical site of every device site"""
    dev = torch.device("cuda")
    s = torch.arange(math.prod(dims), device=dev)
    x, r = [], s
    for d in dims:
        x.append(r % d)
        r = r // d
    nb = [d // b for d, b in zip(dims, block)]
    bc = [xi // b for xi, b in zip(x, block)]
    lex = bc[0] + nb[0] * (bc[1] + nb[1] * (bc[2] + nb[2] * bc[3]))
    loc = [xi % b for xi, b in zip(x, block)]
    par = sum(loc) % 2
    ll = loc[0] + block[0] * (loc[1] + block[1] * (loc[2] + block[2] * loc[3]))
    key = (((sum(bc) % 2) * math.prod(nb) + lex) * 2 + par) * (math.prod(block) // 2) + ll // 2
    return torch.argsort(key)


def _device(f, case, dtype):
    """a field in the device layout of the library, (n, 12, V, 2)"""
    n = f.shape[0]
    d = f.reshape(n, 12, -1)[:, :, _site_order(_ints(case["dims"]), _ints(case["block"]))]
    return torch.view_as_real(d).to(dtype)


def _sap(D, Db, dims, block, b, z, nsweeps, mr, shift):
    x = [torch.arange(d, device="cuda") // w for d, w in zip(dims, block)]
    col = (x[3][:, None, None, None] + x[2][:, None, None] + x[1][:, None] + x[0]) % 2
    split = sum(([d // w, w] for d, w in zip(dims[::-1], block[::-1])), [])
    n = b.shape[0]

    def block_sum(v):                                               # (n, 4, 3, sites) -> one value per block, spread over it
        s = v.sum((1, 2)).reshape([n] + split).sum((2, 4, 6, 8), keepdim=True)
        return s.expand([n] + split).reshape([n, 1, 1] + list(dims[::-1]))

    for _ in range(nsweeps):
        for c in range(2):
            m = (col == c)
            rho = (b - D(z) + shift * z) * m
            for _ in range(mr):
                q = Db(rho) - shift * rho
                qq = block_sum((q.conj() * q).real)
                al = block_sum(q.conj() * rho) / torch.where(qq == 0, 1.0, qq)
                z = z + al * rho
                rho = rho - al * q
    return z


class _Coarse:
    """P from test vectors (N fields) by aggregates and chirality, D_c = P^H D P applied as the three factors"""

    def __init__(self, D, dims, agg, v):
        self.D, self.agg, self.dims = D, agg, dims
        self.cd = [d // a for d, a in zip(dims, agg)]
        q = self._cut(v)
        for _ in range(2):
            q = q @ torch.linalg.inv(_dag(torch.linalg.cholesky(_dag(q) @ q)))
        self.Q = q

    def _cut(self, f):
        """(n, 4, 3, sites) -> (Vc, 2, 6 vol, n)"""
        n, c, a = f.shape[0], self.cd, self.agg
        v = f.reshape(n, 2, 6, c[3], a[3], c[2], a[2], c[1], a[1], c[0], a[0])
        return v.permute(3, 5, 7, 9, 1, 2, 4, 6, 8, 10, 0).reshape(math.prod(c), 2, 6 * math.prod(a), n).contiguous()

    def restrict(self, f):
        return (_dag(self.Q) @ self._cut(f)).permute(3, 0, 1, 2).contiguous()     # (n, Vc, 2, N)

    def prolong(self, x):
        n, c, a = x.shape[0], self.cd, self.agg
        v = self.Q @ x.permute(1, 2, 3, 0).contiguous()
        v = v.reshape(c[3], c[2], c[1], c[0], 2, 6, a[3], a[2], a[1], a[0], n).permute(10, 4, 5, 0, 6, 1, 7, 2, 8, 3, 9)
        return v.reshape([n, 4, 3] + list(self.dims[::-1]))

    def __call__(self, x):
        return torch.cat([self.restrict(self.D(self.prolong(x[i:i + 1]))) for i in range(x.shape[0])])

    def gmres(self, b, iters):
        """iters steps of GMRES from zero, one Krylov space per right-hand side"""
        n, dot = b.shape[0], lambda u, v: (u.conj() * v).sum((1, 2, 3))  # noqa: E731
        one = lambda s: s.reshape(n, 1, 1, 1)  # noqa: E731
        beta = dot(b, b).real.sqrt()
        V = [b / one(beta)]
        H = torch.zeros(n, iters + 1, iters, dtype=C128, device="cuda")
        for j in range(iters):
            w = self(V[j])
            for _ in range(2):
                for i in range(j + 1):
                    h = dot(V[i], w)
                    H[:, i, j] += h
                    w = w - one(h) * V[i]
            H[:, j + 1, j] = dot(w, w).real.sqrt()
            V.append(w / one(H[:, j + 1, j]))
        e = torch.zeros(n, iters + 1, 1, dtype=C128)
        e[:, 0, 0] = beta.cpu()
        y = torch.linalg.lstsq(H.cpu(), e).solution.cuda()
        return sum(one(y[:, j, 0]) * V[j] for j in range(iters))


def _test_vectors(case, seed):
    """N random fields with the upper part of the spectrum damped (eight Richardson steps), on the field that is repeated"""
    base, r = _base(_ints(case["dims"]))
    D, g = _Operator(_links(base, seed)), _gen(seed, 3)
    out = []
    for _ in range(case["ntv"]):
        v = _randn(g, 1, 4, 3, base[3], base[2], base[1], base[0])
        for _ in range(8):
            v = v - 0.2 * D(v)
        out.append(v / torch.linalg.vector_norm(v))
    return torch.cat(out), r


def _rhs(case, seed):
    """canonical Gaussian fields (nrhs, V, 4, 3)"""
    return _randn(_gen(seed, 2), case["nrhs"], math.prod(_ints(case["dims"])), 4, 3)


def _coarse_rhs(case, seed):
    vc = math.prod(d // a for d, a in zip(_ints(case["dims"]), _ints(case["agg"])))
    return _randn(_gen(seed, 4), case["nrhs"], vc, 2, case["ntv"])


# ------------------------------------------------------------------ the cases on the library

def _pack(lat, canon, prec):
    f = lat.field(prec, canon.shape[0])
    mgdd.mgdd_pack(lat.ctx, prec, canon.shape[0], torch.view_as_real(canon.contiguous()), f)
    return f


def prepare(case, seed):
    dims, kind = _ints(case["dims"]), case["kind"]
    lat = mgdd.Lattice(dims, _ints(case["block"]))
    u = torch.view_as_real(_gauge(case, seed))
    s = dict(case=case, lat=lat)
    if kind == "setup_solve":
        s["u"] = u
    else:
        lat.set_gauge(u, MASS, CSW)
    del u
    prec = PREC[case.get("prec", "f64")]
    if kind in ("coarse_solve", "precondition", "build_P"):
        agg = _ints(case["agg"])
        base, r = _test_vectors(case, seed)
        tv = lat.field(mgdd.F64, case["ntv"])
        for k in range(case["ntv"]):                                 # repeated in every direction, then packed
            v = base[k].repeat(1, 1, r[3], r[2], r[1], r[0]).reshape(4, 3, -1).permute(2, 0, 1).contiguous()
            mgdd.mgdd_pack(lat.ctx, mgdd.F64, 1, torch.view_as_real(v), tv[k])
        lat.build_P(agg, tv)
        if kind == "build_P":
            s.update(agg=agg, tv=tv)
    if kind in ("dirac", "sap"):
        s["b"] = _pack(lat, _rhs(case, seed), prec)
        s["z"] = torch.empty_like(s["b"])
    elif kind in ("coarse_solve", "build_P"):
        s["b"] = torch.view_as_real(_coarse_rhs(case, seed)).to(REAL[case["prec"]]).contiguous()
        s["x"] = torch.empty_like(s["b"])
        if kind == "build_P":
            s["f"] = lat.field(prec, 1)
    else:
        s["b"] = _pack(lat, _rhs(case, seed), mgdd.F64)
    if kind in ("solve", "setup_solve"):
        vc = math.prod(d // a for d, a in zip(dims, _ints(case["agg"])))
        s["start"] = torch.view_as_real(_randn(_gen(seed, 5), vc, 2, case["ntv"])).contiguous()
        s["seed"] = int(seed)
        if kind == "solve":
            _setup(s)
    torch.cuda.synchronize()
    return s


def _setup(s):
    c = s["case"]
    s["lat"].setup(_ints(c["agg"]), None, s["start"], nu=3, iota=3, mr_iters=4, n_part2=1,
                   prec=mgdd.F64 if c["precision"] == "f64" else mgdd.F32, ntv=c["ntv"], seed=s["seed"])


def run(s):
    c, lat = s["case"], s["lat"]
    kind = c["kind"]
    if kind == "dirac":
        return lat.dirac(s["b"], s["z"])
    if kind == "sap":
        s["z"].zero_()
        return lat.sap(s["b"], s["z"], c["nsweeps"], c["mr"], c["shift"])
    if kind == "coarse_solve":
        return lat.coarse_solve(s["b"], c["iters"], s["x"])
    if kind == "precondition":
        return lat.precondition(s["b"], PREC[c["prec"]], c["nu"], c["mr"], c["iters"])
    if kind == "build_P":
        lat.build_P(s["agg"], s["tv"])
        return lat.coarse_apply(s["b"], s["x"]), lat.prolong(s["b"], s["f"])
    if kind == "setup_solve":
        lat.set_gauge(s["u"], MASS, CSW)
        _setup(s)
    # twelve digits, so that the solution itself is good to well below single precision
    return lat.solve(s["b"], precision=SOLVE[c["precision"]], restart=20, tol=1e-12, maxit=500)[0]


def work(case):
    """Bytes with every input read and every output written once per step that has to read it again (a coarse operator
    larger than the 256 MB cache is read in every GMRES step), links as two rows, D_c as its five independent blocks."""
    V, n, kind = math.prod(_ints(case["dims"])), case["nrhs"], case["kind"]
    s = {"f64": 8, "f32": 4, "f16": 2}[case.get("prec", "f32")]      # bytes of a real number of a field
    g = 8 if s == 8 else 4                                           # of the links and the clover term
    links = 120 * g
    dirac = 1896
    if kind == "dirac":
        return dict(bytes=V * (links + 48 * s * n), flops=V * n * dirac)

    def sap(sweeps, mr, s, n):
        return V * sweeps * (links + 72 * s * n), V * n * sweeps * ((mr + 1) * dirac + 336 * mr)

    if kind == "sap":
        b, f = sap(case["nsweeps"], case["mr"], s, n)
        return dict(bytes=b, flops=f)
    agg, N = _ints(case["agg"]), case["ntv"]
    vc = V // math.prod(agg)

    def coarse(iters, s, n):
        dc = 5 * (2 * N) ** 2 * 2 * s * vc
        return dc * (iters if dc > 256e6 else 1) + 2 * vc * 4 * N * s * n, iters * n * vc * (72 * (2 * N) ** 2 + 16 * N * 8 * iters)

    def precondition(nu, mr, iters, s, n):
        b1, f1 = coarse(iters, s, n)
        b2, f2 = sap(nu, mr, s, n)
        return b1 + b2 + V * 2 * (N + n) * 24 * s, f1 + f2 + V * n * 192 * N

    def build():
        dc = (2 * N) ** 2 * vc
        hop = sum(1 / a for a in agg)
        return (V * N * (192 + 192 + 96 + 48) + dc * (9 * 24 + 5 * 8),
                V * (192 * N * N * (1 + hop) + N * dirac + 96 * N * N))

    if kind == "coarse_solve":
        b, f = coarse(case["iters"], s, n)
    elif kind == "precondition":
        b, f = precondition(case["nu"], case["mr"], case["iters"], s, n)
    elif kind == "build_P":
        b, f = build()
    else:                                                            # 40 outer iterations of FGMRES(20)
        s = {"f64": 8, "mixed": 4, "mixed_f16": 2}[case["precision"]]
        b, f = precondition(1, 4, 12, s, n)
        b, f = 40 * (b + V * (960 + 384 * n) + V * n * 192 * 24), 40 * (f + V * n * (dirac + 96 * 4 * 10))
        if kind == "setup_solve":
            b1, f1 = sap(6, 4, s, N)
            b2, f2 = build()
            b += b1 + 2 * b2 + V * N * 192 * 20
            f += f1 + 2 * f2 + V * 96 * N * N * 10
    return dict(bytes=b, flops=f)


def exact(case, seed):
    dims, block, kind = _ints(case["dims"]), _ints(case["block"]), case["kind"]
    V = math.prod(dims)
    if kind in ("solve", "setup_solve") and V * case["nrhs"] > 150_000:
        return None
    out = torch.float64
    D = _operator(case, seed)
    if kind in ("dirac", "sap"):
        b = _field(_rhs(case, seed), dims)
        b = torch.view_as_complex(torch.view_as_real(b).to(REAL[case["prec"]]).to(torch.float64))   # as the library gets it
        if kind == "dirac":
            f = torch.cat([D(b[i:i + 1]) for i in range(b.shape[0])])
        else:
            Db = D.blocked(dims, block)
            f = torch.cat([_sap(D, Db, dims, block, b[i:i + 1], torch.zeros_like(b[i:i + 1]), case["nsweeps"], case["mr"],
                                case["shift"]) for i in range(b.shape[0])])
        return _device(f, case, out)
    if kind in ("coarse_solve", "precondition", "build_P"):
        base, r = _test_vectors(case, seed)
        P = _Coarse(D, dims, _ints(case["agg"]), base.repeat(1, 1, 1, r[3], r[2], r[1], r[0]))
        if kind == "precondition":
            b = _field(_rhs(case, seed), dims)
            z = P.prolong(P.gmres(P.restrict(b), case["iters"]))
            Db = D.blocked(dims, block)
            f = torch.cat([_sap(D, Db, dims, block, b[i:i + 1], z[i:i + 1], case["nu"], case["mr"], 0.0)
                           for i in range(b.shape[0])])
            return _device(f, case, out)
        b = torch.view_as_complex(torch.view_as_real(_coarse_rhs(case, seed)).to(REAL[case["prec"]]).to(out))
        if kind == "coarse_solve":
            return torch.view_as_real(P.gmres(b, case["iters"]))
        return torch.view_as_real(P(b)), _device(P.prolong(b), case, out)

    # conjugate gradients on D^H D z = D^H b with two restarts from the iterate
    g5 = torch.tensor([1, 1, -1, -1], dtype=torch.float64, device="cuda").reshape(1, 4, 1, 1, 1, 1, 1)
    found = []
    for b in _field(_rhs(case, seed), dims).split(1):
        z = torch.zeros_like(b)
        for _ in range(3):
            r = b - D(z)
            t = g5 * D(g5 * r)
            p, tt = t, (t.conj() * t).real.sum()
            stop = 1e-22 * tt
            for k in range(2000):
                q = D(p)
                a = tt / (q.conj() * q).real.sum()
                z, r = z + a * p, r - a * q
                t = g5 * D(g5 * r)
                new = (t.conj() * t).real.sum()
                p, tt = t + (new / tt) * p, new
                if k % 25 == 24 and float(tt) < float(stop):
                    break
        found.append(z)
    return _device(torch.cat(found), case, out)
