// The coarse operator D_c = P^H D P (Section 3, Petrov-Galerkin with R = P^H):
// a 9-point stencil of 2N x 2N blocks, built in FP64 on the matrix cores.
//
// Only the forward half is computed. D is gamma5-hermitian and P keeps the
// chiralities apart, so with s = +1 on the first and -1 on the last N coarse
// components
//   D_c(a, a - mu)[i][j] = s_i s_j conj(D_c(a - mu, a)[j][i]),
//   D_c(a, a)[i][j]      = X[i][j] + s_i s_j conj(X[j][i]),
// where X holds half of the clover term and the forward hops that stay inside
// the aggregate. The backward hops, half of the stencil work and 4 of the 9
// products with P^H are not formed.
#include "stencil.h"
#include "transfer.h"

namespace mgdd {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

constexpr int STEP = 16, WAVES = 4;   // sites a step: two 128-byte lines of a component, four sites a wave

// v = U_mu psi (one colour) for the two spins of one chirality, and its image w in the
// other chirality: (1 - gamma_mu) U psi = (v, w) or (w, v). In the chiral
// basis w = sg i sigma_mu v for the space directions (sg = +1 when psi is
// the lower chirality, -1 when it is the upper one) and w = v in time.
template <int MU> __device__ inline void other_chirality(const double2 *v, double sg, double2 *w) {
    const double2 a = v[0], b = v[1];   // one colour of the two spins
    if (MU == 0) {          // (i b, i a)
        w[0] = make_double2(-sg * b.y, sg * b.x);
        w[1] = make_double2(-sg * a.y, sg * a.x);
    } else if (MU == 1) {   // (b, -a)
        w[0] = make_double2(sg * b.x, sg * b.y);
        w[1] = make_double2(-sg * a.x, -sg * a.y);
    } else if (MU == 2) {   // (i a, -i b)
        w[0] = make_double2(-sg * a.y, sg * a.x);
        w[1] = make_double2(sg * b.y, -sg * b.x);
    } else {
        w[0] = a;
        w[1] = b;
    }
}

// same += f v, other += f w of the forward hop in direction MU (same and other
// as in other_chirality); psi: one chirality of a column of P at the
// neighbour, lk: the site's link, `stride` between its entries
template <int MU>
__device__ inline void forward_hop(const double2 *lk, size_t stride, const v2d *psi, double sg, double f, double2 *same, double2 *other) {
#pragma unroll
    for (int r = 0; r < 3; r++) {   // colour r of both spins
        double2 v[2], w[2];
#pragma unroll
        for (int q = 0; q < 2; q++) v[q] = make_double2(0, 0);
#pragma unroll
        for (int b = 0; b < 3; b++) {
            const double2 u = lk[(3 * r + b) * stride];
#pragma unroll
            for (int q = 0; q < 2; q++) cfma(v[q], u, make_double2(psi[3 * q + b][0], psi[3 * q + b][1]));
        }
        other_chirality<MU>(v, sg, w);
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const int c = 3 * q + r;
            same[c] = make_double2(fma(f, v[q].x, same[c].x), fma(f, v[q].y, same[c].y));
            other[c] = make_double2(fma(f, w[q].x, other[c].x), fma(f, w[q].y, other[c].y));
        }
    }
}

// One workgroup per (aggregate a, term t): t = 0 the self term X over all
// sites of a, or each of `parts` workgroups over `per` of them, t = 1 + mu the
// forward hop over the sites of its + mu face. The parts' sums are kept where
// the backward blocks of a belong and added up by dc_parts_kernel.
// Sixteen sites of the list a step, four of them per wave, and the block's
// columns j = (chi', k') in NT tiles of 16 one after the other. Lane (jj, s) =
// (lane % 16, lane / 16) forms D P_j at its wave's site s, all 12 components in
// registers: that is the layout of the B operand of a 16x16x4 FP64 MFMA
// (column jj, summation index s), so the product with P^H needs no exchange;
// the A operand is P_k at the same site, k = lane % 16 of a row tile (RT row
// tiles of 16 test vectors), from LDS, where the workgroup holds the sixteen
// sites' P, links and clover term; the next ones are loaded under the last
// tile's products, as a tile's first hop is under those of the one before. Rows
// past N, columns past 2N and sites past the end of the list are computed from
// clamped addresses; the latter enter as zeros, the others are not stored.
//
// Bound: latency, with one wave per SIMD (its sums of all tiles take half of
// the registers): the matrix cores are busy for 32 %, the vector units for 18 %
// of 24^3 x 48, 3x4x4x4 aggregates, N = 21: 8.1 ms. dc_forward_small_kernel,
// whose waves do not share what they read of P and use half of every line that
// they take from L2 (67 GB against 37 past it), 9.4 ms; one workgroup per
// column with the dot products on the vector units and sums through LDS 29.4 ms.
// Eight sites a step with a wave per tile and half of them, two waves on some
// SIMDs and one on others: 8.5 ms; the same with three waves a SIMD spills. Four
// tiles (N >= 25) spill too, 240 B a lane: P and D_c together of 24^3 x 48, 4^4
// sites, N = 24: 10.9 ms, 25: 15.2, 28: 15.9, 32: 17.6 (one column a workgroup: 38,
// 42, 51, 65).

// LDS place of (component, test vector, site of the step): the sites are
// permuted by the vector, so that the 16 vectors of an A operand lie in all banks
__device__ inline int pk_at(int N, int c, int k, int s) { return (c * N + k) * STEP + (s ^ (k & 15)); }

template <int NT, int RT>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(1))) void dc_forward_kernel(
    Geom g, AggGeom ag, int N, int Va, int parts, int per, const int *__restrict__ agg_sites,
    const int *__restrict__ face_sites,
    const double2 *__restrict__ Up, const double2 *__restrict__ Ap, const double2 *__restrict__ P, double2 *__restrict__ Dc) {
    extern __shared__ double2 pk[];   // [12 N + 72][STEP]: P, links, clover term; at the end [WAVES][sums of a tile]
    constexpr int ROWS = 64 * WAVES / STEP, PER = (96 * NT + ROWS - 1) / ROWS, PERU = (72 + ROWS - 1) / ROWS;
    const int wg = xcd_block(gridDim.x), a = wg / (4 + parts), part = wg % (4 + parts);
    const int t = part < parts ? 0 : part - parts + 1;
    const int n2 = 2 * N, lane = threadIdx.x & 63, s = lane >> 4, wave = threadIdx.x >> 6;
    const size_t V = g.V;
    const int *list = agg_sites + (size_t)a * Va + (t ? 0 : part * per);
    int count = per < Va - part * per ? per : Va - part * per;
    if (t) {
        size_t o = 0;
#pragma unroll
        for (int m = 0; m < 4; m++) {
            if (m == t - 1) {
                count = Va / ag.a[m];
                list = face_sites + o + (size_t)a * count;
            }
            o += V / ag.a[m];
        }
    }
    // the last site coordinate of the aggregate in every direction
    int end[4];
    {
        int r = a;
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int lc = g.L[m] / ag.a[m];
            end[m] = (r % lc + 1) * ag.a[m] - 1;
            r /= lc;
        }
    }
    v4d re[NT][2][RT], im[NT][2][RT];
#pragma unroll
    for (int tl = 0; tl < NT; tl++)
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int rt = 0; rt < RT; rt++) re[tl][h][rt] = im[tl][h][rt] = (v4d){0, 0, 0, 0};
    // the lane's column of a tile (vector, chirality)
    int col[NT];   // 2 vector + chirality
#pragma unroll
    for (int tl = 0; tl < NT; tl++) {
        const int j = 16 * tl + (lane & 15), jc = j < n2 ? j : n2 - 1;
        col[tl] = jc >= N ? 2 * (jc - N) + 1 : 2 * jc;
    }
    int krow[RT];
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
        const int k = 16 * rt + (lane & 15);
        krow[rt] = k < N ? k : N - 1;
    }
    // staging: thread (row, site) = (thread / STEP, thread % STEP), rows 12 k + c
    const int rows = 12 * N;
    const int urow0 = t ? 9 * (t - 1) : 0, urows = t ? 9 : 72;   // of the 36 link and 36 clover rows
    const int ss = threadIdx.x % STEP, row = threadIdx.x / STEP;
    v2d st[PER], su[PERU];
    auto fetch = [&](int q, int row) {
        const int dd = list[q + ss < count ? q + ss : count - 1];
        const double2 *p = P + dd;
#pragma unroll
        for (int i = 0; i < PERU; i++)
            if (i * ROWS < urows) {
                const int rr = row + i * ROWS, r = urow0 + (rr < urows ? rr : urows - 1);
                su[i] = *(const v2d *)((r < 36 ? Up + (size_t)r * V : Ap + (size_t)(r - 36) * V) + dd);
            }
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int r = row + i * ROWS;
            st[i] = *(const v2d *)(p + (size_t)(r < rows ? r : rows - 1) * V);
        }
    };
    auto put = [&](int row) {
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int rr = row + i * ROWS, r = rr < rows ? rr : rows - 1, k = r / 12;
            *(v2d *)(pk + pk_at(N, r - 12 * k, k, ss)) = st[i];
        }
#pragma unroll
        for (int i = 0; i < PERU; i++)
            if (i * ROWS < urows) {
                const int rr = row + i * ROWS, r = urow0 + (rr < urows ? rr : urows - 1);
                *(v2d *)(pk + (rows + r) * STEP + ss) = su[i];
            }
    };
    // the lane's site of a step and where its hops come from: the site itself,
    // with the factor 0 (bit m of out), where a hop leaves the aggregate
    int nb[4], out;
    auto locate = [&](int q) {
        const int qs = q + 4 * wave + s;
        const int d = list[qs < count ? qs : count - 1];
        const int pos = d >> g.lgVb;
        int x[4], bc[4];
        local_coords(g, d & (g.Vb - 1), x);
        unpack_block(g.blk_coord[pos], bc);
        out = qs < count ? 0 : 16;
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const bool leaves = (bc[m] << g.lb[m]) + x[m] == end[m];
            const bool take = t ? t == 1 + m : !leaves;
            nb[m] = d;
            if (take) nb[m] = neighbour(g, pos, x, m, +1);
            else out |= 1 << m;
        }
    };
    v2d psi[2][6];
    auto load_psi = [&](int cl, int dn, v2d *v) {
        const double2 *Pj = P + (size_t)(6 * cl) * V + dn;
#pragma unroll
        for (int c = 0; c < 6; c++) v[c] = *(const v2d *)(Pj + (size_t)c * V);
    };
    auto first = [&]() { return t ? (t == 1 ? nb[0] : t == 2 ? nb[1] : t == 3 ? nb[2] : nb[3]) : nb[0]; };
    fetch(0, row);
    locate(0);
    load_psi(col[0], first(), psi[0]);
    put(row);
    __syncthreads();
    const double2 *lk = pk + rows * STEP + 4 * wave + s;
    for (int q = 0; q < count; q += STEP) {
        const int Nq = N + (int)opaque_zero();   // LDS places are computed in every step, not kept
        const int qn = q + STEP < count ? q + STEP : q;
#pragma unroll
        for (int tl = 0; tl < NT; tl++) {
            const int chi = col[tl] & 1;
            const double sg = chi ? 1.0 : -1.0;
            double2 same[6], other[6];
#pragma unroll
            for (int c = 0; c < 6; c++) same[c] = other[c] = make_double2(0, 0);
            // a hop's operands are loaded while the one before it is computed
            if (t == 0) {
#define HOP(MU)                                                                                  \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    if (MU < 3) load_psi(col[tl], nb[(MU + 1) & 3], psi[(MU + 1) & 1]);                          \
    __builtin_amdgcn_sched_barrier(0);                                                           \
    forward_hop<MU>(lk + 9 * MU * STEP, STEP, psi[MU & 1], sg, out & (1 << MU) ? 0.0 : 1.0, same, other)
                HOP(0);
                HOP(1);
                HOP(2);
                HOP(3);
#undef HOP
            } else if (t == 1) {
                forward_hop<0>(lk, STEP, psi[0], sg, 1.0, same, other);
            } else if (t == 2) {
                forward_hop<1>(lk + 9 * STEP, STEP, psi[0], sg, 1.0, same, other);
            } else if (t == 3) {
                forward_hop<2>(lk + 18 * STEP, STEP, psi[0], sg, 1.0, same, other);
            } else {
                forward_hop<3>(lk + 27 * STEP, STEP, psi[0], sg, 1.0, same, other);
            }
            __builtin_amdgcn_sched_barrier(0);
            // the two chiralities' components of D P_j: same and other, or other and
            // same. (Sums with a factor 0: a choice between the arrays by the lane's
            // chirality would put them in scratch memory)
            const double f = out & 16 ? 0.0 : -0.5, f0 = chi ? 0.0 : f, f1 = chi ? f : 0.0;
            double2 w[2][6];
#pragma unroll
            for (int c = 0; c < 6; c++) {
                w[0][c] = make_double2(fma(f1, other[c].x, f0 * same[c].x), fma(f1, other[c].y, f0 * same[c].y));
                w[1][c] = make_double2(fma(f0, other[c].x, f1 * same[c].x), fma(f0, other[c].y, f1 * same[c].y));
            }
            if (t == 0) {
                double2 in[6];
                const double2 *ck = lk + (36 + 18 * chi) * STEP;
#pragma unroll
                for (int c = 0; c < 6; c++) in[c] = pk[pk_at(Nq, 6 * chi + c, col[tl] >> 1, 4 * wave + s)];
                // the packed Hermitian block row by row: pair 3 + e holds the e-th upper entry
#pragma unroll
                for (int i = 0; i < 6; i++) {
                    const double2 dg = ck[(i / 2) * STEP];
                    double2 ax = cscale(in[i], i & 1 ? dg.y : dg.x);
#pragma unroll
                    for (int k = 0; k < 6; k++) {
                        if (k == i) continue;
                        const double2 e = ck[hpack(k < i ? k : i, k < i ? i : k) / 2 * STEP];
                        if (k < i) cfmac(ax, e, in[k]);
                        else cfma(ax, e, in[k]);
                    }
                    w[0][i] = make_double2(fma(-f0, ax.x, w[0][i].x), fma(-f0, ax.y, w[0][i].y));
                    w[1][i] = make_double2(fma(-f1, ax.x, w[1][i].x), fma(-f1, ax.y, w[1][i].y));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // in flight under the products: the next tile's first hop, or the next
            // step's sites, fields and links
            if (tl + 1 < NT) {
                load_psi(col[tl + 1 < NT ? tl + 1 : 0], first(), psi[0]);
            } else {
                fetch(qn, row + Nq - N);
                locate(qn);
                load_psi(col[0], first(), psi[0]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; h++) {
#pragma unroll
                for (int c = 0; c < 6; c++) {
                    double2 p[RT];
#pragma unroll
                    for (int rt = 0; rt < RT; rt++) p[rt] = pk[pk_at(Nq, 6 * h + c, krow[rt], 4 * wave + s)];
                    // conj(p) w
#pragma unroll
                    for (int rt = 0; rt < RT; rt++) {
                        re[tl][h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[rt].x, w[h][c].x, re[tl][h][rt], 0, 0, 0);
                        im[tl][h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[rt].x, w[h][c].y, im[tl][h][rt], 0, 0, 0);
                    }
#pragma unroll
                    for (int rt = 0; rt < RT; rt++) {
                        re[tl][h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[rt].y, w[h][c].y, re[tl][h][rt], 0, 0, 0);
                        im[tl][h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(-p[rt].y, w[h][c].x, im[tl][h][rt], 0, 0, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        put(row + Nq - N);
        __syncthreads();
    }
    // the waves' sums of a tile: [wave][h][rt][v][lane]; a wave adds up and stores
    // its share of the rows
    double2 *res = Dc + ((size_t)a * 9 + (t ? 2 * t - 1 : 2 * part)) * n2 * n2;
    constexpr int SUMS = 2 * RT * 4;
#pragma unroll
    for (int tl = 0; tl < NT; tl++) {
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int rt = 0; rt < RT; rt++)
#pragma unroll
                for (int v = 0; v < 4; v++)
                    pk[(wave * SUMS + (h * RT + rt) * 4 + v) * 64 + lane] =
                        make_double2(re[tl][h][rt][v], im[tl][h][rt][v]);
        __syncthreads();
        const int j = 16 * tl + (lane & 15);
        for (int e = wave; e < SUMS; e += WAVES) {
            double2 o = pk[e * 64 + lane];
#pragma unroll
            for (int w = 1; w < WAVES; w++) o = cadd(o, pk[(w * SUMS + e) * 64 + lane]);
            const int h = e / (4 * RT), k = 16 * (e / 4 % RT) + 4 * (e & 3) + s;   // row of result register e % 4 in lane (jj, s)
            if (j < n2 && k < N) res[(size_t)j * n2 + h * N + k] = o;
        }
        __syncthreads();
    }
}

// The same for aggregates of fewer than 64 sites, whose lists are one or two
// steps of the kernel above and which are better served by more and smaller
// workgroups: a wave per 16 columns, four sites a step, P from memory, no LDS.
// 16^3 x 32, P and D_c together, this / the kernel above, N = 20: 2^4 sites 4.4
// / 5.8 ms, 2^3 x 4 3.7 / 3.9, 2^2 x 4^2 3.8 / 3.6, 2 x 4^3 2.9 / 2.6; N = 8:
// 1.10 / 1.48, 0.97 / 1.07, 1.05 / 0.98, 0.90 / 0.74.
template <int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void dc_forward_small_kernel(
    Geom g, AggGeom ag, int N, int Va, const int *__restrict__ agg_sites, const int *__restrict__ face_sites,
    const double2 *__restrict__ Up, const double2 *__restrict__ Ap, const double2 *__restrict__ P, double2 *__restrict__ Dc) {
    const int wg = xcd_block(gridDim.x), a = wg / 5, t = wg % 5;
    const int n2 = 2 * N, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, s = lane >> 4;
    const size_t V = g.V;
    const int *list = agg_sites + (size_t)a * Va;
    int count = Va;
    if (t) {
        size_t o = 0;
#pragma unroll
        for (int m = 0; m < 4; m++) {
            if (m == t - 1) {
                count = Va / ag.a[m];
                list = face_sites + o + (size_t)a * count;
            }
            o += V / ag.a[m];
        }
    }
    // the last site coordinate of the aggregate in every direction
    int end[4];
    {
        int r = a;
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const int lc = g.L[m] / ag.a[m];
            end[m] = (r % lc + 1) * ag.a[m] - 1;
            r /= lc;
        }
    }
    const int j = 16 * wave + (lane & 15), jc = j < n2 ? j : n2 - 1, chi = jc >= N;
    const double sg = chi ? 1.0 : -1.0;
    v4d re[2][RT], im[2][RT];
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int rt = 0; rt < RT; rt++) re[h][rt] = im[h][rt] = (v4d){0, 0, 0, 0};
    const double2 *Pj = P + ((size_t)(jc - chi * N) * 12 + 6 * chi) * V;
    const double2 *Pk[RT];
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
        const int k = 16 * rt + (lane & 15);
        Pk[rt] = P + (size_t)(k < N ? k : N - 1) * 12 * V;
    }
    const double2 *Ab = Ap + (size_t)chi * 18 * V;
    for (int q = 0; q < count; q += 4) {
        const bool ok = q + s < count;
        const int d = list[ok ? q + s : count - 1];
        const int pos = d >> g.lgVb;
        int x[4], bc[4];
        local_coords(g, d & (g.Vb - 1), x);
        unpack_block(g.blk_coord[pos], bc);
        double2 same[6], other[6];
#pragma unroll
        for (int c = 0; c < 6; c++) same[c] = other[c] = make_double2(0, 0);
#define HOP(MU)                                                                                   \
    if (t ? t == 1 + MU : (bc[MU] << g.lb[MU]) + x[MU] != end[MU])                                \
    {                                                                                             \
        const double2 *Pn = Pj + neighbour(g, pos, x, MU, +1);                                    \
        double2 u[9];                                                                             \
        v2d psi[6];                                                                               \
        _Pragma("unroll") for (int k = 0; k < 9; k++) u[k] = Up[(size_t)(9 * MU + k) * V + d];     \
        _Pragma("unroll") for (int c = 0; c < 6; c++) psi[c] = *(const v2d *)(Pn + (size_t)c * V); \
        forward_hop<MU>(u, 1, psi, sg, 1.0, same, other);                                         \
        __builtin_amdgcn_sched_barrier(0);   /* one hop's operands in registers at a time */      \
    }
        HOP(0)
        HOP(1)
        HOP(2)
        HOP(3)
#undef HOP
        double f = ok ? -0.5 : 0.0;
#pragma unroll
        for (int c = 0; c < 6; c++) {
            same[c] = cscale(same[c], f);
            other[c] = cscale(other[c], f);
        }
        if (t == 0 && ok) {
            double2 p[18], in[6], ax[6];
#pragma unroll
            for (int e = 0; e < 18; e++) p[e] = Ab[(size_t)e * V + d];
#pragma unroll
            for (int c = 0; c < 6; c++) in[c] = Pj[(size_t)c * V + d];
            herm6_mv<double>(p, in, ax);
#pragma unroll
            for (int c = 0; c < 6; c++) same[c] = cadd(same[c], cscale(ax[c], 0.5));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int c = 0; c < 6; c++) {
                const double2 w = chi == h ? same[c] : other[c];
                double2 p[RT];
#pragma unroll
                for (int rt = 0; rt < RT; rt++) p[rt] = Pk[rt][(size_t)(6 * h + c) * V + d];
                // conj(p) w
#pragma unroll
                for (int rt = 0; rt < RT; rt++) {
                    re[h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[rt].x, w.x, re[h][rt], 0, 0, 0);
                    im[h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[rt].x, w.y, im[h][rt], 0, 0, 0);
                }
#pragma unroll
                for (int rt = 0; rt < RT; rt++) {
                    re[h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[rt].y, w.y, re[h][rt], 0, 0, 0);
                    im[h][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(-p[rt].y, w.x, im[h][rt], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (j >= n2) return;
    double2 *out = Dc + ((size_t)a * 9 + (t ? 2 * t - 1 : 0)) * n2 * n2 + (size_t)j * n2;
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int rt = 0; rt < RT; rt++)
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int k = 16 * rt + 4 * v + s;   // row of result register v in lane (jj, s)
                if (k < N) out[h * N + k] = make_double2(re[h][rt][v], im[h][rt][v]);
            }
}

// the self terms' parts added up in order: block 0 of an aggregate += blocks 2, 4, 6
__global__ __launch_bounds__(256) void dc_parts_kernel(int blk, int parts, double2 *__restrict__ Dc) {
    double2 *B = Dc + (size_t)blockIdx.x * 9 * blk;
    const int e = blockIdx.y * 256 + threadIdx.x;
    if (e >= blk) return;
    double2 v = B[e];
    for (int p = 1; p < parts; p++) v = cadd(v, B[(size_t)2 * p * blk + e]);
    B[e] = v;
}

// The other half of D_c from the forward one, and the FP32 copies: all 9
// blocks, and the compact [Vc][5] (self block and forward hops). One workgroup
// per (a, direction): the self block X + s X^H s in place (every thread holds
// its entries before any is written), a backward block from the forward one of
// the neighbour a - mu. Bound: memory, 24 B of results per entry.
constexpr int FIN_TPB = 256, FIN_PER = 64 * 64 / FIN_TPB;   // 2N <= 64
__global__ __launch_bounds__(FIN_TPB) void dc_finish_kernel(int N, const int *__restrict__ cnbr, double2 *__restrict__ Dc,
                                                            float2 *__restrict__ D32, float2 *__restrict__ H32) {
    const int a = blockIdx.x, dir = blockIdx.y, n2 = 2 * N, blk = n2 * n2;
    double2 *B = Dc + ((size_t)a * 9 + dir) * blk;
    const bool backward = dir && !(dir & 1);
    const double2 *S = backward ? Dc + ((size_t)cnbr[a * 9 + dir] * 9 + dir - 1) * blk : B;
    double2 v[FIN_PER];
#pragma unroll
    for (int q = 0; q < FIN_PER; q++) {
        const int e = q * FIN_TPB + threadIdx.x;
        if (e < blk) {
            const int col = e / n2, row = e - col * n2;
            v[q] = backward ? make_double2(0, 0) : S[e];
            if (dir == 0 || backward) {
                const double2 m = S[(size_t)row * n2 + col];
                const double sg = (row < N) == (col < N) ? 1.0 : -1.0;
                v[q].x += sg * m.x;
                v[q].y -= sg * m.y;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < FIN_PER; q++) {
        const int e = q * FIN_TPB + threadIdx.x;
        if (e < blk) {
            const float2 f = make_float2((float)v[q].x, (float)v[q].y);
            if (dir == 0 || backward) B[e] = v[q];
            D32[((size_t)a * 9 + dir) * blk + e] = f;
            if (!backward) H32[((size_t)a * 5 + (dir + 1) / 2) * blk + e] = f;
        }
    }
}

}  // namespace

int launch_coarse_build(Ctx *c) {
    Level1 &L1 = c->c;
    const Geom &g = c->g;
    AggGeom ag{};
    for (int m = 0; m < 4; m++) ag.a[m] = L1.agg[m];
    const int tiles = (2 * L1.N + 15) / 16;
    const DcSplit split = dc_split(L1.Va, L1.Vc, STEP);
    const size_t stage = (size_t)(12 * L1.N + 72) * STEP * 16, sums = (size_t)WAVES * 2 * (tiles > 2 ? 2 : 1) * 4 * 64 * 16;
    const size_t lds = stage > sums ? stage : sums;
    const bool small = L1.Va < 64 || lds > c->lds_max;
#define FORWARD(NT, RT)                                                                                     \
    dc_forward_kernel<NT, RT><<<(4 + split.parts) * L1.Vc, 64 * WAVES, lds, c->stream>>>(                            \
        g, ag, L1.N, L1.Va, split.parts, split.per, L1.agg_sites, L1.face_sites, (const double2 *)c->U64,               \
        (const double2 *)c->A64, (const double2 *)L1.P64, (double2 *)L1.Dc64)
#define SMALL(RT)                                                                                            \
    dc_forward_small_kernel<RT><<<5 * L1.Vc, 64u * (unsigned)tiles, 0, c->stream>>>(                               \
        g, ag, L1.N, L1.Va, L1.agg_sites, L1.face_sites, (const double2 *)c->U64, (const double2 *)c->A64,   \
        (const double2 *)L1.P64, (double2 *)L1.Dc64)
    if (small) {
        if (tiles <= 2) SMALL(1); else SMALL(2);
    } else if (tiles == 1) {
        FORWARD(1, 1);
    } else if (tiles == 2) {
        FORWARD(2, 1);
    } else if (tiles == 3) {
        FORWARD(3, 2);
    } else {
        FORWARD(4, 2);
    }
#undef SMALL
#undef FORWARD
    int rc = hip_check(c, hipGetLastError(), "D_c forward kernel");
    if (rc) return rc;
    if (!small && split.parts > 1) {
        const int blk = 4 * L1.N * L1.N;
        dc_parts_kernel<<<dim3(L1.Vc, (blk + 255) / 256), 256, 0, c->stream>>>(blk, split.parts, (double2 *)L1.Dc64);
        rc = hip_check(c, hipGetLastError(), "D_c parts kernel");
        if (rc) return rc;
    }
    dc_finish_kernel<<<dim3((unsigned)L1.Vc, 9), FIN_TPB, 0, c->stream>>>(L1.N, L1.cnbr, (double2 *)L1.Dc64,
                                                                        (float2 *)L1.Dc32, (float2 *)L1.Dh32);
    return hip_check(c, hipGetLastError(), "D_c finish kernel");
}

}  // namespace mgdd
