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

// v = U_mu psi for the two spins of one chirality, and its image w in the
// other chirality: (1 - gamma_mu) U psi = (v, w) or (w, v). In the chiral
// basis w = sg i sigma_mu v for the space directions (sg = +1 when psi is
// the lower chirality, -1 when it is the upper one) and w = v in time.
template <int MU> __device__ inline void other_chirality(const double2 *v, double sg, double2 *w) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const double2 a = v[c], b = v[3 + c];
        if (MU == 0) {          // (i b, i a)
            w[c] = make_double2(-sg * b.y, sg * b.x);
            w[3 + c] = make_double2(-sg * a.y, sg * a.x);
        } else if (MU == 1) {   // (b, -a)
            w[c] = make_double2(sg * b.x, sg * b.y);
            w[3 + c] = make_double2(-sg * a.x, -sg * a.y);
        } else if (MU == 2) {   // (i a, -i b)
            w[c] = make_double2(-sg * a.y, sg * a.x);
            w[3 + c] = make_double2(sg * b.y, -sg * b.x);
        } else {
            w[c] = a;
            w[3 + c] = b;
        }
    }
}

// same += v, other += w of the forward hop in direction MU of the half field
// Pj ([6][V]: one chirality of a column of P); same and other as in
// other_chirality
template <int MU>
__device__ inline void forward_hop(const Geom &g, const LinkViews<double> &U, const double2 *__restrict__ Pj,
                                   const int *x, int pos, int d, double sg, double2 *same, double2 *other) {
    const int dn = neighbour(g, pos, x, MU, +1);
    double2 u[9], psi[6], v[6], w[6];
#pragma unroll
    for (int c = 0; c < 6; c++) psi[c] = Pj[(size_t)c * g.V + dn];
    load_link<double, MU>(U, d, u);
    su3_mv<double, false>(u, psi, v);
    su3_mv<double, false>(u, psi + 3, v + 3);
    other_chirality<MU>(v, sg, w);
#pragma unroll
    for (int c = 0; c < 6; c++) {
        same[c] = cadd(same[c], v[c]);
        other[c] = cadd(other[c], w[c]);
    }
    __builtin_amdgcn_sched_barrier(0);   // one hop's operands in registers at a time
}

// One workgroup per (aggregate a, term t): t = 0 the self term X over all
// sites of a, t = 1 + mu the forward hop over the sites of its + mu face.
// Wave w owns the 16 columns j = 16 w .. 16 w + 15 of the block (j = (chi', k')).
// Lane (jj, s) = (lane % 16, lane / 16) forms D P_j at site 4 q + s of the
// list, all 12 components in registers: that is the layout of the B operand of
// a 16x16x4 FP64 MFMA (column jj, summation index s), so the product with P^H
// needs no exchange; the A operand is P_k at the same site, k = lane % 16 of a
// row tile. RT: row tiles of 16 test vectors. Rows past N, columns past 2N and
// sites past the end of the list are computed from clamped addresses; the
// latter enter as zeros, the others are not stored.
//
// Bound: the vector L1's return path (90 % busy: the lanes of a load hold 16
// columns of P, four sites each). 24^3 x 48 lattice, 3x4x4x4 aggregates, N =
// 21: 9.4 ms, the matrix cores busy for 32 % of it (0.2 TFLOP with the padding
// to 32 rows and 48 columns); 29.4 ms as one workgroup per column with the dot
// products on the vector units and sums through LDS. Two sites per lane
// (whole 128-byte lines at once) with the waves split by row chirality took
// 12.5 ms.
template <int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void dc_forward_kernel(
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
    const LinkViews<double> U(Up, V);
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
        forward_hop<MU>(g, U, Pj, x, pos, d, sg, same, other)
        HOP(0);
        HOP(1);
        HOP(2);
        HOP(3);
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
    const unsigned threads = 64u * (unsigned)((2 * L1.N + 15) / 16), nwg = 5u * (unsigned)L1.Vc;
#define FORWARD(RT)                                                                                          \
    dc_forward_kernel<RT><<<nwg, threads, 0, c->stream>>>(g, ag, L1.N, L1.Va, L1.agg_sites, L1.face_sites,  \
                                                          (const double2 *)c->U64, (const double2 *)c->A64, \
                                                          (const double2 *)L1.P64, (double2 *)L1.Dc64)
    if (L1.N <= 16) FORWARD(1);
    else FORWARD(2);
#undef FORWARD
    int rc = hip_check(c, hipGetLastError(), "D_c forward kernel");
    if (rc) return rc;
    dc_finish_kernel<<<dim3((unsigned)L1.Vc, 9), FIN_TPB, 0, c->stream>>>(L1.N, L1.cnbr, (double2 *)L1.Dc64,
                                                                        (float2 *)L1.Dc32, (float2 *)L1.Dh32);
    return hip_check(c, hipGetLastError(), "D_c finish kernel");
}

}  // namespace mgdd
