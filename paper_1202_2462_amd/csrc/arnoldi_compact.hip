// Arnoldi steps of the coarse GMRES (Section 4) on the compact FP32 D_c: per
// coarse site a the self block A(a) and the four forward hops F_mu(a), from
// which the backward hops follow (D_c is gamma5^c-hermitian, s = gamma5^c):
//   (D_c x)(a) = A(a) x(a) + sum_mu F_mu(a) x(a + mu) + sum_mu t_mu(a - mu),
//   t_mu(a) = s F_mu(a)^H s x(a).
// A step forms, where block F_mu(a) is read, both products with it: yf(a), the
// first two sums, and the four vectors t_mu(a), which the next kernel adds to
// its neighbours. So every block is read once per step; forming the backward
// hops where they are needed read each F_mu twice (90 KB instead of 67 KB per
// coarse site at N = 20, and twice the traffic from L2).
//
// Gram-Schmidt is classical with one re-orthogonalisation, coefficients and
// sums in double, every sum in a fixed order. One right-hand side or a few take
// two kernels a step (they are short, so their number counts):
//   stream: v_j = (y - V h2) / |.| at a and its forward neighbours, with h2
//           and the norm from the previous step's sums (the second pass of
//           step j - 1), then the products with the blocks of a, and the sums
//           of <v_k, D_c v_j>, taken with yf at a and with t_mu at a + mu;
//   pass:   y = yf + sum t - V h1 (in double), sums of <v_k, y> and |y|^2.
// With |y|^2 = |y - V h2|^2 + |h2|^2 for the orthonormal V no third kernel has
// to form the norm. More right-hand sides take four: v_j, the products on
// the matrix cores, the sums of <v_k, D_c v_j>, the pass.
// Both forms do the same arithmetic, operation by operation, so that a
// right-hand side gets the same bits alone and among others: a 16x16x4 FP32
// MFMA is the chain of fused multiply-adds over its four summation indices in
// ascending order (checked on the card), and the stream kernel sums in fours;
// the sums in double take the same products in the same order and partition.
#include "lanes.h"
#include "stencil.h"
#include "transfer.h"

namespace mgdd {

namespace {

constexpr int NVMAX = 16;        // basis vectors of a cycle
constexpr int STPB = 256;        // threads of the stream kernel
constexpr int PTPB = 512;        // threads of the pass kernel
constexpr int PGRID = 256;       // workgroups of a pass per right-hand side, at most

typedef float v4f __attribute__((ext_vector_type(4)));

struct Basis {
    const float2 *p[NVMAX];
};

// out[q] = sum_{g < np} part[q stride + g], q < nq <= 4 waves; one wave per q,
// q + waves, ...; read by every thread after the barrier
// U partials at a time in flight (from clamped places; 1: as they come, where
// there are few of them)
template <int WAVES, int U>
__device__ inline void sum_quantities(const double2 *__restrict__ part, size_t stride, int nq, int np, double2 *out) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double v[8];
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int q = wave + WAVES * i;
        if (U == 1 ? q < nq : i * WAVES < nq) {
            const double2 *p = part + (q < nq ? q : nq - 1) * stride;
            for (int g = lane; g < np; g += 64 * U) {
                double2 x[U];
#pragma unroll
                for (int u = 0; u < U; u++) x[u] = p[min(g + 64 * u, np - 1)];
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const bool in = g + 64 * u < np;
                    v[2 * i] += in ? x[u].x : 0.0;
                    v[2 * i + 1] += in ? x[u].y : 0.0;
                }
            }
        }
    }
    const double s = wave_sum8(v);
    const int q = wave + WAVES * (lane >> 4);
    if (!(lane & 7) && q < nq) (lane & 8 ? out[q].y : out[q].x) = s;
    __syncthreads();
}

// |y - V h2|^2 from |y|^2 (the last quantity) and h2; the multiply-adds are
// spelt out, so that every kernel that forms it gets the same bits. Where the
// Krylov space is exhausted (more steps than 2N Vc) the difference is rounding
// noise of either sign: 0 or less ends the basis, and a vector of another length
// than 1 still obeys D V = V H, so that the solution is as good as with the norm
// of the vector itself (42 000 random systems of 1 to 40 dimensions, graded,
// near singular and with invariant subspaces among them: the residuals agree to
// 3e-7 of themselves).
__device__ inline double rest_norm(const double2 *coef, int nk) {
    double nn = coef[nk].x;
#pragma unroll 1
    for (int k = 0; k < nk; k++) nn = fma(-coef[k].y, coef[k].y, fma(-coef[k].x, coef[k].x, nn));
    return nn;
}

// acc += conj(v) u of two entries
__device__ inline void add_products(double2 &acc, v4f v, v4f u) {
    cfmac(acc, make_double2((double)v[0], (double)v[1]), make_double2((double)u[0], (double)u[1]));
    cfmac(acc, make_double2((double)v[2], (double)v[3]), make_double2((double)u[2], (double)u[3]));
}

// Both products sum in batches of four: a batch of the row sums is four
// consecutive columns of one block (the blocks' batches form one list of 5 nb4,
// nb4 = ceil(n2 / 4)), CHAIN consecutive batches are added up, then these in
// four interleaved sums; a batch of the column sums is four rows, added in
// order.
__host__ __device__ inline int row_groups(int n2) { return (n2 + 3) >> 2; }
__host__ __device__ inline int chain_length(int n2) {
    const int nb4 = row_groups(n2), groups = STPB / nb4;
    return (5 * nb4 + groups - 1) / groups;
}

// ---------------------------------------------------------------- one right-hand side or a few
//
// One workgroup per coarse site and right-hand side, the G workgroups of a
// right-hand side taking the sites in turn. Thread (cg, rg) takes the rows
// 4 rg .. 4 rg + 3 of chain cg of the column batches of the site's 5 blocks
// (column-major): a column of 4 rows is 32 contiguous bytes, read once and used
// for both products; the row sums are added over cg, the column sums over rg,
// through LDS. hin: h2 and the squared norm of the previous step ([j + 1][nb][nin]
// partials, the norm last; for j = 0 only the norm of w).
// Bound: reading the blocks (524 MB at 8^3 x 16 coarse sites, N = 20, 103 us at
// the 5.1 TB/s of a large copy): 126 us there, and 10 to 20 us the pass, where
// forming each site's backward hops from its neighbours' blocks took 168 us,
// two passes of 15 us and two sums of 11 us. At 4^3 x 8 sites the chain of
// loads and sums decides: 11.7 and 5 to 7 us (6 to 11 with one partial sum at a
// time in flight) against 11.8, 7.9 and 7.9.
__global__ __launch_bounds__(STPB) __attribute__((amdgpu_waves_per_eu(3))) void arnoldi_stream_kernel(
    int Vc, int N, int nb, const int *__restrict__ cnbr, const float2 *__restrict__ H, const float2 *__restrict__ w,
    const double2 *__restrict__ hin, int nin, Basis V, int j, float2 *__restrict__ vj, float2 *__restrict__ yf,
    float2 *__restrict__ t, double2 *__restrict__ part, double2 *__restrict__ h2, double2 *__restrict__ nr) {
    extern __shared__ float2 sm[];
    __shared__ double2 coef[NVMAX];
    const int n2 = 2 * N, n5 = 5 * n2, NR = row_groups(n2), NBT = 5 * NR, M = chain_length(n2), tid = threadIdx.x;
    const int CG = (NBT + M - 1) / M;       // chains
    float2 *vs = sm;                        // [j + 1][5 n2]: v_k at a and its forward neighbours
    float2 *us = vs + (size_t)(j + 1) * n5; // [5 n2]: yf(a) and t_mu(a)
    float2 *yp = us + n5;                   // [CG][n2]
    float2 *tp = yp + CG * n2;              // [4 n2][NR]
    const int cg = tid / NR, rg = tid - cg * NR, row = 4 * rg;
    const bool active = cg < CG;
    const size_t blk = (size_t)n2 * n2;
    // workgroup g of G and right-hand side sg: the right-hand sides of a g one
    // after the other on its XCD
    const int G = gridDim.x / nb, full = G & ~7;
    int g = blockIdx.x, sg = 0;
    if (nb > 1) {
        const int r = blockIdx.x - full * nb;
        g = r < 0 ? (int)(blockIdx.x / 8 / nb) * 8 + (int)(blockIdx.x & 7) : full + r / nb;
        sg = r < 0 ? (int)(blockIdx.x / 8 % nb) : r % nb;
    }
    const size_t so = (size_t)sg * Vc * n2;
    w += so;
    vj += so;
    yf += so;
    t += 4 * so;
    // the four columns of batch m (4 rows each) through a buffer resource over
    // the site's blocks: past the end reads as 0 (rows past n2 and columns past
    // a block, where n2 is no multiple of 4, are others that the sums below
    // leave out)
    auto columns = [&](int a, int m, v4f (&f)[4][2]) {
        const rsrc_t B = make_rsrc(H + (size_t)a * 5 * blk, 5 * blk * 8);
        const int b = m / NR;
        const unsigned vo = (unsigned)((b * n2 + 4 * (m - b * NR)) * n2 + row) * 8u;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const unsigned so = (unsigned)(q * n2) * 8u;
            f[q][0] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(B, vo, so, 0));
            f[q][1] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(B, vo + 16u, so, 0));
        }
    };
    // in flight while the sums are taken and v_j is formed
    v4f f[4][2];
    columns(__builtin_amdgcn_readfirstlane(xcd_remap(g, Vc)), cg * M, f);
    const int wave = tid >> 6, lane = tid & 63;
    double sc = 0;
    double2 acc[4];
#pragma unroll
    for (int i = 0; i < 4; i++) acc[i] = make_double2(0, 0);
    for (int l = g; l < Vc; l += G) {
        const int a = __builtin_amdgcn_readfirstlane(xcd_remap(l, Vc));
        // the vectors at a and its forward neighbours (5 n2 <= 320 entries), loaded
        // before the coefficients are summed for the first site
        float2 wv[2];
        size_t at[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int e = tid + u * STPB, dd = e / n2, i = e - dd * n2;
            if (e < n5) {
                at[u] = (size_t)cnbr[a * 9 + (dd ? 2 * dd - 1 : 0)] * n2 + i;
                wv[u] = w[at[u]];
#pragma unroll 4
                for (int k = 0; k < j; k++) vs[k * n5 + e] = V.p[k][so + at[u]];
            }
        }
        if (l == g) {
            sum_quantities<STPB / 64, 1>(hin + (size_t)sg * nin, (size_t)nb * nin, j + 1, nin, coef);
            const double nn = rest_norm(coef, j);
            sc = nn > 0 ? 1.0 / sqrt(nn) : 0.0;
            if (g == 0) {
                if (tid == 0) nr[sg] = make_double2(nn, 0);
                if (tid < j) h2[(size_t)tid * nb + sg] = coef[tid];
            }
        }
#pragma unroll
        for (int u = 0; u < 2; u++) {
            const int e = tid + u * STPB;
            if (e < n5) {
                double2 r = make_double2((double)wv[u].x, (double)wv[u].y);
#pragma unroll 4
                for (int k = 0; k < j; k++) {
                    const float2 v = vs[k * n5 + e];
                    cfma(r, cneg(coef[k]), make_double2((double)v.x, (double)v.y));
                }
                const float2 v = make_float2((float)(r.x * sc), (float)(r.y * sc));
                vs[j * n5 + e] = v;
                if (e < n2) vj[at[u]] = v;
            }
        }
        __syncthreads();
        const float2 *x = vs + j * n5;
        if (active) {
            float2 y4[4], x4[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                y4[r] = make_float2(0.f, 0.f);
                x4[r] = row + r < n2 ? x[row + r] : make_float2(0.f, 0.f);
                if (row + r >= N) x4[r] = cneg(x4[r]);
            }
            for (int i = 0; i < M; i++) {
                const int m = cg * M + i;
                if (m >= NBT) break;
                if (i) columns(a, m, f);
                const int b = m / NR, c0 = 4 * (m - b * NR);   // first column of the batch in block b
                float2 xc[4];
#pragma unroll
                for (int q = 0; q < 4; q++) xc[q] = c0 + q < n2 ? x[b * n2 + c0 + q] : make_float2(0.f, 0.f);
                // F(row + r, c0 + q)
                auto F = [&](int q, int r) { return make_float2(f[q][r >> 1][2 * (r & 1)], f[q][r >> 1][2 * (r & 1) + 1]); };
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    float2 z = make_float2(0.f, 0.f);
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        z.x = fmaf(F(q, r).x, xc[q].x, z.x);
                        z.y = fmaf(F(q, r).x, xc[q].y, z.y);
                    }
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        z.x = fmaf(-F(q, r).y, xc[q].y, z.x);
                        z.y = fmaf(F(q, r).y, xc[q].x, z.y);
                    }
                    y4[r] = cadd(y4[r], z);
                }
                if (b)
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        float2 z = make_float2(0.f, 0.f);
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            z.x = fmaf(F(q, r).x, x4[r].x, z.x);
                            z.y = fmaf(F(q, r).x, x4[r].y, z.y);
                        }
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            z.x = fmaf(F(q, r).y, x4[r].y, z.x);
                            z.y = fmaf(-F(q, r).y, x4[r].x, z.y);
                        }
                        if (c0 + q < n2) tp[((b - 1) * n2 + c0 + q) * NR + rg] = z;
                    }
            }
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (row + r < n2) yp[cg * n2 + row + r] = y4[r];
        }
        if (l + G < Vc)   // the next site's
            columns(__builtin_amdgcn_readfirstlane(xcd_remap(l + G, Vc)), cg * M, f);
        __syncthreads();
        // four lanes a row of yf, one thread an entry of t (4 n2 <= 256 of each)
        if (tid < 4 * n2) {
            const int e = tid >> 2;
            float2 s = make_float2(0.f, 0.f), u = s;
#pragma unroll 4
            for (int q = tid & 3; q < CG; q += 4) s = cadd(s, yp[q * n2 + e]);
            s.x += dpp_mov<0xB1>(s.x);
            s.y += dpp_mov<0xB1>(s.y);
            s.x += dpp_mov<0x4E>(s.x);
            s.y += dpp_mov<0x4E>(s.y);
            if (!(tid & 3)) {
                yf[(size_t)a * n2 + e] = s;
                us[e] = s;
            }
#pragma unroll 4
            for (int q = 0; q < NR; q++) u = cadd(u, tp[tid * NR + q]);
            if (tid % n2 >= N) u = cneg(u);
            t[(size_t)a * 4 * n2 + tid] = u;
            us[n2 + tid] = u;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int k = wave + 4 * i;
            if (k <= j)
#pragma unroll 2
                for (int e = 2 * lane; e < n5; e += 128) {
                    const v4f v = *(const v4f *)(vs + k * n5 + e), u = *(const v4f *)(us + e);
                    add_products(acc[i], v, u);
                }
        }
        __syncthreads();
    }
    const double v[8] = {acc[0].x, acc[0].y, acc[1].x, acc[1].y, acc[2].x, acc[2].y, acc[3].x, acc[3].y};
    const double s = wave_sum8(v);
    const int k = wave + 4 * (lane >> 4);
    if (!(lane & 7) && k <= j) {
        double *o = (double *)(part + ((size_t)k * nb + sg) * G + g);
        o[(lane >> 3) & 1] = s;
    }
}

// ---------------------------------------------------------------- several right-hand sides
//
// The same products on the matrix cores (16x16x4 FP32 MFMA, complex products as
// four real ones), one workgroup per (coarse site, 16 right-hand sides): the
// blocks pass through LDS one after the other (the next one's loads in
// flight; one buffer, so that three workgroups share a CU), where wave w < nt
// reads the rows of tile w for yf and wave nt + w the columns of tile w for
// t_mu. Operand layouts as in the coarse apply: A [i][k] in lane i + 16 k,
// B[k][j] in lane j + 16 k, result register v of lane l holds row 4 (l / 16) +
// v of column l % 16. One MFMA is one batch of the stream kernel's sums.
// Bound: the latency of each block's way through LDS (matrix cores 26 %, vector
// units 28 % busy). 6^3 x 12 coarse sites, N = 24, 12 right-hand sides: 161 us,
// and 46 to 181 us the other three kernels; reading the blocks once per
// right-hand side took 725 us and two passes of 92 us.
__device__ inline v4f mma(float a, float b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// LDS row lengths in complex numbers: 2 more than a multiple of 16, so that
// 16 rows of 4 consecutive entries spread over the banks evenly
__host__ __device__ inline int mfma_ldx(int n2) { return (5 * n2 + 15) / 16 * 16 + 2; }
__host__ __device__ inline int mfma_ldb(int n2) { return (n2 + 15) / 16 * 16 + 2; }

__global__ __launch_bounds__(512) void arnoldi_mfma_kernel(int Vc, int N, int nb, const int *__restrict__ cnbr,
                                                           const float2 *__restrict__ H, const float2 *__restrict__ vj,
                                                           float2 *__restrict__ yf, float2 *__restrict__ t) {
    extern __shared__ float2 sm[];
    const int n2 = 2 * N, nt = (n2 + 15) >> 4, LX = mfma_ldx(n2), LB = mfma_ldb(n2), M = chain_length(n2);
    float2 *X = sm;                          // [16 rhs][LX]: v at a and its forward neighbours
    float2 *buf = X + 16 * LX;               // the block at hand, [n2 columns][LB]
    const int a = xcd_block(gridDim.x), r0 = blockIdx.y * 16, tid = threadIdx.x, T = blockDim.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lo = lane & 15, hi = lane >> 4;
    const size_t blk = (size_t)n2 * n2;
    const v4f *B = (const v4f *)(H + (size_t)a * 5 * blk);
    const int npair = n2 * n2 / 2, half = n2 >> 1;
    v4f f[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int p = tid + q * T;
        f[q] = B[p < npair ? p : npair - 1];
    }
    // one wave per vector (n2 <= 64), eight in flight
    const int nw = T >> 6, li = lane < n2 ? lane : n2 - 1;
    for (int p0 = wave; p0 < 80; p0 += 8 * nw) {
        float2 v[8];
        int at[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int p = p0 + u * nw < 80 ? p0 + u * nw : 79, r = p / 5, dd = p - 5 * r;
            at[u] = cnbr[a * 9 + (dd ? 2 * dd - 1 : 0)];
        }
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int p = p0 + u * nw < 80 ? p0 + u * nw : 79, r = r0 + p / 5;
            v[u] = vj[((size_t)(r < nb ? r : nb - 1) * Vc + at[u]) * n2 + li];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int p = p0 + u * nw, r = p / 5, dd = p - 5 * r;
            if (p < 80 && lane < n2) X[r * LX + dd * n2 + lane] = r0 + r < nb ? v[u] : make_float2(0.f, 0.f);
        }
    }
    const v4f zero = {0, 0, 0, 0};
    // row sums: the current chain, and four interleaved sums of chains
    v4f cre = zero, cim = zero, sre[4], sim[4];
#pragma unroll
    for (int q = 0; q < 4; q++) sre[q] = sim[q] = zero;
    int left = M, chain = 0;
    auto end_chain = [&]() {
#pragma unroll
        for (int q = 0; q < 4; q++)
            if ((chain & 3) == q) {
                sre[q] += cre;
                sim[q] += cim;
            }
        cre = cim = zero;
        left = M;
        chain++;
    };
    const bool forward = wave < nt, rhs_ok = r0 + lo < nb;
    const int tile = (forward ? wave : wave - nt) * 16, rc = tile + lo < n2 ? tile + lo : n2 - 1;
    const float2 *Xr = X + lo * LX;
    for (int b = 0; b < 5; b++) {
        if (b) __syncthreads();   // the previous block has been read
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int p = tid + q * T;
            if (p < npair) {
                const int col = p / half, r2 = p - col * half;
                *(v4f *)(buf + col * LB + 2 * r2) = f[q];
            }
        }
        if (b < 4) {
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int p = tid + q * T;
                f[q] = B[(size_t)(b + 1) * npair + (p < npair ? p : npair - 1)];
            }
        }
        __syncthreads();
        // entry k of the batch from k0 on: A the block's, x the vector's, 0 past n2
        if (forward) {
            auto load = [&](int k0, float2 &A, float2 &x) {
                const int k = k0 + hi, kc = k < n2 ? k : n2 - 1;
                A = buf[kc * LB + rc];
                x = Xr[b * n2 + kc];
                if (k >= n2) x = make_float2(0.f, 0.f);
            };
            float2 A, x, An, xn;
            load(0, A, x);
            for (int k0 = 0; k0 < n2; k0 += 4) {
                load(k0 + 4 < n2 ? k0 + 4 : 0, An, xn);
                v4f re = mma(A.x, x.x, zero), im = mma(A.x, x.y, zero);
                re = mma(-A.y, x.y, re);
                im = mma(A.y, x.x, im);
                cre += re;
                cim += im;
                if (!--left) end_chain();
                A = An;
                x = xn;
            }
        } else if (b > 0) {
            auto load = [&](int i0, float2 &A, float2 &x) {
                const int i = i0 + hi, ic = i < n2 ? i : n2 - 1;
                A = buf[rc * LB + ic];
                x = Xr[ic];
                if (i >= N) x = cneg(x);
                if (i >= n2) x = make_float2(0.f, 0.f);
            };
            v4f ure = zero, uim = zero;
            float2 A, x, An, xn;
            load(0, A, x);
            for (int i0 = 0; i0 < n2; i0 += 4) {
                load(i0 + 4 < n2 ? i0 + 4 : 0, An, xn);
                v4f re = mma(A.x, x.x, zero), im = mma(A.x, x.y, zero);
                re = mma(A.y, x.y, re);
                im = mma(-A.y, x.x, im);
                ure += re;
                uim += im;
                A = An;
                x = xn;
            }
            if (rhs_ok) {
                float2 *o = t + (((size_t)(r0 + lo) * Vc + a) * 4 + b - 1) * n2;
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int c = tile + 4 * hi + v;
                    if (c < n2) o[c] = c < N ? make_float2(ure[v], uim[v]) : make_float2(-ure[v], -uim[v]);
                }
            }
        }
    }
    if (forward && rhs_ok) {
        if (left < M) end_chain();
        const v4f re = (sre[0] + sre[1]) + (sre[2] + sre[3]), im = (sim[0] + sim[1]) + (sim[2] + sim[3]);
        float2 *o = yf + ((size_t)(r0 + lo) * Vc + a) * n2;
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int i = tile + 4 * hi + v;
            if (i < n2) o[i] = make_float2(re[v], im[v]);
        }
    }
}

// v_j = (y - V h2) / |.| for several right-hand sides, as the stream kernel
// forms it; stores h2[k nb + segment] and the squared norm
template <int NV>
__global__ __launch_bounds__(PTPB) void arnoldi_vector_kernel(int n, Basis V, int nk, const double2 *__restrict__ pin,
                                                              int npin, const float2 *__restrict__ w,
                                                              float2 *__restrict__ vj, double2 *__restrict__ h2,
                                                              double2 *__restrict__ nr) {
    const int sg = blockIdx.y, nb = gridDim.y, G = gridDim.x, g = blockIdx.x;
    const size_t so = (size_t)sg * n;
    __shared__ double2 coef[NVMAX];
    v4f v[NV], yv;
    auto load = [&](int e) {
        yv = *(const v4f *)(w + so + e);
#pragma unroll
        for (int k = 0; k < NV; k++) v[k] = k < nk ? *(const v4f *)(V.p[k] + so + e) : (v4f){0, 0, 0, 0};
    };
    int e = (g * PTPB + (int)threadIdx.x) * 2;
    if (e < n) load(e);
    sum_quantities<PTPB / 64, 8>(pin + (size_t)sg * npin, (size_t)nb * npin, nk + 1, npin, coef);
    const double nn = rest_norm(coef, nk), sc = nn > 0 ? 1.0 / sqrt(nn) : 0.0;
    if (g == 0) {
        if (threadIdx.x == 0) nr[sg] = make_double2(nn, 0);
        if ((int)threadIdx.x < nk) h2[(size_t)threadIdx.x * nb + sg] = coef[threadIdx.x];
    }
    for (; e < n; e += G * PTPB * 2) {
        double2 r0 = make_double2((double)yv[0], (double)yv[1]), r1 = make_double2((double)yv[2], (double)yv[3]);
#pragma unroll
        for (int k = 0; k < NV; k++)
            if (k < nk) {
                const double2 h = cneg(coef[k]);
                cfma(r0, h, make_double2((double)v[k][0], (double)v[k][1]));
                cfma(r1, h, make_double2((double)v[k][2], (double)v[k][3]));
            }
        *(v4f *)(vj + so + e) = (v4f){(float)(r0.x * sc), (float)(r0.y * sc), (float)(r1.x * sc), (float)(r1.y * sc)};
        if (e + G * PTPB * 2 < n) load(e + G * PTPB * 2);
    }
}

// The sums of <v_k, D_c v_j>, k <= j, for several right-hand sides, from yf and t:
// the products, the workgroups' sites and the order of the stream kernel, so
// that both give the same bits. A lane holds Q pairs of a site's 5 n2 entries
// (128 (Q - 1) < 5 n2 <= 128 Q) for K basis vectors, the next site's in flight.
// part: [k][segment][workgroup]. Grid (G, nb, ceil((j + 1) / 4 K)), G as the
// stream kernel's. Bound: vector instructions (busy for 68 %: every entry of the
// basis is widened and used five times, at its site and from its four backward
// neighbours). 12 right-hand sides, steps 1 to 12, 6^3 x 12 coarse sites,
// N = 24: 16 to 83 us (K = 1: 15 to 85, 4: 20 to 75), 8^3 x 16, N = 20: 39 to
// 269. Sums of <v_k, yf + sum t>, which read the basis once but in another order,
// took 13 to 39 and 31 to 98 us.
template <int Q, int K>
__global__ __launch_bounds__(STPB) void arnoldi_dots_kernel(int Vc, int n2, const int *__restrict__ cnbr, Basis V, int j,
                                                            const float2 *__restrict__ yf, const float2 *__restrict__ t,
                                                            double2 *__restrict__ part) {
    const int k0 = 4 * K * blockIdx.z + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (k0 > j) return;
    const int sg = blockIdx.y, nb = gridDim.y, n5 = 5 * n2;
    const size_t so = (size_t)sg * Vc * n2;
    const float2 *vk[K];
#pragma unroll
    for (int i = 0; i < K; i++) vk[i] = V.p[k0 + 4 * i <= j ? k0 + 4 * i : j] + so;
    // the lane's entries of a site: past the end the last ones, as 0
    int dir[Q], in[Q], ent[Q];
#pragma unroll
    for (int q = 0; q < Q; q++) {
        const int e = 2 * lane + 128 * q < n5 ? 2 * lane + 128 * q : n5 - 2, dd = e / n2;
        dir[q] = dd ? 2 * dd - 1 : 0;
        in[q] = e - dd * n2;
        ent[q] = e - n2;   // of t, or below 0 of yf
    }
    int at[Q];
    v4f u[Q];
    auto fetch = [&](int l) {
        const int a = __builtin_amdgcn_readfirstlane(xcd_remap(l, Vc));
        const float2 *ys = yf + so + (size_t)a * n2 + n2, *ts = t + 4 * (so + (size_t)a * n2);
#pragma unroll
        for (int q = 0; q < Q; q++) at[q] = cnbr[a * 9 + dir[q]];
#pragma unroll
        for (int q = 0; q < Q; q++) u[q] = *(const v4f *)((ent[q] < 0 ? ys : ts) + ent[q]);
    };
    fetch(blockIdx.x);
    double2 acc[K];
#pragma unroll
    for (int i = 0; i < K; i++) acc[i] = make_double2(0, 0);
    for (int l = blockIdx.x; l < Vc; l += gridDim.x) {
        v4f v[K][Q], x[Q];
#pragma unroll
        for (int q = 0; q < Q; q++)
#pragma unroll
            for (int i = 0; i < K; i++) v[i][q] = *(const v4f *)(vk[i] + (size_t)at[q] * n2 + in[q]);
#pragma unroll
        for (int q = 0; q < Q; q++) x[q] = 2 * lane + 128 * q < n5 ? u[q] : (v4f){0, 0, 0, 0};
        __builtin_amdgcn_sched_barrier(0);
        fetch(l + (int)gridDim.x < Vc ? l + (int)gridDim.x : l);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < Q; q++)
#pragma unroll
            for (int i = 0; i < K; i++) add_products(acc[i], v[i][q], x[q]);
    }
#pragma unroll
    for (int i = 0; i < K; i++) {
        const int k = k0 + 4 * i;
        const double re = wave_sum1(acc[i].x), im = wave_sum1(acc[i].y);
        if (lane == 0 && k <= j) part[((size_t)k * nb + sg) * gridDim.x + blockIdx.x] = make_double2(re, im);
    }
}

// ---------------------------------------------------------------- the pass over the basis
//
// z = yf + sum_mu t_mu(a - mu) in double - sum_{k < nk} coef_k v_k, coef
// summed from pin (npin partials each), stored in y = yf, in FP32, and coef by
// workgroup 0 in hout[k nb + segment]; then the sums of <v_k, z> (k < nk) and of
// |z|^2 (as quantity nk) of each workgroup into pout
// [quantity][segment][workgroup]. Grid (G, nb).
template <int NV>
__global__ __launch_bounds__(PTPB) void arnoldi_pass_kernel(int Vc, int n2, const int *__restrict__ cnbr, Basis V,
                                                            int nk, const double2 *__restrict__ pin, int npin,
                                                            float2 *__restrict__ y, const float2 *__restrict__ t,
                                                            double2 *__restrict__ pout, double2 *__restrict__ hout) {
    constexpr int NQ = 2 * NV + 8;   // sums: re, im of every product, then the norm
    const int sg = blockIdx.y, nb = gridDim.y, G = gridDim.x, g = blockIdx.x, n = Vc * n2;
    const size_t so = (size_t)sg * n;
    __shared__ double2 coef[NVMAX];
    __shared__ double red[PTPB / 64][NQ];
    // two elements (n2 is even: of one site); the first pair is loaded while the
    // coefficients are summed
    v4f v[NV], yv, tv[4];
    auto load = [&](int e) {
        yv = *(const v4f *)(y + so + e);
#pragma unroll
        for (int k = 0; k < NV; k++) v[k] = k < nk ? *(const v4f *)(V.p[k] + so + e) : (v4f){0, 0, 0, 0};
        const int a = e / n2, i = e - a * n2;
        const float2 *ts = t + 4 * so + i;
#pragma unroll
        for (int mu = 0; mu < 4; mu++) tv[mu] = *(const v4f *)(ts + (size_t)(cnbr[a * 9 + 2 + 2 * mu] * 4 + mu) * n2);
    };
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; q++) acc[q] = 0;
    int e = (g * PTPB + (int)threadIdx.x) * 2;
    if (e < n) load(e);
    sum_quantities<PTPB / 64, 8>(pin + (size_t)sg * npin, (size_t)nb * npin, nk, npin, coef);
    if (g == 0 && (int)threadIdx.x < nk) hout[(size_t)threadIdx.x * nb + sg] = coef[threadIdx.x];
    for (; e < n; e += G * PTPB * 2) {
        double2 y0 = make_double2((double)yv[0], (double)yv[1]), y1 = make_double2((double)yv[2], (double)yv[3]);
#pragma unroll
        for (int mu = 0; mu < 4; mu++) {
            y0 = cadd(y0, make_double2((double)tv[mu][0], (double)tv[mu][1]));
            y1 = cadd(y1, make_double2((double)tv[mu][2], (double)tv[mu][3]));
        }
#pragma unroll
        for (int k = 0; k < NV; k++)
            if (k < nk) {
                const double2 h = cneg(coef[k]);
                cfma(y0, h, make_double2((double)v[k][0], (double)v[k][1]));
                cfma(y1, h, make_double2((double)v[k][2], (double)v[k][3]));
            }
        yv = (v4f){(float)y0.x, (float)y0.y, (float)y1.x, (float)y1.y};
        *(v4f *)(y + so + e) = yv;
        y0 = make_double2((double)yv[0], (double)yv[1]);
        y1 = make_double2((double)yv[2], (double)yv[3]);
        // the products below widen v again: kept in double it would not fit the registers
#pragma unroll
        for (int k = 0; k < NV; k++) asm volatile("" : "+v"(v[k]));
#pragma unroll
        for (int k = 0; k < NV; k++)
            if (k < nk) {
                double2 d = make_double2(acc[2 * k], acc[2 * k + 1]);
                cfmac(d, make_double2((double)v[k][0], (double)v[k][1]), y0);
                cfmac(d, make_double2((double)v[k][2], (double)v[k][3]), y1);
                acc[2 * k] = d.x;
                acc[2 * k + 1] = d.y;
            }
        acc[2 * NV] += (y0.x * y0.x + y0.y * y0.y) + (y1.x * y1.x + y1.y * y1.y);
        if (e + G * PTPB * 2 < n) load(e + G * PTPB * 2);
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < NQ; q += 8)
        if (q == 2 * NV || q < 2 * nk) {
            const double s = wave_sum8(acc + q);
            if (!(lane & 7)) red[wave][q + (lane >> 3)] = s;
        }
    __syncthreads();
    if ((int)threadIdx.x <= nk) {
        const int q = threadIdx.x;
        const bool norm = q == nk;
        double re = 0, im = 0;
        for (int u = 0; u < PTPB / 64; u++) {
            re += red[u][norm ? 2 * NV : 2 * q];
            im += norm ? 0.0 : red[u][2 * q + 1];
        }
        pout[((size_t)q * nb + sg) * G + g] = make_double2(re, im);
    }
}

// partial sums of |x|^2: pout[segment * G + g]
__global__ __launch_bounds__(PTPB) void arnoldi_norm_kernel(int n, const float2 *__restrict__ x,
                                                            double2 *__restrict__ pout) {
    __shared__ double red[PTPB / 64];
    double s = 0;
    for (int e = blockIdx.x * PTPB + threadIdx.x; e < n; e += gridDim.x * PTPB) {
        const float2 v = x[(size_t)blockIdx.y * n + e];
        s += (double)v.x * v.x + (double)v.y * v.y;
    }
    s = wave_sum1(s);
    if (!(threadIdx.x & 63)) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        s = 0;
        for (int u = 0; u < PTPB / 64; u++) s += red[u];
        pout[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = make_double2(s, 0);
    }
}

// the end of a cycle: nk coefficients of the last second pass and the squared
// norm of the last vector, per segment
__global__ __launch_bounds__(256) void arnoldi_last_kernel(int nk, const double2 *__restrict__ pin, int npin,
                                                           double2 *__restrict__ h2, double2 *__restrict__ nr) {
    __shared__ double2 coef[NVMAX];
    const int sg = blockIdx.x, nb = gridDim.x;
    sum_quantities<4, 8>(pin + (size_t)sg * npin, (size_t)nb * npin, nk + 1, npin, coef);
    if ((int)threadIdx.x < nk) h2[(size_t)threadIdx.x * nb + sg] = coef[threadIdx.x];
    if (threadIdx.x == 0) nr[sg] = make_double2(rest_norm(coef, nk), 0);
}

int pass_grid(size_t n) {
    const size_t g = (n / 2 + PTPB - 1) / PTPB;
    return (int)(g < 1 ? 1 : g > PGRID ? PGRID : g);
}

// the most workgroups of a stream kernel
int stream_most(int Vc) { return Vc < 768 ? Vc : 768; }

size_t stream_lds(int n2, int j) {
    const int NR = row_groups(n2), M = chain_length(n2), CG = (5 * NR + M - 1) / M;
    return 8 * ((size_t)(j + 2) * 5 * n2 + (size_t)CG * n2 + (size_t)4 * n2 * NR);
}

// workgroups of the stream kernel: as many as the LDS lets run at once on the
// 256 CUs, at most 3 per CU (each then takes the same number of sites, and
// the number of partial sums stays small), at most one per site
int stream_grid(int Vc, int n2, int j) {
    const int per = (int)((size_t)160 * 1024 / (stream_lds(n2, j) + 1024));
    const int g = 256 * (per < 1 ? 1 : per > 3 ? 3 : per);
    return Vc < g ? Vc : g;
}

// The stream kernel, each right-hand side reading the blocks, or the matrix
// cores, one read for all of them? The stream takes its time per right-hand
// side, the matrix cores nearly the same for 2 as for 12. 12 steps, stream /
// matrix cores: 2 right-hand sides, 4^3 x 8 coarse sites, N = 20: 373 / 578 us,
// 8^3 x 16: 2.50 / 5.76 ms. They meet between 6 and 7 for three tiles of 16 rows
// (N = 17 .. 24; 8^3 x 16, 6: 6.42 / 6.72 ms, 7: 7.48 / 7.01; 6^3 x 12, N = 24, 6:
// 2.52 / 2.64, 7: 2.91 / 2.76), else between 3 and 4 (8^4, N = 12, 3: 1.26 / 1.41 ms, 4: 1.58 / 1.46; N = 30, 3.69 /
// 3.84, 4.67 / 4.07) and, for the fewest and most vectors, 2 and 3 (N = 8, 2: 0.80
// / 0.88, 3: 1.11 / 0.92; N = 32, 3.17 / 3.79, 4.34 / 3.99). Few sites leave the
// chip idle and the number of kernels decides (2 per step and 4): 128 sites, N =
// 20, 12 right-hand sides: 405 / 501 us; 256, N = 28, 6: 547 / 556, 7: 649 / 567.
bool stream_rhs(int Vc, int n2, int nb) {
    const int tiles = (n2 + 15) / 16, most = tiles == 3 ? 6 : n2 < 24 || n2 > 60 ? 2 : 3;
    return nb <= most || (size_t)Vc * nb <= 1536;
}

}  // namespace

size_t compact_arnoldi_scratch(const StencilOp &op, int m, int nb) {
    const size_t n = (size_t)op.V * 2 * op.N;
    // t, the sums of the products and those of the pass
    return 4 * n * nb * 8 + (size_t)(m + 2) * nb * (stream_most(op.V) + pass_grid(n)) * 16 + 1024;
}

int launch_compact_arnoldi(Ctx *c, const StencilOp &op, int m, int nb, const void *b, void *const *V, void *work0,
                           void *work1, void *scratch, double2 *H1, double2 *H2, double2 *NR) {
    const int Vc = op.V, N = op.N, n2 = 2 * N;
    const size_t n = (size_t)Vc * n2;
    const int G = pass_grid(n);
    if (m + 1 > NVMAX) return fail(c, MGDD_EINVAL, "too many coarse GMRES steps for the fused Arnoldi kernels");
    float2 *t = (float2 *)scratch;
    double2 *part1 = (double2 *)(((uintptr_t)(t + 4 * n * nb) + 255) & ~(uintptr_t)255);
    double2 *part3 = part1 + (size_t)(m + 2) * nb * stream_most(Vc);
    const dim3 grid(G, nb);
    const float2 *H = (const float2 *)op.H32;
    void *work[2] = {work0, work1};
    const void *w = b;
    arnoldi_norm_kernel<<<grid, PTPB, 0, c->stream>>>((int)n, (const float2 *)b, part3);
#define PASS(NV) arnoldi_pass_kernel<NV><<<grid, PTPB, 0, c->stream>>>(Vc, n2, op.nbr, vl, j + 1, part1, gs, y, t, part3, h1)
    const bool stream = stream_rhs(Vc, n2, nb);
    int rc = MGDD_OK;
    for (int j = 0; j < m && !rc; j++) {
        Basis vl{};
        for (int k = 0; k <= j; k++) vl.p[k] = (const float2 *)V[k];
        float2 *y = (float2 *)work[j & 1], *vj = (float2 *)V[j];
        double2 *h1 = H1 + (size_t)j * (m + 1) * nb;
        // algorithmic bytes: the 5 blocks of every coarse site once per launch, per
        // right-hand side w read, y and v_j written and the j earlier basis vectors read
        const double abytes = (double)Vc * (5.0 * n2 * n2 * 8 + nb * (3.0 + j) * n2 * 8);
        double2 *h2p = H2 + (size_t)(j ? j - 1 : 0) * (m + 1) * nb, *nrj = NR + (size_t)j * nb;
        const int gs = stream_grid(Vc, n2, j);
        int slot;
        if (stream) {
            slot = kt_begin(c);
            arnoldi_stream_kernel<<<gs * nb, STPB, stream_lds(n2, j), c->stream>>>(
                Vc, N, nb, op.nbr, H, (const float2 *)w, part3, G, vl, j, vj, y, t, part1, h2p, nrj);
            kt_end(c, slot, KF_COARSE, MGDD_F32, (double)Vc * nb, abytes);
        } else {
#define VECTOR(NV)                                                                                                    \
    arnoldi_vector_kernel<NV><<<grid, PTPB, 0, c->stream>>>((int)n, vl, j, part3, G, (const float2 *)w, vj, h2p, nrj)
            if (j <= 4) VECTOR(4);
            else if (j <= 8) VECTOR(8);
            else VECTOR(16);
#undef VECTOR
            const size_t lds = 8 * ((size_t)16 * mfma_ldx(n2) + (size_t)n2 * mfma_ldb(n2));
            slot = kt_begin(c);
            arnoldi_mfma_kernel<<<dim3(Vc, (nb + 15) / 16), 128 * ((n2 + 15) / 16), lds, c->stream>>>(Vc, N, nb, op.nbr,
                                                                                                    H, vj, y, t);
            kt_end(c, slot, KF_COARSE, MGDD_F32, (double)Vc * nb, abytes);
#define DOTS(Q)                                                                                                  \
    arnoldi_dots_kernel<Q, 2><<<dim3(gs, nb, (j + 8) / 8), STPB, 0, c->stream>>>(Vc, n2, op.nbr, vl, j, y, t, part1)
            if (n2 <= 25) DOTS(1);
            else if (n2 <= 51) DOTS(2);
            else DOTS(3);
#undef DOTS
        }
        if (j < 4) PASS(4);
        else if (j < 8) PASS(8);
        else if (j < 12) PASS(12);
        else PASS(16);
        rc = hip_check(c, hipGetLastError(), "arnoldi");
        w = y;
    }
#undef PASS
    if (!rc) {
        arnoldi_last_kernel<<<nb, 256, 0, c->stream>>>(m, part3, G, H2 + (size_t)(m - 1) * (m + 1) * nb,
                                                       NR + (size_t)m * nb);
        rc = hip_check(c, hipGetLastError(), "arnoldi");
    }
    return rc;
}

}  // namespace mgdd
