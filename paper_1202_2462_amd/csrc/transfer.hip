// Aggregation interpolation (Section 3): P from test vectors by a local
// orthonormalisation per (aggregate, chirality), restriction P^H and
// prolongation P, the tables of the coarse level, and the coarse stencil apply.
// The coarse operator D_c = P^H D P is built in coarse_build.hip.
#include "lanes.h"
#include "stencil.h"
#include "transfer.h"
#include "coarse.h"
#include "level2.h"

namespace mgdd {

namespace {

constexpr int TPB = 256;

template <typename T> __device__ inline T wsum(T v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// sum of (a, b) over the workgroup, identical in every thread (fixed order)
__device__ inline double2 block_sum2(double a, double b, double *red) {
    a = wsum(a);
    b = wsum(b);
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) { red[2 * w] = a; red[2 * w + 1] = b; }
    __syncthreads();
    double A = 0, B = 0;
    for (int i = 0; i < nw; i++) { A += red[2 * i]; B += red[2 * i + 1]; }
    __syncthreads();
    return make_double2(A, B);
}

// ---------------------------------------------------------------- P: local modified Gram-Schmidt
//
// One workgroup per (aggregate, chirality); the (6 * Va) x N block of the test
// vectors is orthonormalised in place, in column order, so that P^H P = 1 on
// the block with a positive real diagonal of R (the unique thin QR).
__global__ __launch_bounds__(TPB) void build_P_kernel(int V, int Va, int N, const int *__restrict__ agg_sites,
                                                      double2 *__restrict__ P, int *__restrict__ flag) {
    __shared__ double red[2 * (TPB / 64)];
    const int a = blockIdx.x, chi = blockIdx.y;
    const int *sites = agg_sites + (size_t)a * Va;
    const size_t fs = (size_t)12 * V;  // field stride
    for (int k = 0; k < N; k++) {
        double2 *w = P + (size_t)k * fs;
        double n0 = 0;
        for (int l = threadIdx.x; l < Va; l += blockDim.x)
            for (int c = 6 * chi; c < 6 * chi + 6; c++) {
                double2 v = w[(size_t)c * V + sites[l]];
                n0 += v.x * v.x + v.y * v.y;
            }
        n0 = block_sum2(n0, 0, red).x;
        for (int j = 0; j < k; j++) {
            const double2 *q = P + (size_t)j * fs;
            double ra = 0, rb = 0;
            for (int l = threadIdx.x; l < Va; l += blockDim.x)
                for (int c = 6 * chi; c < 6 * chi + 6; c++) {
                    size_t e = (size_t)c * V + sites[l];
                    double2 qv = q[e], wv = w[e];
                    ra += qv.x * wv.x + qv.y * wv.y;
                    rb += qv.x * wv.y - qv.y * wv.x;
                }
            double2 r = block_sum2(ra, rb, red);
            for (int l = threadIdx.x; l < Va; l += blockDim.x)
                for (int c = 6 * chi; c < 6 * chi + 6; c++) {
                    size_t e = (size_t)c * V + sites[l];
                    w[e] = csub(w[e], cmul(r, q[e]));
                }
        }
        double nn = 0;
        for (int l = threadIdx.x; l < Va; l += blockDim.x)
            for (int c = 6 * chi; c < 6 * chi + 6; c++) {
                double2 v = w[(size_t)c * V + sites[l]];
                nn += v.x * v.x + v.y * v.y;
            }
        nn = block_sum2(nn, 0, red).x;
        double rkk = sqrt(nn);
        if (!(rkk > 1e-12 * sqrt(n0)) || n0 == 0.0) {
            if (threadIdx.x == 0) atomicExch(flag, 1);
            rkk = 1.0;
        }
        double inv = 1.0 / rkk;
        for (int l = threadIdx.x; l < Va; l += blockDim.x)
            for (int c = 6 * chi; c < 6 * chi + 6; c++) {
                size_t e = (size_t)c * V + sites[l];
                w[e] = cscale(w[e], inv);
            }
    }
}

// The same orthonormalisation for aggregates of at most TPB sites, one thread
// per site and PANEL columns at a time in registers (6 components each): an
// earlier column is loaded once per panel and its products with the PANEL
// columns are summed over the workgroup together (one barrier, two alternating
// LDS slots); within the panel a column's norm and its products with the
// later ones are. Each column still has the earlier ones taken off one after
// the other, so this is modified Gram-Schmidt in column order.
// The test vectors are read from tv and copied to kept (unless null), and P is
// written in every precision while its column is in registers.
// Bound: the reads of the earlier columns (from the Infinity Cache: 256
// workgroups' columns do not fit L2), the streams of tv and P, and the latency
// of the sums. An aggregate's sites cover lines of the field only in part, so
// neighbouring aggregates run on one XCD at the same time, where its L2 puts the
// lines together (24^3 x 48 lattice, 3x4x4x4 aggregates, N = 21: 5.5 ms against
// 8.9 in the order of the launch; with the non-temporal policy, which gives the
// lines up before they are whole, 7.9 in that order). Separate copies and
// conversions took 3.3 ms more than the 4.3 ms without them; one column at a
// time, which reads every earlier column N times over, 10.8 ms.
constexpr int PANEL = 4;

// v[i] <- the sum of v[i] over the workgroup, i < 8
__device__ inline void block_sum8(double *v, double *red) {
    const double s = wave_sum8(v);
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (!(lane & 7)) red[(threadIdx.x >> 6) * 8 + (lane >> 3)] = s;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = red[i];
    for (int w = 1; w < nw; w++)
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] += red[w * 8 + i];
}

__global__ __launch_bounds__(TPB) __attribute__((amdgpu_waves_per_eu(2))) void build_P_panel_kernel(
    int V, int Va, int N, const int *__restrict__ agg_sites, const double2 *tv, double2 *kept, double2 *P,
    float2 *__restrict__ P32, half_cx *__restrict__ P16, int *__restrict__ flag) {
    __shared__ double red[2][8 * (TPB / 64)];
    const int wg = xcd_block(gridDim.x), Vc = gridDim.x >> 1, chi = wg >= Vc, a = wg - chi * Vc;
    const bool active = (int)threadIdx.x < Va;
    const int d = active ? agg_sites[(size_t)a * Va + threadIdx.x] : 0;
    const size_t fs = (size_t)12 * V;  // field stride
    const size_t o = (size_t)6 * chi * V + d;
    int slot = 0;
    auto load = [&](const double2 *F, int k, double2 *v) {
#pragma unroll
        for (int c = 0; c < 6; c++) v[c] = active && k < N ? F[o + (size_t)k * fs + (size_t)c * V] : make_double2(0, 0);
    };
    for (int k0 = 0; k0 < N; k0 += PANEL) {
        double2 w[PANEL][6], q[6], qn[6];
        double n0[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < PANEL; i++) {
            load(tv, k0 + i, w[i]);
#pragma unroll
            for (int c = 0; c < 6; c++) n0[i] += w[i][c].x * w[i][c].x + w[i][c].y * w[i][c].y;
        }
        if (kept && active) {
#pragma unroll
            for (int i = 0; i < PANEL; i++)
                if (k0 + i < N) {
#pragma unroll
                    for (int c = 0; c < 6; c++) kept[o + (size_t)(k0 + i) * fs + (size_t)c * V] = w[i][c];
                }
        }
        if (k0) load(P, 0, q);
        block_sum8(n0, red[slot]);
        slot ^= 1;
        for (int j = 0; j < k0; j++) {
            load(P, j + 1 < k0 ? j + 1 : j, qn);   // while column j is used
            double r[2 * PANEL];
#pragma unroll
            for (int i = 0; i < PANEL; i++) {
                double2 t = make_double2(0, 0);
#pragma unroll
                for (int c = 0; c < 6; c++) cfmac(t, q[c], w[i][c]);
                r[2 * i] = t.x;
                r[2 * i + 1] = t.y;
            }
            block_sum8(r, red[slot]);
            slot ^= 1;
#pragma unroll
            for (int i = 0; i < PANEL; i++)
#pragma unroll
                for (int c = 0; c < 6; c++) cfma(w[i][c], make_double2(-r[2 * i], -r[2 * i + 1]), q[c]);
#pragma unroll
            for (int c = 0; c < 6; c++) q[c] = qn[c];
        }
#pragma unroll
        for (int i = 0; i < PANEL; i++) {
            if (k0 + i >= N) break;
            // r[2 i]: the norm of column i; the others: its products with the later columns
            double r[2 * PANEL] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c < 6; c++) r[2 * i] += w[i][c].x * w[i][c].x + w[i][c].y * w[i][c].y;
#pragma unroll
            for (int m = i + 1; m < PANEL; m++) {
                double2 t = make_double2(0, 0);
#pragma unroll
                for (int c = 0; c < 6; c++) cfmac(t, w[i][c], w[m][c]);
                r[2 * m] = t.x;
                r[2 * m + 1] = t.y;
            }
            block_sum8(r, red[slot]);
            slot ^= 1;
            double rkk = sqrt(r[2 * i]);
            if (!(rkk > 1e-12 * sqrt(n0[i])) || n0[i] == 0.0) {
                if (threadIdx.x == 0) atomicExch(flag, 1);
                rkk = 1.0;
            }
            const double inv = 1.0 / rkk;
#pragma unroll
            for (int c = 0; c < 6; c++) w[i][c] = cscale(w[i][c], inv);
#pragma unroll
            for (int m = i + 1; m < PANEL; m++)
#pragma unroll
                for (int c = 0; c < 6; c++)
                    cfma(w[m][c], make_double2(-r[2 * m] * inv, -r[2 * m + 1] * inv), w[i][c]);
            if (active) {
#pragma unroll
                for (int c = 0; c < 6; c++) {
                    const size_t e = o + (size_t)(k0 + i) * fs + (size_t)c * V;
                    const float2 f = make_float2((float)w[i][c].x, (float)w[i][c].y);
                    half_cx h;
                    h.x = (_Float16)w[i][c].x;
                    h.y = (_Float16)w[i][c].y;
                    P[e] = w[i][c];
                    P32[e] = f;
                    P16[e] = h;
                }
            }
        }
    }
}

// ---------------------------------------------------------------- restriction c = P^H f, prolongation f = P c
//
// T: arithmetic and coarse precision; SP, SF: storage of P and of the fine
// field (T, or half precision with T = float; the fine field rounded once to
// nearest even). R right-hand sides per thread (where fewer exist the last one
// is repeated and not written): a value of P is loaded once for all of them. A
// thread holds one site and one chirality, 6 R complex values in registers, so
// P is read once for up to 12 right-hand sides (FP64: 6); the next column's 6
// values are loaded while one is used. The sums of a right-hand side do not
// depend on R. Bound: reading P for one right-hand side (32^3 x 64, N = 24,
// FP32: 862 and 983 us, 5.8 and 5.1 TB/s; 943 and 1007 us with both chiralities
// in a thread), the vector units for many: 24^3 x 48, N = 24, 12 right-hand
// sides in FP32: restriction 502 us (one workgroup per aggregate and
// right-hand side: 1450 us), prolongation 472 us (one thread per site and
// right-hand side: 1980 us).
template <typename T, typename SP, typename SF, int R>
__global__ __launch_bounds__(TPB) void restrict_kernel(int V, int Va, int N, const int *__restrict__ agg_sites,
                                                             const C<SP> *__restrict__ P, const C<SF> *__restrict__ f,
                                                             C<T> *__restrict__ out, int Vc, int nrhs, int ks,
                                                             int kper) {
    extern __shared__ unsigned char smem[];
    constexpr int NS = (2 * R + 7) / 8 * 8;   // sums per k, rounded up to eights
    T *red = (T *)smem;                       // [waves][kper][NS]
    const int wg = xcd_block(gridDim.x), r0 = blockIdx.y * R;
    const int part = wg % ks, ac = wg / ks, chi = ac & 1, a = ac >> 1;
    const int kb = part * kper, ke = kb + kper < N ? kb + kper : N;
    const int *sites = agg_sites + (size_t)a * Va;
    const size_t fs = (size_t)12 * V;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    auto wide = [](auto v) { return mk<T>((T)v.x, (T)v.y); };
    for (int l0 = 0; l0 < Va; l0 += blockDim.x) {
        const int l = l0 + (int)threadIdx.x;
        const bool active = l < Va;
        const int d = sites[active ? l : Va - 1];
        C<T> fv[R][6];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const C<SF> *fr = f + (size_t)(r0 + r < nrhs ? r0 + r : nrhs - 1) * fs + (size_t)6 * chi * V + d;
#pragma unroll
            for (int c = 0; c < 6; c++) fv[r][c] = wide(fr[(size_t)c * V]);
        }
        const C<SP> *pk = P + (size_t)6 * chi * V + d;
        C<SP> pn[6];
#pragma unroll
        for (int c = 0; c < 6; c++) pn[c] = pk[(size_t)kb * fs + (size_t)c * V];
        for (int k = kb; k < ke; k++) {
            C<T> pv[6];
#pragma unroll
            for (int c = 0; c < 6; c++) pv[c] = active ? wide(pn[c]) : mk<T>(0, 0);
            const size_t kn = (size_t)(k + 1 < ke ? k + 1 : k) * fs;
#pragma unroll
            for (int c = 0; c < 6; c++) pn[c] = pk[kn + (size_t)c * V];
            T s[NS];
#pragma unroll
            for (int q = 0; q < NS; q++) s[q] = 0;
#pragma unroll
            for (int r = 0; r < R; r++) {
                C<T> t = mk<T>(0, 0);
#pragma unroll
                for (int c = 0; c < 6; c++) cfmac(t, pv[c], fv[r][c]);
                s[2 * r] = t.x;
                s[2 * r + 1] = t.y;
            }
            T *o = red + ((size_t)w * kper + (k - kb)) * NS;
#pragma unroll
            for (int q = 0; q < NS; q += 8) {
                const T v = wave_sum8(s + q);
                if (!(lane & 7)) o[q + (lane >> 3)] = l0 ? o[q + (lane >> 3)] + v : v;
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < (ke - kb) * R; i += blockDim.x) {
        const int k = i % (ke - kb), r = i / (ke - kb);
        if (r0 + r >= nrhs) break;
        C<T> v = mk<T>(0, 0);
        for (int q = 0; q < nw; q++) {
            const T *o = red + ((size_t)q * kper + k) * NS + 2 * r;
            v.x += o[0];
            v.y += o[1];
        }
        out[((size_t)(r0 + r) * Vc + a) * 2 * N + chi * N + kb + k] = v;
    }
}

// xcd: neighbouring sites on one XCD, else in the order of the launch
template <typename T, typename SP, typename SF, int R>
__global__ __launch_bounds__(TPB) void prolong_kernel(int V, int Vc, int N, const int *__restrict__ site_agg,
                                                            const C<SP> *__restrict__ P, const C<T> *__restrict__ cin,
                                                            C<SF> *__restrict__ f, int nrhs, int xcd) {
    const int wg = xcd ? xcd_block(gridDim.x) : (int)blockIdx.x, chi = wg & 1, r0 = blockIdx.y * R;
    const int i = (wg >> 1) * TPB + (int)threadIdx.x, d = i < V ? i : V - 1;
    const int a = site_agg[d], au = __builtin_amdgcn_readfirstlane(a);
    const size_t fs = (size_t)12 * V, xs = (size_t)Vc * 2 * N;
    const C<SP> *pk = P + (size_t)6 * chi * V + d;
    C<T> acc[R][6];
#pragma unroll
    for (int r = 0; r < R; r++)
#pragma unroll
        for (int c = 0; c < 6; c++) acc[r][c] = mk<T>(0, 0);
    C<SP> pn[6];
#pragma unroll
    for (int c = 0; c < 6; c++) pn[c] = pk[(size_t)c * V];
    // one aggregate per wave (aggregates that hold whole runs of 64 sites):
    // the coarse values are wave-uniform and come through the scalar cache
    auto columns = [&](int ax) {
        const C<T> *x = cin + ((size_t)r0 * Vc + ax) * 2 * N + (size_t)chi * N;
        for (int k = 0; k < N; k++) {
            C<T> pv[6];
#pragma unroll
            for (int c = 0; c < 6; c++) pv[c] = mk<T>((T)pn[c].x, (T)pn[c].y);
            const size_t kn = (size_t)(k + 1 < N ? k + 1 : k) * fs;
#pragma unroll
            for (int c = 0; c < 6; c++) pn[c] = pk[kn + (size_t)c * V];
#pragma unroll
            for (int r = 0; r < R; r++) {
                const C<T> xv = x[(size_t)(r0 + r < nrhs ? r : nrhs - 1 - r0) * xs + k];
#pragma unroll
                for (int c = 0; c < 6; c++) cfma(acc[r][c], pv[c], xv);
            }
        }
    };
    if (__all(a == au)) columns(au);
    else columns(a);
    if (i >= V) return;
#pragma unroll
    for (int r = 0; r < R; r++) {
        if (r0 + r >= nrhs) break;
        C<SF> *fr = f + (size_t)(r0 + r) * fs + (size_t)6 * chi * V + d;
#pragma unroll
        for (int c = 0; c < 6; c++) fr[(size_t)c * V] = mk<SF>((SF)acc[r][c].x, (SF)acc[r][c].y);
    }
}

// The same with one thread per (site, field) and both chiralities in it, the
// fields of a site in consecutive threads: 12 values of P in flight. The same
// sums, so the same bits.
template <typename T>
__global__ __launch_bounds__(TPB) void prolong_site_kernel(int V, int Vc, int N, const int *__restrict__ site_agg,
                                                           const C<T> *__restrict__ P, const C<T> *__restrict__ cin,
                                                           C<T> *__restrict__ f, int nrhs) {
    const size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= (size_t)V * nrhs) return;
    const int r = (int)(i % nrhs), d = (int)(i / nrhs);
    const int a = site_agg[d];
    const size_t fs = (size_t)12 * V;
    const C<T> *x = cin + ((size_t)r * Vc + a) * 2 * N;
    C<T> acc[12];
#pragma unroll
    for (int c = 0; c < 12; c++) acc[c] = mk<T>(0, 0);
    for (int k = 0; k < N; k++) {
        const C<T> *pk = P + (size_t)k * fs;
        const C<T> x0 = x[k], x1 = x[N + k];
#pragma unroll
        for (int c = 0; c < 12; c++) cfma(acc[c], pk[(size_t)c * V + d], c < 6 ? x0 : x1);
    }
    C<T> *fr = f + (size_t)r * fs;
#pragma unroll
    for (int c = 0; c < 12; c++) fr[(size_t)c * V + d] = acc[c];
}

// ---------------------------------------------------------------- coarse stencil y = D_c x
//
// One workgroup of 1024 threads per (coarse site, right-hand side): the 9 2N
// products of each row are split over floor(1024 / 2N) thread sets
// (dc_row_partial), whose partial rows are then added in set order. Blocks
// are stored column-major, B[a][dir][col][row], so consecutive threads read
// consecutive rows of one column.
template <typename T>
__global__ __launch_bounds__(1024) void coarse_apply_kernel(int Vc, int N, const int *__restrict__ cnbr,
                                                            const C<T> *__restrict__ Dc, const C<T> *__restrict__ x,
                                                            C<T> *__restrict__ y) {
    const int a = blockIdx.x, r = blockIdx.y;
    const int n2 = 2 * N;
    __shared__ C<T> xs[9 * 64];
    __shared__ C<T> part[1024];
    const C<T> *xr = x + (size_t)r * Vc * n2;
    for (int e = threadIdx.x; e < 9 * n2; e += blockDim.x) xs[e] = xr[(size_t)cnbr[a * 9 + e / n2] * n2 + e % n2];
    __syncthreads();
    dc_row_partial<T>(Dc + (size_t)a * 9 * n2 * n2, xs, n2, part);
    __syncthreads();
    const int i = threadIdx.x, nparts = blockDim.x / n2;
    if (i < n2) {
        C<T> acc = mk<T>(0, 0);
        for (int q = 0; q < nparts; q++) acc = cadd(acc, part[q * n2 + i]);
        y[((size_t)r * Vc + a) * n2 + i] = acc;
    }
}

// D_c applied to many right-hand sides on the matrix cores. Per coarse site
// a the product is Y = sum_dir B_dir X_nbr(dir), a (2N x 2N) by (2N x R)
// complex matrix product for R right-hand sides, done as real 16x16x4 MFMA
// tiles: Re Y += Re B Re X - Im B Im X, Im Y += Re B Im X + Im B Re X.
// A wave owns output rows 16t .. 16t+15 of one coarse site for one tile of
// 16 right-hand sides; its A operand (rows of B_dir, column-major blocks)
// streams from HBM, its B operand (4 consecutive entries of 16 neighbour
// vectors) comes through the caches, which the row tiles of a site share.
// Rows and columns past 2N and right-hand sides past nrhs enter as zeros and
// are not written.
template <typename T> struct MfmaTypes;
// Operands of both: A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k.
// Result register v of lane l holds D[row][l % 16] with row = 4 (l / 16) + v
// (FP32) or row = 4 v + l / 16 (FP64).
template <> struct MfmaTypes<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(float a, float b, v4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int row(int v, int kq) { return 4 * kq + v; }
};
template <> struct MfmaTypes<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    __device__ static v4 mma(double a, double b, v4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row(int v, int kq) { return 4 * v + kq; }
};

template <typename T>
__global__ __launch_bounds__(64) void coarse_apply_mfma_kernel(int Vc, int N, int nrhs, int ntiles,
                                                               const int *__restrict__ cnbr,
                                                               const C<T> *__restrict__ Dc,
                                                               const C<T> *__restrict__ x, C<T> *__restrict__ y) {
    using M = MfmaTypes<T>;
    // one wave per (coarse site, row tile, rhs tile); the row tiles of one
    // site are consecutive waves on one XCD, so that they share its L2
    const int w = xcd_block(gridDim.x);
    const int t = w % ntiles, a = w / ntiles, r0 = blockIdx.y * 16;
    const int n2 = 2 * N;
    const int lane = threadIdx.x;
    const int row = t * 16 + (lane & 15), kq = lane >> 4, rl = lane & 15;
    const bool rhs_ok = r0 + rl < nrhs;
    // four independent accumulator chains (Re and Im, two each), so that
    // consecutive MFMAs do not wait for each other's results
    typename M::v4 re0 = {0, 0, 0, 0}, im0 = {0, 0, 0, 0}, re1 = {0, 0, 0, 0}, im1 = {0, 0, 0, 0};
    const C<T> *B = Dc + (size_t)a * 9 * n2 * n2;
    const int nq = (n2 + 3) >> 2;   // k-steps of 4 columns per direction (n2 <= 64)
    for (int dd = 0; dd < 9; dd++) {
        const C<T> *Bd = B + (size_t)dd * n2 * n2;
        const C<T> *xd = x + ((size_t)(r0 + rl) * Vc + cnbr[a * 9 + dd]) * n2;
        // all operands of this direction first, so that their loads overlap
        C<T> av[16], bv[16];
#pragma unroll
        for (int q = 0; q < 16; q++) {
            const int j = 4 * q + kq;
            const bool kin = q < nq && j < n2;
            av[q] = (kin && row < n2) ? Bd[(size_t)j * n2 + row] : mk<T>(0, 0);
            bv[q] = (kin && rhs_ok) ? xd[j] : mk<T>(0, 0);
        }
#pragma unroll
        for (int q = 0; q < 16; q++) {
            if (q < nq) {
                re0 = M::mma(av[q].x, bv[q].x, re0);
                im0 = M::mma(av[q].x, bv[q].y, im0);
                re1 = M::mma(-av[q].y, bv[q].y, re1);
                im1 = M::mma(av[q].y, bv[q].x, im1);
            }
        }
    }
    if (!rhs_ok) return;
    const typename M::v4 re = re0 + re1, im = im0 + im1;
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const int i = t * 16 + M::row(v, kq);
        if (i < n2) y[((size_t)(r0 + rl) * Vc + a) * n2 + i] = mk<T>(re[v], im[v]);
    }
}

}  // namespace

// ---------------------------------------------------------------- host side

// from this many right-hand sides on, D_c is applied on the matrix cores
static int MFMA_MIN_RHS = 4;

// Order in which arnoldi_apply_kernel visits the coarse sites: the coarse GMRES
// step in FP64, and in FP32 where the workspace has no room for the compact
// steps. In FP32 a site reads the forward blocks of its four backward neighbours
// again, so these should still be in the L2 of its XCD, and the XCDs take
// contiguous eighths of the order. Lexicographic order leaves the z and t
// neighbours far behind; here the sites go in 4-D tiles, time fastest within
// a tile, the tiles in lexicographic order. The spatial extents of a tile are
// 4, 3 or 2, whichever divides the coarse extent first; in time, when 8
// divides the time extent, it is one eighth of it (so that each XCD's range
// is a whole number of time slices, their tiles complete: at 12^3 x 24
// coarse sites, 4 x 4 x 4 x 3 tiles cut the coarse step's reads from memory
// by 5 % and its time by about 3 %, where 4^4 tiles gained nothing), else 4,
// 3 or 2 as in space.
static std::vector<int> coarse_visit_order(const int *Lc) {
    int e[4], nt[4];
    for (int m = 0; m < 4; m++) {
        e[m] = Lc[m] % 4 == 0 ? 4 : Lc[m] % 3 == 0 ? 3 : Lc[m] % 2 == 0 ? 2 : 1;
        if (m == 3 && Lc[3] % 8 == 0) e[3] = Lc[3] / 8;
        nt[m] = Lc[m] / e[m];
    }
    const int vt = e[0] * e[1] * e[2] * e[3], ntiles = nt[0] * nt[1] * nt[2] * nt[3];
    std::vector<int> order;
    order.reserve((size_t)vt * ntiles);
    for (int tile = 0; tile < ntiles; tile++) {
        int tc[4], r = tile;
        for (int m = 0; m < 4; m++) { tc[m] = r % nt[m]; r /= nt[m]; }
        for (int i = 0; i < vt; i++) {
            int x[4], q = i;
            x[3] = q % e[3]; q /= e[3];   // time fastest
            for (int m = 0; m < 3; m++) { x[m] = q % e[m]; q /= e[m]; }
            int y[4];
            for (int m = 0; m < 4; m++) y[m] = tc[m] * e[m] + x[m];
            order.push_back(y[0] + Lc[0] * (y[1] + Lc[1] * (y[2] + Lc[2] * y[3])));
        }
    }
    return order;
}

int transfer_setup(Ctx *c, const int *agg, int N) {
    Level1 &L1 = c->c;
    const Geom &g = c->g;
    for (int m = 0; m < 4; m++)
        if (agg[m] <= 0 || g.L[m] % agg[m]) return fail(c, MGDD_ESHAPE, "aggregates must divide the lattice");
    int Va = agg[0] * agg[1] * agg[2] * agg[3];
    if (N <= 0 || N > 32) return fail(c, MGDD_EINVAL, "number of test vectors must be in 1..32");
    if (N > 6 * Va) return fail(c, MGDD_ERANK, "more test vectors than dof per aggregate and chirality");
    int Lc[4];
    for (int m = 0; m < 4; m++) Lc[m] = g.L[m] / agg[m];
    int Vc = Lc[0] * Lc[1] * Lc[2] * Lc[3];
    bool same = L1.agg_sites && L1.N == N && L1.Vc == Vc;
    for (int m = 0; m < 4 && same; m++) same = L1.agg[m] == agg[m];
    if (same) return MGDD_OK;
    // free the previous level (and the third level built on it)
    level2_free(c);
    void *old[] = {L1.P64, L1.P32, L1.P16, L1.Dc64, L1.Dc32, L1.Dh32, L1.cnbr, L1.corder, L1.agg_sites, L1.site_agg,
                   L1.face_sites, L1.tv64};
    (void)hipStreamSynchronize(c->stream);
    for (void *p : old) dfree(c, p);
    L1 = Level1();
    // tables: fine sites of each aggregate in ascending device order (so that
    // consecutive entries are neighbours in memory as far as the aggregate
    // allows), those of them on its + face in each direction, the aggregate
    // of each site
    std::vector<int> agg_sites((size_t)Vc * Va), site_agg(g.V), cnbr((size_t)Vc * 9), nsite(Vc, 0);
    std::vector<int> face[4], nface[4];
    for (int m = 0; m < 4; m++) {
        face[m].resize((size_t)Vc * (Va / agg[m]));
        nface[m].assign(Vc, 0);
    }
    std::vector<uint32_t> coord;
    std::vector<int> bn, lp;
    Geom hg{};
    int block[4] = {1 << g.lb[0], 1 << g.lb[1], 1 << g.lb[2], 1 << g.lb[3]};
    geometry_tables(g.L, block, hg, coord, bn, &lp);
    hg.blk_coord = coord.data();
    hg.blk_nbr = bn.data();
    hg.pos_of_lex = lp.data();
    for (int d = 0; d < g.V; d++) {
        int X[4], ac[4];
        site_coords(hg, d, X);
        for (int m = 0; m < 4; m++) ac[m] = X[m] / agg[m];
        const int a = ac[0] + Lc[0] * (ac[1] + Lc[1] * (ac[2] + Lc[2] * ac[3]));
        agg_sites[(size_t)a * Va + nsite[a]++] = d;
        site_agg[d] = a;
        for (int m = 0; m < 4; m++)
            if (X[m] == ac[m] * agg[m] + agg[m] - 1) face[m][(size_t)a * (Va / agg[m]) + nface[m][a]++] = d;
    }
    for (int a = 0; a < Vc; a++) {
        int t = a, ac[4];
        for (int m = 0; m < 4; m++) { ac[m] = t % Lc[m]; t /= Lc[m]; }
        cnbr[(size_t)a * 9] = a;
        for (int m = 0; m < 4; m++)
            for (int dir = 0; dir < 2; dir++) {
                int y[4] = {ac[0], ac[1], ac[2], ac[3]};
                y[m] = (y[m] + (dir == 0 ? 1 : -1) + Lc[m]) % Lc[m];
                cnbr[(size_t)a * 9 + 1 + 2 * m + dir] = y[0] + Lc[0] * (y[1] + Lc[1] * (y[2] + Lc[2] * y[3]));
            }
    }
    size_t fsz = (size_t)N * 12 * g.V;
    size_t dsz = (size_t)Vc * 9 * 4 * N * N;
    L1.P64 = dalloc(c, fsz * 16);
    L1.tv64 = dalloc(c, fsz * 16);
    L1.P32 = dalloc(c, fsz * 8);
    L1.P16 = dalloc(c, fsz * 4);
    L1.Dc64 = dalloc(c, dsz * 16);
    L1.Dc32 = dalloc(c, dsz * 8);
    L1.Dh32 = dalloc(c, dsz / 9 * 5 * 8);
    L1.cnbr = (int *)dalloc(c, cnbr.size() * sizeof(int));
    const std::vector<int> corder = coarse_visit_order(Lc);
    L1.corder = (int *)dalloc(c, corder.size() * sizeof(int));
    L1.agg_sites = (int *)dalloc(c, agg_sites.size() * sizeof(int));
    L1.site_agg = (int *)dalloc(c, site_agg.size() * sizeof(int));
    std::vector<int> faces;
    for (int m = 0; m < 4; m++) faces.insert(faces.end(), face[m].begin(), face[m].end());
    L1.face_sites = (int *)dalloc(c, faces.size() * sizeof(int));
    if (!L1.P64 || !L1.tv64 || !L1.P32 || !L1.P16 || !L1.Dc64 || !L1.Dc32 || !L1.Dh32 || !L1.cnbr || !L1.corder ||
        !L1.agg_sites || !L1.site_agg || !L1.face_sites)
        return MGDD_ENOMEM;
    int rc = hip_check(c, hipMemcpy(L1.cnbr, cnbr.data(), cnbr.size() * sizeof(int), hipMemcpyHostToDevice), "copy");
    if (!rc) rc = hip_check(c, hipMemcpy(L1.corder, corder.data(), corder.size() * sizeof(int), hipMemcpyHostToDevice), "copy");
    if (!rc) rc = hip_check(c, hipMemcpy(L1.agg_sites, agg_sites.data(), agg_sites.size() * sizeof(int), hipMemcpyHostToDevice), "copy");
    if (!rc) rc = hip_check(c, hipMemcpy(L1.face_sites, faces.data(), faces.size() * sizeof(int), hipMemcpyHostToDevice), "copy");
    if (!rc) rc = hip_check(c, hipMemcpy(L1.site_agg, site_agg.data(), site_agg.size() * sizeof(int), hipMemcpyHostToDevice), "copy");
    if (rc) return rc;
    for (int m = 0; m < 4; m++) { L1.agg[m] = agg[m]; L1.Lc[m] = Lc[m]; }
    L1.Vc = Vc;
    L1.Va = Va;
    L1.N = N;
    return MGDD_OK;
}

// memory of the current device, aligned for 16-byte loads
static bool kernel_readable(const void *p) {
    hipPointerAttribute_t at;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return at.type == hipMemoryTypeDevice && at.device == dev && !((uintptr_t)p & 15);
}

int launch_build_P(Ctx *c, const void *tv64) {
    Level1 &L1 = c->c;
    const Geom &g = c->g;
    const size_t fsz = (size_t)L1.N * 12 * g.V;
    const bool panel = L1.Va <= TPB, keep = tv64 != L1.tv64;
    // the panel kernel reads the caller's vectors itself, keeps the copy of
    // them and writes every form of P (24^3 x 48, N = 21: 5.5 ms; with two
    // copies before and two conversions after it 7.6 ms); a copy also takes
    // memory that a kernel's 16-byte loads may not
    const bool direct = panel && (!keep || kernel_readable(tv64));
    int rc = MGDD_OK;
    if (!direct) {
        rc = hip_check(c, hipMemcpyAsync(L1.P64, tv64, fsz * 16, hipMemcpyDeviceToDevice, c->stream), "copy");
        if (!rc && keep)
            rc = hip_check(c, hipMemcpyAsync(L1.tv64, tv64, fsz * 16, hipMemcpyDeviceToDevice, c->stream), "copy");
        if (rc) return rc;
    }
    int *flag = (int *)ensure_scratch(c, sizeof(int));
    if (!flag) return MGDD_ENOMEM;
    rc = hip_check(c, hipMemsetAsync(flag, 0, sizeof(int), c->stream), "memset");
    if (rc) return rc;
    if (panel)
        build_P_panel_kernel<<<2 * L1.Vc, (unsigned)((L1.Va + 63) / 64 * 64), 0, c->stream>>>(
            g.V, L1.Va, L1.N, L1.agg_sites, (const double2 *)(direct ? tv64 : L1.P64),
            direct && keep ? (double2 *)L1.tv64 : nullptr,
            (double2 *)L1.P64, (float2 *)L1.P32, (half_cx *)L1.P16, flag);
    else
        build_P_kernel<<<dim3(L1.Vc, 2), TPB, 0, c->stream>>>(g.V, L1.Va, L1.N, L1.agg_sites, (double2 *)L1.P64, flag);
    rc = hip_check(c, hipGetLastError(), "build_P kernel");
    if (rc) return rc;
    int hflag = 0;
    rc = hip_check(c, hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, c->stream), "copy");
    if (!rc) rc = hip_check(c, hipStreamSynchronize(c->stream), "sync");
    if (rc) return rc;
    if (hflag) return fail(c, MGDD_ERANK, "test vectors are rank deficient on some aggregate");
    if (!panel) {
        rc = launch_convert(c, MGDD_F64, MGDD_F32, fsz, L1.P64, L1.P32);
        if (!rc) rc = launch_convert(c, MGDD_F64, MGDD_F16, fsz, L1.P64, L1.P16);
    }
    return rc;
}

// right-hand sides per thread for nrhs of them: the registers hold 12 (FP64:
// 6); the fewest that take them in the same number of groups
static int rhs_per_thread(int prec, int nrhs) {
    const int most = prec == MGDD_F64 ? 6 : 12, groups = (nrhs + most - 1) / most, need = (nrhs + groups - 1) / groups;
    return need <= 2 ? need : need <= 4 ? 4 : need <= 6 ? 6 : need <= 8 ? 8 : 12;
}

#define MULTI_R(F, T, SP, SF)             \
    do {                                  \
        if (R == 1) F(T, SP, SF, 1);      \
        else if (R == 2) F(T, SP, SF, 2); \
        else if (R == 4) F(T, SP, SF, 4); \
        else F(T, SP, SF, 6);             \
    } while (0)
#define MULTI_R12(F, T, SP, SF)            \
    do {                                   \
        if (R <= 6) MULTI_R(F, T, SP, SF); \
        else if (R == 8) F(T, SP, SF, 8);  \
        else F(T, SP, SF, 12);             \
    } while (0)
#define MULTI(F)                                                  \
    do {                                                          \
        if (prec == MGDD_F64) MULTI_R(F, double, double, double); \
        else if (prec == MGDD_F32) MULTI_R12(F, float, float, float); \
        else MULTI_R12(F, float, _Float16, _Float16);             \
    } while (0)

int launch_restrict(Ctx *c, int prec, int nrhs, const void *fine, void *coarse) {
    const Level1 &L1 = c->c;
    const void *P = prec == MGDD_F64 ? L1.P64 : prec == MGDD_F32 ? L1.P32 : L1.P16;
    const int R = rhs_per_thread(prec, nrhs), groups = (nrhs + R - 1) / R;
    const RestrictSplit split = restrict_split(L1.N, (size_t)L1.Vc * 2 * groups);
    const int ks = split.parts, kper = split.per, ns = (2 * R + 7) / 8 * 8;
    const unsigned threads = L1.Va >= TPB ? TPB : (unsigned)((L1.Va + 63) / 64 * 64);
    const size_t lds = (size_t)(threads / 64) * kper * ns * (prec == MGDD_F64 ? 8 : 4);
    const dim3 grid((unsigned)(L1.Vc * 2 * ks), (unsigned)groups);
#define RESTRICT(T, SP, SF, RR)                                                                          \
    restrict_kernel<T, SP, SF, RR><<<grid, threads, lds, c->stream>>>(                                   \
        c->g.V, L1.Va, L1.N, L1.agg_sites, (const C<SP> *)P, (const C<SF> *)fine, (C<T> *)coarse, L1.Vc, nrhs, ks, kper)
    MULTI(RESTRICT);
#undef RESTRICT
    return hip_check(c, hipGetLastError(), "restrict kernel");
}

// One field in FP32 or FP64 and two in FP64 are served better by a thread per
// site and field on lattices whose P comes from memory: FP64, N = 20, 16^3 x 32, 1
// and 2 fields: 87 and 101 us against 96 and 111; 24^3 x 48, N = 28, 6^2 x 4^2 sites
// an aggregate: 677 and 703 against 692 and 748; FP32, 1 field: 347 against 353.
// Not so below 131072 sites (16^4: 43.9 and 60 against 39.2 and 42; FP32 20.5
// against 19.3), nor one field on 2^20 sites or more (32^3 x 64, N = 20: 1740
// against 1617, FP32 850 against 822).
static bool prolong_by_site(const Ctx *c, int prec, int nrhs) {
    if (c->g.V < 131072 || prec == MGDD_F16) return false;
    return nrhs == 1 ? c->g.V < 1 << 20 : nrhs == 2 && prec == MGDD_F64;
}

int launch_prolong(Ctx *c, int prec, int nrhs, const void *coarse, void *fine) {
    const Level1 &L1 = c->c;
    const void *P = prec == MGDD_F64 ? L1.P64 : prec == MGDD_F32 ? L1.P32 : L1.P16;
    const unsigned nwg = (unsigned)((c->g.V + TPB - 1) / TPB);
    // A P that fits the Infinity Cache (256 MB) is read from it the faster with an
    // XCD's sites together (16^3 x 32, N = 20, FP32, 1 right-hand side: 38 us, in the
    // order of the launch 41.6), one from memory with all XCDs' streams together
    // (24^3 x 48, N = 24, FP32, 2: 326 against 342 us).
    const bool cached = (size_t)12 * c->g.V * L1.N * csize(prec) <= 256000000;
    if (prolong_by_site(c, prec, nrhs)) {
        const unsigned n = (unsigned)(((size_t)c->g.V * nrhs + TPB - 1) / TPB);
        if (prec == MGDD_F64)
            prolong_site_kernel<double><<<n, TPB, 0, c->stream>>>(c->g.V, L1.Vc, L1.N, L1.site_agg, (const double2 *)P,
                                                                  (const double2 *)coarse, (double2 *)fine, nrhs);
        else
            prolong_site_kernel<float><<<n, TPB, 0, c->stream>>>(c->g.V, L1.Vc, L1.N, L1.site_agg, (const float2 *)P,
                                                                 (const float2 *)coarse, (float2 *)fine, nrhs);
        return hip_check(c, hipGetLastError(), "prolong kernel");
    }
    // few sites: smaller groups, so that every CU has a workgroup (8^4, 12
    // right-hand sides, FP32: 6.8 us, with all in one thread 11.2; 8^3 x 16 11.0 and
    // 21.7; 16^2 x 8^2 14.6 and 23.6)
    int R = rhs_per_thread(prec, nrhs);
    while (R > 1 && 2 * nwg * ((nrhs + R - 1) / R) < 256) R = R > 8 ? 8 : R > 2 ? R - 2 : 1;
    const dim3 grid(2 * nwg, (unsigned)((nrhs + R - 1) / R));
#define PROLONG(T, SP, SF, RR)                                                                               \
    prolong_kernel<T, SP, SF, RR><<<grid, TPB, 0, c->stream>>>(c->g.V, L1.Vc, L1.N, L1.site_agg,             \
                                                               (const C<SP> *)P, (const C<T> *)coarse,       \
                                                               (C<SF> *)fine, nrhs, cached)
    MULTI(PROLONG);
#undef PROLONG
    return hip_check(c, hipGetLastError(), "prolong kernel");
}
#undef MULTI
#undef MULTI_R12
#undef MULTI_R

int launch_stencil_apply(Ctx *c, const StencilOp &op, int prec, int nrhs, const void *in, void *out) {
    if (nrhs >= MFMA_MIN_RHS) {
        const int ntiles = (2 * op.N + 15) / 16;
        dim3 grid(op.V * ntiles, (nrhs + 15) / 16);
        if (prec == MGDD_F64)
            coarse_apply_mfma_kernel<double><<<grid, 64, 0, c->stream>>>(
                op.V, op.N, nrhs, ntiles, op.nbr, (const double2 *)op.D64, (const double2 *)in, (double2 *)out);
        else
            coarse_apply_mfma_kernel<float><<<grid, 64, 0, c->stream>>>(
                op.V, op.N, nrhs, ntiles, op.nbr, (const float2 *)op.D32, (const float2 *)in, (float2 *)out);
        return hip_check(c, hipGetLastError(), "coarse apply kernel (MFMA)");
    }
    dim3 grid(op.V, nrhs);
    if (prec == MGDD_F64)
        coarse_apply_kernel<double><<<grid, 1024, 0, c->stream>>>(op.V, op.N, op.nbr, (const double2 *)op.D64,
                                                                 (const double2 *)in, (double2 *)out);
    else
        coarse_apply_kernel<float><<<grid, 1024, 0, c->stream>>>(op.V, op.N, op.nbr, (const float2 *)op.D32,
                                                                (const float2 *)in, (float2 *)out);
    return hip_check(c, hipGetLastError(), "coarse apply kernel");
}

int launch_coarse_apply(Ctx *c, int prec, int nrhs, const void *in, void *out) {
    return launch_stencil_apply(c, level1_op(c), prec, nrhs, in, out);
}

}  // namespace mgdd
