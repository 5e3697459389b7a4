// Wilson-clover operator D = A - 1/2 H (Section 1): one thread per site,
// site-major loads of the 8 neighbour spinors and links, spin projection to
// half spinors before the SU(3) products.
#include "dirac.h"
#include "lanes.h"
#include "stencil.h"

namespace mgdd {

namespace {

constexpr int TPB = 256;

// One thread per (site, right-hand side). Workgroup w covers TPB sites of one
// right-hand side; the right-hand sides of one range of sites are consecutive
// workgroups on one XCD, so the links and the clover term of those sites come
// from HBM once and from L2 for the other right-hand sides.
// S: storage type of the spinors (T, or _Float16 with T = float: half
// storage, FP32 arithmetic, links and clover term in FP32)
template <typename T, typename S = T> struct SpinorView { using type = FieldView<T>; };
template <> struct SpinorView<float, _Float16> { using type = HalfFieldView; };

// STAGE (lattice blocks of TPB sites, so that a workgroup is one block): the
// workgroup first puts its own spinors in LDS, and the neighbours inside the
// block (three quarters of them for 4^4 blocks) are read from there; only the
// neighbours outside the block are read from memory, where the cache need not
// have kept them since another workgroup read them.
// RECON: the links are special unitary, rows 0 and 1 are read and row 2 is
// rebuilt (a third fewer link bytes); antiperiodic: the sign of the time
// links at the boundary, which the rebuilt row must carry
template <typename T, typename S = T, bool RECON = false, bool STAGE = false>
__global__ __launch_bounds__(TPB) void dirac_kernel(Geom g, const C<T> *__restrict__ Up, const C<T> *__restrict__ Ap,
                                                    const C<S> *__restrict__ in, C<S> *__restrict__ out, int nrhs,
                                                    int nwg, int antiperiodic) {
    const int w = xcd_block(nwg);
    const int r = w % nrhs;
    const int i = (w / nrhs) * TPB + threadIdx.x;
    if (!STAGE && i >= g.V) return;  // staged: V is a multiple of TPB
    const int d = site_in_lex_block_order(g, i);
    int nbr[8];
    site_neighbours(g, d, nbr);
    T sf = 1, sb = 1;
    if (RECON) time_link_signs<T>(g, d, antiperiodic, sf, sb);
    const size_t V = g.V;
    LinkViews<T> U(Up, V);
    CloverViews<T> A(Ap, V);
    using FV = typename SpinorView<T, S>::type;
    FV f(in + (size_t)r * 12 * V, V, 12), o(out + (size_t)r * 12 * V, V, 12);
    C<T> acc[12], psi[12], res[12];
    load_spinor<T>(f, d, psi);
    if (STAGE) {
        __shared__ C<T> sp[12 * TPB];
#pragma unroll
        for (int k = 0; k < 12; k++) sp[k * TPB + (d & (TPB - 1))] = psi[k];
        __syncthreads();
        hop_sum_staged<T, T, RECON, TPB>(U, (const C<T> *)in + (size_t)r * 12 * V, V, sp, d >> g.lgVb, g.lgVb, d,
                                         nbr, acc, sf, sb);
    } else {
        hop_sum<T, RECON>(U, f, d, nbr, acc, sf, sb);
    }
    clover_mv<T, true>(A, d, psi, res);
#pragma unroll
    for (int k = 0; k < 12; k++) res[k] = csub(res[k], cscale(acc[k], (T)0.5));
    store_spinor<T, true>(o, d, res);
}

// FP32 or half-precision spinors (S) read as FP64 (the widening is exact)
template <typename S> struct WidenView {
    typename F32Store<S>::view f;
    __device__ WidenView(const C<S> *base, size_t V, int ncomp) : f((const float2 *)base, V, ncomp) {}
    __device__ double2 ld(int comp, int site, unsigned salt = 0) const {
        const float2 v = f.ld(comp, site, salt);
        return make_double2((double)v.x, (double)v.y);
    }
};

// dirac_kernel<double> with FP32 or half-precision input (S): the FP64 apply
// of such a field without a converted copy
template <bool RECON, bool STAGE, typename S = float>
__global__ __launch_bounds__(TPB) void dirac_widen_kernel(Geom g, const double2 *__restrict__ Up,
                                                          const double2 *__restrict__ Ap, const C<S> *__restrict__ in,
                                                          double2 *__restrict__ out, int nrhs, int nwg,
                                                          int antiperiodic) {
    const int w = xcd_block(nwg);
    const int r = w % nrhs;
    const int i = (w / nrhs) * TPB + threadIdx.x;
    if (!STAGE && i >= g.V) return;
    const int d = site_in_lex_block_order(g, i);
    int nbr[8];
    site_neighbours(g, d, nbr);
    double sf = 1, sb = 1;
    if (RECON) time_link_signs<double>(g, d, antiperiodic, sf, sb);
    const size_t V = g.V;
    LinkViews<double> U(Up, V);
    CloverViews<double> A(Ap, V);
    WidenView<S> f(in + (size_t)r * 12 * V, V, 12);
    FieldView<double> o(out + (size_t)r * 12 * V, V, 12);
    double2 acc[12], psi[12], res[12];
    if (STAGE) {
        __shared__ C<S> sp[12 * TPB];
        const C<S> *fin = in + (size_t)r * 12 * V;
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const float2 v = f.f.ld(k, d);   // exact: back to S unchanged below
            sp[k * TPB + (d & (TPB - 1))] = mk<S>((S)v.x, (S)v.y);
            psi[k] = make_double2((double)v.x, (double)v.y);
        }
        __syncthreads();
        hop_sum_staged<double, S, RECON, TPB>(U, fin, V, sp, d >> g.lgVb, g.lgVb, d, nbr, acc, sf, sb);
    } else {
        hop_sum<double, RECON>(U, f, d, nbr, acc, sf, sb);
        load_spinor<double>(f, d, psi);
    }
    clover_mv<double, true>(A, d, psi, res);
#pragma unroll
    for (int k = 0; k < 12; k++) res[k] = csub(res[k], cscale(acc[k], 0.5));
    store_spinor<double, true>(o, d, res);
}

// ---- several right-hand sides, blocks of TPB sites: R of them per thread

// raw components of a field stored as S
template <typename S> struct RawView {
    rsrc_t r;
    unsigned cs;
    __device__ RawView(const C<S> *base, size_t V) : r(make_rsrc(base, 12 * V * sizeof(C<S>))) {
        cs = (unsigned)(V * sizeof(C<S>));
    }
    __device__ C<S> ld(int comp, int site) const {
        const unsigned vo = (unsigned)site * (unsigned)sizeof(C<S>), so = comp * cs;
        if constexpr (sizeof(S) == 2) return __builtin_bit_cast(C<S>, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
        else return BIO<S>::ld(r, vo, so);
    }
};

// a where b is +0, b where a is
__device__ inline half_cx either(half_cx a, half_cx b) {
    return __builtin_bit_cast(half_cx, __builtin_bit_cast(unsigned, a) | __builtin_bit_cast(unsigned, b));
}
__device__ inline float2 either(float2 a, float2 b) {
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    return __builtin_bit_cast(float2, make_uint2(x.x | y.x, x.y | y.y));
}
__device__ inline double2 either(double2 a, double2 b) {
    const uint4 x = __builtin_bit_cast(uint4, a), y = __builtin_bit_cast(uint4, b);
    return __builtin_bit_cast(double2, make_uint4(x.x | y.x, x.y | y.y, x.z | y.z, x.w | y.w));
}

constexpr int OUT = TPB, RS = TPB + 2;   // the zero slot; LDS sites of a component

template <typename T, typename S, bool RECON, int R> struct BlockHops {
    LinkViews<T> U;
    const C<S> *in, *sp;
    size_t V;
    int d, ln[8], nd[8], nb[8];
    T sf, sb;
    C<T> acc[R][12], u[9], gu[9];
    C<S> gm[12];
    __device__ BlockHops(const C<T> *Up, size_t v) : U(Up, v), V(v) {}

    // neighbour M's spinor of right-hand side q when it is outside the block
    // (0 otherwise: an offset past the field)
    template <int M> __device__ void load_spinor(int q) {
        const RawView<S> f(in + (size_t)q * 12 * V, V);
#pragma unroll
        for (int k = 0; k < 12; k++) gm[k] = f.ld(k, nd[M]);
    }
    template <int M> __device__ void load_link() {
#pragma unroll
        for (int k = 0; k < (RECON ? 6 : 9); k++) gu[k] = U.template get<M / 2>().ld(k, M & 1 ? nb[M] : d);
    }
    // hop M of every right-hand side; the reads of the next one's operands from
    // memory run under its arithmetic (the branch, always taken, keeps the
    // scheduler from holding more than one step's operands)
    template <int M> __device__ void step() {
#pragma unroll
        for (int q = 0; q < R; q++)
            if (opaque_zero() == 0) {
                if (q == 0) {
#pragma unroll
                    for (int k = 0; k < (RECON ? 6 : 9); k++) u[k] = gu[k];
                }
                C<T> psi[12];
#pragma unroll
                for (int k = 0; k < 12; k++) psi[k] = widen_to(either(sp[(12 * q + k) * RS + ln[M]], gm[k]), T());
                __builtin_amdgcn_sched_barrier(0);
                if (q + 1 < R) {
                    load_spinor<M>(q + 1);
                } else if (M < 7) {
                    load_link<(M + 1) & 7>();
                    load_spinor<(M + 1) & 7>(0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (q == 0 && RECON) su3_row2<T>(u, M == 6 ? sf : M == 7 ? sb : (T)1);
                hop<T, M / 2, !(M & 1)>(acc[q], u, psi);
            }
    }
};

// The apply for nrhs > 1: a link and the clover term are read, and the link's
// third row rebuilt, once for R right-hand sides; the workgroup's spinors are in
// LDS as they are stored (S), a neighbour outside the block is the zero slot
// there and comes from memory, one step ahead. Every right-hand side goes
// through the operations of dirac_kernel in the same order, so that it gets
// the same bits from both. Bound: what misses L2. The workgroups in flight
// hold as much in LDS as the 4 MB of L2, so that most of a block's halo comes
// from beyond it (24^3 x 48, FP32, 12 right-hand sides: 4.0 GB read of the
// 1.1 GB that are there once). Before (R = 1) and after, 24^3 x 48: FP32 12
// right-hand sides 1106 -> 839 us, half storage 861 -> 588, FP64 4 621 -> 520.
// Not faster: the groups of one range of sites one after the other instead of
// together, links or clover term with the non-temporal policy (2 - 10 % slower).
template <typename T, typename S, typename O, bool RECON, int R, int WAVES>
__global__ __launch_bounds__(TPB) __attribute__((amdgpu_waves_per_eu(WAVES))) void dirac_block_kernel(
    Geom g, const C<T> *__restrict__ Up, const C<T> *__restrict__ Ap, const C<S> *__restrict__ in, C<O> *__restrict__ out,
    int nrhs, int ngr, int nwg, int antiperiodic) {
    __shared__ C<S> sp[R * 12 * RS];
    const int w = xcd_block(nwg);
    const int gr = w % ngr, r0 = min(gr * R, nrhs - R), first = gr * R - r0;   // the last group overlaps the one before
    const int d = site_in_lex_block_order(g, (w / ngr) * TPB + threadIdx.x), l = d & (TPB - 1);
    const size_t V = g.V;
    BlockHops<T, S, RECON, R> H(Up, V);
    H.in = in + (size_t)r0 * 12 * V;
    H.sp = sp;
    H.d = d;
    site_neighbours(g, d, H.nb);
#pragma unroll
    for (int m = 0; m < 8; m++) {
        const bool inside = (H.nb[m] ^ d) < TPB;
        H.ln[m] = inside ? H.nb[m] & (TPB - 1) : OUT;
        H.nd[m] = inside ? 12 * g.V : H.nb[m];
    }
    H.sf = H.sb = 1;
    if (RECON) time_link_signs<T>(g, d, antiperiodic, H.sf, H.sb);
#pragma unroll
    for (int q = 0; q < R; q++) {
        const RawView<S> f(H.in + (size_t)q * 12 * V, V);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            sp[(12 * q + k) * RS + l] = f.ld(k, d);
            H.acc[q][k] = mk<T>(0, 0);
        }
    }
    if (l < 12 * R) sp[l * RS + OUT] = mk<S>(0, 0);
    H.template load_link<0>();
    H.template load_spinor<0>(0);
    __syncthreads();
    H.template step<0>();
    H.template step<1>();
    H.template step<2>();
    H.template step<3>();
    H.template step<4>();
    H.template step<5>();
    H.template step<6>();
    H.template step<7>();
    const CloverViews<T> A(Ap, V);
#pragma unroll
    for (int h = 0; h < 2; h++) {
        C<T> p[18];
#pragma unroll
        for (int k = 0; k < 18; k++) p[k] = (h ? A.a1 : A.a0).ld(k, d);
#pragma unroll
        for (int q = 0; q < R; q++)
            if (q >= first) {
                C<T> psi[6], res[6];
#pragma unroll
                for (int k = 0; k < 6; k++) psi[k] = widen_to(sp[(12 * q + 6 * h + k) * RS + l], T());
                herm6_mv<T>(p, psi, res);
                const typename SpinorView<T, O>::type o(out + (size_t)(r0 + q) * 12 * V, V, 12);
#pragma unroll
                for (int k = 0; k < 6; k++)
                    o.template st<true>(6 * h + k, d, csub(res[k], cscale(H.acc[q][6 * h + k], (T)0.5)));
            }
    }
}

// ---- few sites: four lanes per site, one per direction

// h = (1 -+ gamma_mu) psi, upper half, and d, the 12 components that a hop with w
// = U h (or U^H h) adds to the sum: the two halves of hop() in stencil.h
template <typename T, int MU, bool FWD> __device__ inline void quad_project(const C<T> *psi, C<T> *h) {
    const C<T> *u0 = psi, *u1 = psi + 3, *l0 = psi + 6, *l1 = psi + 9;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const C<T> f0 = MU == 0 ? ci(l1[a]) : MU == 1 ? l1[a] : MU == 2 ? ci(l0[a]) : l0[a];
        const C<T> f1 = MU == 0 ? ci(l0[a]) : MU == 1 ? cneg(l0[a]) : MU == 2 ? cneg(ci(l1[a])) : l1[a];
        h[a] = FWD ? cadd(u0[a], f0) : csub(u0[a], f0);
        h[3 + a] = FWD ? cadd(u1[a], f1) : csub(u1[a], f1);
    }
}
template <typename T, int MU, bool FWD> __device__ inline void quad_lower(const C<T> *w, C<T> *d) {
#pragma unroll
    for (int a = 0; a < 3; a++) {
        // B^H w: (i w1, i w0), (w1, -w0), (i w0, -i w1), (-w0, -w1)
        const C<T> b0 = MU == 0 ? ci(w[3 + a]) : MU == 1 ? w[3 + a] : MU == 2 ? ci(w[a]) : cneg(w[a]);
        const C<T> b1 = MU == 0 ? ci(w[a]) : MU == 1 ? cneg(w[a]) : MU == 2 ? cneg(ci(w[3 + a])) : cneg(w[3 + a]);
        d[a] = FWD ? cneg(b0) : b0;
        d[3 + a] = FWD ? cneg(b1) : b1;
    }
}

// Lane mu of a site forms its forward and its backward hop, all its operands
// in flight at once; the sum then goes from lane to lane in the order of
// dirac_kernel's, so that both give the same bits. A lane finishes three
// components of the result. Bound: the latency of one chain of loads, where
// dirac_kernel has eight (and 16 of 256 CUs at work on 8^4 sites): 8^4, FP64, pass
// after pass 5.3 us against 11.6, the first on a new field after 2 GB of other
// traffic, waited for, 18.0 against 28.2.
constexpr int QSITES = 16;   // sites of a workgroup, one wave
template <typename T, typename S, typename O, bool RECON>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1))) void dirac_quad_kernel(
    Geom g, const C<T> *__restrict__ Up, const C<T> *__restrict__ Ap, const C<S> *__restrict__ in, C<O> *__restrict__ out,
    int antiperiodic) {
    __shared__ C<T> sum[12][QSITES];
    const int lane = threadIdx.x, m = lane & 3, ls = lane >> 2, h = m >> 1;
    const int i = blockIdx.x * QSITES + ls, d = i < g.V ? i : g.V - 1;
    const size_t V = g.V;
    in += (size_t)blockIdx.y * 12 * V;
    const int pos = d >> g.lgVb;
    int x[4], nf, nb, t;
    local_coords(g, d & (g.Vb - 1), x);
    t = (int)((g.blk_coord[pos] >> 24) << g.lb[3]) + x[3];
    {
        int xf[4], xb[4];
        bool fin = false, bin = false;
#pragma unroll
        for (int mu = 0; mu < 4; mu++) {
            const int bm = 1 << g.lb[mu];
            xf[mu] = mu == m ? (x[mu] + 1) & (bm - 1) : x[mu];
            xb[mu] = mu == m ? (x[mu] - 1) & (bm - 1) : x[mu];
            if (mu == m) {
                fin = x[mu] + 1 < bm || g.nb[mu] == 1;
                bin = x[mu] > 0 || g.nb[mu] == 1;
            }
        }
        const int pf = g.blk_nbr[pos * 8 + 2 * m], pb = g.blk_nbr[pos * 8 + 2 * m + 1];
        nf = ((fin ? pos : pf) << g.lgVb) + local_index(g, xf);
        nb = ((bin ? pos : pb) << g.lgVb) + local_index(g, xb);
    }
    const T sf = antiperiodic && m == 3 && t == g.L[3] - 1 ? (T)-1 : (T)1;
    const T sb = antiperiodic && m == 3 && t == 0 ? (T)-1 : (T)1;
    C<S> rf[12], rb[12], ro[6];
    C<T> uf[9], ub[9], p[18];
    const C<T> *Um = Up + (size_t)(9 * m) * V, *Ah = Ap + (size_t)(18 * h) * V;
#pragma unroll
    for (int k = 0; k < 12; k++) rf[k] = in[(size_t)k * V + nf];
#pragma unroll
    for (int k = 0; k < (RECON ? 6 : 9); k++) uf[k] = Um[(size_t)k * V + d];
#pragma unroll
    for (int k = 0; k < 12; k++) rb[k] = in[(size_t)k * V + nb];
#pragma unroll
    for (int k = 0; k < (RECON ? 6 : 9); k++) ub[k] = Um[(size_t)k * V + nb];
#pragma unroll
    for (int k = 0; k < 6; k++) ro[k] = in[(size_t)(6 * h + k) * V + d];
#pragma unroll
    for (int k = 0; k < 18; k++) p[k] = Ah[(size_t)k * V + d];
    __builtin_amdgcn_sched_barrier(0);
    C<T> hf[6], hb[6], wf[6], wb[6], df[6], db[6];
    {
        C<T> pf[12], pb[12];
#pragma unroll
        for (int k = 0; k < 12; k++) {
            pf[k] = widen_to(rf[k], T());
            pb[k] = widen_to(rb[k], T());
        }
#define PROJECT(MU)                          \
    if (m == MU) {                           \
        quad_project<T, MU, true>(pf, hf);   \
        quad_project<T, MU, false>(pb, hb);  \
    }
        PROJECT(0)
        PROJECT(1)
        PROJECT(2)
        PROJECT(3)
#undef PROJECT
    }
    if (RECON) {
        su3_row2<T>(uf, sf);
        su3_row2<T>(ub, sb);
    }
    su3_mv<T, false>(uf, hf, wf);
    su3_mv<T, false>(uf, hf + 3, wf + 3);
    su3_mv<T, true>(ub, hb, wb);
    su3_mv<T, true>(ub, hb + 3, wb + 3);
#define LOWER(MU)                           \
    if (m == MU) {                          \
        quad_lower<T, MU, true>(wf, df);    \
        quad_lower<T, MU, false>(wb, db);   \
    }
    LOWER(0)
    LOWER(1)
    LOWER(2)
    LOWER(3)
#undef LOWER
    C<T> acc[12];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const C<T> a = k < 6 ? wf[k] : df[k - 6], b = k < 6 ? wb[k] : db[k - 6];
        acc[k] = cadd(cadd(mk<T>(0, 0), a), b);
#pragma unroll
        for (int step = 0; step < 3; step++)   // from the lane before: lane 3 has the sum at the end
            acc[k] = cadd(cadd(mk<T>(dpp_mov<0x90>(acc[k].x), dpp_mov<0x90>(acc[k].y)), a), b);
    }
    if (m == 3)
#pragma unroll
        for (int k = 0; k < 12; k++) sum[k][ls] = acc[k];
    __syncthreads();
    C<T> own[6], res[6];
#pragma unroll
    for (int k = 0; k < 6; k++) own[k] = widen_to(ro[k], T());
    herm6_mv<T>(p, own, res);
    const typename SpinorView<T, O>::type o(out + (size_t)blockIdx.y * 12 * V, V, 12);
    if (i < g.V)
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const C<T> r = m & 1 ? res[3 + k] : res[k];
            o.st_lane(k, d, (unsigned)(3 * m) * o.cs, csub(r, cscale(sum[3 * m + k][ls], (T)0.5)));
        }
}

}  // namespace

// algorithmic bytes of one apply per site: links (two rows of each when they
// are rebuilt) and clover term once per launch, spinors in and out per field
static double dirac_launch_bytes(const Ctx *c, int prec, size_t in_bytes, size_t out_bytes, int nrhs) {
    const double real = prec == MGDD_F64 ? 8.0 : 4.0;
    const double links = 4 * (c->links_su3 ? 6 : 9) * 2 * real, clover = 72 * real;
    return (double)c->g.V * (links + clover + (double)(in_bytes + out_bytes) * nrhs);
}

// The staged kernels take one workgroup per lattice block: blocks of TPB
// sites. -1: an option the context cannot run.
static int dirac_staged(Ctx *c) {
    if (c->dirac_stage == 1 && c->g.Vb != TPB) {
        fail(c, MGDD_ESHAPE, "the staged Wilson-clover apply needs blocks of 256 sites");
        return -1;
    }
    return c->dirac_stage >= 0 && c->g.Vb == TPB ? 1 : 0;
}

// Right-hand sides per thread, 1: dirac_kernel / dirac_widen_kernel. FP32
// arithmetic: the count of 2 and 3 that takes less (24^3 x 48, 2: 71 us, 3: 66
// us each, the last group's repeated ones included; against 93). FP64: 2 (130
// against 155 us each), the one repeated of an odd count costing more than
// that up to 5 of them (3: 490 against 484 us). With fewer than 192 workgroups
// the chip is better filled by one each (8^4, FP32, 12 right-hand sides, 64
// workgroups: 18 against 11 us; 8^2 x 16^2, 6: 128 18.6, 192 14.3 against 18.4).
static int rhs_per_thread(const Ctx *c, bool f64, int nrhs) {
    const int two = (nrhs + 1) / 2, three = (nrhs + 2) / 3, nblk = c->g.V / TPB;
    if (nrhs < 2 || (f64 && nrhs % 2 && nrhs < 7)) return 1;
    if (!f64 && 66 * 3 * three <= 71 * 2 * two && nblk * three >= 192) return 3;
    return nblk * two >= 192 ? 2 : 1;
}

template <typename T, typename S, typename O, int R, int WAVES>
static void launch_block(Ctx *c, const void *U, const void *A, const void *in, void *out, int nrhs) {
    const int ngr = (nrhs + R - 1) / R, nwg = c->g.V / TPB * ngr, anti = c->t_antiperiodic ? 1 : 0;
#define BLOCK(RECON)                                                                                            \
    dirac_block_kernel<T, S, O, RECON, R, WAVES><<<nwg, TPB, 0, c->stream>>>(                                   \
        c->g, (const C<T> *)U, (const C<T> *)A, (const C<S> *)in, (C<O> *)out, nrhs, ngr, nwg, anti)
    if (c->links_su3) BLOCK(true); else BLOCK(false);
#undef BLOCK
}

// Four lanes per site up to 16384 sites of all right-hand sides together, where
// the other kernels leave most CUs idle and take the time of their chain of
// loads (8^4, 1 right-hand side, FP64 6.0 against 10.3 us, FP32 5.4 against 9.0,
// half storage 5.5 / 8.9; 4: 9.8 / 12.0, 7.9 / 9.0, 7.2 / 8.8; 8^2 x 16^2: 9.1 /
// 12.9, 7.7 / 9.9, 7.0 / 9.2). Past that its four lanes per site, each with the
// registers of a wave per SIMD, are too many: 32768 sites, 8 x 16^3: 17.1 against
// 15.1, 11.6 / 10.8, 10.1 / 10.3; 8^2 x 16^2, 2: 16.7 / 14.2, 11.5 / 10.2.
static bool few_sites(const Ctx *c, int nrhs) { return c->dirac_stage == 0 && (size_t)c->g.V * nrhs <= 16384; }

template <typename T, typename S, typename O>
static void launch_quad(Ctx *c, const void *U, const void *A, const void *in, void *out, int nrhs) {
    const dim3 grid((c->g.V + QSITES - 1) / QSITES, nrhs);
    const int anti = c->t_antiperiodic ? 1 : 0;
#define QUAD(RECON)                                                                                                  \
    dirac_quad_kernel<T, S, O, RECON><<<grid, 64, 0, c->stream>>>(c->g, (const C<T> *)U, (const C<T> *)A,            \
                                                                  (const C<S> *)in, (C<O> *)out, anti)
    if (c->links_su3) QUAD(true); else QUAD(false);
#undef QUAD
}

int launch_dirac_widen(Ctx *c, int nrhs, const void *in32, void *out64, int in_prec) {
    int nwg = ((c->g.V + TPB - 1) / TPB) * nrhs;
    const int anti = c->t_antiperiodic ? 1 : 0;
    const int st = dirac_staged(c);
    if (st < 0) return MGDD_ESHAPE;
    const bool stage = st == 1;
    const int slot = kt_begin(c);
    if (few_sites(c, nrhs)) {
        if (in_prec == MGDD_F16) launch_quad<double, _Float16, double>(c, c->U64, c->A64, in32, out64, nrhs);
        else launch_quad<double, float, double>(c, c->U64, c->A64, in32, out64, nrhs);
    } else if (stage && rhs_per_thread(c, true, nrhs) == 2) {   // 16^3 x 32, 4 right-hand sides: 102 -> 78 us
        if (in_prec == MGDD_F16) launch_block<double, _Float16, double, 2, 1>(c, c->U64, c->A64, in32, out64, nrhs);
        else launch_block<double, float, double, 2, 1>(c, c->U64, c->A64, in32, out64, nrhs);
    } else {
#define WIDEN(R, G, S)                                                                                                \
    dirac_widen_kernel<R, G, S><<<nwg, TPB, 0, c->stream>>>(c->g, (const double2 *)c->U64, (const double2 *)c->A64,  \
                                                            (const C<S> *)in32, (double2 *)out64, nrhs, nwg, anti)
#define WIDEN_S(S)                                                                                                    \
    do {                                                                                                              \
        if (c->links_su3) {                                                                                           \
            if (stage) WIDEN(true, true, S); else WIDEN(true, false, S);                                              \
        } else {                                                                                                      \
            if (stage) WIDEN(false, true, S); else WIDEN(false, false, S);                                            \
        }                                                                                                             \
    } while (0)
    if (in_prec == MGDD_F16) WIDEN_S(_Float16); else WIDEN_S(float);
    }
#undef WIDEN_S
#undef WIDEN
    kt_end(c, slot, KF_DIRAC, MGDD_F64, (double)c->g.V * nrhs,
           dirac_launch_bytes(c, MGDD_F64, 12 * csize(in_prec), 192, nrhs));
    return hip_check(c, hipGetLastError(), "dirac kernel");
}

int launch_dirac(Ctx *c, int prec, int nrhs, const void *in, void *out) {
    int nwg = ((c->g.V + TPB - 1) / TPB) * nrhs;
    const int anti = c->t_antiperiodic ? 1 : 0;
    const int st = dirac_staged(c);
    if (st < 0) return MGDD_ESHAPE;
    const bool stage = st == 1;
    const int slot = kt_begin(c);
#define DIRAC(T, S, R, G)                                                                                             \
    dirac_kernel<T, S, R, G><<<nwg, TPB, 0, c->stream>>>(c->g, (const C<T> *)(prec == MGDD_F64 ? c->U64 : c->U32),    \
                                                         (const C<T> *)(prec == MGDD_F64 ? c->A64 : c->A32),          \
                                                         (const C<S> *)in, (C<S> *)out, nrhs, nwg, anti)
#define DIRAC_STAGED(T)                                                                                               \
    do {                                                                                                              \
        if (c->links_su3) {                                                                                           \
            if (stage) DIRAC(T, T, true, true); else DIRAC(T, T, true, false);                                        \
        } else {                                                                                                      \
            if (stage) DIRAC(T, T, false, true); else DIRAC(T, T, false, false);                                      \
        }                                                                                                             \
    } while (0)
    const int per = stage ? rhs_per_thread(c, prec == MGDD_F64, nrhs) : 1;
    if (few_sites(c, nrhs)) {
        if (prec == MGDD_F64) launch_quad<double, double, double>(c, c->U64, c->A64, in, out, nrhs);
        else if (prec == MGDD_F32) launch_quad<float, float, float>(c, c->U32, c->A32, in, out, nrhs);
        else launch_quad<float, _Float16, _Float16>(c, c->U32, c->A32, in, out, nrhs);
    } else if (per > 1) {
        if (prec == MGDD_F64) launch_block<double, double, double, 2, 1>(c, c->U64, c->A64, in, out, nrhs);
        else if (prec == MGDD_F32 && per == 2) launch_block<float, float, float, 2, 3>(c, c->U32, c->A32, in, out, nrhs);
        else if (prec == MGDD_F32) launch_block<float, float, float, 3, 2>(c, c->U32, c->A32, in, out, nrhs);
        else if (per == 2) launch_block<float, _Float16, _Float16, 2, 3>(c, c->U32, c->A32, in, out, nrhs);
        else launch_block<float, _Float16, _Float16, 3, 2>(c, c->U32, c->A32, in, out, nrhs);
    } else if (prec == MGDD_F64) {
        DIRAC_STAGED(double);
    } else if (prec == MGDD_F32) {
        DIRAC_STAGED(float);
    } else {
        if (c->links_su3) DIRAC(float, _Float16, true, false); else DIRAC(float, _Float16, false, false);
    }
#undef DIRAC_STAGED
#undef DIRAC
    const size_t sp = 12 * csize(prec);
    kt_end(c, slot, KF_DIRAC, prec, (double)c->g.V * nrhs, dirac_launch_bytes(c, prec, sp, sp, nrhs));
    return hip_check(c, hipGetLastError(), "dirac kernel");
}

}  // namespace mgdd
