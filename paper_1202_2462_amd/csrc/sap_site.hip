// Red-Black Schwarz colour step (Section 2, Algorithm 2.1) with minimal-residual
// block solves for special unitary links: one workgroup per lattice block, one
// lane per site, all 12 components of rho, e and q in registers. rho and the
// first two rows of the block's forward links are in LDS (74.6 KB for a 4^4
// block in FP32: two blocks per CU, one's memory phase under the other's MR
// steps); row 2 is rebuilt where a link is used.
//
// The hops of one direction are taken together: with w_f = U h_f and S = w_f +
// U^H h_b in one chain, the upper spins receive S and the lower ones B^H (S -
// 2 w_f). A neighbour outside the block is a zero spinor (the slot after the
// block's sites), so that every lane runs the same instructions; in the residual
// it is read from memory, the arithmetic being shared.
//
// Bound: issue of vector instructions (48^3 x 96: busy for 76 %; 1245 B per site
// update between L2 and memory of 768 that are there once). One sweep of 32^3 x
// 64, 4 MR steps, FP32: 646 us; with two lanes per site, which exchange half of
// each hop sum and select by chirality, 763 us.
#include "lanes.h"
#include "schwarz.h"
#include "stencil.h"

namespace mgdd {

namespace {

// h = (1 - gamma_mu) psi (FWD) or (1 + gamma_mu) psi, upper half
template <int MU, bool FWD> __device__ inline void project(const float2 *psi, float2 *h) {
    const float2 *u0 = psi, *u1 = psi + 3, *l0 = psi + 6, *l1 = psi + 9;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        // -B l of the forward hop: (i l1, i l0), (l1, -l0), (i l0, -i l1), (l0, l1)
        const float2 f0 = MU == 0 ? ci(l1[a]) : MU == 1 ? l1[a] : MU == 2 ? ci(l0[a]) : l0[a];
        const float2 f1 = MU == 0 ? ci(l0[a]) : MU == 1 ? cneg(l0[a]) : MU == 2 ? cneg(ci(l1[a])) : l1[a];
        h[a] = FWD ? cadd(u0[a], f0) : csub(u0[a], f0);
        h[3 + a] = FWD ? cadd(u1[a], f1) : csub(u1[a], f1);
    }
}

// w = U h of the forward hop of direction MU: psi the forward neighbour's
// spinor, u the site's link, its third row rebuilt here (sign: see su3_row2)
template <int MU> __device__ inline void forward_half(const float2 *psi, float2 *u, float sign, float2 *w) {
    float2 h[6];
    su3_row2<float>(u, sign);
    project<MU, true>(psi, h);
    su3_mv<float, false>(u, h, w);
    su3_mv<float, false>(u, h + 3, w + 3);
}

// acc += both hops of direction MU (acc = for MU = 0): w of the forward one,
// psi and u the backward neighbour's spinor and link
template <int MU>
__device__ inline void add_hops(float2 *acc, const float2 *w, const float2 *psi, float2 *u, float sign) {
    float2 h[6], s[6];
    su3_row2<float>(u, sign);
    project<MU, false>(psi, h);
#pragma unroll
    for (int q = 0; q < 2; q++)
#pragma unroll
        for (int a = 0; a < 3; a++) {
            float2 v = w[3 * q + a];
#pragma unroll
            for (int b = 0; b < 3; b++) cfmac(v, u[b * 3 + a], h[3 * q + b]);
            s[3 * q + a] = v;
        }
    // d = w_b - w_f = S - 2 w_f; B^H d = (i d1, i d0), (d1, -d0), (i d0, -i d1), (-d0, -d1)
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const float2 d0 = make_float2(fmaf(-2.f, w[a].x, s[a].x), fmaf(-2.f, w[a].y, s[a].y));
        const float2 d1 = make_float2(fmaf(-2.f, w[3 + a].x, s[3 + a].x), fmaf(-2.f, w[3 + a].y, s[3 + a].y));
        const float2 b0 = MU == 0 ? ci(d1) : MU == 1 ? d1 : MU == 2 ? ci(d0) : cneg(d0);
        const float2 b1 = MU == 0 ? ci(d0) : MU == 1 ? cneg(d0) : MU == 2 ? cneg(ci(d1)) : cneg(d1);
        if (MU == 0) {
            acc[a] = s[a];
            acc[3 + a] = s[3 + a];
            acc[6 + a] = b0;
            acc[9 + a] = b1;
        } else {
            acc[a] = cadd(acc[a], s[a]);
            acc[3 + a] = cadd(acc[3 + a], s[3 + a]);
            acc[6 + a] = cadd(acc[6 + a], b0);
            acc[9 + a] = cadd(acc[9 + a], b1);
        }
    }
}

// a where b is +0, b where a is
__device__ inline float2 either(float2 a, float2 b) {
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    return __builtin_bit_cast(float2, make_uint2(x.x | y.x, x.y | y.y));
}

// sums of (a, b, c) over the workgroup, in every lane: lane permutations in
// each wave, then the waves' sums in order; one barrier. red: 4 values a wave
template <int NW> __device__ inline void block_sum(float &a, float &b, float &c, float *red) {
    float v = swap_add<16>(swap_add<32>(a, b), swap_add<32>(c, c));   // rows of 16 lanes: a, c, b, c
    v += dpp_mov<0x128>(v);
    v = sum_of_8(v);
    const int lane = threadIdx.x & 63;
    if (!(lane & 15)) red[(threadIdx.x >> 6) * 4 + (lane >> 4)] = v;
    __syncthreads();
    a = red[0];
    c = red[1];
    b = red[2];
#pragma unroll
    for (int w = 1; w < NW; w++) {
        a += red[4 * w];
        c += red[4 * w + 1];
        b += red[4 * w + 2];
    }
}

// S: storage of the spinor fields (FP32, or half precision with FP32
// arithmetic, z rounded once when it is stored); SHIFT: a nonzero shift
template <int VB, typename S, bool SHIFT>
__global__ __launch_bounds__(VB) __attribute__((amdgpu_waves_per_eu(2, 2))) void sap_site_kernel(
    Geom g, const float2 *__restrict__ Up, const float2 *__restrict__ Ap, const void *__restrict__ b,
    void *__restrict__ z, int colour, int mr, float2 shift, int antiperiodic) {
    using FV = typename F32Store<S>::view;
    constexpr int RS = VB + 4, LS = VB + 2, OUT = VB;   // OUT: the zero slot
    extern __shared__ unsigned char smem[];
    float2 *rl = (float2 *)smem;                // [12][RS]: z, then rho
    float2 *lk = rl + 12 * RS;                // [4][6][LS]: rows 0, 1 of each site's forward links
    float *red = (float *)(lk + 24 * LS);           // [4 VB / 64]
    const size_t V = g.V;
    const int pos = (colour ? g.ncol0 : 0) + xcd_block(gridDim.x);
    const int l = threadIdx.x, d = pos * VB + l;
    const size_t roff = (size_t)blockIdx.y * 12 * V * F32Store<S>::ESZ;   // bytes
    const LinkViews<float> U(Up, V);
    const CloverViews<float> A(Ap, V);
    const FV bf((const float2 *)((const char *)b + roff), V, 12), zf((const float2 *)((const char *)z + roff), V, 12);

    // neighbours: local index (wrapped), OUT when it lies outside the block
    int x[4], lw[8], ln[8];
    local_coords(g, l, x);
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const int mu = q >> 1, bm = 1 << g.lb[mu];
        int y[4] = {x[0], x[1], x[2], x[3]};
        y[mu] += q & 1 ? -1 : 1;
        const bool in = (y[mu] >= 0 && y[mu] < bm) || g.nb[mu] == 1;
        y[mu] &= bm - 1;
        lw[q] = local_index(g, y);
        ln[q] = in ? lw[q] : OUT;
    }
    float sf = 1, sb = 1;
    {
        const int t = (int)((g.blk_coord[pos] >> 24) << g.lb[3]) + x[3];
        if (antiperiodic && t == g.L[3] - 1) sf = -1;
        if (antiperiodic && t == 0) sb = -1;
    }

    // data read or written once (links, z, b) with the non-temporal policy, so
    // that the clover rows, which every MR step reads again, stay in L2
#define STAGE(MU)                                                                                     \
    _Pragma("unroll") for (int k = 0; k < 6; k++) lk[(6 * MU + k) * LS + l] = U.template get<MU>().template ld<true>(k, d)
    STAGE(0);
    STAGE(1);
    STAGE(2);
    STAGE(3);
#undef STAGE
    float2 zs[12];
#pragma unroll
    for (int c = 0; c < 12; c++) {
        zs[c] = zf.template ld<true>(c, d);
        rl[c * RS + l] = zs[c];
    }
    if (l < 12) rl[l * RS + OUT] = make_float2(0.f, 0.f);
    if (l < 24) lk[l * LS + OUT] = make_float2(0.f, 0.f);
    __syncthreads();

    // r = b - (D - shift) z
    float2 rho[12], e[12], acc[12];
#pragma unroll
    for (int c = 0; c < 12; c++) acc[c] = make_float2(0.f, 0.f);
    // a neighbour inside the block from LDS (memory: an offset past the field,
    // which reads as 0), one outside from memory (LDS: the zero slot); a
    // direction's reads from memory are in flight while the one before it is
    // computed, the clover term's during the last
    const int none = 12 * g.V;
    float2 gf[12], gb[12], gu[6], a0[18], a1[18];
#define FROM_MEMORY(MU)                                                                                          \
    {                                                                                                            \
        const int nf = ln[2 * MU] == OUT ? g.blk_nbr[pos * 8 + 2 * MU] * VB + lw[2 * MU] : none;                 \
        const int nb = ln[2 * MU + 1] == OUT ? g.blk_nbr[pos * 8 + 2 * MU + 1] * VB + lw[2 * MU + 1] : none;     \
        _Pragma("unroll") for (int c = 0; c < 12; c++) gf[c] = zf.ld(c, nf);                                     \
        _Pragma("unroll") for (int c = 0; c < 12; c++) gb[c] = zf.ld(c, nb);                                     \
        _Pragma("unroll") for (int k = 0; k < 6; k++) gu[k] = U.template get<MU>().ld(k, nb);                    \
    }
#define RESIDUAL(MU, NEXT)                                                                                       \
    if (opaque_zero() == 0) {                                                                                    \
        float2 pf[12], pb[12], uf[9], ub[9], w[6];                                                                 \
        const int f = ln[2 * MU], bk = ln[2 * MU + 1];                                                           \
        _Pragma("unroll") for (int c = 0; c < 12; c++) pf[c] = either(rl[c * RS + f], gf[c]);                    \
        _Pragma("unroll") for (int k = 0; k < 6; k++) uf[k] = lk[(6 * MU + k) * LS + l];                         \
        _Pragma("unroll") for (int c = 0; c < 12; c++) pb[c] = either(rl[c * RS + bk], gb[c]);                   \
        _Pragma("unroll") for (int k = 0; k < 6; k++) ub[k] = either(lk[(6 * MU + k) * LS + bk], gu[k]);         \
        __builtin_amdgcn_sched_barrier(0);                                                                       \
        NEXT;                                                                                                    \
        __builtin_amdgcn_sched_barrier(0);                                                                       \
        forward_half<MU>(pf, uf, MU == 3 ? sf : 1.f, w);                                                     \
        add_hops<MU>(acc, w, pb, ub, MU == 3 ? sb : 1.f);                                                    \
    }
    FROM_MEMORY(0)
    RESIDUAL(0, FROM_MEMORY(1))
    RESIDUAL(1, FROM_MEMORY(2))
    RESIDUAL(2, FROM_MEMORY(3))
    RESIDUAL(3, _Pragma("unroll") for (int k = 0; k < 18; k++) {
        a0[k] = A.a0.template ld<true>(k, d);
        a1[k] = A.a1.template ld<true>(k, d);
    })
#undef RESIDUAL
#undef FROM_MEMORY
    herm6_mv<float>(a0, zs, rho);
    herm6_mv<float>(a1, zs + 6, rho + 6);
#pragma unroll
    for (int c = 0; c < 12; c++) {
        float2 az = make_float2(fmaf(-0.5f, acc[c].x, rho[c].x), fmaf(-0.5f, acc[c].y, rho[c].y));
        if (SHIFT) cfma(az, cneg(shift), zs[c]);
        rho[c] = csub(bf.template ld<true>(c, d), az);
        e[c] = make_float2(0.f, 0.f);
    }
    __syncthreads();   // every lane has read z from LDS
#pragma unroll
    for (int c = 0; c < 12; c++) rl[c * RS + l] = rho[c];
    __syncthreads();

    for (int it = 0; it < mr; it++) {
        float2 q[12];
        // the LDS reads of a hop run under the arithmetic of the one before it
        float2 pf[12], uf[9];
#define READ_FORWARD(MU)                                                                            \
    {                                                                                               \
        _Pragma("unroll") for (int c = 0; c < 12; c++) pf[c] = rl[c * RS + ln[2 * MU]];             \
        _Pragma("unroll") for (int k = 0; k < 6; k++) uf[k] = lk[(6 * MU + k) * LS + l];            \
    }
#define BLOCK_HOPS(MU, NEXT)                                                                        \
    if (opaque_zero() == 0) {                                                                       \
        float2 pb[12], ub[9], w[6];                                                                   \
        _Pragma("unroll") for (int c = 0; c < 12; c++) pb[c] = rl[c * RS + ln[2 * MU + 1]];         \
        _Pragma("unroll") for (int k = 0; k < 6; k++) ub[k] = lk[(6 * MU + k) * LS + ln[2 * MU + 1]]; \
        __builtin_amdgcn_sched_barrier(0);                                                          \
        forward_half<MU>(pf, uf, MU == 3 ? sf : 1.f, w);                                        \
        __builtin_amdgcn_sched_barrier(0);                                                          \
        NEXT;                                                                                       \
        __builtin_amdgcn_sched_barrier(0);                                                          \
        add_hops<MU>(acc, w, pb, ub, MU == 3 ? sb : 1.f);                                       \
    }
        READ_FORWARD(0)
        BLOCK_HOPS(0, READ_FORWARD(1))
        BLOCK_HOPS(1, READ_FORWARD(2))
        BLOCK_HOPS(2, READ_FORWARD(3))
        BLOCK_HOPS(3, )
#undef READ_FORWARD
#undef BLOCK_HOPS
        herm6_mv<float>(a0, rho, q);
        herm6_mv<float>(a1, rho + 6, q + 6);
        float sa = 0, sr = 0, si = 0;
#pragma unroll
        for (int c = 0; c < 12; c++) {
            q[c] = make_float2(fmaf(-0.5f, acc[c].x, q[c].x), fmaf(-0.5f, acc[c].y, q[c].y));
            if (SHIFT) cfma(q[c], cneg(shift), rho[c]);
            // |q|^2 and conj(q) rho
            sa = fmaf(q[c].x, q[c].x, sa);
            sa = fmaf(q[c].y, q[c].y, sa);
            sr = fmaf(q[c].x, rho[c].x, sr);
            sr = fmaf(q[c].y, rho[c].y, sr);
            si = fmaf(q[c].x, rho[c].y, si);
            si = fmaf(-q[c].y, rho[c].x, si);
        }
        block_sum<VB / 64>(sa, sr, si, red);
        if (sa == 0.f) break;
        const float2 alpha = make_float2(sr / sa, si / sa), minus = cneg(alpha);
#pragma unroll
        for (int c = 0; c < 12; c++) {
            cfma(e[c], alpha, rho[c]);
            cfma(rho[c], minus, q[c]);
        }
        if (it + 1 < mr) {
#pragma unroll
            for (int c = 0; c < 12; c++) rl[c * RS + l] = rho[c];
            __syncthreads();
        }
    }
#pragma unroll
    for (int c = 0; c < 12; c++) zf.template st<true>(c, d, cadd(zf.template ld<true>(c, d), e[c]));
}

}  // namespace

size_t sap_site_lds(int Vb) { return 8 * (12 * ((size_t)Vb + 4) + 24 * ((size_t)Vb + 2)) + 4 * 4 * (Vb / 64); }

int launch_sap_site(Ctx *c, int prec, int nrhs, int col, int mr, double sre, double sim, const void *b, void *z) {
    const Geom &g = c->g;
    const dim3 grid(col ? g.nblocks - g.ncol0 : g.ncol0, nrhs);
    const size_t lds = sap_site_lds(g.Vb);
    const bool shifted = sre != 0 || sim != 0;
    const int anti = c->t_antiperiodic ? 1 : 0;
#define SITE32(VB, S, SH)                                                                                        \
    sap_site_kernel<VB, S, SH><<<grid, VB, lds, c->stream>>>(g, (const float2 *)c->U32, (const float2 *)c->A32, b, z, \
                                                             col, mr, make_float2((float)sre, (float)sim), anti)
#define SITE(VB)                                                                  \
    do {                                                                          \
        if (prec == MGDD_F32) {                                                   \
            if (shifted) SITE32(VB, float, true); else SITE32(VB, float, false);  \
        } else {                                                                  \
            if (shifted) SITE32(VB, _Float16, true); else SITE32(VB, _Float16, false); \
        }                                                                         \
    } while (0)
    if (g.Vb == 256) SITE(256);
    else if (g.Vb == 128) SITE(128);
    else SITE(64);
#undef SITE
#undef SITE32
    return hip_check(c, hipGetLastError(), "sap kernel");
}

}  // namespace mgdd
