// Aggregation interpolation, restriction, prolongation and the coarse
// operator (see transfer.hip).
#pragma once

#include "mgdd_internal.h"

namespace mgdd {

struct AggGeom {
    int a[4];
};

// A 9-point stencil operator with 2N x 2N complex blocks per site (D_c on the
// coarse lattice, D_cc on the level-3 lattice): sites, N, neighbour table
// [V][9] (self first), blocks [V][9][col][row] in FP64 and FP32.
struct StencilOp {
    int V = 0, N = 0;
    const int *nbr = nullptr;
    const void *D64 = nullptr, *D32 = nullptr;
    const void *H32 = nullptr;   // [V][5][col][row] FP32 self and forward blocks, or null
    const int *order = nullptr;  // [V] visiting order of the sites (null: index order)
};
inline StencilOp level1_op(const Ctx *c) {
    StencilOp o;
    o.V = c->c.Vc;
    o.N = c->c.N;
    o.nbr = c->c.cnbr;
    o.D64 = c->c.Dc64;
    o.D32 = c->c.Dc32;
    o.H32 = c->c.Dh32;
    o.order = c->c.corder;
    return o;
}
inline StencilOp level2_op(const Ctx *c) {
    StencilOp o;
    o.V = c->c2.Vcc;
    o.N = c->c2.N2;
    o.nbr = c->c2.cnbr2;
    o.D64 = c->c2.Dcc64;
    o.D32 = c->c2.Dcc32;
    return o;
}
int launch_stencil_apply(Ctx *c, const StencilOp &op, int prec, int nrhs, const void *in, void *out);

// tables and buffers of the coarse level for aggregates agg and N test vectors
int transfer_setup(Ctx *c, const int *agg, int N);
// P from N FP64 fine fields (device layout); FP32 copy made too. MGDD_ERANK if rank deficient.
int launch_build_P(Ctx *c, const void *tv64);
int launch_restrict(Ctx *c, int prec, int nrhs, const void *fine, void *coarse);

// How a restriction divides the N test vectors of an (aggregate, chirality)
// pair: `parts` workgroups of `per` consecutive ones, the last with what is
// left, none with nothing (the kernel loads a part's first column of P at once).
// Few workgroups (one per pair and group of right-hand sides): up to 4 parts,
// so that the launch fills the chip.
struct RestrictSplit {
    int parts, per;
};
inline RestrictSplit restrict_split(int N, size_t workgroups) {
    int ks = 1;
    while (ks < 4 && ks < N && workgroups * ks < 1024) ks *= 2;
    const int per = (N + ks - 1) / ks;
    return {(N + per - 1) / per, per};
}
int launch_prolong(Ctx *c, int prec, int nrhs, const void *coarse, void *fine);
int launch_coarse_build(Ctx *c);

// How the D_c build divides the Va sites of an aggregate's self term: `parts`
// (at most 4) workgroups of `per` sites, the last with what is left, none with
// nothing; per is a multiple of the kernel's step. Up to 512 aggregates the
// self terms, four times as long as the hops on 4^4 sites and with four hops a
// site, would be what the launch waits for. P and D_c together, one part / four: 16
// aggregates (8^4), N = 8: 176 / 104 us, N = 20: 468 / 235; 512 (16^3 x 32), N =
// 8: 662 / 573, N = 20: 2.18 / 1.99 ms. More fill the chip either way: 24^3 x 48,
// 3x4x4x4 sites, N = 21: 13.45 / 13.68 ms.
struct DcSplit {
    int parts, per;
};
inline DcSplit dc_split(int Va, int Vc, int step) {
    const int steps = (Va + step - 1) / step, most = Vc <= 512 ? 4 : 1, per = (steps + most - 1) / most;
    return {(steps + per - 1) / per, per * step};
}
int launch_coarse_apply(Ctx *c, int prec, int nrhs, const void *in, void *out);

// Fused Arnoldi process on D_c for the coarse GMRES (arnoldi.hip); m <= 15.
constexpr int ARNOLDI_FUSED_MAX_STEPS = 15;
size_t coarse_arnoldi_scratch(const StencilOp &op, int m, int nb);
// The same on a compact FP32 D_c (op.H32) with every block read once per step
// (arnoldi_compact.hip); scratch: compact_arnoldi_scratch bytes.
size_t compact_arnoldi_scratch(const StencilOp &op, int m, int nb);
int launch_compact_arnoldi(Ctx *c, const StencilOp &op, int m, int nb, const void *b, void *const *V, void *work0,
                           void *work1, void *scratch, double2 *H1, double2 *H2, double2 *NR);
// w <- w - V V^H w twice (nb segments of n), three passes; k <= 64 vectors.
constexpr int FUSED_CGS2_MAX = 64;
int fused_cgs2(Ctx *c, int p, size_t n, int nb, void *const *V, int k, void *w, double2 *h1, double2 *h2,
               double2 *nrm);
int launch_coarse_arnoldi(Ctx *c, const StencilOp &op, int p, int m, int nb, const void *b, void *const *V,
                          void *work0, void *work1, void *scratch, double2 *H1, double2 *H2, double2 *NR);
// Least squares of a GMRES cycle on the device (arnoldi.hip): coef[i][s] = y_i
// of min ||beta e_1 - H y|| from the Gram-Schmidt outputs h1, h2, nr of m
// steps (the layout of launch_coarse_arnoldi); *status (may be null) set to
// 1 on a non-finite result. m <= LSQ_MAX_STEPS.
constexpr int LSQ_MAX_STEPS = 32;
int launch_hessenberg_lsq(Ctx *c, int m, int nb, const double2 *h1, const double2 *h2, const double2 *nr, double2 *coef,
                          int *status);

}  // namespace mgdd
