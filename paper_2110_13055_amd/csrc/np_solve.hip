// np_solve.hip -- implicit ion transport: backward-Euler steps and the steady
// state of the Nernst-Planck equations, Eq. (3), with the adsorption law of
// Eq. (6), for a frozen flow and potential (the paper discretises Eq. 3 with
// an implicit finite-volume method, Sec. 2).
//
// The cell balance is the explicit step's: Scharfetter-Gummel face fluxes
// F = alpha C_P - beta C_N with alpha = D Bs(Pe) + w/2, beta = D Bs(Pe) -
// w/2 (w the face-normal drift, Bs(x) = (x/2) coth(x/2)), k_eff C_P on
// electrode faces, the inlet ghost at c0, the open or Dirichlet outlet. The
// coefficients are evaluated in FP32 exactly as the explicit step does; the
// operator is applied in FP64. For species s the outflow is A_s C - b_s; a
// backward-Euler step solves (I/dt + A_s) C' = C/dt + b_s and the steady
// state A_s C = b_s, both by BiCGSTAB (van der Vorst 1992) with right
// preconditioning (block_solve below), both species in the same kernels with
// their own scalars, side by side in memory: one load brings a node's pair.
// Persistent workgroups and fixed-order partial sums as in pot.hip: every
// workgroup derives the same scalars, and the iterate does not depend on
// timing or on how often the host checks.
//
// Iteration k (species s, M the preconditioner). The vectors are FP64; the
// preconditioned directions p^ = M p and s^ = M s are FP32 numbers, the same
// ones where A is applied and where x is updated, so that their rounding
// changes M and not the balance of x and r. s replaces r.
//   dir     stop test on |r_k|; beta = (rho_k / rho_{k-1}) (alpha / omega);
//           p = r + beta (p - omega v); p^ = M p
//   apply   v = A p^; partial rhat . v
//   sdir    alpha = rho_k / (rhat . v); s = r - alpha v; s^ = M s
//   apply   t = A s^; partials t . s, t . t
//   update  omega = (t . s) / (t . t); x += alpha p^ + omega s^;
//           r = s - omega t; partials rho_{k+1} = rhat . r, |r|^2
// A species whose residual met the tolerance is frozen (its partials stop
// changing, so every later test repeats the decision; its scalars are zero,
// which keeps its x and r).
#include <algorithm>

#include "cdi_internal.h"
#include "device_common.h"
#include "np_solve_internal.h"
#include "reduce_common.h"

namespace cdi {

namespace {

// Partial-sum regions, 2 species x G doubles each.
enum { kRv = 0, kTs = 1, kTt = 2, kRho0 = 3, kRho1 = 4, kRr = 5, kBb = 6, kRegions = 7 };

__device__ inline double *reg(const NpsArgs &a, int r, int s) { return a.part + ((size_t)r * 2 + s) * a.G; }

__device__ __forceinline__ float of_species(float2 c, int s) { return s ? c.y : c.x; }
__device__ __forceinline__ double of_species(double2 c, int s) { return s ? c.y : c.x; }

// alpha, beta of a face from the half drift hw (the explicit step's Bs).
__device__ inline void sg_coef(float D, float invD2, float hw, float &al, float &be)
{
    const float pe = hw * invD2;
    const float x2 = pe * pe;
    float bs;
    if (x2 < 0.25f) {
        bs = fmaf(x2, fmaf(x2, fmaf(x2, 1.f / 30240.f, -1.f / 720.f), 1.f / 12.f), 1.f);
    } else {
        const float a = fabsf(pe);
        const float e = __expf(a);
        bs = 0.5f * a * (e + 1.f) * __builtin_amdgcn_rcpf(e - 1.f);
    }
    const float db = D * bs;
    al = db + hw;
    be = db - hw;
}

// Faces of node n: neighbour map values, and per species the coefficient of
// the node's own concentration (al) and either the neighbour's (be, fluid
// faces) or the ghost's constant term (be, open x-end faces), so that a
// face's outflow is al C_P - be C_N or al C_P - be; b = the sum of the ghost
// terms (the constant inflow); diag = sum of al.
template <class L>
struct NpNode {
    int m[2 * L::D];
    float al[2][2 * L::D], be[2][2 * L::D];
    double b[2];
    float diag[2];
    float adv;  // largest half drift of the flow across a face to a fluid cell
};

// Its neighbours, from the list when the instance has one built with the ions'
// x periodicity (read with the node's data), else through the coordinates and
// the map.
template <class L>
__device__ __forceinline__ void np_faces(const Grid &g, const Phys &p, int n, NpNode<L> &c)
{
    constexpr int D = L::D;
    const int P = g.P;
    if (g.nbr && (p.npx == kNpxPeriodic) == (g.periodic_x != 0)) {
#pragma unroll
        for (int k = 0; k < 2 * D; ++k) c.m[k] = ldu(g.nbr + (size_t)k * P, (uint32_t)n);
    } else {
        int x, y, z;
        unpack_xyz(g, ldu(g.fluid, (uint32_t)n), x, y, z);
        NbCtx ctx;
        nb_ctx<L>(g, x, y, z, p.npx == kNpxPeriodic, ctx);
#pragma unroll
        for (int k = 0; k < 2 * D; ++k) c.m[k] = nb_get<L>(g, ctx, k + 1);
    }
}

// Its coefficients, after np_faces. Every load is issued before the per-face
// branches (a load inside a divergent branch waits for its data before the
// next face starts): the flux (and potential) of each neighbour, at the node
// itself where the face is not fluid.
template <class L>
__device__ __forceinline__ void np_coefs(const Grid &g, const Phys &p, const float *j, int n, NpNode<L> &c)
{
    constexpr int D = L::D;
    const int P = g.P;
    float jP[3], jN[2 * D], psiN[2 * D];
    jP[0] = ldu(j, (uint32_t)n);
    jP[1] = ldu(j + P, (uint32_t)n);
    jP[2] = D == 3 ? ldu(j + (size_t)2 * P, (uint32_t)n) : 0.f;
    const float psiP = p.psi ? ldu(p.psi, (uint32_t)n) : 0.f;
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
        const uint32_t q = (uint32_t)(c.m[k] >= 0 ? c.m[k] : n);
        jN[k] = ldu(j + (size_t)(k >> 1) * P, q);
        psiN[k] = p.psi ? ldu(p.psi, q) : 0.f;
    }
    const float invD2[2] = {2.f * p.invD[0], 2.f * p.invD[1]};
    const float hzD[2] = {0.5f * p.z[0] * p.D[0], 0.5f * p.z[1] * p.D[1]};
    c.b[0] = c.b[1] = 0.0;
    c.adv = 0.f;
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
        const int i = k + 1;
        const int axis = k >> 1;
        const int sgi = (k & 1) ? -1 : 1;
        const float sg = (float)sgi;
        const int m = c.m[k];
#pragma unroll
        for (int s = 0; s < 2; ++s) c.al[s][k] = c.be[s][k] = 0.f;
        if (m == kOutside) {  // an open x end (the ions are not periodic)
            if (p.npx == kNpxClosed) continue;
            const float dpsi = p.psi ? 0.f : -sg * p.dpsi_dx;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float al, be;
                if (sgi < 0) {  // inlet: ghost at c0, inflow u_in
                    sg_coef(p.D[s], invD2[s], -0.5f * p.u_in - hzD[s] * dpsi, al, be);
                    be *= p.c0;
                } else if (p.npx == kNpxDirichlet) {
                    sg_coef(p.D[s], invD2[s], 0.5f * jP[0] - hzD[s] * dpsi, al, be);
                    be *= p.c_out;
                } else {  // open outlet: drift carries C_P out, or feed c0 in
                    const float w = 2.f * (0.5f * jP[0] - hzD[s] * dpsi);
                    al = fmaxf(w, 0.f);
                    be = -fminf(w, 0.f) * p.c0;
                }
                c.al[s][k] = al;
                c.be[s][k] = be;
                c.b[s] += (double)be;
            }
        } else if (m == kElectrode) {
#pragma unroll
            for (int s = 0; s < 2; ++s) c.al[s][k] = p.keff[s];
        } else if (m >= 0) {
            const float hun = 0.25f * (jP[axis] + jN[k]) * sg;
            c.adv = fmaxf(c.adv, fabsf(hun));
            const bool mig = p.psi || axis == 0;  // the ramp has no y/z gradient
            const float dpsi = p.psi ? psiN[k] - psiP : -sg * p.dpsi_dx;
#pragma unroll
            for (int s = 0; s < 2; ++s) sg_coef(p.D[s], invD2[s], mig ? hun - hzD[s] * dpsi : hun, c.al[s][k], c.be[s][k]);
        }
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        float d = 0.f;
#pragma unroll
        for (int k = 0; k < 2 * D; ++k) d += c.al[s][k];
        c.diag[s] = d;
    }
}

template <class L>
__device__ inline void np_node(const Grid &g, const Phys &p, const float *j, int n, NpNode<L> &c)
{
    np_faces<L>(g, p, n, c);
    np_coefs<L>(g, p, j, n, c);
}

template <class L>
__global__ __launch_bounds__(kTile) void nps_setup_kernel(NpsArgs a)
{
    __shared__ double sm[kTile / 64];
    int t0, t1;
    tile_range(a.g.P / kTile, t0, t1);
    double bb[2] = {0, 0}, rho[2] = {0, 0}, rr[2] = {0, 0};
    float adv = 0.f;
    double range = a.p.psi ? 0.0 : 16.0 * fabs((double)a.p.dpsi_dx);  // (16 voxels of a brick)
    for (int t = t0; t < t1; ++t) {
        const int n = t * kTile + threadIdx.x;
        if (a.p.psi) {  // the range in the tile's block
            float lo = INFINITY, hi = -INFINITY;
#pragma unroll
            for (int q = 0; q < kBlockTiles; ++q) {
                const int m = (t / kBlockTiles * kBlockTiles + q) * kTile + (int)threadIdx.x;
                const float v = a.p.psi[m < a.g.n_f ? m : t * kTile];
                lo = fminf(lo, v);
                hi = fmaxf(hi, v);
            }
            range = fmax(range, wg_max(hi, sm) + wg_max(-lo, sm));
        }
        double xv[2] = {0, 0}, rv[2] = {0, 0};
        float di[2] = {0, 0};
        if (n < a.g.n_f) {
            NpNode<L> c;
            np_node<L>(a.g, a.p, a.j, n, c);
            adv = fmaxf(adv, c.adv);
            float2 cN[2 * L::D];
#pragma unroll
            for (int k = 0; k < 2 * L::D; ++k) cN[k] = a.C[c.m[k] >= 0 ? c.m[k] : n];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                xv[s] = of_species(a.C[n], s);
                double ax = (c.diag[s] + a.idt) * xv[s];
#pragma unroll
                for (int k = 0; k < 2 * L::D; ++k)
                    if (c.m[k] >= 0) ax -= (double)c.be[s][k] * (double)of_species(cN[k], s);
                const double rhs = a.idt * xv[s] + c.b[s];
                rv[s] = rhs - ax;
                const float d = (float)(c.diag[s] + a.idt);
                di[s] = 1.f / (d > 0.f ? d : 1.f);  // (no outflow at all: an isolated closed pocket)
                bb[s] += rhs * rhs;
                rho[s] += rv[s] * rv[s];
                rr[s] += rv[s] * rv[s];
            }
        }
        stu(a.x, (uint32_t)n, make_double2(xv[0], xv[1]));
        stu(a.r, (uint32_t)n, make_double2(rv[0], rv[1]));
        stu(a.rh, (uint32_t)n, make_double2(rv[0], rv[1]));
        stu(a.di, (uint32_t)n, make_float2(di[0], di[1]));
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const double s_bb = wg_sum(bb[s], sm), s_rho = wg_sum(rho[s], sm), s_rr = wg_sum(rr[s], sm);
        if (threadIdx.x == 0) {
            reg(a, kBb, s)[blockIdx.x] = s_bb;
            reg(a, kRho0, s)[blockIdx.x] = s_rho;
            reg(a, kRr, s)[blockIdx.x] = s_rr;
            // iteration -1 leaves alpha = omega = 1: r.v = rho_0, t.s = t.t = 1
            reg(a, kRv, s)[blockIdx.x] = s_rho;
            reg(a, kTs, s)[blockIdx.x] = blockIdx.x == 0 ? 1.0 : 0.0;
            reg(a, kTt, s)[blockIdx.x] = blockIdx.x == 0 ? 1.0 : 0.0;
        }
    }
    const double s_pe = wg_max(2.0 * adv * fmaxf(a.p.invD[0], a.p.invD[1]), sm);
    if (threadIdx.x == 0) {  // (free until the first update)
        reg(a, kRho1, 0)[blockIdx.x] = s_pe;
        reg(a, kRho1, 1)[blockIdx.x] = range * fmaxf(fabsf(a.p.z[0]), fabsf(a.p.z[1]));
    }
}

__global__ __launch_bounds__(kTile) void nps_state_kernel(NpsArgs a, int G, double tol)
{
    __shared__ double sm[kTile / 64];
    for (int q = 0; q < 2; ++q) {
        double v = 0;
        for (int k = threadIdx.x; k < G; k += blockDim.x) v = fmax(v, reg(a, kRho1, q)[k]);
        v = wg_max(v, sm);
        if (threadIdx.x == 0) a.state[q ? kNsRange : kNsPe] = v;
    }
    for (int s = 0; s < 2; ++s) {
        const double bb = region_sum(a.part + ((size_t)kBb * 2 + s) * G, G, sm);
        const double rr = region_sum(a.part + ((size_t)kRr * 2 + s) * G, G, sm);
        if (threadIdx.x == 0) {
            a.state[kNsBb + s] = bb;
            a.state[kNsThr + s] = tol * tol * bb;
            a.state[kNsRr + s] = rr;
            a.state[kNsIters + s] = 0;
            a.state[kNsScale + s] = rr > 0.0 && isfinite(rr) ? ldexp(1.0, -ilogb(sqrt(rr))) : 1.0;
            a.state[kNsActive + s] = rr <= tol * tol * bb ? 0.0 : 1.0;
        }
    }
    if (threadIdx.x == 0) a.state[kNsDone] = (a.state[kNsActive] == 0 && a.state[kNsActive + 1] == 0) ? 1.0 : 0.0;
}

// The preconditioner: M is block diagonal over blocks of kBlockNodes
// consecutive nodes (16 x 16 x 7 voxels of a brick at porosity 0.6), in a block
// a few sweeps towards A_b z = r from z = 0, on FP32 numbers, with r scaled by a
// power of two per solve (which scales M). With A_b = D - O (D the diagonal, O >=
// 0): what leaves a cell enters its neighbours, so that the columns of O D^-1 sum
// to at most 1 and the eigenvalues of D^-1 A_b lie in the disc |lambda - 1| <= 1.
// They are real, in (0, 2), without a flow: the drift in a potential is a gradient
// and A_b similar to a symmetric matrix, through weights e^(z psi). A flow adds
// imaginary parts of up to half of its cell Peclet number.
//   Chebyshev: the kChebSteps-th iterate of the Chebyshev iteration for D^-1 A_b
//   on [kChebLow, 2]. Its residual polynomial stays below 1 in the ellipse with
//   these foci that goes through 0, whose half height is 0.447, and reaches 16
//   at 1 +- i. Taken while the flow's largest |Pe| is below kChebMaxPe, twice
//   that height, and the potential's range in a block is below kChebMaxRange, half
//   of where the weights' ratio e^range begins to tell (a uniform field of 25 thermal
//   voltages a block: 60 iterations, 35: 64, 47: 75, 59: no convergence).
//   plain: z <- D^-1 (r + O z), kPlainSweeps terms of the Neumann series. O D^-1 is
//   not negative and its powers' columns sum to at most 1: no drift amplifies. An
//   odd number, as after an even one nothing is left of lambda = 2.
// Iterations and ms of steady solves to 1e-10, with the diagonal, Chebyshev and
// plain sweeps: 192^3, flow of |Pe| 0.3: 299 and 129, 108 and 49, 123 and 57; 192^3,
// electrode at -4 thermal voltages: 318 and 105, 112 and 37, 131 and 44; 64^3,
// |Pe| 0.9: 205 and 11.8, 79 and 4.3, 74 and 4.4; 3.6: 157 and 9.1, 51 and 2.9, 57
// and 3.4; 9 and 60: 154 and 9.1, 133 and 8.3, Chebyshev breaks down, 42 and 2.6,
// 25 and 1.5. (5, 6, 7 and 10 plain sweeps
// at |Pe| 4, 96^3: 58, 49, 48 and 41 iterations, nine 42.) The blocks take the cells'
// own coefficients: a diffusion-only block does as well in weak fields and fails
// in steep ones (no convergence at -20). The coefficients are formed again from flux and
// potential where they are needed, 16 bytes a node instead of 48 for stored
// ones. The sweeps run on the block in LDS; what bounds the direction kernels
// is their streams (116 and 100 bytes a node) about as much as their arithmetic.
// 192^3, 4.2 M nodes, to 1e-10: 141 -> 52 ms, 300 -> 118 iterations of 383 ->
// 372 us.
constexpr double kChebMaxPe = 0.89, kChebMaxRange = 25.0;
constexpr int kPlainSweeps = 9;

// Nodes per thread of the direction kernels: two. A node's row and its loads
// take about 45 registers; at four a thread only two workgroups of 256 fit a
// compute unit (per iteration of 4.2 M nodes, p^ and s^: 124 and 109 us at four,
// 95 and 72 at two, 108 and 87 at one; capped at 168 or 128 registers the four
// spill, 148 and 95, 231 and 220).
constexpr int kDirNodes = 2, kDirThreads = kBlockNodes / kDirNodes;

template <class L>
struct BlockRows {
    float be[kDirNodes][2][2 * L::D];   // off the diagonal, 0 outside the block
    uint16_t lm[kDirNodes][2 * L::D];   // the neighbours' places in the block (the node's own where be = 0)
    float dinv[kDirNodes][2];
};

// The rows of this thread's nodes (zero beyond the lattice): only the
// coefficients of neighbours in the block, straight through.
template <class L>
__device__ __forceinline__ void block_rows(const NpsArgs &a, int base, BlockRows<L> &b)
{
    constexpr int F = 2 * L::D;
    const Phys &p = a.p;
    const int P = a.g.P;
    const float invD2[2] = {2.f * p.invD[0], 2.f * p.invD[1]};
    const float hzD[2] = {0.5f * p.z[0] * p.D[0], 0.5f * p.z[1] * p.D[1]};
    NpNode<L> c[kDirNodes];
#pragma unroll
    for (int j = 0; j < kDirNodes; ++j) {
        const int n = base + j * kDirThreads + (int)threadIdx.x;
        np_faces<L>(a.g, p, n < a.g.n_f ? n : a.g.n_f - 1, c[j]);
    }
#pragma unroll
    for (int j = 0; j < kDirNodes; ++j) {
        const int own = j * kDirThreads + (int)threadIdx.x;
        const bool on = base + own < a.g.n_f;
        const uint32_t n = on ? (uint32_t)(base + own) : 0u;
        bool in[F];
        float jP[L::D], jN[F], psiN[F];
#pragma unroll
        for (int d = 0; d < L::D; ++d) jP[d] = ldu(a.j + (size_t)d * P, n);
        const float psiP = p.psi ? ldu(p.psi, n) : 0.f;
        const float2 di = ldu(a.di, n);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const uint32_t l = (uint32_t)(c[j].m[f] - base);  // (beyond the block for negative values too)
            in[f] = on && c[j].m[f] >= 0 && l < (uint32_t)kBlockNodes;
            b.lm[j][f] = (uint16_t)(in[f] ? l : (uint32_t)own);
            const uint32_t q = in[f] ? (uint32_t)c[j].m[f] : n;
            jN[f] = ldu(a.j + (size_t)(f >> 1) * P, q);
            psiN[f] = p.psi ? ldu(p.psi, q) : 0.f;
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const float sg = (f & 1) ? -1.f : 1.f;
            const float hun = 0.25f * (jP[f >> 1] + jN[f]) * sg;
            const float dpsi = p.psi ? psiN[f] - psiP : (f >> 1) == 0 ? -sg * p.dpsi_dx : 0.f;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                float al, be;
                sg_coef(p.D[s], invD2[s], hun - hzD[s] * dpsi, al, be);
                b.be[j][s][f] = in[f] ? be : 0.f;
            }
        }
        b.dinv[j][0] = on ? di.x : 0.f;
        b.dinv[j][1] = on ? di.y : 0.f;
    }
}

// z = M r of this thread's nodes, PLAIN or Chebyshev sweeps. zs: two buffers of a block.
template <class L, int PLAIN>
__device__ __forceinline__ void block_solve(const float (&r)[kDirNodes][2], const BlockRows<L> &b,
                                            float2 (*zs)[kBlockNodes], float (&z)[kDirNodes][2])
{
    constexpr ChebCoef c = cheb_coef();
    float d[kDirNodes][2];
#pragma unroll
    for (int j = 0; j < kDirNodes; ++j)
#pragma unroll
        for (int s = 0; s < 2; ++s) z[j][s] = d[j][s] = (PLAIN ? 1.f : c.first) * (r[j][s] * b.dinv[j][s]);
#pragma unroll
    for (int k = 1; k < (PLAIN ? kPlainSweeps : kChebSteps); ++k) {
        float2 *const q = zs[k & 1];
#pragma unroll
        for (int j = 0; j < kDirNodes; ++j) q[j * kDirThreads + threadIdx.x] = make_float2(z[j][0], z[j][1]);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kDirNodes; ++j) {
            float y[2] = {r[j][0], r[j][1]};
#pragma unroll
            for (int f = 0; f < 2 * L::D; ++f) {
                const float2 v = q[b.lm[j][f]];
                y[0] = fmaf(b.be[j][0][f], v.x, y[0]);
                y[1] = fmaf(b.be[j][1][f], v.y, y[1]);
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (PLAIN) {
                    z[j][s] = b.dinv[j][s] * y[s];
                    continue;
                }
                d[j][s] = fmaf(c.r[k], fmaf(b.dinv[j][s], y[s], -z[j][s]), c.d[k] * d[j][s]);
                z[j][s] += d[j][s];
            }
            keep_order();  // one node's gathers at a time (all at once take 48 more registers)
        }
    }
}

// The two halves of an iteration that make a direction. WHICH 0 (dir): the
// stop test, p and p^ = M p; WHICH 1 (sdir): s = r - alpha v and s^ = M s.
template <class L, int WHICH, int PLAIN>
__global__ __launch_bounds__(kDirThreads) void nps_dir_kernel(NpsArgs a, int k)
{
    __shared__ double sm[12 * (kDirThreads / 64)];
    __shared__ int stop;
    __shared__ float2 zs[2][kBlockNodes];
    if (stopped_at(a.state, kNsDone, &stop)) return;
    const int G = a.G;
    const int now = k & 1 ? kRho1 : kRho0, old = k & 1 ? kRho0 : kRho1;
    bool act[2];
    double beta[2] = {0, 0}, omega[2] = {0, 0}, alpha[2] = {0, 0};
    if (WHICH == 0) {
        const double *const regions[12] = {reg(a, kRr, 0),  reg(a, kRr, 1),  reg(a, now, 0), reg(a, now, 1),
                                           reg(a, old, 0),  reg(a, old, 1),  reg(a, kRv, 0), reg(a, kRv, 1),
                                           reg(a, kTs, 0),  reg(a, kTs, 1),  reg(a, kTt, 0), reg(a, kTt, 1)};
        double t[12];
        region_sums(regions, G, sm, t);
        bool bad = false;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            act[s] = !(t[s] <= a.state[kNsThr + s]);
            if (k == 0 || !act[s]) continue;  // p = r
            const double om = t[8 + s] / t[10 + s];
            const double be = (t[2 + s] / t[4 + s]) * ((t[4 + s] / t[6 + s]) / om);
            if (!(isfinite(be) && isfinite(t[s]))) bad = true;
            omega[s] = om;
            beta[s] = be;
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            for (int s = 0; s < 2; ++s) {
                a.state[kNsActive + s] = act[s] ? 1.0 : 0.0;
                a.state[kNsRr + s] = t[s];
                if (act[s]) a.state[kNsIters + s] = k;
            }
            if (bad) a.state[kNsDone] = 2.0;
            else if (!act[0] && !act[1]) a.state[kNsDone] = 1.0;
        }
        if (bad || (!act[0] && !act[1])) return;
    } else {
        const double *const regions[4] = {reg(a, now, 0), reg(a, now, 1), reg(a, kRv, 0), reg(a, kRv, 1)};
        double t[4];
        region_sums(regions, G, sm, t);
#pragma unroll
        for (int s = 0; s < 2; ++s)
            if (a.state[kNsActive + s] != 0.0) alpha[s] = t[s] / t[2 + s];
    }
    const double scale[2] = {a.state[kNsScale], a.state[kNsScale + 1]};
    int b0, b1;
    tile_range((a.g.P + kBlockNodes - 1) / kBlockNodes, b0, b1);
    for (int blk = b0; blk < b1; ++blk) {
        const int base = blk * kBlockNodes;
        BlockRows<L> rows;
        block_rows<L>(a, base, rows);
        float rf[kDirNodes][2], z[kDirNodes][2];
#pragma unroll
        for (int j = 0; j < kDirNodes; ++j) {
            const int n = base + j * kDirThreads + (int)threadIdx.x;
            double2 w = make_double2(0, 0);
            if (n < a.g.n_f) {
                w = ldu(a.r, (uint32_t)n);
                if (WHICH == 0) {
                    if (k > 0) {
                        const double2 v = ldu(a.v, (uint32_t)n), p = ldu(a.pv, (uint32_t)n);
                        w.x += beta[0] * (p.x - omega[0] * v.x);
                        w.y += beta[1] * (p.y - omega[1] * v.y);
                    }
                    stu(a.pv, (uint32_t)n, w);
                } else {
                    const double2 v = ldu(a.v, (uint32_t)n);
                    w.x -= alpha[0] * v.x;
                    w.y -= alpha[1] * v.y;
                    stu(a.r, (uint32_t)n, w);
                }
            }
            rf[j][0] = (float)(w.x * scale[0]);
            rf[j][1] = (float)(w.y * scale[1]);
        }
        keep_order();
        __syncthreads();  // the sweeps of the block before may still read zs
        block_solve<L, PLAIN>(rf, rows, zs, z);
#pragma unroll
        for (int j = 0; j < kDirNodes; ++j) {
            const int n = base + j * kDirThreads + (int)threadIdx.x;
            if (n < a.g.n_f) stu(WHICH == 0 ? a.ph : a.sh, (uint32_t)n, make_float2(z[j][0], z[j][1]));
        }
    }
}

// y = (idt I + A) in (in = p^ or s^), with partials: WHICH 0 (y = v): rhat . v;
// WHICH 1 (y = t): t . s, t . t.
template <class L, int WHICH>
__global__ __launch_bounds__(kTile) void nps_apply_kernel(NpsArgs a)
{
    __shared__ double sm[kTile / 64];
    __shared__ int stop;
    if (stopped_at(a.state, kNsDone, &stop)) return;
    const bool act[2] = {a.state[kNsActive] != 0.0, a.state[kNsActive + 1] != 0.0};
    const float2 *in = WHICH == 0 ? a.ph : a.sh;
    double2 *out = WHICH == 0 ? a.v : a.t;
    int t0, t1;
    tile_range(a.g.P / kTile, t0, t1);
    double d0[2] = {0, 0}, d1[2] = {0, 0};
    for (int t = t0; t < t1; ++t) {
        const int n = t * kTile + threadIdx.x;
        if (n >= a.g.n_f) continue;
        NpNode<L> c;
        np_faces<L>(a.g, a.p, n, c);
        // the neighbours' pairs, all gathered before any is used (the node's
        // own where the face is not fluid; not applied there)
        float2 vN[2 * L::D];
#pragma unroll
        for (int f = 0; f < 2 * L::D; ++f) vN[f] = ldu(in, (uint32_t)(c.m[f] >= 0 ? c.m[f] : n));
        const float2 vP = ldu(in, (uint32_t)n);
        const double2 w = ldu(WHICH == 0 ? a.rh : a.r, (uint32_t)n);
        np_coefs<L>(a.g, a.p, a.j, n, c);
        double y[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            y[s] = ((double)c.diag[s] + a.idt) * (double)of_species(vP, s);
#pragma unroll
            for (int f = 0; f < 2 * L::D; ++f)
                if (c.m[f] >= 0) y[s] -= (double)c.be[s][f] * (double)of_species(vN[f], s);
            d0[s] += y[s] * of_species(w, s);
            if (WHICH == 1) d1[s] += y[s] * y[s];
        }
        stu(out, (uint32_t)n, make_double2(y[0], y[1]));
    }
    const int G = a.G;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (!act[s]) continue;  // a frozen species keeps its last partials
        const double s0 = wg_sum(d0[s], sm);
        const double s1 = WHICH == 1 ? wg_sum(d1[s], sm) : 0.0;
        if (threadIdx.x == 0) {
            if (WHICH == 0) {
                a.part[((size_t)kRv * 2 + s) * G + blockIdx.x] = s0;
            } else {
                a.part[((size_t)kTs * 2 + s) * G + blockIdx.x] = s0;
                a.part[((size_t)kTt * 2 + s) * G + blockIdx.x] = s1;
            }
        }
    }
}

// x += alpha p^ + omega s^; r = s - omega t; partials rho_{k+1}, |r|^2. Bound
// by its streams (112 bytes a node).
__global__ __launch_bounds__(kTile) void nps_update_kernel(NpsArgs a, int k)
{
    __shared__ double sm[8 * (kTile / 64)];
    __shared__ int stop;
    if (stopped_at(a.state, kNsDone, &stop)) return;
    const bool act[2] = {a.state[kNsActive] != 0.0, a.state[kNsActive + 1] != 0.0};
    const int G = a.G, now = k & 1 ? kRho1 : kRho0;
    const double *const regions[8] = {reg(a, now, 0), reg(a, now, 1), reg(a, kRv, 0), reg(a, kRv, 1),
                                      reg(a, kTs, 0), reg(a, kTs, 1), reg(a, kTt, 0), reg(a, kTt, 1)};
    double t8[8], alpha[2], omega[2];
    region_sums(regions, G, sm, t8);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        alpha[s] = act[s] ? t8[s] / t8[2 + s] : 0.0;
        omega[s] = act[s] ? t8[4 + s] / t8[6 + s] : 0.0;
    }
    int t0, t1;
    tile_range(a.g.P / kTile, t0, t1);
    double rho[2] = {0, 0}, rr[2] = {0, 0};
    for (int t = t0; t < t1; ++t) {
        const int n = t * kTile + threadIdx.x;
        if (n >= a.g.n_f) continue;
        const uint32_t q = (uint32_t)n;
        const float2 ph = ldu(a.ph, q), sh = ldu(a.sh, q);
        double2 x = ldu(a.x, q), r = ldu(a.r, q);
        const double2 tv = ldu(a.t, q), rh = ldu(a.rh, q);
        x.x += alpha[0] * (double)ph.x + omega[0] * (double)sh.x;
        x.y += alpha[1] * (double)ph.y + omega[1] * (double)sh.y;
        r.x -= omega[0] * tv.x;
        r.y -= omega[1] * tv.y;
        stu(a.x, q, x);
        stu(a.r, q, r);
        rho[0] += rh.x * r.x;
        rho[1] += rh.y * r.y;
        rr[0] += r.x * r.x;
        rr[1] += r.y * r.y;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (!act[s]) continue;
        const double s_rho = wg_sum(rho[s], sm), s_rr = wg_sum(rr[s], sm);
        if (threadIdx.x == 0) {
            a.part[((size_t)(k & 1 ? kRho0 : kRho1) * 2 + s) * G + blockIdx.x] = s_rho;
            a.part[((size_t)kRr * 2 + s) * G + blockIdx.x] = s_rr;
        }
    }
}

// The stop test before iteration k, alone (one workgroup).
__global__ __launch_bounds__(kTile) void nps_check_kernel(NpsArgs a, int k, int G)
{
    __shared__ double sm[kTile / 64];
    if (a.state[kNsDone] != 0.0) return;
    bool act[2];
    for (int s = 0; s < 2; ++s) {
        const double rr = region_sum(a.part + ((size_t)kRr * 2 + s) * G, G, sm);
        act[s] = !(rr <= a.state[kNsThr + s]);
        if (threadIdx.x == 0) {
            if (!isfinite(rr)) a.state[kNsDone] = 2.0;
            a.state[kNsRr + s] = rr;
            if (act[s]) a.state[kNsIters + s] = k;
        }
    }
    if (threadIdx.x == 0 && a.state[kNsDone] == 0.0 && !act[0] && !act[1]) a.state[kNsDone] = 1.0;
}

// The FP64 solution as FP32 concentrations with their remainders.
__global__ __launch_bounds__(kTile) void nps_store_kernel(const double2 *x, float2 *C, __half2 *Clo, int n_f)
{
    const int n = blockIdx.x * kTile + threadIdx.x;
    if (n >= n_f) return;
    const double2 v = x[n];
    const float2 c = make_float2((float)v.x, (float)v.y);
    C[n] = c;
    Clo[n] = __halves2half2(lo_encode((float)(v.x - c.x)), lo_encode((float)(v.y - c.y)));
}

// Rates of adsorption, inflow and outflow of C (per tile, FP64).
template <class L>
__global__ __launch_bounds__(kTile) void nps_rates_kernel(Grid g, Phys p, const float2 *C, const float *j, double scale,
                                                          double *acc, double *part)
{
    __shared__ double sm[(kTile / 64) * 6];
    const int tile = blockIdx.x;
    const int n = tile * kTile + threadIdx.x;
    const int P = g.P;
    double v[6] = {0, 0, 0, 0, 0, 0};
    if (n < g.n_f) {
        NpNode<L> c;
        np_node<L>(g, p, j, n, c);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const double cp = (double)of_species(C[n], s);
#pragma unroll
            for (int f = 0; f < 2 * L::D; ++f) {
                const int m = c.m[f];
                if (m == kElectrode) {
                    v[s] += (double)c.al[s][f] * cp;  // adsorbed
                } else if (m == kOutside) {
                    const double F = (double)c.al[s][f] * cp - (double)c.be[s][f];
                    if (f & 1)
                        v[2 + s] -= F;  // the -x face is the inlet: inflow
                    else
                        v[4 + s] += F;  // outflow
                }
            }
        }
    }
    double out[6];
    block_sum<6>(v, sm, out);
    if (threadIdx.x == 0) {
        if (acc) {
            double *a = acc + (size_t)tile * 8;
            for (int k = 0; k < 6; ++k) a[k] += scale * out[k];
        } else {
            for (int k = 0; k < 6; ++k) part[(size_t)tile * 6 + k] = out[k];
        }
    }
}

}  // namespace

uint64_t nps_part_doubles() { return (uint64_t)kRegions * 2 * kNpsMaxWorkgroups; }

int nps_plain(double pe, double range) { return !(pe <= kChebMaxPe && range <= kChebMaxRange); }

hipError_t nps_workgroups(int dim, int ntiles, int *G)
{
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const void *k = dim == 2 ? (const void *)nps_apply_kernel<D2Q9, 1> : (const void *)nps_apply_kernel<D3Q19, 1>;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kTile, 0);
    if (e != hipSuccess) return e;
    // at most 4 per CU (steady ions at 192^3: 50.2 ms at 4, 55.5 at 6, 54.8 at
    // 8): fewer tiles in flight per XCD leave more of its L2 to the neighbours'
    // lines
    if (per_cu > kNpsWorkgroupsPerCU) per_cu = kNpsWorkgroupsPerCU;
    long long g = (long long)cus * (per_cu > 0 ? per_cu : 1);
    g = g < kNpsMaxWorkgroups ? g : kNpsMaxWorkgroups;
    *G = (int)(ntiles < g ? ntiles : g);
    return hipSuccess;
}

template <class L>
const void *dir_kernel(int which, int plain)
{
    return plain ? (which ? (const void *)nps_dir_kernel<L, 1, 1> : (const void *)nps_dir_kernel<L, 0, 1>)
                 : (which ? (const void *)nps_dir_kernel<L, 1, 0> : (const void *)nps_dir_kernel<L, 0, 0>);
}

// As many workgroups as are resident together, none left over for a second wave.
hipError_t nps_dir_workgroups(int dim, int ntiles, int plain, int *Gd)
{
    int dev = 0, cus = 0, fit = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    for (int w = 0; w < 2 && e == hipSuccess; ++w) {
        const void *k = dim == 2 ? dir_kernel<D2Q9>(w, plain) : dir_kernel<D3Q19>(w, plain);
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, k, kDirThreads, 0);
        const long long most = (long long)cus * std::min(std::max(fit, 1), kNpsWorkgroupsPerCU);
        const long long blocks = ((long long)ntiles + kBlockTiles - 1) / kBlockTiles;
        Gd[w] = (int)std::min(std::min(blocks, most), (long long)kNpsMaxWorkgroups);
    }
    return e;
}

hipError_t launch_nps_setup(int dim, const NpsArgs &a, double tol, hipStream_t s)
{
    if (dim == 2)
        nps_setup_kernel<D2Q9><<<a.G, kTile, 0, s>>>(a);
    else
        nps_setup_kernel<D3Q19><<<a.G, kTile, 0, s>>>(a);
    nps_state_kernel<<<1, kTile, 0, s>>>(a, a.G, tol);
    return hipGetLastError();
}

template <class L, int PLAIN>
void iter_l(const NpsArgs &a, int k, hipStream_t s)
{
    nps_dir_kernel<L, 0, PLAIN><<<a.Gd[0], kDirThreads, 0, s>>>(a, k);
    nps_apply_kernel<L, 0><<<a.G, kTile, 0, s>>>(a);
    nps_dir_kernel<L, 1, PLAIN><<<a.Gd[1], kDirThreads, 0, s>>>(a, k);
    nps_apply_kernel<L, 1><<<a.G, kTile, 0, s>>>(a);
}

hipError_t launch_nps_iter(int dim, const NpsArgs &a, int k, hipStream_t s)
{
    if (dim == 2)
        a.plain ? iter_l<D2Q9, 1>(a, k, s) : iter_l<D2Q9, 0>(a, k, s);
    else
        a.plain ? iter_l<D3Q19, 1>(a, k, s) : iter_l<D3Q19, 0>(a, k, s);
    nps_update_kernel<<<a.G, kTile, 0, s>>>(a, k);
    return hipGetLastError();
}

hipError_t launch_nps_check(const NpsArgs &a, int k, hipStream_t s)
{
    nps_check_kernel<<<1, kTile, 0, s>>>(a, k, a.G);
    return hipGetLastError();
}

hipError_t launch_nps_store(const NpsArgs &a, float2 *Cout, __half2 *Clo, hipStream_t s)
{
    const int tiles = a.g.P / kTile;
    if (tiles > 0) nps_store_kernel<<<tiles, kTile, 0, s>>>(a.x, Cout, Clo, a.g.n_f);
    return hipGetLastError();
}

hipError_t launch_nps_rates(int dim, const Grid &g, const Phys &p, const float2 *C, const float *j, double scale,
                            double *acc, double *part, double *out, hipStream_t s)
{
    const int tiles = g.P / kTile;
    if (tiles == 0) return hipSuccess;
    if (dim == 2)
        nps_rates_kernel<D2Q9><<<tiles, kTile, 0, s>>>(g, p, C, j, scale, acc, part);
    else
        nps_rates_kernel<D3Q19><<<tiles, kTile, 0, s>>>(g, p, C, j, scale, acc, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !out) return e;
    return launch_reduce_tiles(part, tiles, 6, 6, out, s);
}

}  // namespace cdi
