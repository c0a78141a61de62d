// step.hip -- the hot path: one lattice Boltzmann step (Eq. 7 with the BGK
// collision of Eq. 8, half-way bounce-back at solid faces) fused with one
// explicit finite-volume Nernst-Planck step (Eq. 3) and the adsorption flux
// of Eq. (6), over the compacted fluid nodes. The AA storage rules and the
// FP16 deviation format are described in device_common.h.
//
// The ions see the mass flux j = rho u. In a fused step the Nernst-Planck
// part reads the flux of the previous step (jin, or the FP16 moments) for the
// node and its face neighbours, while the LBM part writes the flux of this
// step. Face fluxes are Scharfetter-Gummel; the two sides of a face compute
// exactly opposite values, so solute is conserved to the rounding of the
// update. Per tile, the adsorbed / inflow / outflow amounts of the step are
// summed over each wave's 64 nodes in FP32, then over the tile's waves in
// FP64, in a fixed order, and added to that tile's own FP64 accumulator slot.
//
// Inlet/outlet planes (x = 0 and x = nx - 1): the node one plane inside owns
// the post-streaming populations the extrapolation needs, so its thread also
// advances the boundary node (no separate pass over the scattered planes).
#include "device_common.h"

namespace cdi {

namespace {

// Odd AA parity with FP32 or FP16 populations: the tile stages the slots of
// its own 256 nodes in LDS. Every slot has exactly one reader, which is also
// its writer (the AA rule above), so a slot whose reader lies in the tile is
// read from and written to LDS, and the owner loads it before and stores it
// after the step, both coalesced; a slot read by a node of another tile is
// left to that node's global load and store. Nodes of the inlet/outlet planes
// (advanced by their interior partner under extrapolation) write through
// global memory, so their slots are never stored back by an owner. On the
// 512^3 electrode about 29 % of the slots lie outside their reader's tile;
// staged, the FP32 fused odd step took 3.39 ms instead of 3.73, the FP32
// flow-only one 2.55 instead of 2.87, the FP16 fused one 2.76 instead of
// 2.87 (its flow-only step gains about 1 %).
// On lattices whose working set stays largely in the memory-side cache the
// extra work and barrier do not pay (96^3 to 160^3 electrodes stepped 5-13 %
// slower staged), so the host stages an instance's odd steps only from a
// tile count on (Grid::stage_odd); kStageOdd names the steps that may be
// staged.
//
// Stage layout: Q planes of kTile elements in the storage type, then kTile
// spare elements, one per thread. Every lane issues the LDS access (a lane
// whose slot lies outside the tile reads or writes its spare element) and
// only the global access is predicated; the stage is addressed through a
// pointer in the LDS address space, so that the compiler cannot fold an LDS
// and a global load into one generic-address access (which goes through the
// vector memory path and waits on both counters).
template <class L, int ST, int ODD, int LBM, int NP>
constexpr bool kStageOdd = LBM && ODD == 1 && kPlain<ST>;

template <int ST>
using StageT = typename std::conditional<kHalfPop<ST>, uint16_t, float>::type;  // FP16 as its bits

typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
template <int ST>
using LdsT = typename std::conditional<kHalfPop<ST>, lds_u16, lds_f32>::type;

template <class L>
constexpr int kStageElems = (L::Q + 1) * kTile;

template <int ST>
__device__ __forceinline__ float pop_float(StageT<ST> v)
{
    if constexpr (kHalfPop<ST>) return __half2float(__ushort_as_half(v));
    else return v;
}

template <int ST>
__device__ __forceinline__ StageT<ST> pop_stored(float v)
{
    if constexpr (kHalfPop<ST>) return __half_as_ushort(__float2half_rn(v));
    else return v;
}

// Where the staged odd step finds and leaves its populations: slot i is plane i
// of the neighbour along e_i, or plane opp(i) of the node itself where that is
// solid; the population opp(i) arrives in it and the one sent along e_i leaves
// through it. The slot's place in the stage, the thread's spare element when
// another tile owns it (never so where the neighbour is solid), is formed once
// for the three uses below. Formed at each, with the lanes' masks kept in scalar
// registers that spilled, longer address sums and a source term of a dozen
// operations per direction, a forced FP32 odd step issued 1500 vector
// instructions a wave instead of 1130 and took 251 us instead of 234 (5.2 M
// nodes); the FP16 fused one at 45 M nodes 795 instead of 735.
template <class L, int ST>
struct StageSlots {
    static constexpr uint32_t kBytes = sizeof(StageT<ST>);
    static constexpr uint32_t kSpare = L::Q * kTile * kBytes;  // from here on: another tile's
    uint32_t own, two[(L::Q - 1) / 2];                         // byte offsets, those of i and opp(i) in one word
    __device__ __forceinline__ uint32_t at(int i) const
    {
        return i == 0 ? own : (i & 1 ? two[(i - 1) / 2] & 0xffffu : two[(i - 1) / 2] >> 16);
    }
    __device__ __forceinline__ bool outside(int i) const { return i != 0 && at(i) >= kSpare; }
};

template <class L, int ST>
__device__ __forceinline__ void stage_slots(const Nbrs<L> &nb, int base, StageSlots<L, ST> &s)
{
    constexpr uint32_t B = StageSlots<L, ST>::kBytes;
    s.own = threadIdx.x * B;
    auto slot = [&](int i) {
        const uint32_t loc = (uint32_t)(nb.n[i] - base);
        return loc < (uint32_t)kTile ? loc * B + (nb.fl[i] ? i * kTile * B : L::opp[i] * kTile * B)
                                     : StageSlots<L, ST>::kSpare + s.own;
    };
#pragma unroll
    for (int i = 1; i < L::Q; i += 2) s.two[(i - 1) / 2] = slot(i) | slot(i + 1) << 16;
}

template <int ST>
__device__ __forceinline__ LdsT<ST> *stage_at(LdsT<ST> *stage, uint32_t byte)
{
    typedef __attribute__((address_space(3))) char lds_char;
    return (LdsT<ST> *)((lds_char *)stage + byte);
}

// The slots' lanes are told apart by a comparison where they are needed: kept
// from one use to the next the masks do not fit the scalar registers.
template <class L, int ST>
__device__ __forceinline__ void stage_forget(StageSlots<L, ST> &s)
{
#pragma unroll
    for (int i = 0; i < (L::Q - 1) / 2; ++i) asm volatile("" : "+v"(s.two[i]));
}

// The stored values behind the Q incoming populations of node n (odd
// parity): all stage reads first, then the global loads of the slots outside
// the tile (into the same registers, for those lanes only), so that the
// stage reads are waited for once rather than before every global load.
template <class L, int ST>
__device__ __forceinline__ void staged_gather(const void *F, const Nbrs<L> &nb, LdsT<ST> *stage,
                                              const StageSlots<L, ST> &s, StageT<ST> (&raw)[L::Q])
{
#pragma unroll
    for (int i = 0; i < L::Q; ++i) raw[i] = *stage_at<ST>(stage, s.at(L::opp[i]));
#pragma unroll
    for (int i = 1; i < L::Q; ++i) {
        const int j = L::opp[i];
        if (s.outside(j)) raw[i] = *pop_at<L::Q, StageT<ST>>(F, j, nb.n[j]);
    }
}

// Store outgoing value v of direction i (odd parity); lds_ok false for the
// nodes whose slots go through global memory (what they leave in the stage is
// not stored back).
template <class L, int ST>
__device__ __forceinline__ void staged_scatter(void *F, const Nbrs<L> &nb, int i, float v, LdsT<ST> *stage,
                                               const StageSlots<L, ST> &s, bool lds_ok)
{
    const StageT<ST> r = pop_stored<ST>(v);
    *stage_at<ST>(stage, s.at(i)) = r;
    if (s.outside(i))
        *pop_at<L::Q, StageT<ST>>(F, i, nb.n[i]) = r;
    else if (!lds_ok)  // rare
        st_pair<kHalfPop<ST>, L::Q>(F, L::opp[i], i, nb.n[i], i == 0 || !nb.fl[i], v);
}

// Moments, residual terms, collision and the AA store of one node whose
// incoming populations (minus w_i) are f (sums: their moments, where they were
// summed already); NP: also store the mass flux j for
// the ions of the next step (FP32; the other storages carry it in Mout).
// FP32 storage: f_i - w_i (1 + pr.rout) on entry, and values stored relative
// to the plane references of pr (see PlaneRef); the other storages pass zeros.
template <class L, int ST, int ODD, int NP, bool STAGE = false>
__device__ __attribute__((always_inline)) inline void lbm_node(const Phys &p, const Bufs &b, int P, int n, const Nbrs<L> &nb,
                                const float (&f)[L::Q], const PlaneRef &pr, double (&res)[2], const MomSums *sums,
                                LdsT<ST> *stage = nullptr, const StageSlots<L, ST> *slots = nullptr, bool lds_ok = false)
{
    constexpr int Q = L::Q, D = L::D;
    float drho, jx, jy, jz;  // drho: rho - 1 - pr.rout
    if (sums) {
        drho = sums->d;
        jx = sums->jx;
        jy = sums->jy;
        jz = sums->jz;
    } else {
        lat_moments<L>(f, drho, jx, jy, jz);
    }
    if (p.forced) {  // Guo forcing: u = (sum e f + F/2) / rho
        jx += 0.5f * p.F[0];
        jy += 0.5f * p.F[1];
        jz += 0.5f * p.F[2];
    }
    const float rho = 1.f + pr.rout + drho;
    const float rinv = __builtin_amdgcn_rcpf(rho);
    const float ux = jx * rinv, uy = jy * rinv, uz = jz * rinv;
    if (b.flags & kResid) {
        float px, py, pz;
        if (!kPlain<ST>) {
            const float4 m = ldu(b.Min, (uint32_t)n);
            px = m.y;
            py = m.z;
            pz = m.w;
        } else {
            px = ldu(b.ubuf, (uint32_t)n);
            py = ldu(b.ubuf + P, (uint32_t)n);
            pz = D == 3 ? ldu(b.ubuf + 2 * (size_t)P, (uint32_t)n) : 0.f;
        }
        const double dx = (double)ux - px, dy = (double)uy - py, dz = (double)uz - pz;
        res[0] += dx * dx + dy * dy + dz * dz;
        res[1] += (double)ux * ux + (double)uy * uy + (double)uz * uz;
    }
    if (kPlain<ST> && (b.flags & kStoreU)) {
        stu(b.ubuf, (uint32_t)n, ux);
        stu(b.ubuf + P, (uint32_t)n, uy);
        if (D == 3) stu(b.ubuf + 2 * (size_t)P, (uint32_t)n, uz);
        stu(b.ubuf + (size_t)D * P, (uint32_t)n, pr.rout + drho);  // rho - 1, for the plane references
    }
    if (!kPlain<ST>) stu(b.Mout, (uint32_t)n, make_float4(drho, ux, uy, uz));
    if (NP && kPlain<ST>) {
        stu(b.jout, (uint32_t)n, jx);
        stu(b.jout + P, (uint32_t)n, jy);
        if (D == 3) stu(b.jout + 2 * (size_t)P, (uint32_t)n, jz);
    }
    const EqTerms eq = eq_terms(drho, rho, ux, uy, uz, p.linear_eq);
    const float om = p.omega;
    // FP16 populations are stored times hs
    const float sc = kPlain<ST> && kHalfPop<ST> ? p.hs : 1.f;
    if (kPlain<ST> && om == 1.f && !p.forced) {
        // tau = 1: BGK (Eq. 8) relaxes every population to the equilibrium
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const float v = sc * stored_pop<L, ODD>(feq_dir<L>(i, eq, ux, uy, uz), i, nb, pr);
            if (STAGE)
                staged_scatter<L, ST>(b.f, nb, i, v, stage, *slots, lds_ok);
            else
                scatter<L, ST, ODD>(ODD == kPull ? b.f2 : b.f, P, nb, n, i, v);
        }
        return;
    }
    // Guo, Zheng & Shi (2002) source term, coef w_i (3 (e_i - u) + 9 (e_i . u)
    // e_i) . F, as w_i ((e_i . G) (1 + 3 e_i . u) - u . G) with G = 3 coef F: four
    // operations a direction. Fused steps keep a branch per direction, which
    // stops the scheduler from spreading all of them over the registers (FP16
    // fused, 45 M nodes, even and odd: 410 and 735 us against 435 and 726
    // without it; FP32 flow, forced, 5.2 M nodes: 133 and 234 against 127 and 235)
    const float fc = 3.f * p.fcoef;
    const float Gx = fc * p.F[0], Gy = fc * p.F[1], Gz = D == 3 ? fc * p.F[2] : 0.f;
    const float uG = fmaf(ux, Gx, fmaf(uy, Gy, uz * Gz));
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const float fe = feq_dir<L>(i, eq, ux, uy, uz);
        float src = 0.f;
        if (p.forced) {
            const float eu = lat_dot<L>(i, ux, uy, uz);
            src = L::w[i] * (i == 0 ? -uG : fmaf(lat_dot<L>(i, Gx, Gy, Gz), fmaf(3.f, eu, 1.f), -uG));
            if (NP) asm volatile("" : "+v"(src));
        }
        float out;
        if (ST == kF16)
            out = ((1.f - om) * (f[i] - fe) + src) * p.hs;
        else
            out = sc * stored_pop<L, ODD>(f[i] - om * (f[i] - fe) + src, i, nb, pr);
        if (STAGE)
            staged_scatter<L, ST>(b.f, nb, i, out, stage, *slots, lds_ok);
        else
            scatter<L, ST, ODD>(ODD == kPull ? b.f2 : b.f, P, nb, n, i, out);
    }
}

// Moments of a node's state (dr: rho - 1 - rout) to the moments buffer, and
// its residual terms: a whole flow step of the moment storages, whose
// post-collision state is the equilibrium of Mout.
template <class L>
__device__ __forceinline__ void moment_node(const Bufs &b, int n, float dr, float jx, float jy, float jz, float rout,
                                            double (&res)[2])
{
    const float rinv = __builtin_amdgcn_rcpf(1.f + rout + dr);
    const float ux = jx * rinv, uy = jy * rinv, uz = jz * rinv;
    if (b.flags & kResid) {
        const float4 m = ldu(b.Min, (uint32_t)n);
        const double dx = (double)ux - m.y, dy = (double)uy - m.z, dz = (double)uz - m.w;
        res[0] += dx * dx + dy * dy + dz * dz;
        res[1] += (double)ux * ux + (double)uy * uy + (double)uz * uz;
    }
    stu(b.Mout, (uint32_t)n, make_float4(dr, ux, uy, uz));
}

// Moments of the FP16 deviations, kept apart from those of the equilibria so
// that with zero deviations (tau = 1) both storages round the same sums.
template <int ST>
struct DevSums : MomSums {
    __device__ __forceinline__ void add_to(MomSums &s) const
    {
        if constexpr (!kMoments<ST>) {
            s.d += this->d;
            s.jx += this->jx;
            s.jy += this->jy;
            s.jz += this->jz;
        }
    }
};

// What leaves node n through its faces in one explicit ion step, per species
// (out), and the part through open x ends (fi in, fo out).
struct IonFlux {
    float out[2] = {0.f, 0.f}, fi[2] = {0.f, 0.f}, fo[2] = {0.f, 0.f};
    float ads = 0.f;  // adsorbing faces
};

// The fluxes to fluid cells with no potential field, a ramp that is not steep
// and hardly a face beyond the series' range. on: the faces to fluid cells; jn the neighbours' flux along the face's
// axis, cn their concentrations (0 where the face is not fluid: its flux is
// formed and multiplied by 0). Straight-line code, without a branch
// per face; y and z faces, where the ramp has no gradient, share the half drift
// h between the species. Returns whether every face of the lane is within the
// series' range.
template <class L>
__device__ __forceinline__ bool ion_faces(const Phys &p, const bool (&on)[2 * L::D], const float (&cP)[2],
                                          const float (&jP)[3], const float2 (&cn)[2 * L::D],
                                          const float (&jn)[2 * L::D], IonFlux &f)
{
    float wx = 0.f, wyz = 0.f;
#pragma unroll
    for (int k = 0; k < 2 * L::D; ++k) {
        const float h = ((k & 1) ? -0.25f : 0.25f) * (jP[k >> 1] + jn[k]);  // (x faces: less the ramp's part)
        if (k < 2)
            wx = fmaxf(wx, fabsf(h));
        else
            wyz = fmaxf(wyz, fabsf(h));
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const float F = sg_series(p.D[s], p.sgc[s], k < 2 ? h + ((k & 1) ? -p.hr[s] : p.hr[s]) : h, cP[s],
                                      s ? cn[k].y : cn[k].x);
            f.out[s] = fmaf(on[k] ? 1.f : 0.f, F, f.out[s]);
        }
    }
    const float w = fmaxf(wyz, wx + fmaxf(fabsf(p.hr[0]), fabsf(p.hr[1])));
    return w * w <= p.h2_max;
}

// The same fluxes where ion_faces was out of its range: a rolled loop that
// looks everything up again, so that the rare case costs the steps no
// registers. Faces within the series' range take the series, as their other
// cell does.
template <class L, int ST>
__device__ __forceinline__ void ion_faces_wide(const Grid &g, const Phys &p, const Bufs &b, int x, int y, int z, bool jm,
                                               const bool (&end)[2], float c0, float c1, float j0, float j1, float j2,
                                               IonFlux &f)
{
    f.out[0] = f.out[1] = 0.f;
#pragma unroll 1
    for (int k = 0; k < 2 * L::D; ++k) {
        const int m = nb_map<L>(g, x, y, z, k + 1, g.periodic_x);
        if (m < 0 || (k == 0 && end[0]) || (k == 1 && end[1])) continue;
        const int axis = k >> 1;
        float jN;
        if (jm) {
            const float4 mm = ldu(b.Min, (uint32_t)m);
            float r = 1.f + mm.x;
            if (ST == kMomR) {
                int xm = x + (k == 0) - (k == 1);
                xm = xm < 0 ? g.nx - 1 : (xm >= g.nx ? 0 : xm);
                r = 1.f + ldu(b.rin, (uint32_t)xm) + mm.x;
            }
            jN = r * (axis == 0 ? mm.y : (axis == 1 ? mm.z : mm.w));
        } else {
            jN = ldu(b.jin + (size_t)axis * g.P, (uint32_t)m);
        }
        const float sg = (k & 1) ? -1.f : 1.f;
        const float h = 0.25f * sg * ((axis == 0 ? j0 : (axis == 1 ? j1 : j2)) + jN);
        const float2 cm = ld_conc<ST>(b.Cin, (uint32_t)m);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const float hs = axis == 0 ? h + sg * p.hr[s] : h, cp = s ? c1 : c0, cn = s ? cm.y : cm.x;
            f.out[s] += hs * hs <= p.h2_max ? sg_series(p.D[s], p.sgc[s], hs, cp, cn)
                                            : sg_flux(p.D[s], 2.f * p.invD[s], hs, cp, cn);
        }
    }
}

// The same values in line, for flows that take many faces beyond the series'
// range. Bound by the number of vector memory instructions like ion_faces, whose
// detour adds dependent ones (160^3, every tile beyond: ion step 53 -> 37 us,
// fused with moments 84 -> 67, FP16 101 -> 84, FP32 populations 158 -> 142,
// a batch of 16 cubes 45 -> 30; with the potential's form in the same kernel 41).
template <class L>
__device__ __forceinline__ void ion_faces_far(const Phys &p, const bool (&on)[2 * L::D], const float (&cP)[2],
                                              const float (&jP)[3], const float2 (&cn)[2 * L::D],
                                              const float (&jn)[2 * L::D], IonFlux &f)
{
#pragma unroll
    for (int k = 0; k < 2 * L::D; ++k) {
        if (on[k]) {
            const float h = ((k & 1) ? -0.25f : 0.25f) * (jP[k >> 1] + jn[k]);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float hs = k < 2 ? h + ((k & 1) ? -p.hr[s] : p.hr[s]) : h, cN = s ? cn[k].y : cn[k].x;
                f.out[s] += hs * hs <= p.h2_max ? sg_series(p.D[s], p.sgc[s], hs, cP[s], cN)
                                                : sg_flux(p.D[s], 2.f * p.invD[s], hs, cP[s], cN);
            }
        }
    }
}

// The fluxes in a potential field (psi; the migration of every face from the
// potential's difference) or in a steep ramp.
template <class L>
__device__ __forceinline__ void ion_faces_any(const Phys &p, bool psi, const bool (&on)[2 * L::D], const float (&cP)[2],
                                              const float (&jP)[3], float psiP, const float2 (&cn)[2 * L::D],
                                              const float (&jn)[2 * L::D], const float (&psin)[2 * L::D], IonFlux &f)
{
    const float invD2[2] = {2.f * p.invD[0], 2.f * p.invD[1]};
    const float hzD[2] = {0.5f * p.z[0] * p.D[0], 0.5f * p.z[1] * p.D[1]};
#pragma unroll
    for (int k = 0; k < 2 * L::D; ++k) {
        if (on[k]) {
            const float q = ((k & 1) ? -0.25f : 0.25f) * (jP[k >> 1] + jn[k]);
            const float d = psi ? psin[k] - psiP : (k == 0 ? -p.dpsi_dx : (k == 1 ? p.dpsi_dx : 0.f));
#pragma unroll
            for (int s = 0; s < 2; ++s)
                f.out[s] += sg_flux(p.D[s], invD2[s], q - hzD[s] * d, cP[s], s ? cn[k].y : cn[k].x);
        }
    }
}

// The x-end face on side sgi of a node at (x, y, z) on that end, where the
// ions' treatment of the end is not the lattice's own wrap: the inlet ghost,
// the open or Dirichlet outlet, or (periodic ions, open flow) the cell at the
// other end. jm: the neighbours' flux comes from the moments buffer.
template <class L, int ST>
__device__ __forceinline__ void ion_end_face(const Grid &g, const Phys &p, const Bufs &b, int sgi, int x, int y,
                                                       int z, bool jm, bool psi, float c0, float c1, float jP0,
                                                       float psiP, IonFlux &f)
{
    if (p.npx == kNpxClosed) return;
    const float sg = (float)sgi, cP[2] = {c0, c1};
    const float hzD[2] = {0.5f * p.z[0] * p.D[0], 0.5f * p.z[1] * p.D[1]};
    float dpsi = psi ? 0.f : -sg * p.dpsi_dx;
    if (p.npx == kNpxPeriodic) {
        const int m = nb_map<L>(g, x, y, z, sgi > 0 ? 1 : 2, true);
        if (m == kElectrode) f.ads += 1.f;
        if (m < 0) return;
        float jN;
        if (jm) {
            const float4 mm = ldu(b.Min, (uint32_t)m);
            // (relative to the other end's plane, with plane references)
            jN = (ST == kMomR ? 1.f + ldu(b.rin, (uint32_t)(sgi < 0 ? g.nx - 1 : 0)) + mm.x : 1.f + mm.x) * mm.y;
        } else {
            jN = ldu(b.jin, (uint32_t)m);
        }
        if (psi) dpsi = ldu(p.psi, (uint32_t)m) - psiP;
        const float2 cm = ld_conc<ST>(b.Cin, (uint32_t)m);
#pragma unroll
        for (int s = 0; s < 2; ++s)
            f.out[s] += sg_flux(p.D[s], 2.f * p.invD[s], 0.25f * (jP0 + jN) * sg - hzD[s] * dpsi, cP[s], s ? cm.y : cm.x);
        return;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        if (sgi < 0) {  // inlet face: ghost at c0, inflow u_in
            const float F = sg_flux(p.D[s], 2.f * p.invD[s], -0.5f * p.u_in - hzD[s] * dpsi, cP[s], p.c0);
            f.out[s] += F;
            f.fi[s] -= F;
        } else {  // outlet face
            const float hw = 0.5f * jP0 - hzD[s] * dpsi;
            float F;
            if (p.npx == kNpxDirichlet) {
                F = sg_flux(p.D[s], 2.f * p.invD[s], hw, cP[s], p.c_out);
            } else {  // open: drift carries C_P out, or feed c0 in
                const float w = 2.f * hw;
                F = fmaxf(w, 0.f) * cP[s] + fminf(w, 0.f) * p.c0;
            }
            f.out[s] += F;
            f.fo[s] += F;
        }
    }
}

// One 256-node tile of one instance (all threads of the workgroup call it;
// sm: (kTile/64)*6 doubles of LDS; stg: the stage of kStageOdd steps).
// PSI: the form of the ions' fluxes: in a ramp (0), in a potential field or a
// steep ramp, in a flow that takes many faces beyond the series' range, or as p
// says.
constexpr int kPsiField = 1, kPsiFar = 2, kPsiAny = 3;

template <class L, int ST, int ODD, int LBM, int NP, int PSI, int STG = 0>
__device__ __attribute__((always_inline)) inline void step_tile(const Grid &g, const Phys &p, const Bufs &b, int tile, double *sm,
                                                             StageT<ST> *stage)
{
    constexpr int Q = L::Q, D = L::D, F = 2 * L::D;
    constexpr bool kStage = STG && kStageOdd<L, ST, ODD, LBM, NP>;
    LdsT<ST> *const stg = (LdsT<ST> *)stage;
    const int base = tile * kTile;
    const int n = tile * kTile + threadIdx.x;
    const bool active = n < g.n_f;
    const int P = g.P;
    float acc[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    bool at_end = false;
    double res[2] = {0, 0};

    // coordinates and neighbours of the node
    int x = 0, y = 0, z = 0;
    Nbrs<L> nb;
    bool inert = false;             // a face may be an inert solid
    bool end[2] = {false, false};  // the +x / -x face is an end of the ions' own
    bool edge = false;
    // odd parity, staged: the node's own slots are loaded between its
    // coordinates and its neighbours' rows (the three in flight together: each
    // wait is for the earliest), and stored into the stage after the lookups
    // are issued
    StageT<ST> own[kStage ? Q : 1];
    // ion-only steps read their faces' neighbours from the list, when the
    // instance has one: one dependent load fewer (512^3 electrode: 0.82 ms
    // against 0.87 through the rows). Steps with a flow, whose nodes need their
    // coordinates anyway, look them up in the rows (fused: moments 1.61 ms
    // against 1.80, FP32 2.73 against 2.88, FP16 2.29 against 2.30)
    constexpr bool need_all = LBM && (ODD || !kPlain<ST>);
    const bool list = !LBM && g.nbr;
    const bool coords = LBM || !list;
    if (active) {
        uint32_t packed = 0;
        if (coords) packed = ldu(g.fluid, (uint32_t)n);
        if constexpr (kStage) {
#pragma unroll
            for (int q = 0; q < Q; ++q) own[q] = *pop_at<Q, StageT<ST>>(b.f, q, n);
        }
        if (coords) unpack_xyz(g, packed, x, y, z);
        edge = LBM && g.inout && (b.flags & kNee) && (x <= 1 || x >= g.nx - 2);
        if (list) {  // precomputed: independent of the coordinates
            nb.n[0] = n;
            nb.fl[0] = true;
            int m[F + 1];
#pragma unroll
            for (int i = 1; i <= F; ++i) m[i] = ldu(g.nbr + (size_t)(i - 1) * P, (uint32_t)n);
            keep_order();
#pragma unroll
            for (int i = 1; i <= F; ++i) {
                set_nbr<L>(nb, i, m[i], n);
                inert = inert || m[i] == kInert;
            }
            end[0] = !g.periodic_x && m[1] == kOutside;
            end[1] = !g.periodic_x && m[2] == kOutside;
        } else if (need_all || NP) {
            nb_rows<L, need_all>(g, x, y, z, n, nb, inert);
            end[0] = !g.periodic_x && x == g.nx - 1;
            end[1] = !g.periodic_x && x == 0;
        } else if (edge) {  // an even flow step looks at its x neighbours only there
            set_nbr<L>(nb, 1, nb_map<L>(g, x, y, z, 1, g.periodic_x), n);
            set_nbr<L>(nb, 2, nb_map<L>(g, x, y, z, 2, g.periodic_x), n);
        }
        if constexpr (kStage) {
#pragma unroll
            for (int q = 0; q < Q; ++q) stg[q * kTile + threadIdx.x] = own[q];
        }
    }

    // Fused step, in this order: the ions' own and face-neighbour
    // concentrations (and with FP32 populations their mass fluxes) are loaded;
    // the flow's incoming populations are gathered; the ion update (which
    // needs only the previous step's flux) is computed and stored; then the
    // collision. The ions' loads overlap the flow's, and the ions' inputs
    // are dead before the collision's register peak. With the moment buffers
    // the face neighbours' moments are loaded once for both parts (the flow's
    // emitters, the ions' mass flux). Measured on the 512^3 electrode against
    // loading the ions' inputs after the flow's stores: FP32 -16 %, moments
    // -17 %, FP16 deviations -16 % per fused step. An ion-only step loads them
    // the same way, all before its faces.
    constexpr bool kEarlyJ = kPlain<ST> || !LBM;  // the ions' flux is the stored one
    // with a potential field, the neighbours' potential too, where the flux
    // is loaded early (ion-only step 1.18 -> 0.96 ms, FP32 fused 3.50 ->
    // 3.27 ms on the 512^3 electrode, same waves per SIMD); not in the
    // batched kernels, whose per-instance descriptor leaves no registers to
    // spare (their ion-only and FP16 / moment fused forms lose a wave per
    // SIMD, which costs the served requests, all in the ramp, 10 %)
    constexpr bool kEarlyPsi = kEarlyJ && PSI == kPsiField;
    const int form = PSI != kPsiAny ? PSI : p.psi || p.steep ? kPsiField : p.far ? kPsiFar : 0;
    const bool psi = (PSI == kPsiField || PSI == kPsiAny) && p.psi;
    float cP[2] = {0.f, 0.f}, jP[3] = {0.f, 0.f, 0.f};
    __half2 elo = __floats2half2_rn(0.f, 0.f);
    float2 cn[F];
    float jn[F], psin[F];
    if (NP && active) {
        const float2 c = ld_conc<ST>(b.Cin, (uint32_t)n);
        cP[0] = c.x;
        cP[1] = c.y;
        elo = ldu(b.Clin, (uint32_t)n);
        if (kEarlyJ) {
            jP[0] = ldu(b.jin, (uint32_t)n);
            jP[1] = ldu(b.jin + P, (uint32_t)n);
            jP[2] = D == 3 ? ldu(b.jin + 2 * (size_t)P, (uint32_t)n) : 0.f;
        }
#pragma unroll
        for (int k = 0; k < F; ++k) {
            const uint32_t q = (uint32_t)nb.n[k + 1];
            // (loaded for the lanes whose face is fluid: with the node's own
            // values in the others, FP32 fused steps took 2 % longer)
            cn[k] = make_float2(0.f, 0.f);
            jn[k] = 0.f;
            if (nb.fl[k + 1]) {
                cn[k] = ld_conc<ST>(b.Cin, q);
                if (kEarlyJ) jn[k] = ldu(b.jin + (size_t)(k >> 1) * P, q);
            }
            psin[k] = kEarlyPsi && p.psi ? ldu(p.psi, q) : 0.f;
        }
        keep_order();
    }
    StageSlots<L, ST> slots;
    if (kStage) {
        if (active) stage_slots<L, ST>(nb, base, slots);
        __syncthreads();
    }
    const bool nee = g.inout && (b.flags & kNee);
    // fused, with the moment buffers: the ions' flux is in the moments (else,
    // on the first step of a call, in jin)
    const bool jm = LBM && !kPlain<ST> && (b.flags & kJFromM);

    // the flow's incoming populations (the collision follows the ions)
    float f[kMoments<ST> ? 1 : Q];
    MomSums sums;  // with the moment buffers: their moments
    bool do_flow = false;
    PlaneRef pr{};  // the node's plane references
    if (LBM && active) {
        // a boundary node with a fluid interior neighbour is advanced by that neighbour
        do_flow = !(edge && ((x == 0 && nb.fl[1]) || (x == g.nx - 1 && nb.fl[2])));
        if (kRefs<ST>) pr = plane_ref<ST == kMomR ? 0 : ODD>(g, b.rin, b.rout, x);
        if (!kPlain<ST>) {
            // The emitters' moments in groups whose loads are issued together
            // (the node's own where the emitter is solid), then used; one at a
            // time each load waited for its data before the next was issued.
            // Fused: the node and its faces first, shared with the ions, then
            // the edge directions in groups of 6 (512^3 electrode: 1.60 ms;
            // groups of 4 1.66, of 12 1.61 and, with plane references, 2.02
            // against 1.84); flow only: groups of 10 (1.05 ms; all 18 at once
            // 1.10, groups of 6 1.09).
            DevSums<ST> dsums;
            auto eval = [&](int i, float4 m) {
                const float gi = emitter_g<L, ST>(i, i != 0 && nb.fl[L::opp[i]], m, p, pr);
                if constexpr (!kMoments<ST>) {
                    const float dev = gather_raw<L, ST, ODD>(b.f, P, nb, n, i) * p.hs_inv;
                    f[i] = fmaf(L::w[i], gi, dev);
                    add_plain<L>(dsums, i, dev);
                }
                return gi;
            };
            auto use = [&](int i, float4 m, float4 mo) {  // directions i (odd) and i + 1
                static_assert(L::opp[1] == 2 && L::opp[Q - 2] == Q - 1, "opposite directions are neighbours");
                const float gi = eval(i, m);
                add_pair<L>(sums, i, gi, eval(i + 1, mo));
            };
            auto load = [&](int i) { return ldu(b.Min, (uint32_t)(i == 0 ? n : nb.n[L::opp[i]])); };
            constexpr int kG = NP ? 6 : 10, i1 = NP ? F + 1 : 1;
            if (NP) {
                float4 mg[F + 1];
#pragma unroll
                for (int i = 0; i <= F; ++i) mg[i] = load(i);
                keep_order();
                if (jm) {
                    auto rho_of = [&](int k, float mx) {  // face k's emitter (k < 0: the node)
                        if (ST != kMomR) return 1.f + mx;
                        return 1.f + (k < 0 || k > 1 || !nb.fl[k + 1] ? pr.rin[1] : pr.rin[k == 0 ? 0 : 2]) + mx;
                    };
                    const float r = rho_of(-1, mg[0].x);
                    jP[0] = r * mg[0].y;
                    jP[1] = r * mg[0].z;
                    jP[2] = D == 3 ? r * mg[0].w : 0.f;
#pragma unroll
                    for (int k = 0; k < F; ++k) {
                        const float4 m = mg[L::opp[k + 1]];
                        jn[k] = rho_of(k, m.x) * (k < 2 ? m.y : (k < 4 ? m.z : m.w));
                    }
                } else if (!kEarlyJ) {
                    jP[0] = ldu(b.jin, (uint32_t)n);
                    jP[1] = ldu(b.jin + P, (uint32_t)n);
                    jP[2] = D == 3 ? ldu(b.jin + 2 * (size_t)P, (uint32_t)n) : 0.f;
#pragma unroll
                    for (int k = 0; k < F; ++k)
                        jn[k] = ldu(b.jin + (size_t)(k >> 1) * P, (uint32_t)nb.n[k + 1]);
                }
                add_rest<L>(sums, eval(0, mg[0]));
#pragma unroll
                for (int i = 1; i < F; i += 2) use(i, mg[i], mg[i + 1]);
            }
#pragma unroll
            for (int i0 = i1; i0 < Q; i0 += kG) {
                float4 mg[kG];
#pragma unroll
                for (int u = 0; u < kG; ++u)
                    if (i0 + u < Q) mg[u] = load(i0 + u);
                float4 m0 = make_float4(0.f, 0.f, 0.f, 0.f);
                if (!NP && i0 == i1) m0 = load(0);
                keep_order();
                if (!NP && i0 == i1) add_rest<L>(sums, eval(0, m0));
#pragma unroll
                for (int u = 0; u < kG; u += 2)
                    if (i0 + u < Q) use(i0 + u, mg[u], mg[u + 1]);
            }
            dsums.add_to(sums);
        } else if (do_flow) {
            if (kStage) {
                const float sc = kHalfPop<ST> ? p.hs_inv : 1.f;
                StageT<ST> raw[Q];
                staged_gather<L, ST>(b.f, nb, stg, slots, raw);
                stage_forget(slots);
#pragma unroll
                for (int i = 0; i < Q; ++i) f[i] = rel_pop<L, ODD>(sc * pop_float<ST>(raw[i]), i, nb, pr);
            } else {
#pragma unroll
                for (int i = 0; i < Q; ++i)
                    f[i] = rel_pop<L, ODD>(gather<L, ST, ODD>(b.f, P, nb, n, i, b.Min, p, pr), i, nb, pr);
            }
        }
    }

    // the ions: face fluxes of the explicit finite-volume update
    if (NP && active) {
        IonFlux fx;
        bool on[F];  // faces to fluid cells
        if (g.periodic_x && p.npx != kNpxPeriodic) {  // a periodic lattice whose ions have ends
            if (!coords) unpack_xyz(g, ldu(g.fluid, (uint32_t)n), x, y, z);
            end[0] = x == g.nx - 1;
            end[1] = x == 0;
        }
        // the adsorbing faces: not fluid, no end, and not inert
#pragma unroll
        for (int k = 0; k < F; ++k) {
            const bool e = k < 2 && end[k & 1];
            fx.ads += nb.fl[k + 1] || e ? 0.f : 1.f;
            on[k] = nb.fl[k + 1] && !e;
        }
        if (inert) {  // rare
            if (!coords) unpack_xyz(g, ldu(g.fluid, (uint32_t)n), x, y, z);
            int m[F];
#pragma unroll
            for (int k = 0; k < F; ++k) m[k] = nb_map<L>(g, x, y, z, k + 1, g.periodic_x);
#pragma unroll
            for (int k = 0; k < F; ++k) fx.ads -= m[k] == kInert && !(k < 2 && end[k & 1]) ? 1.f : 0.f;
        }
        float psiP = 0.f;
        if (form == kPsiField) {
            if (psi) {
                psiP = ldu(p.psi, (uint32_t)n);
                if (!kEarlyPsi) {
#pragma unroll
                    for (int k = 0; k < F; ++k) psin[k] = ldu(p.psi, (uint32_t)nb.n[k + 1]);
                }
            }
            ion_faces_any<L>(p, psi, on, cP, jP, psiP, cn, jn, psin, fx);
        } else if (form == kPsiFar) {
            ion_faces_far<L>(p, on, cP, jP, cn, jn, fx);
        } else if (!ion_faces<L>(p, on, cP, jP, cn, jn, fx)) {  // rare
            if (!coords) unpack_xyz(g, ldu(g.fluid, (uint32_t)n), x, y, z);
            ion_faces_wide<L, ST>(g, p, b, x, y, z, jm, end, cP[0], cP[1], jP[0], jP[1], jP[2], fx);
        }
        at_end = end[0] || end[1];
        if (at_end) {  // (not both: nx >= 4)
            if (!coords) unpack_xyz(g, ldu(g.fluid, (uint32_t)n), x, y, z);
            ion_end_face<L, ST>(g, p, b, end[0] ? 1 : -1, x, y, z, jm, psi, cP[0], cP[1], jP[0], psiP, fx);
        }
        const float fa[2] = {fx.ads * (p.keff[0] * cP[0]), fx.ads * (p.keff[1] * cP[1])};
        // forward Euler into value + remainder (see lo_encode)
        float e0, e1;
        const float c0 = two_sum(cP[0], lo_decode(__low2half(elo)) - p.dt * (fx.out[0] + fa[0]), e0);
        const float c1 = two_sum(cP[1], lo_decode(__high2half(elo)) - p.dt * (fx.out[1] + fa[1]), e1);
        st_conc<ST>(b.Cout, (uint32_t)n, make_float2(c0, c1));
        stu(b.Clout, (uint32_t)n, __halves2half2(lo_encode(e0), lo_encode(e1)));
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            acc[s] = p.dt * fa[s];
            acc[2 + s] = p.dt * fx.fi[s];
            acc[4 + s] = p.dt * fx.fo[s];
        }
    }

    // the flow: collide and stream (and the residual terms on request)
    if (LBM && do_flow) {
        if constexpr (kMoments<ST>)
            moment_node<L>(b, n, sums.d, sums.jx, sums.jy, sums.jz, pr.rout, res);
        else
            lbm_node<L, ST, ODD, NP, kStage>(p, b, P, n, nb, f, pr, res, kPlain<ST> ? nullptr : &sums, stg, &slots,
                                             !(nee && (x == 0 || x == g.nx - 1)));
        const bool inl = edge && x == 1 && nb.fl[2];
        const bool outl = edge && x == g.nx - 2 && nb.fl[1];
        if (inl || outl) {
            // the boundary node's moments are the target equilibrium's: the
            // extrapolated non-equilibrium part carries none
            const int bn = inl ? nb.n[2] : nb.n[1];
            const int xb = inl ? 0 : g.nx - 1;
            PlaneRef pb{};
            if (kRefs<ST>) pb = plane_ref<ODD>(g, b.rin, b.rout, xb);
            MomSums sb;
            if constexpr (!kPlain<ST>) sb = nee_moments(p, inl, sums, pr.rout, pb.rout);
            if constexpr (kMoments<ST>) {
                moment_node<L>(b, bn, sb.d, sb.jx, sb.jy, sb.jz, pb.rout, res);
            } else {
                Nbrs<L> nbb;
                nbb.n[0] = bn;
                nbb.fl[0] = true;
#pragma unroll
                for (int i = 1; i < Q; ++i) set_nbr<L>(nbb, i, nb_map<L>(g, xb, y, z, i, false), bn);  // rare path
                float fb[Q];
                nee_populations<L>(p, inl, f, fb, pr.rout, pb.rout);
                lbm_node<L, ST, ODD, NP>(p, b, P, bn, nbb, fb, pb, res, kPlain<ST> ? nullptr : &sb);
            }
        }
    }
    if (kStage) {
        // the owner stores back each slot whose reader (and writer) is in the
        // tile: node x - e_q for slot q when that voxel is fluid, else the node
        __syncthreads();
        if (active) {
            stage_forget(slots);
            const bool end0 = nee && (x == 0 || x == g.nx - 1), endm = nee && x == 1, endp = nee && x == g.nx - 2;
            // all stage reads first, then the stores (one wait for the reads)
            StageT<ST> v[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) v[q] = stg[q * kTile + threadIdx.x];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int r = L::opp[q];
                const bool fl = q != 0 && nb.fl[r];
                const bool end = L::ex[q] == 0 || !fl ? end0 : (L::ex[q] > 0 ? endm : endp);  // the reader's plane
                if (!slots.outside(r) && !end) *pop_at<Q, StageT<ST>>(b.f, q, n) = v[q];
            }
        }
    }
    if (LBM && (b.flags & kResid)) {
        double s[2];
        block_sum<2>(res, sm, s);
        if (threadIdx.x == 0) {
            b.resid[2 * (size_t)tile] = s[0];
            b.resid[2 * (size_t)tile + 1] = s[1];
        }
        __syncthreads();
    }

    if (NP) tile_accumulate(acc, at_end, sm, b.acc + (size_t)tile * 8);
}

template <class L, int ST, int ODD, int LBM, int NP, int STG, int PSI>
__global__ __launch_bounds__(kTile) void step_kernel(Grid g, Phys p, Bufs b)
{
    __shared__ double sm[kTileSums];
    __shared__ StageT<ST> stage[STG ? kStageElems<L> : 1];
    extern __shared__ double lds_pad[];  // sized at launch: occupancy cap only
    (void)lds_pad;
    if (NP) tile_sums_init(sm);
    step_tile<L, ST, ODD, LBM, NP, PSI, STG>(g, p, b, block_tile(g), sm, stage);
}

// A batch member's descriptor is read from memory, and a pointer read from
// memory is a generic address to the compiler: its accesses become flat
// instructions, which take the vector memory path and count on both wait
// counters. Read through the constant address space (the descriptors do not
// change during a launch), the pointers are known to address global memory
// and their accesses are global ones.
__device__ __forceinline__ void load_inst(const BatchInst *inst, int k, Grid &g, Phys &p, Bufs &b)
{
    g = inst[k].g;
    p = inst[k].p;
    b = inst[k].b;
    typedef const __attribute__((address_space(4))) BatchInst const_inst_t;
    const_inst_t &c = ((const_inst_t *)inst)[k];
    g.fluid = c.g.fluid;
    g.map = c.g.map;
    g.sched = c.g.sched;
    g.nbr = c.g.nbr;
    g.rows = c.g.rows;
    p.psi = c.p.psi;
    b.f = c.b.f;
    b.f2 = c.b.f2;
    b.Min = c.b.Min;
    b.Mout = c.b.Mout;
    b.jin = c.b.jin;
    b.jout = c.b.jout;
    b.Cin = c.b.Cin;
    b.Cout = c.b.Cout;
    b.Clin = c.b.Clin;
    b.Clout = c.b.Clout;
    b.acc = c.b.acc;
    b.resid = c.b.resid;
    b.ubuf = c.b.ubuf;
    b.rin = c.b.rin;
    b.rout = c.b.rout;
}

// Many instances in one persistent launch per step class (LBM parity and
// mode): workgroup w takes entries w, w + G, w + 2G, ... of the class's list
// of (instance, tile) pairs. Each instance carries its own lattice,
// parameters and buffers, so uneven sizes share the launch; the descriptor is
// copied once per tile into registers. Tile results do not depend on which
// workgroup computes them.
template <class L, int ST, int ODD, int LBM, int NP, int PSI>
__global__ __launch_bounds__(kTile) void batch_kernel(const BatchInst *__restrict__ inst,
                                                      const int2 *__restrict__ tiles, int ntiles)
{
    __shared__ double sm[kTileSums];
    extern __shared__ double lds_pad[];
    (void)lds_pad;
    if (NP) tile_sums_init(sm);
    // workgroups are dealt round-robin over the 8 XCDs: each XCD takes one
    // contiguous eighth of the list, so neighbouring tiles share its L2
    const int G = (int)gridDim.x, w = (int)blockIdx.x;
    int lo = 0, hi = ntiles, first = w, stride = G;
    if (G >= 8) {
        const int x = w & 7;
        lo = (int)((int64_t)ntiles * x / 8);
        hi = (int)((int64_t)ntiles * (x + 1) / 8);
        first = lo + (w >> 3);
        stride = (G - x + 7) >> 3;
    }
    for (int q = first; q < hi; q += stride) {
        const int2 e = tiles[q];
        Grid g;
        Phys p;
        Bufs b;
        load_inst(inst, e.x, g, p, b);
        step_tile<L, ST, ODD, LBM, NP, PSI>(g, p, b, e.y, sm, nullptr);  // not staged
        if (NP && q + stride < hi) __syncthreads();  // the next tile reuses the sums
    }
}

// Dynamic LDS of an occupancy cap (pad bytes beside the kernels' own small
// scratch), less what a staged odd step declares itself, so that the cap
// admits the same number of workgroups per CU for every step class.
template <class L, int ST, int STG>
size_t cap_lds(int pad)
{
    const size_t stage = STG ? sizeof(StageT<ST>) * kStageElems<L> : 0;
    return (size_t)pad > stage ? (size_t)pad - stage : 0;
}

// Form of the flow-only kernels, which read no concentrations.
template <int ST>
constexpr int kFlowForm = ST == kH16L ? kH16 : ST;

template <class L, int ST>
void launch_batch_t(int cls, const BatchInst *inst, const int2 *tiles, int ntiles, int wg, int pad,
                    hipStream_t s)
{
    const size_t lds = (size_t)pad;
    constexpr int F = kFlowForm<ST>, R = ST == kH16L ? kPsiAny : 0;  // (kH16L: rare)
    constexpr int O1 = kMoments<ST> ? 0 : 1, OP = kMoments<ST> ? 0 : kPull;  // the moment forms have no parity
#define BK(S, O, NP, PSI) batch_kernel<L, S, O, 1, NP, PSI><<<wg, kTile, lds, s>>>(inst, tiles, ntiles)
    switch (cls) {
    case kClassFlowEven: BK(F, 0, 0, 0); break;
    case kClassFlowOdd: BK(F, O1, 0, 0); break;
    case kClassFlowPull: BK(F, OP, 0, 0); break;
    case kClassFusedEven: BK(ST, 0, 1, R); break;
    case kClassFusedOdd: BK(ST, O1, 1, R); break;
    case kClassFusedPull: BK(ST, OP, 1, R); break;
    case kClassAny + kClassFusedEven: BK(ST, 0, 1, kPsiAny); break;
    case kClassAny + kClassFusedOdd: BK(ST, O1, 1, kPsiAny); break;
    default: BK(ST, OP, 1, kPsiAny); break;
    }
#undef BK
}

template <class L, int ST, int ODD, int LBM, int NP, int PSI>
void launch_psi(const Grid &g, const Phys &p, const Bufs &b, hipStream_t s)
{
    const unsigned T = (unsigned)(g.P / kTile);
    if constexpr (kStageOdd<L, ST, ODD, LBM, NP>) {
        if (g.stage_odd) {
            step_kernel<L, ST, ODD, LBM, NP, 1, PSI><<<T, kTile, cap_lds<L, ST, 1>(g.lds_pad), s>>>(g, p, b);
            return;
        }
    }
    step_kernel<L, ST, ODD, LBM, NP, 0, PSI><<<T, kTile, (size_t)g.lds_pad, s>>>(g, p, b);
}

// Kernels of their own for ions in a potential field or a steep ramp, and for
// flows with many faces beyond the series' range, whose code would cost the
// others registers.
template <class L, int ST, int ODD, int LBM, int NP>
void launch_t(const Grid &g, const Phys &p, const Bufs &b, hipStream_t s)
{
    if (NP && (p.psi || p.steep))
        launch_psi<L, ST, ODD, LBM, NP, NP * kPsiField>(g, p, b, s);
    else if (NP && p.far)
        launch_psi<L, ST, ODD, LBM, NP, NP * kPsiFar>(g, p, b, s);
    else
        launch_psi<L, ST, ODD, LBM, NP, 0>(g, p, b, s);
}

template <class L, int ST, int ODD>
void launch_mode(int lbm, int np, const Grid &g, const Phys &p, const Bufs &b, hipStream_t s)
{
    if (lbm && np)
        launch_t<L, ST, ODD, 1, 1>(g, p, b, s);
    else if (lbm)
        launch_t<L, kFlowForm<ST>, ODD, 1, 0>(g, p, b, s);
    else
        launch_t<L, ST == kH16L ? kH16L : kF32, 0, 0, 1>(g, p, b, s);
}

template <class L, int ST>
void launch_form(int odd, int lbm, int np, const Grid &g, const Phys &p, const Bufs &b, hipStream_t s)
{
    if constexpr (kMoments<ST>) {  // no parity
        launch_mode<L, ST, 0>(lbm, np, g, p, b, s);
    } else {
        if (odd == kPull)
            launch_mode<L, ST, kPull>(lbm, np, g, p, b, s);
        else if (odd)
            launch_mode<L, ST, 1>(lbm, np, g, p, b, s);
        else
            launch_mode<L, ST, 0>(lbm, np, g, p, b, s);
    }
}

template <class L>
void launch_prec(int st, int odd, int lbm, int np, const Grid &g, const Phys &p, const Bufs &b,
                 hipStream_t s)
{
    switch (st) {
    case kMom: launch_form<L, kMom>(odd, lbm, np, g, p, b, s); break;
    case kMomR: launch_form<L, kMomR>(odd, lbm, np, g, p, b, s); break;
    case kH16: launch_form<L, kH16>(odd, lbm, np, g, p, b, s); break;
    case kH16L: launch_form<L, kH16L>(odd, lbm, np, g, p, b, s); break;
    case kF16: launch_form<L, kF16>(odd, lbm, np, g, p, b, s); break;
    default: launch_form<L, kF32>(odd, lbm, np, g, p, b, s); break;
    }
}

template <class L>
void launch_batch_l(int cls, const BatchInst *inst, const int2 *tiles, int ntiles, int wg, int pad,
                    hipStream_t s)
{
    if (cls >= kClassIons) {
        if (cls == kClassIonsL)
            batch_kernel<L, kH16L, 0, 0, 1, kPsiAny><<<wg, kTile, (size_t)pad, s>>>(inst, tiles, ntiles);
        else if (cls == kClassIonsAny)
            batch_kernel<L, kF32, 0, 0, 1, kPsiAny><<<wg, kTile, (size_t)pad, s>>>(inst, tiles, ntiles);
        else
            batch_kernel<L, kF32, 0, 0, 1, 0><<<wg, kTile, (size_t)pad, s>>>(inst, tiles, ntiles);
        return;
    }
    const int k = cls % kClassesPerForm;
    switch (cls / kClassesPerForm) {
    case kMom: launch_batch_t<L, kMom>(k, inst, tiles, ntiles, wg, pad, s); break;
    case kMomR: launch_batch_t<L, kMomR>(k, inst, tiles, ntiles, wg, pad, s); break;
    case kH16: launch_batch_t<L, kH16>(k, inst, tiles, ntiles, wg, pad, s); break;
    case kH16L: launch_batch_t<L, kH16L>(k, inst, tiles, ntiles, wg, pad, s); break;
    case kF16: launch_batch_t<L, kF16>(k, inst, tiles, ntiles, wg, pad, s); break;
    default: launch_batch_t<L, kF32>(k, inst, tiles, ntiles, wg, pad, s); break;
    }
}

}  // namespace

hipError_t launch_batch(int dim, int cls, const BatchInst *inst, const int2 *tiles, int ntiles,
                        int workgroups, int lds_pad, hipStream_t s)
{
    if (ntiles <= 0 || workgroups <= 0) return hipSuccess;
    if (cls < 0 || cls >= kClasses) return hipErrorInvalidValue;
    if (dim == 2)
        launch_batch_l<D2Q9>(cls, inst, tiles, ntiles, workgroups, lds_pad, s);
    else
        launch_batch_l<D3Q19>(cls, inst, tiles, ntiles, workgroups, lds_pad, s);
    return hipGetLastError();
}

hipError_t launch_step(int dim, int st, int odd, int lbm, int np, const Grid &g, const Phys &p,
                       const Bufs &b, hipStream_t s)
{
    if (g.P <= 0) return hipSuccess;
    if (st < 0 || st >= kForms) return hipErrorInvalidValue;
    if (dim == 2)
        launch_prec<D2Q9>(st, odd, lbm, np, g, p, b, s);
    else
        launch_prec<D3Q19>(st, odd, lbm, np, g, p, b, s);
    return hipGetLastError();
}

}  // namespace cdi
