// device_common.h -- device helpers shared by the step and auxiliary kernels:
// neighbour lookup through the fluid index map, the BGK equilibrium, the AA
// storage rules, the inlet/outlet extrapolation and block reductions.
//
// AA storage rules (Bailey et al. 2009). With the stored state at parity 0
// ("A"), the post-streaming population f_i(x) sits in node x, slot i; a step
// reads it there, collides, and writes f*_i back into node x, slot opp(i).
// With the state at parity 1 ("B"), f_i(x) sits in node x - e_i, slot opp(i)
// when that voxel is fluid, else in node x, slot i (it was reflected); a step
// reads it there and writes f*_i into node x + e_i, slot i (fluid), or into
// node x, slot opp(i) (half-way bounce-back off a solid face, the no-flow
// rule). Each node reads and writes the same set of slots, so a step is
// race-free in place.
//
// FP16 storage keeps, instead of f - w_i, the post-collision deviation from
// the emitting node's equilibrium, times hs; the emitter's moments
// (rho - 1, u) are kept in FP32. The emitter of f_i(x) is x - e_i if that
// voxel is fluid, else x itself (which sent it in direction opp(i)).
//
// Pull streaming (ODD = kPull) keeps two arrays: a step reads f_i(x) from
// node x - e_i, slot i of the input array when that voxel is fluid, else from
// node x, slot opp(i) (its own reflected population), and writes f*_i into
// node x, slot i of the output array.
//
// Moment storage keeps the moments alone: with tau = 1 and no body force the
// BGK post-collision populations are exactly the equilibrium of the node's
// moments (the FP16 deviations above are then identically zero), so f_i(x)
// is the emitter's equilibrium and no population is stored; the AA parity
// plays no role.
#pragma once

#include "cdi_internal.h"

namespace cdi {

// Element idx of an array whose base is the same for the whole wave. The
// address is formed as base + a 32-bit byte offset, which the hardware takes
// as a scalar base plus one vector offset: no 64-bit address arithmetic per
// lane, and one offset serves every array indexed by the same node. The host
// keeps idx * sizeof(T) below 2^32.
template <class T>
__device__ __forceinline__ T ldu(const T *base, uint32_t idx)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + idx * (uint32_t)sizeof(T));
}

template <class T>
__device__ __forceinline__ void stu(T *base, uint32_t idx, T v)
{
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + idx * (uint32_t)sizeof(T)) = v;
}

// Both species' concentrations of node n.
template <int ST>
__device__ __forceinline__ float2 ld_conc(const float2 *C, uint32_t n)
{
    static_assert(ST == kH16L || offset_elem(ST) >= (int)sizeof(float2), "a pair's byte offset has to fit");
    if constexpr (ST == kH16L) return C[n];
    else return ldu(C, n);
}

template <int ST>
__device__ __forceinline__ void st_conc(float2 *C, uint32_t n, float2 v)
{
    if constexpr (ST == kH16L) C[n] = v;
    else stu(C, n, v);
}

// No instruction is scheduled across this point: loads written before it are
// issued before what uses them. (Left alone, the scheduler moves each load down
// to its use to save registers, two in flight at a time.)
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0); }

// blockIdx -> tile: workgroups are dealt round-robin over the 8 XCDs, each
// with its own L2; this keeps consecutive tiles on one XCD so that the y/z
// neighbours a tile touches were mostly fetched by the same L2.
__device__ inline int xcd_tile(int b, int nb)
{
    const int q = nb >> 3, r = nb & 7;
    const int xcd = b & 7, k = b >> 3;
    return xcd * q + (xcd < r ? xcd : r) + k;
}

// Tile processed by this workgroup: its XCD-local position, through the
// (band, z) schedule when there is one.
__device__ inline int block_tile(const Grid &g)
{
    const int pos = xcd_tile(blockIdx.x, gridDim.x);
    return g.sched ? g.sched[pos] : pos;
}

// map value of the neighbour of (x,y,z) along direction i: fluid index,
// kElectrode, kInert, or kOutside past an open x end. y and z wrap.
template <class L>
__device__ inline int nb_map(const Grid &g, int x, int y, int z, int i, bool periodic_x)
{
    int xn = x + L::ex[i];
    if (xn < 0 || xn >= g.nx) {
        if (!periodic_x) return kOutside;
        xn = xn < 0 ? xn + g.nx : xn - g.nx;
    }
    int yn = y + L::ey[i];
    yn = yn < 0 ? yn + g.ny : (yn >= g.ny ? yn - g.ny : yn);
    int zn = z;
    if (L::D == 3) {
        zn = z + L::ez[i];
        zn = zn < 0 ? zn + g.nz : (zn >= g.nz ? zn - g.nz : zn);
    }
    return g.map[brick_index(g.bk, xn, yn, zn)];
}

__device__ inline void unpack_xyz(const Grid &g, uint32_t c, int &x, int &y, int &z)
{
    x = (int)(c & ((1u << g.bk.cbx) - 1));
    y = (int)((c >> g.bk.cbx) & ((1u << g.bk.cby) - 1));
    z = (int)(c >> (g.bk.cbx + g.bk.cby));
}

// Neighbour lookup context of one voxel: for each axis and offset -1/0/+1,
// that axis's share of the neighbour's brick-ordered index. The brick part
// (above the in-brick bits) and the in-brick part occupy disjoint bits, so a
// neighbour's index is the plain sum of its three axis shares: one three-way
// add per lattice direction (the shares are kept as byte offsets into the
// map, below 2^32 for 2^30 voxels). Coordinates wrap on every axis (the index is
// always in range); xo marks offsets beyond an open x end.
struct NbCtx {
    uint32_t X[3], Y[3], Z[3];
    bool xo[3];
};

template <class L>
__device__ inline void nb_ctx(const Grid &g, int x, int y, int z, bool periodic_x, NbCtx &c)
{
    const Bricks &k = g.bk;
    const int V = k.bsx + k.bsy + k.bsz;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        int xn = x + d - 1;
        bool out = false;
        if (xn < 0 || xn >= g.nx) {
            out = !periodic_x;
            xn = xn < 0 ? xn + g.nx : xn - g.nx;
        }
        c.xo[d] = out;
        c.X[d] = (((uint32_t)(xn >> k.bsx) << V) | (uint32_t)(xn & ((1 << k.bsx) - 1))) << 2;
        int yn = y + d - 1;
        yn = yn < 0 ? yn + g.ny : (yn >= g.ny ? yn - g.ny : yn);
        // brick-row products as 24-bit multiplies (full rate; the 32-bit
        // multiply issues at a quarter): below 2^30 voxels, no brick count or
        // brick index reaches 2^24
        c.Y[d] = ((__umul24((uint32_t)(yn >> k.bsy), (uint32_t)k.nbx) << V) |
                  ((uint32_t)(yn & ((1 << k.bsy) - 1)) << k.bsx)) << 2;
        if (L::D == 3) {
            int zn = z + d - 1;
            zn = zn < 0 ? zn + g.nz : (zn >= g.nz ? zn - g.nz : zn);
            c.Z[d] = ((__umul24((uint32_t)(zn >> k.bsz), (uint32_t)(k.nbx * k.nby)) << V) |
                      ((uint32_t)(zn & ((1 << k.bsz) - 1)) << (k.bsx + k.bsy))) << 2;
        } else {
            c.Z[d] = 0;
        }
    }
}

// map value of the neighbour along direction i (see nb_map). Past an open x
// end the wrapped voxel is read (always in range) and replaced by kOutside.
template <class L>
__device__ inline int nb_get(const Grid &g, const NbCtx &c, int i)
{
    const int dx = L::ex[i] + 1, dy = L::ey[i] + 1, dz = L::ez[i] + 1;
    const int m = *reinterpret_cast<const int *>(reinterpret_cast<const char *>(g.map) + (c.X[dx] + c.Y[dy] + c.Z[dz]));
    return (L::ex[i] != 0 && c.xo[dx]) ? kOutside : m;
}

// A node's neighbours: n[i] the node along direction i, the node itself where
// that voxel is not fluid (fl[i] false).
template <class L>
struct Nbrs {
    int n[L::Q];
    bool fl[L::Q];
};

template <class L>
__device__ __forceinline__ void set_nbr(Nbrs<L> &nb, int i, int m, int self)
{
    nb.fl[i] = m >= 0;
    nb.n[i] = m >= 0 ? m : self;
}

// Neighbours of node n at (x, y, z) from the lattice's rows (see cdi_internal.h): all
// directions (ALL) or the faces. inert: a row of its faces holds an inert solid.
template <class L, int ALL>
__device__ __forceinline__ void nb_rows(const Grid &g, int x, int y, int z, int n, Nbrs<L> &nb, bool &inert)
{
    const Bricks &k = g.bk;
    const int S = k.bsy + k.bsz, xi = x & ((1 << k.bsx) - 1);
    uint32_t Y[3], Z[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {  // row shares of the three y and z, as byte offsets
        int yn = y + d - 1;
        yn = yn < 0 ? yn + g.ny : (yn >= g.ny ? yn - g.ny : yn);
        Y[d] = ((__umul24((uint32_t)(yn >> k.bsy), (uint32_t)k.nbx) << S) | (uint32_t)(yn & ((1 << k.bsy) - 1))) << 4;
        if (L::D == 3) {
            int zn = z + d - 1;
            zn = zn < 0 ? zn + g.nz : (zn >= g.nz ? zn - g.nz : zn);
            Z[d] = ((__umul24((uint32_t)(zn >> k.bsz), (uint32_t)(k.nbx * k.nby)) << S) |
                    ((uint32_t)(zn & ((1 << k.bsz) - 1)) << k.bsy)) << 4;
        } else {
            Z[d] = 0;
        }
    }
    const uint32_t X = (uint32_t)(x >> k.bsx) << (S + 4);
    // rows by (ey + 1) + 3 (ez + 1); the edges and corners of the y-z square
    // hold one direction each with ALL, none otherwise
    int4 r[9];
    uint32_t t[9];
    int c[9];
#pragma unroll
    for (int q = 0; q < (L::D == 3 ? 9 : 3); ++q) {
        const int s = L::D == 3 ? q : q + 3;
        const int dy = s % 3, dz = s / 3;
        const bool corner = dy != 1 && dz != 1;
        if (corner && !ALL) continue;
        const char *at = reinterpret_cast<const char *>(g.rows) + (X + Y[dy] + Z[dz]);
        if (s == 4 || (!corner && ALL)) {
            r[s] = *reinterpret_cast<const int4 *>(at);
        } else {
            const int2 h = *reinterpret_cast<const int2 *>(at);
            r[s] = make_int4(h.x, h.y, 0, 0);
        }
    }
    const bool first = xi == 0, last = xi == (1 << k.bsx) - 1 || x == g.nx - 1;
#pragma unroll
    for (int q = 0; q < (L::D == 3 ? 9 : 3); ++q) {
        const int s = L::D == 3 ? q : q + 3;
        const bool corner = s % 3 != 1 && s / 3 != 1;
        if (corner && !ALL) continue;
        t[s] = (uint32_t)r[s].y >> xi;  // bits 0, 1, 2: x - 1, x, x + 1
        c[s] = s == 4 ? n : r[s].x + __popc(((uint32_t)r[s].y >> 1) & ((1u << xi) - 1u));
    }
    nb.n[0] = n;
    nb.fl[0] = true;
#pragma unroll
    for (int i = 1; i < (ALL ? L::Q : 2 * L::D + 1); ++i) {
        const int s = (L::ey[i] + 1) + 3 * (L::ez[i] + 1);
        int m;
        if (L::ex[i] == 0)
            m = c[s];
        else if (L::ex[i] < 0)
            m = first ? r[s].z : c[s] - 1;
        else
            m = last ? r[s].w : c[s] + (int)((t[s] >> 1) & 1u);
        nb.fl[i] = (t[s] >> (L::ex[i] + 1)) & 1u;
        nb.n[i] = nb.fl[i] ? m : n;
    }
    int any = r[4].y | r[3].y | r[5].y;
    if (L::D == 3) any |= r[1].y | r[7].y;
    inert = any < 0;
}

// acc + c v for a lattice vector component c (-1, 0 or 1 on D2Q9 and D3Q19;
// a constant once a direction loop is unrolled): the product with 0 is
// dropped and the others become an add or a subtraction. The compiler may not
// drop 0 * v by itself (under IEEE rules it is NaN for an infinite v); the
// value is the same, up to the sign of a zero.
__device__ __forceinline__ float lat_add(float acc, int c, float v)
{
    return c == 0 ? acc : (c > 0 ? acc + v : acc - v);
}

// e_i . u, from -0 (the exact additive identity: -0 + v is v for every v).
template <class L>
__device__ __forceinline__ float lat_dot(int i, float ux, float uy, float uz)
{
    return lat_add(lat_add(lat_add(-0.f, L::ex[i], ux), L::ey[i], uy), L::ez[i], uz);
}

// Zeroth and first moments of f: d = sum_i f_i, j = sum_i e_i f_i.
template <class L>
__device__ __forceinline__ void lat_moments(const float (&f)[L::Q], float &d, float &jx, float &jy, float &jz)
{
    d = jx = jy = jz = -0.f;
#pragma unroll
    for (int i = 0; i < L::Q; ++i) {
        d += f[i];
        jx = lat_add(jx, L::ex[i], f[i]);
        jy = lat_add(jy, L::ey[i], f[i]);
        jz = lat_add(jz, L::ez[i], f[i]);
    }
}

// 1 / rho from rho - 1: the hardware reciprocal (within 1 ulp), one
// instruction where an IEEE division takes ten. Every kernel that forms u =
// j / rho uses it, so they all form the same u.
__device__ __forceinline__ float inv_rho(float drho) { return __builtin_amdgcn_rcpf(1.f + drho); }

// BGK equilibrium less w_i (1 + R), R a reference density deviation, split
// into per-node terms so that a direction costs two fused multiply-adds and
// a product: with dr = rho - 1 - R it is w_i (a + e.u (b + c e.u)), where
// a = dr - (3/2) rho u.u, b = 3 rho and c = (9/2) rho; the linear (Stokes)
// part has a = dr and c = 0.
struct EqTerms {
    float a, b, c;
};

__device__ inline EqTerms eq_terms(float dr, float rho, float ux, float uy, float uz, int linear)
{
    if (linear) return EqTerms{dr, 3.f * rho, 0.f};
    const float uu = ux * ux + uy * uy + uz * uz;
    return EqTerms{fmaf(-1.5f * rho, uu, dr), 3.f * rho, 4.5f * rho};
}

__device__ __forceinline__ float feq_eu(float w, const EqTerms &t, float eu)
{
    return w * fmaf(eu, fmaf(t.c, eu, t.b), t.a);
}

// direction i of the node whose terms are t
template <class L>
__device__ __forceinline__ float feq_dir(int i, const EqTerms &t, float ux, float uy, float uz)
{
    return feq_eu(L::w[i], t, lat_dot<L>(i, ux, uy, uz));
}

// FP32 population storage holds f_i - w_i (1 + R[x_s]), where x_s is the x
// plane of the node whose slot holds the value (pull streaming: the emitter,
// the node that collided it; AA: the node written to) and R[x] is a reference
// density deviation per x plane (the plane mean of rho - 1, renewed now and
// then: the stored values then carry only the local fluctuations, which FP32
// rounds far more finely than f - w_i near a pressure drop). A step reads
// with table Rin and writes with table Rout (equal except on the step that
// renews R) and works with g_i = f_i - w_i (1 + Rout[x]) = stored +
// w_i (Rin[x_s] - Rout[x]). A value written into the slot of the neighbour
// x + e_i (AA, odd parity) is stored as g + w_i (Rout[x] - Rout[x + e_x]).
struct PlaneRef {
    float rout;   // Rout[x]
    float dIn[3]; // Rin[x - ex] - Rout[x], ex = -1, 0, 1
    float dOut[3];// Rout[x] - Rout[x + ex]
    float rin[3]; // Rin[x - ex] (a node's density is formed with its plane's own value
                  // wherever two nodes have to agree on it: rout + dIn rounds)
};

// (dOut only for the odd AA parity, which writes into neighbours' slots)
template <int ODD>
__device__ inline PlaneRef plane_ref(const Grid &g, const float *rin, const float *rout, int x)
{
    PlaneRef r{};
    if (!rin) return r;
    const int xm = x > 0 ? x - 1 : (g.periodic_x ? g.nx - 1 : 0);
    const int xp = x < g.nx - 1 ? x + 1 : (g.periodic_x ? 0 : g.nx - 1);
    r.rout = ldu(rout, (uint32_t)x);
    r.rin[0] = ldu(rin, (uint32_t)xp);  // ex = -1: the slot's node is at x + 1
    r.rin[1] = ldu(rin, (uint32_t)x);
    r.rin[2] = ldu(rin, (uint32_t)xm);  // ex = +1: at x - 1
#pragma unroll
    for (int k = 0; k < 3; ++k) r.dIn[k] = r.rin[k] - r.rout;
    if (ODD == 1) {
        r.dOut[0] = r.rout - ldu(rout, (uint32_t)xm);
        r.dOut[2] = r.rout - ldu(rout, (uint32_t)xp);
    }
    return r;
}

// g_i from the stored value read for direction i (ODD: the kernels' parity
// argument) of a node whose neighbours are nb.
template <class L, int ODD>
__device__ __forceinline__ float rel_pop(float raw, int i, const Nbrs<L> &nb, const PlaneRef &r)
{
    const bool fl = (i != 0) && nb.fl[L::opp[i]];
    const bool there = ODD != 0 && fl;  // pull or odd parity: read in the emitter's slot
    return raw + L::w[i] * (there ? r.dIn[L::ex[i] + 1] : r.dIn[1]);
}

// The value to store for outgoing g_i (relative to Rout[x]).
template <class L, int ODD>
__device__ __forceinline__ float stored_pop(float g, int i, const Nbrs<L> &nb, const PlaneRef &r)
{
    if (ODD != 1 || i == 0) return g;  // written into the node's own slot
    return nb.fl[i] ? g + L::w[i] * r.dOut[L::ex[i] + 1] : g;
}

// Populations are stored in blocks of 64 nodes, one wave: block k holds the
// Q directions of nodes 64k .. 64k + 63, direction by direction (64
// consecutive values each). A wave's access to one direction is one
// contiguous run of 256 bytes (FP32) as with whole planes, but the Q streams
// of a block lie in one region of Q x 256 bytes instead of Q planes far
// apart. Measured on the 512^3 electrode against whole planes of P values:
// FP32 fused step 3 % and flow-only step 6 % faster (blocks of 256 nodes:
// 0.5 % slower than 64). P is a multiple of the 256-node tile, so every block
// is whole.
constexpr int kPopBlockLog = 6;

// (the node's part, one 64-bit product, and the direction's constant part
// apart, so that a node's Q accesses share the first and fold the second
// into the instructions' offsets)
template <int Q, class T>
__device__ __forceinline__ const T *pop_at(const void *F, int q, int n)
{
    const uint32_t first = (uint32_t)n & ~((1u << kPopBlockLog) - 1);  // of the block
    const char *const node = reinterpret_cast<const char *>(F) + (uint64_t)(uint32_t)n * sizeof(T) +
                             (uint64_t)first * (uint32_t)((Q - 1) * sizeof(T));
    return reinterpret_cast<const T *>(node) + (q << kPopBlockLog);
}
template <int Q, class T>
__device__ __forceinline__ T *pop_at(void *F, int q, int n)
{
    return const_cast<T *>(pop_at<Q, T>(const_cast<const void *>(F), q, n));
}

// Value of direction a or b (one of the two per lane) at node m.
template <int FP16, int Q>
__device__ __forceinline__ float ld_pair(const void *F, int a, int b, int m, bool first)
{
    const int q = first ? a : b;
    if (FP16) return __half2float(*pop_at<Q, __half>(F, q, m));
    return *pop_at<Q, float>(F, q, m);
}

template <int FP16, int Q>
__device__ __forceinline__ void st_pair(void *F, int a, int b, int m, bool first, float v)
{
    const int q = first ? a : b;
    if (FP16)
        *pop_at<Q, __half>(F, q, m) = __float2half_rn(v);
    else
        *pop_at<Q, float>(F, q, m) = v;
}

// Stored value behind the incoming population i of node n (FP32 f - w_i or
// the scaled FP16 deviation; nothing with moment storage).
template <class L, int ST, int ODD>
__device__ inline float gather_raw(const void *F, int P, const Nbrs<L> &nb, int n, int i)
{
    if (kMoments<ST>) return 0.f;
    constexpr bool H = kHalfPop<ST>;
    const int j = L::opp[i];
    const bool fl = i != 0 && nb.fl[j];
    // pull: plane i of the emitter x - e_i, or the node's own reflected plane j
    if (ODD == kPull) return ld_pair<H, L::Q>(F, i, j, i == 0 ? n : nb.n[j], fl);
    // AA: plane i of the node itself, or (odd parity, fluid emitter) plane j of the emitter
    return ld_pair<H, L::Q>(F, i, j, !ODD || i == 0 ? n : nb.n[j], !ODD || i == 0 || !fl);
}

// FP16 and moment storage: the incoming population of direction i before its
// weight, (f_i - w_i) / w_i less the FP16 deviation, from the emitter's
// moments m: dr + rho (E (+-3 + 4.5 E) - 1.5 u.u), E = e_i . u. The emitter
// x - e_i sent it along e_i; a reflected one (fl false) was sent by x along
// e_opp(i) = -e_i, which only flips the sign of e.u (w_opp(i) = w_i). The
// linear (Stokes) equilibrium drops the squares by uniform factors, without a
// branch per direction (in which the compiler also split the moments' loads).
// kMomR: m.x is relative to the emitter's plane, the result to Rout of the
// node's.
template <class L, int ST>
__device__ __forceinline__ float emitter_g(int i, bool fl, float4 m, const Phys &p, const PlaneRef &pr)
{
    const float c2 = p.linear_eq ? 0.f : 4.5f, c1 = p.linear_eq ? 0.f : -1.5f;
    float dr = m.x, rho;
    if (ST == kMomR) {
        dr = m.x + (fl ? pr.dIn[L::ex[i] + 1] : pr.dIn[1]);
        rho = 1.f + pr.rout + dr;
    } else {
        rho = 1.f + m.x;
    }
    const float uu = fmaf(m.w, m.w, fmaf(m.z, m.z, m.y * m.y));
    if (i == 0) return fmaf(rho, c1 * uu, dr);
    const float E = lat_dot<L>(i, m.y, m.z, m.w);
    return fmaf(rho, fmaf(c1, uu, E * fmaf(c2, E, fl ? 3.f : -3.f)), dr);
}

// Zeroth and first moments accumulated from g, the rest direction and then
// each direction i (odd) with its opposite i + 1: their sum and difference are
// formed first, so that equal values cancel in the first moments exactly
// (accumulated one by one with fused multiply-adds they leave the rounding of w
// g: 40 % more velocity error after 100 steps); and from the FP16 deviations.
struct MomSums {
    float d = 0.f, jx = 0.f, jy = 0.f, jz = 0.f;
};
template <class L>
__device__ __forceinline__ void add_rest(MomSums &s, float g)
{
    s.d = fmaf(L::w[0], g, s.d);
}
template <class L>
__device__ __forceinline__ void add_pair(MomSums &s, int i, float g, float h)
{
    const float t = g - h;
    s.d = fmaf(L::w[i], g + h, s.d);
    if (L::ex[i]) s.jx = fmaf(L::w[i] * L::ex[i], t, s.jx);
    if (L::ey[i]) s.jy = fmaf(L::w[i] * L::ey[i], t, s.jy);
    if (L::ez[i]) s.jz = fmaf(L::w[i] * L::ez[i], t, s.jz);
}
template <class L>
__device__ __forceinline__ void add_plain(MomSums &s, int i, float v)
{
    s.d += v;
    s.jx = lat_add(s.jx, L::ex[i], v);
    s.jy = lat_add(s.jy, L::ey[i], v);
    s.jz = lat_add(s.jz, L::ez[i], v);
}

// f_i - w_i of an emitter with deviation dev (0 with moment storage).
template <class L, int ST>
__device__ __forceinline__ float from_emitter(float dev, int i, bool fl, float4 m, const Phys &p, const PlaneRef &pr)
{
    return fmaf(L::w[i], emitter_g<L, ST>(i, fl, m, p, pr), dev);
}

// Incoming f_i - w_i of node n (nb: n's neighbours; M: the
// emitters' moments, FP16 and moment storage; pr: kMomR).
template <class L, int ST, int ODD>
__device__ inline float gather(const void *F, int P, const Nbrs<L> &nb, int n, int i, const float4 *M,
                               const Phys &p, const PlaneRef &pr)
{
    const float raw = gather_raw<L, ST, ODD>(F, P, nb, n, i);
    if (ST == kF32) return raw;
    if (kPlain<ST>) return raw * p.hs_inv;
    const int j = L::opp[i];
    return from_emitter<L, ST>(raw * p.hs_inv, i, i != 0 && nb.fl[j], ldu(M, (uint32_t)(i == 0 ? n : nb.n[j])), p, pr);
}

// Store the outgoing value of direction i (FP32: f* - w_i; FP16: scaled
// deviation; moment storage: nothing). F: the array written.
template <class L, int ST, int ODD>
__device__ inline void scatter(void *F, int P, const Nbrs<L> &nb, int n, int i, float v)
{
    if (kMoments<ST>) return;
    constexpr bool H = kHalfPop<ST>;
    const int j = L::opp[i];
    if (ODD == kPull)
        st_pair<H, L::Q>(F, i, i, n, true, v);  // the node's own slot i
    else
        // even parity (or the rest direction): the node's own plane opp(i); odd
        // parity: plane i of the fluid neighbour x + e_i, else (reflected) plane opp(i)
        st_pair<H, L::Q>(F, j, i, !ODD || i == 0 ? n : nb.n[i], !ODD || i == 0 || !nb.fl[i], v);
}

// Non-equilibrium extrapolation (Guo, Zheng & Shi 2002) for the inlet
// (velocity u_in) or outlet (density rho_out) node next to the interior node
// whose post-streaming populations are fc: the boundary takes the target
// equilibrium plus the interior node's non-equilibrium part. fc is relative to
// the interior node's reference rc (fc_i = f_i - w_i (1 + rc)), fb is returned
// relative to the boundary node's rb (0 and 0 for f - w_i storage).
template <class L>
__device__ inline void nee_populations(const Phys &p, bool inlet, const float (&fc)[L::Q], float (&fb)[L::Q],
                                       float rc = 0.f, float rb = 0.f)
{
    float dr, jx, jy, jz;
    lat_moments<L>(fc, dr, jx, jy, jz);
    const float rho = 1.f + rc + dr;
    const float ri = __builtin_amdgcn_rcpf(rho);
    const float ux = jx * ri, uy = jy * ri, uz = jz * ri;
    // target: inlet (rho of the interior node, u_in), outlet (rho_out, u of the interior node)
    const float trho = inlet ? rho : p.rho_out;
    const float tx = inlet ? p.u_in : ux, ty = inlet ? 0.f : uy, tz = inlet ? 0.f : uz;
    const float tdr = inlet ? (rc + dr) - rb : (p.rho_out - 1.f) - rb;
    const EqTerms te = eq_terms(tdr, trho, tx, ty, tz, p.linear_eq), ce = eq_terms(dr, rho, ux, uy, uz, p.linear_eq);
#pragma unroll
    for (int i = 0; i < L::Q; ++i)
        fb[i] = feq_dir<L>(i, te, tx, ty, tz) + (fc[i] - feq_dir<L>(i, ce, ux, uy, uz));
}

// The moments of the populations nee_populations gives, from those of the
// interior node (c, relative to rc): the target equilibrium's.
__device__ __forceinline__ MomSums nee_moments(const Phys &p, bool inlet, const MomSums &c, float rc, float rb)
{
    const float rho = 1.f + rc + c.d, ri = __builtin_amdgcn_rcpf(rho);
    MomSums t;
    t.d = inlet ? (rc + c.d) - rb : (p.rho_out - 1.f) - rb;
    t.jx = inlet ? rho * p.u_in : p.rho_out * (c.jx * ri);
    t.jy = inlet ? 0.f : p.rho_out * (c.jy * ri);
    t.jz = inlet ? 0.f : p.rho_out * (c.jz * ri);
    return t;
}

// Concentrations are stored as an FP32 value and an FP16 remainder per
// species (times 2^24): value + remainder carry the explicit update's sum to
// about 2^-35 of C, so increments far below half an FP32 ulp accumulate in the
// remainder instead of being dropped. (Rounded to FP32 alone, the update
// stalls wherever a cell's change per step falls below half an ulp, which
// near a steady state left C up to 1e-3 off after 20000 steps.) A remainder
// too large for FP16 (|C| beyond 2^15) is dropped.
__device__ __forceinline__ float lo_decode(__half h) { return __half2float(h) * (1.f / 16777216.f); }
__device__ __forceinline__ __half lo_encode(float lo)
{
    const float t = lo * 16777216.f;
    return __float2half_rn(fabsf(t) < 65000.f ? t : 0.f);
}

// a + b = s + e exactly, s = fl(a + b) (Knuth's TwoSum).
__device__ __forceinline__ float two_sum(float a, float b, float &e)
{
    const float s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
    return s;
}

// Scharfetter-Gummel flux from P to N with normal drift w, Pe = w / D:
// D [B(-Pe) C_P - B(Pe) C_N], B(x) = x / (e^x - 1). With Bs(x) = B(x) + x/2 =
// (x/2) coth(x/2), an even function, this is exactly
//   D Bs(Pe) (C_P - C_N) + (w/2) (C_P + C_N):
// a symmetric diffusive part and a central advective part, with no sign
// cases. Seen from N the operands are C_P - C_N negated, the same C_P + C_N,
// the same Pe^2 and w/2 negated, so the two cells of a face form exactly
// opposite values. Bs needs only Pe^2: below |Pe| = 1/2 its series
// 1 + x^2/12 - x^4/720 + x^6/30240 (next term below 3e-8 there), above the
// closed form with the hardware exponential (e^|x| - 1 >= 0.64, no
// cancellation). hw = w / 2, invD2 = 2 / D.
__device__ inline float sg_flux(float D, float invD2, float hw, float cp, float cn)
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
    return fmaf(D * bs, cp - cn, hw * (cp + cn));
}

// The same flux through a face in a ramp or no potential, in the steps' own
// form: D Bs as a series in h^2 = (w / 2)^2 whose coefficients (c, per
// species) carry D, so that it takes four fused multiply-adds. For |Pe| <= 1
// (the next term of Bs is below 2.1e-8 there).
__device__ __forceinline__ float sg_series(float D, const float (&c)[4], float h, float cp, float cn)
{
    const float h2 = h * h;
    const float db = fmaf(h2, fmaf(h2, fmaf(h2, fmaf(h2, c[3], c[2]), c[1]), c[0]), D);
    return fmaf(db, cp - cn, h * (cp + cn));
}

// Sum of v over the wave in a fixed order, the same value in every lane:
// neighbouring pairs, then quads, then eights and rows of 16 by DPP lane
// permutations within each row of 16 lanes (VALU only, no LDS), then the four
// rows' sums, each read from the row's first lane, in row order. Every lane
// of the wave must be active.
template <int CTRL>
__device__ __forceinline__ float dpp_plus(float v)
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v = dpp_plus<0xB1>(v);   // quad_perm [1,0,3,2]: pairs
    v = dpp_plus<0x4E>(v);   // quad_perm [2,3,0,1]: quads
    v = dpp_plus<0x124>(v);  // row_ror:4: two quads
    v = dpp_plus<0x128>(v);  // row_ror:8: the row of 16
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
    return ((r0 + r1) + r2) + r3;
}

// Per-tile FP64 accumulation of the ions' six per-lane FP32 amounts (adsorbed,
// in, out per species): each wave sums its lanes (wave_sum) and leaves the sums
// in LDS; the wave that comes last adds them in wave order in FP64, lane k
// amount k, to the tile's accumulators. No barrier: the other waves end at
// once instead of waiting for the slowest (512^3 electrode, fused moment step:
// 1.57 ms; 1.62 with the accumulators read early by every wave). sm: kTileSums
// doubles, tile_sums_init before the first tile; a barrier between two tiles.
constexpr int kTileWaves = kTile / 64, kTileSums = kTileWaves * 6 + 1;

__device__ inline void tile_sums_init(double *sm)
{
    if (threadIdx.x == 0) *reinterpret_cast<int *>(sm + kTileWaves * 6) = 0;
    __syncthreads();
}

// at_end: this lane's node has an open x end (amounts 2 .. 5 are 0 elsewhere).
__device__ inline void tile_accumulate(const float (&v)[6], bool at_end, double *sm, double *acc)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool ads = __any(v[0] != 0.f || v[1] != 0.f), ends = __any(at_end);
    float w[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (ads) {
        w[0] = wave_sum(v[0]);
        w[1] = wave_sum(v[1]);
    }
    if (ends) {
#pragma unroll
        for (int k = 2; k < 6; ++k) w[k] = wave_sum(v[k]);
    }
    int *count = reinterpret_cast<int *>(sm + kTileWaves * 6);
    int before = 0;
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 6; ++k) sm[wave * 6 + k] = (double)w[k];
        before = __hip_atomic_fetch_add(count, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (__builtin_amdgcn_readfirstlane(before) != kTileWaves - 1) return;
    // the last wave
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (lane < 6) {
        double t = 0;
        for (int q = 0; q < kTileWaves; ++q) t += sm[q * 6 + lane];
        if (t != 0.0) acc[lane] += t;
    }
    if (lane == 0) *count = 0;
}

// Sum over the block in a fixed order (wave shuffles, then the waves in
// order); the result is valid in thread 0. sm holds (blockDim/64) * N doubles.
template <int N>
__device__ inline void block_sum(double (&v)[N], double *sm, double (&out)[N])
{
    // a wave whose lanes all hold 0 (most waves, for the inlet/outlet and
    // adsorption amounts) skips the shuffles: its sum is 0 either way
#pragma unroll
    for (int k = 0; k < N; ++k)
        if (__ballot(v[k] != 0.0))
            for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < N; ++k) sm[wave * N + k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = blockDim.x >> 6;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            double s = 0;
            for (int w = 0; w < nw; ++w) s += sm[w * N + k];
            out[k] = s;
        }
    }
}

}  // namespace cdi
