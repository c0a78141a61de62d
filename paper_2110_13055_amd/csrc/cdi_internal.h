// cdi_internal.h -- lattice tables, kernel argument blocks and launcher
// declarations shared by the HIP translation units of libcdi.
//
// Data layout in device memory (N_f fluid nodes, stride P = N_f rounded up to
// a whole number of 256-node tiles):
//   populations  Q x P values in blocks of 64 nodes (block k: the Q
//                directions of nodes 64k .. 64k + 63, 64 values each), FP32
//                f - w_i(1 + R[x]) or FP16 scaled values; none with moment
//                storage
//   moments      FP16 and moment storage: float4 (rho - 1, ux, uy, uz) per
//                node, double buffered (the moments of the previous step
//                belong to the emitters of the populations now stored)
//   jbuf         advecting mass flux j = rho u for the ions, d planes of P,
//                double buffered (fused steps read one and write the other)
//   conc         both species of a node as a float2, double buffered (Jacobi
//                update)
//   acc          per tile 8 doubles: A_na, A_cl, In_na, In_cl, Out_na, Out_cl
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>

namespace cdi {

constexpr int kTile = 256;  // fluid nodes per tile (= threads per block)

// D2Q9; directions 1..4 are the faces +x, -x, +y, -y.
struct D2Q9 {
    static constexpr int D = 2, Q = 9;
    static constexpr int ex[9] = {0, 1, -1, 0, 0, 1, -1, 1, -1};
    static constexpr int ey[9] = {0, 0, 0, 1, -1, 1, -1, -1, 1};
    static constexpr int ez[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    static constexpr int opp[9] = {0, 2, 1, 4, 3, 6, 5, 8, 7};
    static constexpr float w[9] = {4.f / 9, 1.f / 9, 1.f / 9, 1.f / 9, 1.f / 9,
                                   1.f / 36, 1.f / 36, 1.f / 36, 1.f / 36};
};

// D3Q19; directions 1..6 are the faces +x, -x, +y, -y, +z, -z.
struct D3Q19 {
    static constexpr int D = 3, Q = 19;
    static constexpr int ex[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
    static constexpr int ey[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
    static constexpr int ez[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
    static constexpr int opp[19] = {0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17};
    static constexpr float w[19] = {1.f / 3,  1.f / 18, 1.f / 18, 1.f / 18, 1.f / 18, 1.f / 18, 1.f / 18,
                                    1.f / 36, 1.f / 36, 1.f / 36, 1.f / 36, 1.f / 36, 1.f / 36,
                                    1.f / 36, 1.f / 36, 1.f / 36, 1.f / 36, 1.f / 36, 1.f / 36};
};

// map values of non-fluid voxels
constexpr int kElectrode = -1;
constexpr int kInert = -2;
constexpr int kOutside = -3;  // beyond an open x end

// Nernst-Planck x-end treatments (same numbering as the public enum)
constexpr int kNpxInletOutlet = 0, kNpxPeriodic = 1, kNpxClosed = 2, kNpxDirichlet = 3;

// step flags
constexpr int kStoreU = 1;    // write u of the incoming state to ubuf
constexpr int kResid = 2;     // accumulate |u - ubuf|^2 and |u|^2 per tile
constexpr int kJFromM = 4;    // FP16/moment fused: ions read j from the moments buffer
constexpr int kNee = 8;       // the stored state carries inlet/outlet extrapolation
                              // (every state after the first step)

// Internal node order: fluid nodes are numbered brick by brick (bricks of
// 2^bsx x 2^bsy x 2^bsz voxels, bricks in x-fastest order, voxels inside a
// brick x-fastest), so that a workgroup's nodes and most of their lattice
// neighbours share a small block of memory. The public numbering (fields
// handed to the caller, the fluid index map) stays lexicographic.
struct Bricks {
    int bsx, bsy, bsz;  // log2 of the brick edge lengths
    int nbx, nby, nbz;  // bricks along each axis (padded)
    int cbx, cby;       // bits of x and y in a packed node coordinate
};

// Packed node coordinates: x | y << cbx | z << (cbx + cby), 32 bits.
__host__ __device__ inline uint32_t pack_xyz(const Bricks &k, int x, int y, int z)
{
    return (uint32_t)x | ((uint32_t)y << k.cbx) | ((uint32_t)z << (k.cbx + k.cby));
}

__host__ __device__ inline int64_t brick_index(const Bricks &k, int x, int y, int z)
{
    const int64_t b = ((int64_t)(z >> k.bsz) * k.nby + (y >> k.bsy)) * k.nbx + (x >> k.bsx);
    const int l = ((((z & ((1 << k.bsz) - 1)) << k.bsy) | (y & ((1 << k.bsy) - 1))) << k.bsx) |
                  (x & ((1 << k.bsx) - 1));
    return (b << (k.bsx + k.bsy + k.bsz)) | l;
}

struct Grid {
    int nx, ny, nz;
    int n_f;         // fluid nodes
    int P;           // plane stride (multiple of kTile)
    int periodic_x;  // LBM periodic in x (body-force drive)
    int inout;       // inlet/outlet planes at x = 0 and x = nx - 1
    Bricks bk;
    const uint32_t *fluid;  // internal node -> packed (x, y, z)
    const int *map;         // brick-ordered voxel -> internal node, or kElectrode / kInert
    // Tile schedule: XCD-local position -> tile. Tiles are ordered by
    // (band of rows, z) so the planes above and below a tile were visited
    // shortly before by the same XCD and are still in its L2.
    const int *sched;
    // Optional neighbour list: map value of the face neighbour of node n along
    // direction i in nbr[(i - 1) * P + n] (i = 1 .. 2 d), so that an ion-only
    // step reads it with the node's other data instead of after its coordinates.
    const int *nbr;
    // The lattice's rows (below): what the steps that do not read the list
    // look their neighbours up in.
    const int4 *rows;
    // dynamic LDS reserved per step workgroup: caps the workgroups resident
    // per CU (and so the working set the L2 must hold); 0 = no cap
    int lds_pad;
    // odd AA steps of the storages that allow it stage the tile's population
    // slots in LDS (set by the host from the tuning and the tile count)
    int stage_odd;
};

// A row: the 2^bsx voxels along x at one (y, z) of a brick, in the order of
// the brick enumeration, as one int4:
//   x  node index of the row's first fluid voxel (its fluid voxels are
//      consecutive nodes)
//   y  fluid bits: bit 0 the voxel before the row, bit 1 + i voxel i, then the
//      voxel after the row's last one; bit 31: the row holds an inert solid
//   z  map value of the voxel before the row (wrapped, or kOutside beyond an
//      open x end)
//   w  map value of the voxel after it
// A node's three neighbours in one row are its rank among the row's bits and
// the nodes beside it, so a step loads 9 rows (D3Q19) instead of 18 map
// entries, and 1 B per voxel instead of 4.
static_assert(sizeof(int4) == 16, "a row is 16 bytes");

struct Phys {
    float omega;       // 1 / tau
    float fcoef;       // 1 - 1/(2 tau), Guo source prefactor
    float F[3];        // body-force density
    int forced;
    int linear_eq;
    // Nernst-Planck
    float D[2], invD[2], z[2], keff[2];
    float c0, c_out, u_in;
    float rho_out;     // outlet density of the flow
    float dpsi_dx;     // ramp drop per cell (dpsi / nx)
    // Scharfetter-Gummel series in the half drift h (see sg_series): D Bs =
    // D + c1 h^2 + .. + c4 h^8 per species, valid while h^2 <= h2_max (|Pe| <= 1
    // for both species); hr: the ramp's half drift across an x face; steep: the
    // ramp alone comes near that bound; far: the flow takes faces beyond it (as of
    // the last positivity check; chooses between kernels of the same results)
    float sgc[2][4], h2_max, hr[2];
    int steep, far;
    int npx;
    float dt;
    const float *psi;  // optional field (fluid order), else ramp
    // FP16 deviation scale
    float hs, hs_inv;
};

// Buffers of one step; multi-plane fields are P apart (structure of arrays).
struct Bufs {
    void *f;        // populations: the array read (and, AA streaming, written)
    void *f2;       // pull streaming: the array written
    const float4 *Min;
    float4 *Mout;
    const float *jin;
    float *jout;
    const float2 *Cin;  // both species of a node together: a neighbour's pair is one load
    float2 *Cout;
    const __half2 *Clin;  // the concentrations' FP16 remainders (see lo_encode), per node
    __half2 *Clout;
    double *acc;
    double *resid;
    float *ubuf;    // FP32 storage: u (d planes) and rho - 1 (plane d) of the state, on kStoreU
    // FP32 storage: reference density deviation per x plane of the values read
    // and of the values written (see PlaneRef); nullptr: zero
    const float *rin;
    const float *rout;
    int flags;
};

// Storage of the lattice state (values of cdi_params.precision): FP32
// populations and FP16 populations (both relative to the plane references,
// the FP16 ones scaled; the ions' flux in its own buffer), FP16 deviations
// from the emitter's equilibrium with FP32 moment buffers, moments only.
// kMomR: moments only, with rho - 1 relative to the plane references (see
// PlaneRef): the kernels of an FP32 instance held as moments once its
// references have been renewed. kH16L: FP16 populations of an instance beyond
// 2^29 nodes, whose ion kernels form the concentrations' addresses in 64 bits.
constexpr int kF32 = 0, kF16 = 1, kMom = 2, kH16 = 3, kMomR = 4, kH16L = 5, kForms = 6;
// The widest element that a form's kernels address by node with a 32-bit byte
// offset (ldu, stu): a moment, the concentrations' pair, or one FP32 value.
constexpr int offset_elem(int form)
{
    return form == kF16 || form == kMom || form == kMomR ? 16 : form == kH16L ? 4 : 8;
}
// Whether that offset fits for an instance of P nodes.
constexpr bool offsets_fit(int form, int64_t P) { return P * offset_elem(form) <= 4294967295LL; }
template <int ST>
constexpr bool kMoments = ST == kMom || ST == kMomR;  // no populations stored
template <int ST>
constexpr bool kRefs = ST == kF32 || ST == kH16 || ST == kH16L || ST == kMomR;  // relative to the plane references
template <int ST>
constexpr bool kPlain = ST == kF32 || ST == kH16 || ST == kH16L;  // populations relative to the plane references
template <int ST>
constexpr bool kHalfPop = ST == kF16 || ST == kH16 || ST == kH16L;  // populations stored in FP16

// One instance of a batched launch.
constexpr int kModeIdle = 0, kModeFlow = 1, kModeIons = 2, kModeFused = 3;
struct BatchInst {
    Grid g;
    Phys p;
    Bufs b;
};
// Step classes of a batched step (kernel variants): per storage form, LBM
// only or fused by parity (class kClassesPerForm * form + ...; the moment
// forms have no parity and use the even ones), and ions only (kClassIonsL: of
// kH16L members). While no member is in a potential field, a steep ramp or a flow
// beyond the flux series' range, the ion-carrying classes take kernels without the
// code of those fluxes, which costs registers; else the ones kClassAny further on.
constexpr int kClassFlowEven = 0, kClassFlowOdd = 1, kClassFlowPull = 2, kClassFusedEven = 3, kClassFusedOdd = 4,
              kClassFusedPull = 5, kClassAny = 3, kClassesPerForm = 9, kClassIons = kForms * kClassesPerForm,
              kClassIonsAny = kClassIons + 1, kClassIonsL = kClassIons + 2, kClasses = kClassIons + 3;

// Value of the kernels' parity argument for pull streaming (AA uses 0 / 1).
constexpr int kPull = 2;

// ------------------------------------------------------------ launchers
// Every launcher enqueues on `stream` and returns hipGetLastError().
hipError_t launch_init_labels(uint8_t *labels, int nx, int ny, int nz, int walls2d, hipStream_t s);
hipError_t launch_voxelize(uint8_t *labels, const int64_t *prims, int64_t nprims, int dim, int nx,
                           int ny, int nz, int walls_y, int buffer_x, hipStream_t s);
hipError_t launch_compact(const uint8_t *labels, int64_t nvox, int *map, int *fluid, int *blk,
                          int64_t *nfluid, hipStream_t s);
int64_t compact_blocks(int64_t nvox);
// Internal (brick-ordered) numbering of the fluid voxels: imap over the
// brick enumeration, ifluid[node] = lexicographic voxel, and lex2int[k] =
// internal node of lexicographic fluid node k (needs the lexicographic map).
hipError_t launch_compact_bricks(const uint8_t *labels, const int *lexmap, int nx, int ny, int nz,
                                 const Bricks &bk, int *imap, uint32_t *ifluid, int *lex2int, int *blk,
                                 int64_t *nfluid, hipStream_t s);
int64_t brick_enum_size(const Bricks &bk);
// Reorder d planes between the internal (stride P) and lexicographic (stride
// n_f) node orders. to_lex: dst[c*n_f + k] = src[c*P + lex2int[k]]; else the
// inverse scatter.
hipError_t launch_permute(const float *src, float *dst, const int *lex2int, int n_f, int P, int d,
                          int to_lex, hipStream_t s);
// The same between two planes in lexicographic order and a float2 per node.
hipError_t launch_permute_pairs(float *lex, float2 *pairs, const int *lex2int, int n_f, int to_lex, hipStream_t s);

// Streaming kernels of known traffic over bytes (a multiple of 16): copy,
// XOR checksum of every 8 KiB block of src into dst (16 bytes per block),
// fill with a 32-bit value.
constexpr int kStreamCopy = 0, kStreamRead = 1, kStreamFill = 2;
constexpr uint64_t kStreamReadBlock = 8192;
hipError_t launch_stream(int mode, void *dst, const void *src, uint64_t bytes, uint32_t value, hipStream_t s);

hipError_t launch_fill_f32(float *p, float v, int64_t n, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s);
hipError_t launch_fill_f64(double *p, double v, int64_t n, hipStream_t s);

// One LBM and/or Nernst-Planck step over all fluid nodes.
//   dim 2/3, st = storage form (kF32 ...), odd = AA parity of the stored state
//   or kPull, lbm/np switches.
hipError_t launch_step(int dim, int st, int odd, int lbm, int np, const Grid &g, const Phys &p,
                       const Bufs &b, hipStream_t s);
// One step of the instances of one step class in one persistent launch of
// `workgroups` workgroups over the class's (instance, tile) list (inst and
// tiles in device memory).
hipError_t launch_batch(int dim, int cls, const BatchInst *inst, const int2 *tiles, int ntiles,
                        int workgroups, int lds_pad, hipStream_t s);
// Moments of the stored state: rho (nullable), u (nullable, d planes),
// j (nullable, d planes); rref: the FP32 plane references of the state
// (nullptr: zero).
hipError_t launch_moments(int dim, int st, int odd, int nee, const Grid &g, const Phys &p,
                          const void *f, const float4 *M, const float *rref, float *rho, float *u, float *j,
                          hipStream_t s);
// Plane references: rref[x] = base[x] + mean of drho (rho - 1 - base of the
// fluid nodes in node order, value n at drho[n * stride]; base nullptr: zero)
// over the fluid voxels of plane x, 0 where the plane holds none; FP64 sums
// in a fixed order (one workgroup per plane).
hipError_t launch_plane_means(const Grid &g, const float *drho, int stride, const float *base, float *rref,
                              hipStream_t s);
// Packed coordinates of the first node of every tile (host-side tile schedule).
hipError_t launch_tile_heads(const Grid &g, uint32_t *heads, hipStream_t s);
// The rows of the lattice (Grid::rows), brick_enum_size / 2^bsx of them.
int64_t row_count(const Bricks &bk);
hipError_t launch_build_rows(const Grid &g, int4 *rows, hipStream_t s);
// Both species from two planes of P to a float2 per node.
hipError_t launch_pair_planes(const float *src, float2 *dst, int P, hipStream_t s);
// Neighbour list of every fluid node (see Grid::nbr), 2 d planes of P.
hipError_t launch_build_nbr(int dim, const Grid &g, int *nbr, hipStream_t s);
// j = rho u from the moments buffer (FP16 and moment storage; rref: the
// plane references its densities are relative to, nullptr: zero).
hipError_t launch_j_from_m(int dim, const Grid &g, const float4 *M, const float *rref, float *j, hipStream_t s);
// The FP32 populations of a state held as moments (M, relative to the plane
// references rref, nullptr: zero), in the nodes' own slots: those of an AA state
// of parity 1, or (pull) of a pull-streaming one. F and M do not overlap.
hipError_t launch_pops_from_m(int dim, const Grid &g, int pull, int linear_eq, const float4 *M, const float *rref,
                              float *F, hipStream_t s);
// Deterministic single-block sums: out[k] = sum_t in[t*stride + k], k < width.
hipError_t launch_reduce_tiles(const double *in, int ntiles, int stride, int width, double *out,
                               hipStream_t s);
// FP64 sum of each concentration field with its remainders (solute mass): out[0..1].
hipError_t launch_mass(const Grid &g, const float2 *C, const __half2 *Clo, double *part, double *out, hipStream_t s);
// max over nodes/species of dt * (sum of outflow coefficients), out[0]; the
// share of the tiles with a face beyond the flux series' range, out[1] (0 in a
// potential field and in a steep ramp).
hipError_t launch_stability(int dim, const Grid &g, const Phys &p, const float *j, double *part,
                            double *out, hipStream_t s);

}  // namespace cdi
