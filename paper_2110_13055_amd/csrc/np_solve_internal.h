// np_solve_internal.h -- argument block and launchers of the implicit ion
// transport (np_solve.hip): backward-Euler steps and the steady state of the
// Nernst-Planck equations, Eq. (3), on a frozen flow and potential.
#pragma once

#include "cdi_internal.h"

namespace cdi {

constexpr int kNpsMaxWorkgroups = 4096;
constexpr int kNpsWorkgroupsPerCU = 4;  // cap on resident solver workgroups per compute unit

// Solver state (doubles): per species s, active flag (1 while iterating),
// iterations done, |r|^2 of the last test, |rhs|^2, tol^2 |rhs|^2; then a
// global stop code.
enum {
    kNsActive = 0,  // + s
    kNsIters = 2,   // + s
    kNsRr = 4,      // + s
    kNsBb = 6,      // + s
    kNsThr = 8,     // + s
    kNsDone = 10,   // 0 running, 1 converged, 2 diverged / breakdown
    kNsScale = 11,  // + s: the power of two that brings |r_0| to 1 to 2
    kNsPe = 13,     // largest |Pe| of the flow across a face between fluid cells
    kNsRange = 14,  // largest range of the potential within a block, thermal voltages times |z|
    kNsSlots = 15
};

struct NpsArgs {
    Grid g;
    Phys p;
    const float2 *C;   // concentrations of the state the step starts from
    const float *j;    // frozen advecting mass flux (d planes of P)
    int G, Gd[2];      // workgroups (nps_workgroups, nps_dir_workgroups)
    int plain;         // the preconditioner's sweeps (nps_plain), set after the set-up
    double idt;        // 1 / dt of a backward-Euler step, 0 for the steady state
    // FP64 vectors of P, both species of a node side by side (r holds s between
    // the halves of an iteration), and the preconditioned directions
    double2 *x, *r, *rh, *pv, *v, *t;
    float2 *ph, *sh;
    float2 *di;        // reciprocal diagonals of (I/dt + A)
    double *part;      // per-workgroup partial sums (nps_part_doubles)
    double *state;     // kNsSlots doubles
    double *acc;       // the solver's per-tile accumulators (rates pass)
};

uint64_t nps_part_doubles();
// Workgroups of the kernels that leave partial sums, and of the two direction kernels.
hipError_t nps_workgroups(int dim, int ntiles, int *G);
hipError_t nps_dir_workgroups(int dim, int ntiles, int plain, int *Gd);
// Whether a system with these kNsPe and kNsRange takes plain sweeps (np_solve.hip).
int nps_plain(double pe, double range);
// x = C, r = rhat = C idt + b - A x, reciprocal diagonals, |rhs|^2, rho_0, the drift's
// measures and the state.
hipError_t launch_nps_setup(int dim, const NpsArgs &a, double tol, hipStream_t s);
// BiCGSTAB iteration k (direction, A p, s, A s, update); returns at once after the stop.
hipError_t launch_nps_iter(int dim, const NpsArgs &a, int k, hipStream_t s);
// The stop test before iteration k (one workgroup).
hipError_t launch_nps_check(const NpsArgs &a, int k, hipStream_t s);
// C_out = (float) x for the fluid nodes.
hipError_t launch_nps_store(const NpsArgs &a, float2 *Cout, __half2 *Clo, hipStream_t s);
// Rates of adsorption, inflow and outflow of the concentrations C (FP64 per
// tile), times scale, added to acc (scale = dt of an implicit step) or
// written to part and reduced into out[0..5] (out != nullptr).
hipError_t launch_nps_rates(int dim, const Grid &g, const Phys &p, const float2 *C, const float *j, double scale,
                            double *acc, double *part, double *out, hipStream_t s);

}  // namespace cdi
