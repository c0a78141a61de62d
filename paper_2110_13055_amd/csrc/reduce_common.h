// reduce_common.h -- the persistent-workgroup machinery of the Krylov
// solvers (pot.hip, np_solve.hip): XCD-contiguous tile ranges, fixed-order
// workgroup sums and the totals of per-workgroup partial sums.
#pragma once

#include "cdi_internal.h"
#include "device_common.h"

namespace cdi {

// Contiguous tile range of this workgroup at its XCD-contiguous position:
// an XCD sweeps one contiguous eighth of the lattice.
__device__ inline void tile_range(int ntiles, int &t0, int &t1)
{
    const long long G = gridDim.x;
    const long long c = xcd_tile(blockIdx.x, gridDim.x);
    t0 = (int)(c * ntiles / G);
    t1 = (int)((c + 1) * ntiles / G);
}

// Sum of v over the workgroup in a fixed order, returned to every thread.
__device__ inline double wg_sum(double v, double *sm)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();  // sm may still be read from a previous call
    if (lane == 0) sm[wave] = v;
    __syncthreads();
    double s = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += sm[w];
    return s;
}

// Largest v over the workgroup, returned to every thread.
__device__ inline double wg_max(double v, double *sm)
{
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();  // sm may still be read from a previous call
    if (lane == 0) sm[wave] = v;
    __syncthreads();
    double s = sm[0];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) s = fmax(s, sm[w]);
    return s;
}

// Whether the solve has stopped (state[slot] != 0), read once per workgroup
// so that all its waves take the same branch.
__device__ inline bool stopped_at(const double *state, int slot, int *flag)
{
    if (threadIdx.x == 0) *flag = state[slot] != 0.0;
    __syncthreads();
    return *flag != 0;
}

// Totals of N partial-sum regions (G values each), the same in every workgroup:
// all loads first, then one pass through LDS. sm: N * waves.
template <int N>
__device__ inline void region_sums(const double *const (&part)[N], int G, double *sm, double (&out)[N])
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = 0;
    for (int k = threadIdx.x; k < G; k += blockDim.x)
#pragma unroll
        for (int i = 0; i < N; ++i) out[i] += part[i][k];
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) out[i] += __shfl_xor(out[i], off, 64);
    __syncthreads();  // sm may still be read from a previous call
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < N; ++i) sm[i * waves + wave] = out[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        out[i] = 0;
        for (int w = 0; w < waves; ++w) out[i] += sm[i * waves + w];
    }
}

// Total of a partial-sum region (G values), the same in every workgroup.
__device__ inline double region_sum(const double *part, int G, double *sm)
{
    double v = 0;
    for (int k = threadIdx.x; k < G; k += blockDim.x) v += part[k];
    return wg_sum(v, sm);
}

// Chebyshev sweeps of the solvers' block preconditioners: kChebSteps steps on
// [kChebLow, 2] over blocks of kBlockNodes consecutive nodes. The spectrum of the
// diagonally scaled matrix is real and ends at 2 for the potential and for ions
// without drift; with drift np_solve.hip says how far they may be taken. Whole solves (steady ions at 192^3,
// Laplace at 256^3, a coupled 96x80x88 run): six steps on [0.1, 2] 50.2, 9.4 and
// 11.9 ms; four on [0.2, 2] 64.6, 10.6 and 12.3; eight on [0.06, 2] 48.9, 9.2 and 12.2.
constexpr int kBlockTiles = 4, kBlockNodes = kBlockTiles * kTile;
constexpr int kChebSteps = 6;
constexpr double kChebLow = 0.1;

struct ChebCoef {
    float first, d[kChebSteps], r[kChebSteps];
};
constexpr ChebCoef cheb_coef()
{
    ChebCoef c{};
    const double th = (2.0 + kChebLow) / 2, de = (2.0 - kChebLow) / 2, s = th / de;
    double rho = 1 / s;
    c.first = (float)(1 / th);
    for (int k = 1; k < kChebSteps; ++k) {
        const double rn = 1 / (2 * s - rho);
        c.d[k] = (float)(rn * rho);
        c.r[k] = (float)(2 * rn / de);
        rho = rn;
    }
    return c;
}

}  // namespace cdi
