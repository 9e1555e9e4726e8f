// diag_dev.h -- sums of the diagnostics, shared by the FP64 and the FP32 particle stores.
//
// Every sum is taken by at most SUM_ROWS workgroups over contiguous ranges of the particles (or of the
// grid), whose partials one workgroup adds in a fixed order: a diagnostic of a given particle order is
// reproducible bit for bit.
#pragma once
#include <algorithm>

#include "pic_internal.h"

namespace pic {

constexpr int DT = 256;          // threads of the diagnostics' kernels
constexpr int SUM_ROWS = 1024;   // four workgroups per compute unit; more rows only lengthen the reduction
constexpr int SUM_RESULTS = 64;  // doubles at the start of the reduction buffer: the results, before the partials

inline int sum_rows(int64_t n) { return (int)std::min<int64_t>(std::max<int64_t>(nblocks(n, DT), 1), SUM_ROWS); }

// sums of a workgroup's NV values to out[0 .. NV): across each wave in registers, then its waves
template <int NV> __device__ inline void block_sums(double v[NV], double *out) {
    __shared__ double s[DT / 64][NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double t = v[k];
        for (int h = 32; h > 0; h >>= 1) t += __shfl_down(t, h);
        if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6][k] = t;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double t = s[0][threadIdx.x];
        for (int w = 1; w < DT / 64; ++w) t += s[w][threadIdx.x];
        out[threadIdx.x] = t;
    }
}

// the workgroup's contiguous range of n
__device__ inline void row_range(int64_t n, int64_t &a, int64_t &b) {
    a = n * blockIdx.x / gridDim.x;
    b = n * (blockIdx.x + 1) / gridDim.x;
}

// pass 1: count, w, w x, w y, w z, w ux, w uy, w uz, w cos kz, w sin kz, w cos 2kz, w sin 2kz, w (gamma - 1)
__device__ inline void moment1_add(double v[13], double w, double x, double y, double z, double ux, double uy,
                                   double uz, double kb) {
    double s1, c1, s2, c2;
    sincos(kb * z, &s1, &c1);
    sincos(2.0 * kb * z, &s2, &c2);
    v[0] += 1.0;
    v[1] += w;
    v[2] += w * x;
    v[3] += w * y;
    v[4] += w * z;
    v[5] += w * ux;
    v[6] += w * uy;
    v[7] += w * uz;
    v[8] += w * c1;
    v[9] += w * s1;
    v[10] += w * c2;
    v[11] += w * s2;
    v[12] += w * (sqrt(1.0 + ux * ux + uy * uy + uz * uz) - 1.0);
}

// pass 2: central second moments about the means m1[2 + k] / m1[1] of pass 1
struct Means {
    double m[6];
    __device__ Means() {}
    __device__ Means(const double *m1) {
        for (int k = 0; k < 6; ++k) m[k] = m1[2 + k] / m1[1];
    }
};
__device__ inline void moment2_add(double v[8], const Means &M, double w, double x, double y, double z, double ux,
                                   double uy, double uz) {
    const double dx = x - M.m[0], dy = y - M.m[1], dz = z - M.m[2];
    const double a = ux - M.m[3], b = uy - M.m[4], c = uz - M.m[5];
    v[0] += w * dx * dx;
    v[1] += w * dy * dy;
    v[2] += w * dz * dz;
    v[3] += w * a * a;
    v[4] += w * b * b;
    v[5] += w * c * c;
    v[6] += w * dx * a;
    v[7] += w * dy * b;
}

// count and kinetic energy m w (gamma - 1) of a plasma particle (mobile ions: w < 0, mass mi)
__device__ inline void kinetic_add(double v[2], double w, double ux, double uy, double uz, double mi) {
    v[0] += 1.0;
    v[1] += (w < 0.0 ? -mi * w : w) * (sqrt(1.0 + ux * ux + uy * uy + uz * uz) - 1.0);
}

// The wave's sums of 16 values, value l / 4 in lane l: a lane gives the half of its values that it does
// not keep to the lane that keeps them, so that 17 exchanges do for the 96 of 16 sums by themselves.
__device__ inline double wave_sums16(double v[16]) {
    const int lane = __lane_id();
#pragma unroll
    for (int d = 32, n = 8; d >= 4; d >>= 1, n >>= 1) {
        const bool up = lane & d;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const double keep = up ? v[k + n] : v[k], give = up ? v[k] : v[k + n];
            v[k] = keep + __shfl_xor(give, d);
        }
    }
    v[0] += __shfl_xor(v[0], 2);
    return v[0] + __shfl_xor(v[0], 1);
}

// the 16 values of a particle in its lab group
__device__ inline void lab_group_values(const Params &P, double t, double x, double y, double z, double ux, double uy,
                                        double uz, double w, double v[LAB_GROUP_VALUES]) {
    double L[8];
    lab_of(P, t, x, y, z, ux, uy, uz, L);
    v[0] = 1.0;
    v[1] = w;
    v[2] = w * L[3];
    v[3] = v[4] = L[3];
    v[5] = w * L[2];
    v[6] = w * L[2] * L[2];
    v[7] = w * L[0];
    v[8] = w * L[0] * L[0];
    v[9] = w * L[1];
    v[10] = w * L[1] * L[1];
    v[11] = w * L[4];
    v[12] = w * L[4] * L[4];
    v[13] = w * L[5];
    v[14] = w * L[5] * L[5];
    v[15] = w * L[7];
}

// added to group g of a block's LDS table (lab_table_*) by one lane
__device__ inline void lab_group_lane(double *tab, int g, const double v[LAB_GROUP_VALUES]) {
    double *e = tab + LAB_GROUP_VALUES * g;
#pragma unroll
    for (int k = 0; k < LAB_GROUP_VALUES; ++k) {
        if (k == 3)
            atomicMin(&e[k], v[k]);
        else if (k == 4)
            atomicMax(&e[k], v[k]);
        else
            atomicAdd(&e[k], v[k]);
    }
}

// a particle into the table, by its lane
__device__ inline void lab_group_add(double *tab, const LabGroupSpec &G, const Params &P, double t, double x, double y,
                                     double z, double ux, double uy, double uz, double w) {
    const int g = lab_group_of(G, z, uz);
    if (g < 0) return;
    double v[LAB_GROUP_VALUES];
    lab_group_values(P, t, x, y, z, ux, uy, uz, w, v);
    lab_group_lane(tab, g, v);
}

// The same called by every lane of a wave, `in` where it has a particle.  Neighbouring particles share
// groups, and 64 lanes adding to one entry add one
// after the other; a group of eight lanes or more is summed across the wave and added once.  The
// beam of 4.2 M particles in 64 slices: 8.0 ms lane by lane, 0.34 ms with a sum of each value by
// itself, 0.16 ms with wave_sums16.
__device__ inline void lab_group_add_wave(double *tab, const LabGroupSpec &G, const Params &P, double t, bool in,
                                          double x, double y, double z, double ux, double uy, double uz, double w) {
    const int g = in ? lab_group_of(G, z, uz) : -1;
    bool mine = g >= 0;
    double v[LAB_GROUP_VALUES];
    lab_group_values(P, t, x, y, z, ux, uy, uz, w, v);
    unsigned long long todo = __ballot(mine);
    while (todo) {
        const int lead = __ffsll(todo) - 1, lg = __builtin_amdgcn_readlane(g, lead);
        const bool here = mine && g == lg;
        const unsigned long long gm = __ballot(here);
        todo &= ~gm;
        if (__popcll(gm) < 8) continue;  // left to the lanes themselves
        double *e = tab + LAB_GROUP_VALUES * lg, r[LAB_GROUP_VALUES];
#pragma unroll
        for (int k = 0; k < LAB_GROUP_VALUES; ++k) r[k] = here && k != 3 && k != 4 ? v[k] : 0.0;
        const double sum = wave_sums16(r);
        // the least t in the lower half of the wave, the least -t in the upper one
        const int lane = __lane_id(), k = lane >> 2;
        const double tt = here ? v[3] : INFINITY, nt = here ? -v[3] : INFINITY;
        double m = fmin(lane < 32 ? tt : nt, __shfl_xor(lane < 32 ? nt : tt, 32));
        for (int h = 16; h > 0; h >>= 1) m = fmin(m, __shfl_xor(m, h));
        if ((lane & 3) == 0 && k != 3 && k != 4) atomicAdd(&e[k], sum);
        if (lane == 0) atomicMin(&e[3], m);
        if (lane == 32) atomicMax(&e[4], -m);
        if (here) mine = false;
    }
    if (mine) lab_group_lane(tab, g, v);
}

void lab_groups_clear(double *out, int ng, hipStream_t st);  // k_diag.hip

// k_split32.hip: partials of the FP32 store's sums into part, one row per workgroup; return the rows
int split_moments1(Ctx &c, double kb, double *part);
int split_moments2(Ctx &c, const double *m1, double *part);  // after split_moments1 on the same state
int split_plasma_kinetic(Ctx &c, double *part);
void split_rho(Ctx &c, double *rho, int mask);

}  // namespace pic
