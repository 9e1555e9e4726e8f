// k_adjoint.hip -- exact discrete adjoint of one FP64 step, for gradients of
// the final bunching factor with respect to the undulator K and the plasma
// density.  The step is reversed one sub-operation at a time:
//   window shift -> E update with Mur faces -> second B half step ->
//   deposit (ion current) -> move -> push -> gather (+ external field) ->
//   first B half step.
// Discrete events (window shift, removal, injection) are those the forward
// step takes from state n; the forward state is recomputed, never stored.
// The external field is linear in K and every plasma weight is linear in n0,
// so K dL/dK = sum <lam_field_at_particle, external field> and
// n0 dL/dn0 = sum <lam_J, J_plasma + J_ions>.
// Adjoint fields are kept in the ring order of the forward fields.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "tiles64.h"

namespace pic {

constexpr int AT = 256;
constexpr int PT = 512;  // threads of the particle kernel

// A sum with its rounding error carried along (Knuth's two-sum).  The gradients are small
// differences of large sums -- the plasma electrons' current against the ions', a bunching wave's
// adjoint over a uniform lattice -- whose plain FP64 sums left 1e-6 of the density gradient to the
// order of their terms on the 64x64x256 workload.
struct Sum2 {
    double hi, lo;
    __host__ __device__ void add(double v, double e = 0.0) {
        const double s = hi + v, b = s - hi;
        lo += ((hi - (s - b)) + (v - b)) + e;
        hi = s;
    }
    __host__ __device__ double value() const { return hi + lo; }
};

// the workgroup's sum, in thread 0; red: one entry per wave
template <int NT> __device__ inline Sum2 block_sum2(Sum2 v, Sum2 *red) {
    for (int k = 32; k > 0; k >>= 1) {
        const double h = __shfl_down(v.hi, k), l = __shfl_down(v.lo, k);
        v.add(h, l);
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < NT / 64; ++w) v.add(red[w].hi, red[w].lo);
    __syncthreads();
    return v;
}

struct Lam {  // views into the caller's adjoint vector
    double *x[3], *u[3];
};

static Lam lam_view(double *lam, int64_t off, int64_t cap) {
    Lam L;
    uint64_t c = (uint64_t)std::max<int64_t>(cap, 1);
    for (int d = 0; d < 3; ++d) {
        L.x[d] = lam + off + d * c;
        L.u[d] = lam + off + (3 + d) * c;
    }
    return L;
}

// ---------------------------------------------------------------- fields
__device__ inline int plane_of(const Params &P, int64_t o, int k0r, int &i, int &j, int &p) {
    i = (int)(o % P.nx);
    int64_t r = o / P.nx;
    j = (int)(r % P.ny);
    p = (int)(r / P.ny);
    int l = p - k0r;
    return l < 0 ? l + P.nz : l;
}

// adjoint of the E^{n+1} values produced by the interior update (Mur terms folded in)
__device__ inline double lam_eff(const Params &P, const double *lE, int c, int i, int j, int l, int k0r, int shift,
                                 int fm, double cm) {
    if (l < 0 || l >= P.nz) return 0.0;
    int p = ring_plane(l, k0r, P.nz);
    int64_t o = cell_index(P, i, j, p);
    if (c == 2) return l == P.nz - 1 ? 0.0 : lE[o];
    if (l == 0 || l == P.nz - 1) return 0.0;
    double v = lE[o];
    if (l == 1 && !shift) v += cm * lE[cell_index(P, i, j, ring_plane(0, k0r, P.nz))];
    if (l == P.nz - 2 && fm) v += cm * lE[cell_index(P, i, j, ring_plane(P.nz - 1, k0r, P.nz))];
    return v;
}

// fm: the forward applied the Mur condition at the front face (window at rest)
__global__ void __launch_bounds__(AT) k_adj_e(Params P, int k0r, int shift, int fm, double cm, const double *lEx,
                                              const double *lEy, const double *lEz, double *nEx, double *nEy,
                                              double *nEz, double *lBx, double *lBy, double *lBz, double *Jx,
                                              double *Jy, double *Jz) {
    int64_t o = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (o >= P.nc) return;
    int i, j, p;
    int l = plane_of(P, o, k0r, i, j, p);
    const double *lE[3] = {lEx, lEy, lEz};
    double *nE[3] = {nEx, nEy, nEz}, *J[3] = {Jx, Jy, Jz};
    double dt = P.dt;
    double e[3];
    for (int c = 0; c < 3; ++c) {
        e[c] = lam_eff(P, lE[c], c, i, j, l, k0r, shift, fm, cm);
        double n = e[c];
        if (c < 2) {
            if (l == 0 && !shift) n += -cm * lE[c][o];
            if (l == 1 && !shift) n += lE[c][cell_index(P, i, j, ring_plane(0, k0r, P.nz))];
            if (l == P.nz - 1) n += fm ? -cm * lE[c][o] : lE[c][o];  // Mur, or the face kept
            if (l == P.nz - 2 && fm) n += lE[c][cell_index(P, i, j, ring_plane(P.nz - 1, k0r, P.nz))];
        } else if (l == P.nz - 1)
            n += lE[2][o];  // untouched outside half plane
        nE[c][o] = n;
        J[c][o] = -dt * e[c];
    }
    // lam_B += dt * (transpose of the curl of B in the E update)
    double ex_l1 = lam_eff(P, lEx, 0, i, j, l + 1, k0r, shift, fm, cm);
    double ey_l1 = lam_eff(P, lEy, 1, i, j, l + 1, k0r, shift, fm, cm);
    double ez_j1 = lam_eff(P, lEz, 2, i, j + 1, l, k0r, shift, fm, cm);
    double ez_i1 = lam_eff(P, lEz, 2, i + 1, j, l, k0r, shift, fm, cm);
    double ex_j1 = lam_eff(P, lEx, 0, i, j + 1, l, k0r, shift, fm, cm);
    double ey_i1 = lam_eff(P, lEy, 1, i + 1, j, l, k0r, shift, fm, cm);
    lBx[o] += dt * (e[1] - ey_l1 - e[2] + ez_j1);
    lBy[o] += dt * (-e[0] + ex_l1 + e[2] - ez_i1);
    lBz[o] += dt * (e[0] - ex_j1 - e[1] + ey_i1);
}

// The step's last pass: the new lam_E to its place, and the scratch in J cleared.
struct AdjLast {
    double *lE[3], *J[3];
};

// lam_E += transpose of (B <- B - h curl E) applied to lam_B.  LAST: into its place, with what goes with
// it (one pass for this one, three copies and three fills).
template <bool LAST>
__global__ void __launch_bounds__(AT) k_adj_bhalf(Params P, int k0r, double h, const double *lBx, const double *lBy,
                                                  const double *lBz, double *nEx, double *nEy, double *nEz,
                                                  AdjLast A) {
    int64_t o = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (o >= P.nc) return;
    int i, j, p;
    int l = plane_of(P, o, k0r, i, j, p);
    // lam of Bx, By at (i, j, l') with l' = nz-1 does not feed E (those half planes are not updated)
    auto bxy = [&](const double *a, int ii, int jj, int ll) -> double {
        if (ll < 0 || ll >= P.nz - 1) return 0.0;
        return a[cell_index(P, ii, jj, ring_plane(ll, k0r, P.nz))];
    };
    auto bz = [&](int ii, int jj, int ll) -> double { return lBz[cell_index(P, ii, jj, ring_plane(ll, k0r, P.nz))]; };
    double *d[3] = {LAST ? A.lE[0] : nEx, LAST ? A.lE[1] : nEy, LAST ? A.lE[2] : nEz};
    d[0][o] = nEx[o] + h * (bxy(lBy, i, j, l) - bxy(lBy, i, j, l - 1) - bz(i, j, l) + bz(i, j - 1, l));
    d[1][o] = nEy[o] + h * (bz(i, j, l) - bz(i - 1, j, l) - bxy(lBx, i, j, l) + bxy(lBx, i, j, l - 1));
    d[2][o] = nEz[o] + h * (bxy(lBx, i, j, l) - bxy(lBx, i, j - 1, l) - bxy(lBy, i, j, l) + bxy(lBy, i - 1, j, l));
    if (LAST)
        for (int k = 0; k < 3; ++k) A.J[k][o] = 0.0;
}

__global__ void k_zero_plane(int64_t plane, int p, double *a0, double *a1, double *a2, double *b0, double *b1,
                             double *b2) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= plane) return;
    int64_t o = (int64_t)p * plane + s;
    a0[o] = a1[o] = a2[o] = 0.0;
    b0[o] = b1[o] = b2[o] = 0.0;
}

// <lam_Jz, J_ion>: sum over cells of lam_Jz times the ion profile of the cell's plane
__global__ void __launch_bounds__(AT) k_ion_dot(Params P, int k0r, const double *lJz, const double *jion, Sum2 *out) {
    __shared__ Sum2 red[AT / 64];
    Sum2 v{0.0, 0.0};
    for (int64_t o = (int64_t)blockIdx.x * AT + threadIdx.x; o < P.nc; o += (int64_t)gridDim.x * AT) {
        int p = (int)(o / P.plane);
        int l = p - k0r;
        if (l < 0) l += P.nz;
        if (l != P.nz - 1) v.add(lJz[o] * jion[l]);
    }
    v = block_sum2<AT>(v, red);
    if (threadIdx.x == 0) out[blockIdx.x] = v;
}

// ---------------------------------------------------------------- particle reverse
// The transpose of one component's gather: lam times its weights into the adjoint field's box L, and
// lam times its derivatives along x, y, z from the field's box F added to gX.
template <class G, int K>
__device__ inline void gather_adj(const double *F, double *L, const double wi[3][3], const double wh[3][3],
                                  const double di[3][3], const double dh[3][3], const int bi[3], const int bh[3],
                                  double lam, double gX[3]) {
    if (!__any(lam != 0.0)) return;
    constexpr bool hx = G::half(K, 0), hy = G::half(K, 1), hz = G::half(K, 2);
    constexpr int SY = G::FX, SZ = G::FX * G::FY;
    const int o = K * G::NB + (hx ? bh[0] : bi[0]) + SY * (hy ? bh[1] : bi[1]) + SZ * (hz ? bh[2] : bi[2]);
    const double *f = F + o;
    double *l = L + o;
    const double *wx = hx ? wh[0] : wi[0], *wy = hy ? wh[1] : wi[1], *wz = hz ? wh[2] : wi[2];
    const double *dx = hx ? dh[0] : di[0], *dy = hy ? dh[1] : di[1], *dz = hz ? dh[2] : di[2];
    double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double lc = lam * wz[c];
        double p = 0.0, px = 0.0, py = 0.0;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const int r = SY * b + SZ * c;
            const double r0 = f[r], r1 = f[r + 1], r2 = f[r + 2], lb = lc * wy[b];
            atomicAdd(&l[r], lb * wx[0]);
            atomicAdd(&l[r + 1], lb * wx[1]);
            atomicAdd(&l[r + 2], lb * wx[2]);
            const double q = fma(wx[2], r2, fma(wx[1], r1, wx[0] * r0));
            p = fma(wy[b], q, p);
            py = fma(dy[b], q, py);
            px = fma(wy[b], fma(dx[2], r2, fma(dx[1], r1, dx[0] * r0)), px);
        }
        gz = fma(dz[c], p, gz);
        gy = fma(wz[c], py, gy);
        gx = fma(wz[c], px, gx);
    }
    gX[0] = fma(lam, gx, gX[0]);
    gX[1] = fma(lam, gy, gX[1]);
    gX[2] = fma(lam, gz, gX[2]);
    asm volatile("" : "+v"(gX[0]), "+v"(gX[1]), "+v"(gX[2]));  // summed here, not after the other components' reads
    __builtin_amdgcn_sched_barrier(0);
}

// Adjoint of one component of the Esirkepov current, J_c(m, a, b) = f P_c[m] A_c[a][b]: returns
// <lam_J, J> of the particle and adds the derivatives with respect to S0 and DS.  Nodes that no
// lane of the wave reaches (the windows' last, without a crossing) are left out: their weights and
// the weights' derivatives vanish, and what the last node along the axis adds to every P_c[m]'s
// factor alike drops out, the DS and their derivatives summing to zero.
template <class G, int C>
__device__ inline double deposit_grad(const double *Ls, const int jb[3], const double S0[3][4], const double DS[3][4],
                                      const bool cross[3], double f, double gS0[3][4], double gDS[3][4]) {
    constexpr int CA = (C + 1) % 3, CB = (C + 2) % 3;
    constexpr int ST[3] = {1, G::jx(C), G::jx(C) * G::jy(C)};
    const double *o = Ls + G::jofs(C) + jb[0] + ST[1] * jb[1] + ST[2] * jb[2];
    const bool m2 = __any(cross[C]), a3 = __any(cross[CA]), b3 = __any(cross[CB]);
    double val = 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (a == 3 && !a3) break;
        const double sa = S0[CA][a], da = DS[CA][a];
        double ga = 0.0, gda = 0.0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (b == 3 && !b3) break;
            const double *e = o + ST[CA] * a + ST[CB] * b;
            const double l2 = m2 ? f * e[2 * ST[C]] : 0.0;
            const double l1 = fma(f, e[ST[C]], l2), l0 = fma(f, e[0], l1);
            const double sb = S0[CB][b], db = DS[CB][b];
            const double ub = fma(0.5, db, sb), vb = fma(1.0 / 3.0, db, 0.5 * sb);
            const double A = fma(sa, ub, da * vb);
            const double gA = fma(DS[C][2], l2, fma(DS[C][1], l1, DS[C][0] * l0));
            val = fma(A, gA, val);
            gDS[C][0] = fma(A, l0, gDS[C][0]);
            gDS[C][1] = fma(A, l1, gDS[C][1]);
            gDS[C][2] = fma(A, l2, gDS[C][2]);
            ga = fma(gA, ub, ga);
            gda = fma(gA, vb, gda);
            gS0[CB][b] = fma(gA, fma(0.5, da, sa), gS0[CB][b]);
            gDS[CB][b] = fma(gA, fma(1.0 / 3.0, da, 0.5 * sa), gDS[CB][b]);
        }
        gS0[CA][a] += ga;
        gDS[CA][a] += gda;
        // each row is finished before the next one's reads
        asm volatile("" : "+v"(val), "+v"(gDS[C][0]), "+v"(gDS[C][1]), "+v"(gDS[C][2]), "+v"(gS0[CB][0]),
                     "+v"(gS0[CB][1]), "+v"(gS0[CB][2]), "+v"(gDS[CB][0]), "+v"(gDS[CB][1]), "+v"(gDS[CB][2]));
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    return val;
}

__device__ inline void push_boris_adj(double dt, const double u[3], const double E[3], const double B[3],
                                      const double lo[3], double lu[3], double lE[3], double lB[3]) {
    double a = -0.5 * dt;
    double um[3], T[3], Sv[3], up[3], c[3];
    for (int d = 0; d < 3; ++d) um[d] = u[d] + a * E[d];
    double gm = sqrt(1.0 + dot3(um, um));
    for (int d = 0; d < 3; ++d) T[d] = a * B[d] / gm;
    double tt = dot3(T, T);
    for (int d = 0; d < 3; ++d) Sv[d] = 2.0 * T[d] / (1.0 + tt);
    cross3(um, T, c);
    for (int d = 0; d < 3; ++d) up[d] = um[d] + c[d];
    double lum[3], lup[3], lS[3], lT[3], tmp[3];
    for (int d = 0; d < 3; ++d) {
        lE[d] = a * lo[d];
        lum[d] = lo[d];
    }
    cross3(Sv, lo, lup);
    cross3(lo, up, lS);
    cross3(T, lup, tmp);
    for (int d = 0; d < 3; ++d) lum[d] += lup[d] + tmp[d];
    cross3(lup, um, lT);
    double TS = dot3(T, lS), den = 1.0 + tt;
    for (int d = 0; d < 3; ++d) lT[d] += 2.0 * lS[d] / den - 4.0 * T[d] * TS / (den * den);
    double lgm = -a * dot3(B, lT) / (gm * gm);
    for (int d = 0; d < 3; ++d) lB[d] = a * lT[d] / gm;
    for (int d = 0; d < 3; ++d) lum[d] += lgm * um[d] / gm;
    for (int d = 0; d < 3; ++d) {
        lu[d] = lum[d];
        lE[d] += a * lum[d];
    }
}

__device__ inline void push_vay_adj(double dt, const double u[3], const double E[3], const double B[3],
                                    const double lo[3], double lu[3], double lE[3], double lB[3]) {
    double a = -0.5 * dt;
    double g0 = sqrt(1.0 + dot3(u, u));
    double v0[3], c[3], u1[3], tau[3], t[3], w[3];
    for (int d = 0; d < 3; ++d) v0[d] = u[d] / g0;
    cross3(v0, B, c);
    for (int d = 0; d < 3; ++d) u1[d] = u[d] + 2.0 * a * E[d] + a * c[d];
    for (int d = 0; d < 3; ++d) tau[d] = a * B[d];
    double us = dot3(u1, tau), tau2 = dot3(tau, tau);
    double sig = 1.0 + dot3(u1, u1) - tau2;
    double D = sqrt(sig * sig + 4.0 * (tau2 + us * us));
    double gn = sqrt(0.5 * (sig + D));
    for (int d = 0; d < 3; ++d) t[d] = tau[d] / gn;
    double sf = 1.0 / (1.0 + dot3(t, t));
    double ut = dot3(u1, t);
    cross3(u1, t, c);
    for (int d = 0; d < 3; ++d) w[d] = u1[d] + ut * t[d] + c[d];
    double lsf = dot3(lo, w), lw[3], lu1[3], lt[3], ltau[3], tmp[3];
    for (int d = 0; d < 3; ++d) lw[d] = sf * lo[d];
    double tlw = dot3(t, lw);
    cross3(t, lw, tmp);
    for (int d = 0; d < 3; ++d) lu1[d] = lw[d] + tlw * t[d] + tmp[d];
    cross3(lw, u1, tmp);
    for (int d = 0; d < 3; ++d) lt[d] = tlw * u1[d] + ut * lw[d] + tmp[d];
    for (int d = 0; d < 3; ++d) lt[d] += -2.0 * lsf * sf * sf * t[d];
    double lgn = -dot3(tau, lt) / (gn * gn);
    for (int d = 0; d < 3; ++d) ltau[d] = lt[d] / gn;
    double lsig = lgn / (4.0 * gn), lD = lgn / (4.0 * gn);
    lsig += lD * sig / D;
    double ltau2 = lD * 2.0 / D, lus = lD * 4.0 * us / D;
    ltau2 += -lsig;
    for (int d = 0; d < 3; ++d) lu1[d] += 2.0 * lsig * u1[d];
    for (int d = 0; d < 3; ++d) {
        ltau[d] += 2.0 * ltau2 * tau[d] + lus * u1[d];
        lu1[d] += lus * tau[d];
    }
    for (int d = 0; d < 3; ++d) lB[d] = a * ltau[d];
    double lv0[3];
    cross3(B, lu1, lv0);
    cross3(lu1, v0, tmp);
    for (int d = 0; d < 3; ++d) {
        lv0[d] *= a;
        lB[d] += a * tmp[d];
        lE[d] = 2.0 * a * lu1[d];
        lu[d] = lu1[d];
    }
    double uv = dot3(u, lv0);
    for (int d = 0; d < 3; ++d) lu[d] += lv0[d] / g0 - u[d] * uv / (g0 * g0 * g0);
}

// adjoint of the particles that no list holds (dead slots, and live ones that the step takes out): zero
__global__ void __launch_bounds__(AT) k_adj_dead(int64_t n, const uint32_t *key, int64_t nb, double *lb, int64_t capb,
                                                 double *lp, int64_t capp) {
    const int64_t q = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (q >= n || key[q] != NO_BIN) return;
    double *l = q < nb ? lb + q : lp + (q - nb);
    const int64_t cap = q < nb ? capb : capp;
    for (int d = 0; d < 6; ++d) l[d * cap] = 0.0;
}

// the nodes of an adjoint field's box to the grid, cleared
template <class G> __device__ inline void flush_nodes(const Params &P, int k0r, const Item64 &I, double *L,
                                                      double *const dst[6]) {
    int e = threadIdx.x;
    opaque64(e);
    for (; e < G::NB; e += PT) {
        const int y = e / G::FX, a = e - y * G::FX, c = y / G::FY, b = y - c * G::FY;
        const int l = I.t0z - 1 + c;
        const bool in = l >= 0 && l < P.nz;
        const int64_t o = in ? cell_near(P, I.t0x - 1 + a, I.t0y - 1 + b, ring_plane(l, k0r, P.nz)) : 0;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double v = L[k * G::NB + e];
            L[k * G::NB + e] = 0.0;
            if (in && v != 0.0) atomicAdd(&dst[k][o], v);
        }
    }
}

// lam_J of the tile into LDS
template <class G, int K> __device__ inline void stage_lj(const Params &P, int k0r, const Item64 &I, const double *src,
                                                          double *L) {
    constexpr int X = G::jx(K), Y = G::jy(K), N = G::jsize(K), R = (N + PT - 1) / PT;
    double v[R];
    int e0 = threadIdx.x;
    opaque64(e0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = e0 + r * PT, y = e / X, a = e - y * X, c = y / Y, b = y - c * Y, l = I.t0z - 2 + c;
        const bool in = e < N && l >= 0 && l < P.nz;
        v[r] = in ? src[cell_near(P, I.t0x - 2 + a, I.t0y - 2 + b, ring_plane(l, k0r, P.nz))] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (e0 + r * PT < N) L[G::jofs(K) + e0 + r * PT] = v[r];
}

// The particles' part of the reverse step, tile by tile through the lists of k_tiles64.hip: E^n, B^n
// and lam_J staged in LDS (74 KB), the adjoint fields' contributions summed in LDS boxes (41 KB) and
// added to the grid once per item.  One thread per particle over the grid, with 162 global FP64
// atomics each, took 15.0 ms on the 64x64x256 workload (1 M beam, 2 M plasma particles); this takes
// 0.90 ms.  Bound: VALU (about 3500 instructions a wave) on one workgroup a CU, which is what the
// LDS boxes leave: 512 threads, two waves a SIMD.  The fields are gathered twice, before the push and
// with the scatter: keeping the first pass's 18 derivatives costs more in spills than 162 LDS reads.
template <class G>
__global__ void __launch_bounds__(PT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_adj_particles(Params P, StepCtx S, Bounds64 W, Species64 sb, Species64 sp, TileList T, double *lamb, double *lamp,
                FieldsT<double> f, double *nEx, double *nEy, double *nEz, double *lBx, double *lBy, double *lBz,
                const double *lJx, const double *lJy, const double *lJz, Sum2 *part) {
    extern __shared__ __align__(16) double sma[];
    __shared__ int s_item;
    __shared__ Sum2 red[PT / 64];
    double *F = sma, *L = F + G::NF, *Ls = L + G::NF;  // fields, adjoint fields, lam_J
    const uint32_t tid = threadIdx.x;
    for (int e = tid; e < G::NF; e += PT) L[e] = 0.0;
    Sum2 gK{0.0, 0.0}, gn{0.0, 0.0};
    ItemQueue64 Q;
    if (tid == 0) s_item = Q.first(T);
    __syncthreads();
    int cur = __builtin_amdgcn_readfirstlane(s_item);
    while (cur >= 0) {
        const Item64 I = item64(T, cur, G::TX, G::TY, G::TZ);
        {
            Stage64<G, PT> st;
            st.load(P, S.k0r, I, f);
            stage_lj<G, 0>(P, S.k0r, I, lJx, Ls);
            stage_lj<G, 1>(P, S.k0r, I, lJy, Ls);
            stage_lj<G, 2>(P, S.k0r, I, lJz, Ls);
            st.store(F);
        }
        __syncthreads();
        if (tid == 0) Q.claim(T);
        for (uint32_t e = I.begin + tid; e < I.end; e += PT) {
            const Raw64 r = load_raw64(sb, sp, T.list[e]);
            int c0[3], bi[3];
            double wi[3][3], fl[3], E[3], B[3];
            for (int d = 0; d < 3; ++d) fl[d] = floor(r.X[d]);
            cell_in_tile64(P, W, I, fl, c0);
            {
                double wh[3][3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    bi[d] = c0[d] + near_int(r.X[d], fl[d], wi[d]);
                    weights3<double>(r.X[d] - 0.5 - fl[d], wh[d]);
                }
                E[0] = gather_lds<G, 0>(F, wi, wh, bi, c0);
                E[1] = gather_lds<G, 1>(F, wi, wh, bi, c0);
                E[2] = gather_lds<G, 2>(F, wi, wh, bi, c0);
                B[0] = gather_lds<G, 3>(F, wi, wh, bi, c0);
                B[1] = gather_lds<G, 4>(F, wi, wh, bi, c0);
                B[2] = gather_lds<G, 5>(F, wi, wh, bi, c0);
            }
            double Ee[3], Be[3], dEe[3], dBe[3];
            ext_field64(P, r.X[2], S.t, Ee, Be, dEe, dBe);
            for (int d = 0; d < 3; ++d) {
                E[d] += Ee[d];
                B[d] += Be[d];
            }
            double Un[3], X1[3];
            push<double>(P.pusher, -0.5 * P.dt, r.U, E, B, Un);
            const double g = sqrt(1.0 + dot3(Un, Un));
            for (int d = 0; d < 3; ++d) X1[d] = r.X[d] + P.dt * Un[d] / g;
            const bool beam = r.id < (uint32_t)sb.n;
            const int64_t cap = beam ? sb.cap : sp.cap;
            double *const lq = beam ? lamb + r.id : lamp + (r.id - (uint32_t)sb.n);
            if (!(isfinite(X1[0]) && isfinite(X1[1]) && isfinite(X1[2]))) {
                // the forward step dropped this particle without a deposit
                for (int d = 0; d < 6; ++d) lq[d * cap] = 0.0;
                continue;
            }
            const bool alive1 = !(X1[2] < W.lo || X1[2] >= W.hi);
            double gX[3] = {0.0, 0.0, 0.0}, gX1[3], lun[3];
            for (int d = 0; d < 3; ++d) {
                const double lx = lq[d * cap], lu1 = lq[(3 + d) * cap];  // loaded by all, then selected
                gX1[d] = alive1 ? lx : 0.0;
                lun[d] = alive1 ? lu1 : 0.0;
            }
            {
                double S0[3][4], DS[3][4], gS0[3][4], gDS[3][4];
                int jb[3];
                bool cross[3], h0[3], h1[3];
                double d1[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const int n0 = bi[d] - c0[d];
                    double w1[3];
                    const int n1 = near_int(X1[d], fl[d], w1), lo = n0 < n1 ? n0 : n1;
                    d1[d] = X1[d] - fl[d] - (double)n1;
                    h0[d] = n0 > lo;
                    h1[d] = n1 > lo;
                    cross[d] = n0 != n1;
                    jb[d] = c0[d] + lo + 1;  // box node of offset lo - 1, origin -2
                    window4(wi[d], h0[d], S0[d]);
                    window4(w1, h1[d], DS[d]);
                    for (int m = 0; m < 4; ++m) {
                        DS[d][m] -= S0[d][m];
                        gS0[d][m] = 0.0;
                        gDS[d][m] = 0.0;
                    }
                }
                const double fq = r.w / P.dt;
                double val = deposit_grad<G, 0>(Ls, jb, S0, DS, cross, fq, gS0, gDS);
                val += deposit_grad<G, 1>(Ls, jb, S0, DS, cross, fq, gS0, gDS);
                val += deposit_grad<G, 2>(Ls, jb, S0, DS, cross, fq, gS0, gDS);
                gn.add(beam ? 0.0 : val);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    double dw[3], w4[4];
                    dweights3(r.X[d] - fl[d] - (double)(bi[d] - c0[d]), dw);
                    window4(dw, h0[d], w4);
                    for (int m = 0; m < 4; ++m) gX[d] += (gS0[d][m] - gDS[d][m]) * w4[m];
                    dweights3(d1[d], dw);
                    window4(dw, h1[d], w4);
                    for (int m = 0; m < 4; ++m) gX1[d] += gDS[d][m] * w4[m];
                }
            }
            const double ug = dot3(Un, gX1);
            for (int d = 0; d < 3; ++d) {
                gX[d] += gX1[d];
                lun[d] += P.dt * (gX1[d] / g - Un[d] * ug / (g * g * g));
            }
            double lu[3], lEp[3], lBp[3];
            if (P.pusher == 1)
                push_vay_adj(P.dt, r.U, E, B, lun, lu, lEp, lBp);
            else
                push_boris_adj(P.dt, r.U, E, B, lun, lu, lEp, lBp);
            gK.add(dot3(lEp, Ee) + dot3(lBp, Be));
            gX[2] += dot3(lEp, dEe) + dot3(lBp, dBe);
            double wh[3][3], di[3][3], dh[3][3];  // the weights again: kept from the gather they would be spilled
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                double x = r.X[d];
                asm volatile("" : "+v"(x));
                const double oi = x - fl[d] - (double)(bi[d] - c0[d]), oh = x - 0.5 - fl[d];
                weights3<double>(oi, wi[d]);
                dweights3(oi, di[d]);
                weights3<double>(oh, wh[d]);
                dweights3(oh, dh[d]);
            }
            gather_adj<G, 0>(F, L, wi, wh, di, dh, bi, c0, lEp[0], gX);
            gather_adj<G, 1>(F, L, wi, wh, di, dh, bi, c0, lEp[1], gX);
            gather_adj<G, 2>(F, L, wi, wh, di, dh, bi, c0, lEp[2], gX);
            gather_adj<G, 3>(F, L, wi, wh, di, dh, bi, c0, lBp[0], gX);
            gather_adj<G, 4>(F, L, wi, wh, di, dh, bi, c0, lBp[1], gX);
            gather_adj<G, 5>(F, L, wi, wh, di, dh, bi, c0, lBp[2], gX);
            for (int d = 0; d < 3; ++d) {
                lq[d * cap] = gX[d];
                lq[(3 + d) * cap] = lu[d];
            }
        }
        if (tid == 0) s_item = Q.resolve(T);
        __syncthreads();
        cur = __builtin_amdgcn_readfirstlane(s_item);
        double *const dst[6] = {nEx, nEy, nEz, lBx, lBy, lBz};
        flush_nodes<G>(P, S.k0r, I, L, dst);
    }
    gK = block_sum2<PT>(gK, red);
    gn = block_sum2<PT>(gn, red);
    if (tid == 0) {
        part[2 * blockIdx.x] = gK;
        part[2 * blockIdx.x + 1] = gn;
    }
}

template <class G> static constexpr int adj_lds() { return 8 * (2 * G::NF + G::NJ); }

pic_status adjoint_setup(Ctx &c) {
    const bool flat = tiles64_flat(c.P);
    PIC_HIP(c, hipFuncSetAttribute(flat ? (const void *)k_adj_particles<Geom2D> : (const void *)k_adj_particles<Geom3D>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   flat ? adj_lds<Geom2D>() : adj_lds<Geom3D>()));
    return PIC_OK;
}

__global__ void k_zero_slots(Lam L, int64_t a, int64_t b) {
    int64_t q = a + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= b) return;
    for (int d = 0; d < 3; ++d) {
        L.x[d][q] = 0.0;
        L.u[d][q] = 0.0;
    }
}

// ---------------------------------------------------------------- seed
__global__ void __launch_bounds__(AT) k_bunch_sums(Part64 p, int64_t n, double kb, double *out) {
    __shared__ double s[3][AT];
    double v[3] = {0, 0, 0};
    int64_t q = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (q < n && p.alive[q]) {
        double sn, cs;
        sincos(kb * p.z[q], &sn, &cs);
        v[0] = p.w[q];
        v[1] = p.w[q] * cs;
        v[2] = p.w[q] * sn;
    }
    for (int k = 0; k < 3; ++k) s[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int h = AT / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h)
            for (int k = 0; k < 3; ++k) s[k][threadIdx.x] += s[k][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int k = 0; k < 3; ++k) out[3 * blockIdx.x + k] = s[k][0];
}

__global__ void k_bunch_seed(Part64 p, int64_t n, double kb, double C, double Sn, double A, double W, double *lz) {
    int64_t q = (int64_t)blockIdx.x * AT + threadIdx.x;
    if (q >= n || !p.alive[q]) return;
    double sn, cs;
    sincos(kb * p.z[q], &sn, &cs);
    lz[q] = p.w[q] * kb * (-C * sn + Sn * cs) / (A * W);
}

pic_status adjoint_seed(Ctx &c, double kb, double *lam, double *loss) {
    int64_t len = 6 * (std::max<int64_t>(c.cap_b, 1) + std::max<int64_t>(c.cap_p, 1)) + 6 * c.P.nc;
    PIC_HIP(c, hipMemsetAsync(lam, 0, 8 * (uint64_t)len, c.st));
    int64_t n = c.nb_slots;
    double C = 0, Sn = 0, W = 0;
    if (n > 0) {
        int nblk = nblocks(n, AT);
        hipLaunchKernelGGL(k_bunch_sums, dim3(nblk), dim3(AT), 0, c.st, c.b64, n, kb, c.red);
        std::vector<double> h(3 * (size_t)nblk);
        PIC_HIP(c, hipMemcpyAsync(h.data(), c.red, 24 * (uint64_t)nblk, hipMemcpyDeviceToHost, c.st));
        PIC_HIP(c, hipStreamSynchronize(c.st));
        for (int b = 0; b < nblk; ++b) {
            W += h[3 * b];
            C += h[3 * b + 1];
            Sn += h[3 * b + 2];
        }
    }
    if (W <= 0) {
        c.err = "adjoint seed: no beam particles";
        return PIC_ESTATE;
    }
    double A = sqrt(C * C + Sn * Sn);
    *loss = A / W;
    Lam L = lam_view(lam, 0, c.cap_b);
    hipLaunchKernelGGL(k_bunch_seed, dim3(nblocks(n, AT)), dim3(AT), 0, c.st, c.b64, n, kb, C, Sn, A, W, L.x[2]);
    PIC_HIP(c, hipStreamSynchronize(c.st));
    return PIC_OK;
}

// slots of plasma after the forward step's injection (host replay of the sheet logic)
static int64_t plasma_slots_after(const Ctx &c, const StepCtx &S) {
    if (!c.P.has_plasma) return c.np_slots;
    int64_t sheet = sheet_particles(c.P);
    double hi = (double)(S.k0n + c.P.nz - 4);
    int64_t l = c.sh_hi, n = c.np_slots;
    while (sheet_z(l, c.P.ppz, c.P.bR, S.t1) < hi) {
        if (sheet_weight(c.P, l) != 0.0) n += sheet;
        ++l;
    }
    return n;
}

pic_status adjoint_step(Ctx &c, double *lam, double grad[2]) {
    const Params &P = c.P;
    StepCtx S = make_step_ctx(c);
    uint64_t cb = (uint64_t)std::max<int64_t>(c.cap_b, 1), cp = (uint64_t)std::max<int64_t>(c.cap_p, 1);
    Lam Lb = lam_view(lam, 0, c.cap_b), Lp = lam_view(lam, 6 * cb, c.cap_p);
    double *lE[3], *lB[3], *nE[3], *Bn[3];
    for (int k = 0; k < 3; ++k) {
        lE[k] = lam + 6 * (cb + cp) + k * P.nc;
        lB[k] = lam + 6 * (cb + cp) + (3 + k) * P.nc;
        nE[k] = c.adj + k * P.nc;
        Bn[k] = c.adj + (3 + k) * P.nc;
    }
    // slots injected during step n carry no adjoint into state n
    int64_t np1 = std::min<int64_t>(plasma_slots_after(c, S), c.cap_p);
    if (np1 > c.np_slots)
        hipLaunchKernelGGL(k_zero_slots, dim3(nblocks(np1 - c.np_slots, AT)), dim3(AT), 0, c.st, Lp, c.np_slots, np1);
    // B^n = B^{n-1/2} - (dt/2) curl E^n
    FieldsT<double> f, fn;
    for (int k = 0; k < 3; ++k) {
        f.E[k] = fn.E[k] = c.E64[k];
        f.B[k] = c.B64[k];
        fn.B[k] = Bn[k];
    }
    launch_bhalf<double>(P, S.k0r, f, fn, 0.5 * P.dt, c.jion64, c.st);
    // window shift: the back plane became the empty front plane
    if (S.shift)
        hipLaunchKernelGGL(k_zero_plane, dim3(nblocks(P.plane, 256)), dim3(256), 0, c.st, (int64_t)P.plane, S.k0r,
                           lE[0], lE[1], lE[2], lB[0], lB[1], lB[2]);
    // E update with Mur faces
    double cm = (P.dt - 1.0) / (P.dt + 1.0);
    int nb = nblocks(P.nc, AT);
    hipLaunchKernelGGL(k_adj_e, dim3(nb), dim3(AT), 0, c.st, P, S.k0r, S.shift, (int)(c.bw <= 0.0), cm, lE[0], lE[1],
                       lE[2], nE[0], nE[1],
                       nE[2], lB[0], lB[1], lB[2], c.J64[0], c.J64[1], c.J64[2]);
    // second half step
    const AdjLast last{{lE[0], lE[1], lE[2]}, {c.J64[0], c.J64[1], c.J64[2]}};
    hipLaunchKernelGGL(k_adj_bhalf<false>, dim3(nb), dim3(AT), 0, c.st, P, S.k0r, 0.5 * P.dt, lB[0], lB[1], lB[2],
                       nE[0], nE[1], nE[2], last);
    // the partial sums, read back together at the end: the ions' (none: zero), then the particles'
    Sum2 *const part = (Sum2 *)c.adj_part;
    int parts = 0, ion_parts = 0;
    // ion current: n0 dL/dn0 += <lam_Jz, J_ion>
    if (P.ions && c.sh_hi > c.sh_lo) {
        launch_ion64(P, c.sh_lo, c.sh_hi - c.sh_lo, S.t, S.t1, S.k0, c.jion64, c.st);
        parts = ion_parts = 256;
        hipLaunchKernelGGL(k_ion_dot, dim3(ion_parts), dim3(AT), 0, c.st, P, S.k0r, c.J64[2], c.jion64, part);
    }
    // particles
    const Species64 b{c.b64.x, (int64_t)cb, c.nb_slots}, p{c.p64.x, (int64_t)cp, c.np_slots};
    const int64_t n = b.n + p.n;
    if (n > 0) {
        const int grid = std::min(c.ncu, 512);
        const bool flat = tiles64_flat(P);
        tiles64_build(c, b, p, grid, false);
        hipLaunchKernelGGL(k_adj_dead, dim3(nblocks(n, AT)), dim3(AT), 0, c.st, n, c.tiles.key, b.n, Lb.x[0], b.cap,
                           Lp.x[0], p.cap);
        const Bounds64 W(P, S.k0, S.k0n);
        auto launch = [&](auto kernel, int lds) {
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(PT), lds, c.st, P, S, W, b, p, c.tiles, Lb.x[0], Lp.x[0], fn,
                               nE[0], nE[1], nE[2], lB[0], lB[1], lB[2], c.J64[0], c.J64[1], c.J64[2], part + ion_parts);
        };
        if (flat)
            launch(k_adj_particles<Geom2D>, adj_lds<Geom2D>());
        else
            launch(k_adj_particles<Geom3D>, adj_lds<Geom3D>());
        parts += 2 * grid;
    }
    // first half step, then the new lam_E
    hipLaunchKernelGGL(k_adj_bhalf<true>, dim3(nb), dim3(AT), 0, c.st, P, S.k0r, 0.5 * P.dt, lB[0], lB[1], lB[2],
                       nE[0], nE[1], nE[2], last);
    Sum2 h[ADJ_PARTS], gn{0.0, 0.0}, gK{0.0, 0.0};
    if (parts) PIC_HIP(c, hipMemcpyAsync(h, part, sizeof(Sum2) * parts, hipMemcpyDeviceToHost, c.st));
    PIC_HIP(c, hipStreamSynchronize(c.st));
    for (int k = 0; k < ion_parts; ++k) gn.add(h[k].hi, h[k].lo);
    for (int k = ion_parts; k < parts; k += 2) {
        gK.add(h[k].hi, h[k].lo);
        gn.add(h[k + 1].hi, h[k + 1].lo);
    }
    grad[0] += gK.value();
    grad[1] += gn.value();
    return PIC_OK;
}

}  // namespace pic
