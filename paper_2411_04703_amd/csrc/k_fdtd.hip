// k_fdtd.hip -- Yee FDTD in normalised units on the ring-buffered moving window.
//
// Maxwell's curl equations with electron and ion currents (section 1,
// Eq. Max1, Max2 of the paper; Gaussian factors absorbed by the units):
//   B <- B - (dt/2) curl E      (twice per step, around the particle push)
//   E <- E + dt (curl B - J)
// Yee staggering: Ex(i+1/2,j,k) Ey(i,j+1/2,k) Ez(i,j,k+1/2), Bx(i,j+1/2,k+1/2)
// By(i+1/2,j,k+1/2) Bz(i+1/2,j+1/2,k).  x, y periodic.  z: nz logical planes
// stored as a ring (logical plane l lives in ring plane (l + k0) mod nz).  The
// z boundaries absorb (section 1): first-order Mur on the tangential E at the
// back face, and at the front face while the window is at rest; a moving
// window's front face keeps its tangential E, and the half planes beyond it
// stay zero.
// One thread per cell, x fastest: every array access is coalesced along x.  The
// grid is (cells of a plane, ring planes): the ring plane is the block's y
// index and (i, j) come from 32-bit arithmetic on the in-plane index.
#include "pic_internal.h"

namespace pic {

template <typename JT> __device__ inline double jvalue(JT v, double finv);
template <> __device__ inline double jvalue<double>(double v, double) { return v; }
template <> __device__ inline double jvalue<long long>(long long v, double finv) { return (double)v * finv; }

// in-plane index s = i + nx j of the calling thread, false past the plane's end
__device__ inline bool plane_cell(const Params &P, int &i, int &j) {
    const int s = (int)blockIdx.x * (int)blockDim.x + (int)threadIdx.x;
    if (s >= P.plane) return false;
    j = s / P.nx;
    i = s - j * P.nx;
    return true;
}

// g: where the new B goes (f itself, or another set beside E); profile: an nz-long array to clear, or null
template <typename T>
__global__ void __launch_bounds__(256) k_bhalf(Params P, int k0r, FieldsT<T> f, FieldsT<T> g, T h, T *profile) {
    int i, j;
    if (!plane_cell(P, i, j)) return;
    const int p = (int)blockIdx.y;
    const int64_t o = (int64_t)p * P.plane + i + (int64_t)P.nx * j;
    int l = p - k0r;
    if (l < 0) l += P.nz;
    int64_t oi = o + ((i + 1 == P.nx) ? 1 - P.nx : 1);
    int64_t oj = o + ((j + 1 == P.ny) ? (int64_t)(1 - P.ny) * P.nx : P.nx);
    const T *Ex = f.E[0], *Ey = f.E[1], *Ez = f.E[2];
    T ex = Ex[o], ey = Ey[o], ez = Ez[o];
    T bx = f.B[0][o], by = f.B[1][o];
    if (l != P.nz - 1) {
        int64_t ol = o + ((p + 1 == P.nz) ? -(int64_t)(P.nz - 1) * P.plane : (int64_t)P.plane);
        bx -= h * ((Ez[oj] - ez) - (Ey[ol] - ey));
        by -= h * ((Ex[ol] - ex) - (Ez[oi] - ez));
    }
    g.B[0][o] = bx;
    g.B[1][o] = by;
    g.B[2][o] = f.B[2][o] - h * ((Ey[oi] - ey) - (Ex[oj] - ex));
    if (profile && i == 0 && j == 0) profile[p] = T(0);
}

// Also the Mur faces: tangential E on logical planes 0 and nz - 1, which no other thread reads or writes,
// from the threads of the planes beside them, which hold the old and the new value there -- the back
// face unless the window shifts after this step (k_shift), the front face only while the window is at
// rest: a moving window's front keeps its tangential E (zero; the planes enter empty), since a
// static-face Mur condition at a face that jumps forward every step or two is unstable with plasma
// streaming in.  (As a pass of its own over saved planes it was one more launch a step, 4 us.)
template <typename T, typename JT>
__global__ void __launch_bounds__(256) k_eupdate(Params P, int k0r, int shift, int front_mur, FieldsT<T> f, JT *Jx,
                                                 JT *Jy, JT *Jz, const JT *jion, T dt, T cm) {
    int i, j;
    if (!plane_cell(P, i, j)) return;
    const int p = (int)blockIdx.y;
    const int64_t o = (int64_t)p * P.plane + i + (int64_t)P.nx * j;
    int l = p - k0r;
    if (l < 0) l += P.nz;
    int64_t oi = o - ((i == 0) ? 1 - P.nx : 1);
    int64_t oj = o - ((j == 0) ? (int64_t)(1 - P.ny) * P.nx : P.nx);
    int64_t ol = o - ((p == 0) ? -(int64_t)(P.nz - 1) * P.plane : (int64_t)P.plane);
    const T *Bx = f.B[0], *By = f.B[1], *Bz = f.B[2];
    T bx = Bx[o], by = By[o], bz = Bz[o];
    double jx = jvalue<JT>(Jx[o], P.finv), jy = jvalue<JT>(Jy[o], P.finv), jz = jvalue<JT>(Jz[o], P.finv);
    Jx[o] = JT(0);
    Jy[o] = JT(0);
    Jz[o] = JT(0);
    if (l != 0 && l != P.nz - 1) {
        const T ex = f.E[0][o], ey = f.E[1][o];
        const T nx = ex + dt * ((bz - Bz[oj]) - (by - By[ol]) - (T)jx);
        const T ny = ey + dt * ((bx - Bx[ol]) - (bz - Bz[oi]) - (T)jy);
        f.E[0][o] = nx;
        f.E[1][o] = ny;
        if (l == 1 && !shift) {
            f.E[0][ol] = ex + cm * (nx - f.E[0][ol]);
            f.E[1][ol] = ey + cm * (ny - f.E[1][ol]);
        }
        if (l == P.nz - 2 && front_mur) {
            const int64_t ot = o + ((p + 1 == P.nz) ? -(int64_t)(P.nz - 1) * P.plane : (int64_t)P.plane);
            f.E[0][ot] = ex + cm * (nx - f.E[0][ot]);
            f.E[1][ot] = ey + cm * (ny - f.E[1][ot]);
        }
    }
    if (l != P.nz - 1) {
        double jt = jz + (jion ? jvalue<JT>(jion[l], P.finv) : 0.0);
        f.E[2][o] += dt * ((by - By[oi]) - (bx - Bx[oj]) - (T)jt);
    }
}

// The window shifts after this step: the back plane becomes the new front plane, which enters empty.
template <typename T>
__global__ void k_shift(Params P, int k0r, FieldsT<T> f) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= P.plane) return;
    for (int c = 0; c < 3; ++c) {
        f.E[c][k0r * (int64_t)P.plane + s] = T(0);
        f.B[c][k0r * (int64_t)P.plane + s] = T(0);
    }
}

// The field part of an FP32 step in one pass: B by a full step (B^(n-1/2) -> B^(n+1/2), what k_bhalf
// does with h = dt), E by a step with the new B and the currents, the Mur faces and the shift (as
// k_eupdate and k_shift), from the fields `f` into `g`.  A thread forms the new B of its cell and
// the six components of it that E needs from the neighbours before it (loads that hit in L1), so that
// nothing waits for a whole pass over B; the old fields stay as they are, which is why `g` is a second
// set.  The threads of planes 1 and nz - 2 hold what the Mur faces beside them need and write those.
// The currents are cleared where they are not zero.
// Bound: HBM, 96 bytes a cell for 120 in two passes.  Workgroups go round the 8 XCDs, so that workgroup
// k works on block k / 8 of the (k mod 8)th eighth of the planes and neighbours share an L2.
template <typename T, typename JT>
__global__ void __launch_bounds__(256) k_fields(Params P, int k0r, int shift, int front_mur, int nbx, FieldsT<T> f,
                                                FieldsT<T> g, JT *Jx, JT *Jy, JT *Jz, const JT *jion, T dt, T cm) {
    uint32_t w = blockIdx.x;
    if (gridDim.x % 8 == 0) w = (w % 8) * (gridDim.x / 8) + w / 8;
    const int p = (int)(w / (uint32_t)nbx), s = (int)(w % (uint32_t)nbx) * 256 + (int)threadIdx.x;
    if (s >= P.plane) return;
    const int j = s / P.nx, i = s - j * P.nx;
    int l = p - k0r;
    if (l < 0) l += P.nz;
    const uint32_t pl = (uint32_t)P.plane;
    const uint32_t x0 = (uint32_t)i, xp = i + 1 == P.nx ? 0 : x0 + 1, xm = i == 0 ? P.nx - 1 : x0 - 1;
    const uint32_t y0 = (uint32_t)(j * P.nx), yp = j + 1 == P.ny ? 0 : y0 + P.nx, ym = j == 0 ? (P.ny - 1) * P.nx : y0 - P.nx;
    const uint32_t z0 = pl * (uint32_t)p, zp = p + 1 == P.nz ? 0 : z0 + pl, zm = p == 0 ? pl * (P.nz - 1) : z0 - pl;
    const T *Ex = f.E[0], *Ey = f.E[1], *Ez = f.E[2], *Bx = f.B[0], *By = f.B[1], *Bz = f.B[2];
    const uint32_t o = x0 + y0 + z0, oxm = xm + y0 + z0, oym = x0 + ym + z0, ozm = x0 + y0 + zm;
    const bool top = l == P.nz - 1;
    auto step_b = [&](T b, T d1, T d2) { return fma(-dt, d1 - d2, b); };
    const T ex = Ex[o], ey = Ey[o], ez = Ez[o];
    T bx = Bx[o], by = By[o], bz = Bz[o];
    if (!top) {
        const uint32_t ozp = x0 + y0 + zp;
        bx = step_b(bx, Ez[x0 + yp + z0] - ez, Ey[ozp] - ey);
        by = step_b(by, Ex[ozp] - ex, Ez[xp + y0 + z0] - ez);
    }
    bz = step_b(bz, Ey[xp + y0 + z0] - ey, Ex[x0 + yp + z0] - ex);
    const JT ix = Jx[o], iy = Jy[o], iz = Jz[o];
    if (ix != JT(0)) Jx[o] = JT(0);
    if (iy != JT(0)) Jy[o] = JT(0);
    if (iz != JT(0)) Jz[o] = JT(0);
    T nx = ex, ny = ey, nz = ez;
    if (!top) {
        const T exm = Ex[oxm], ezm = Ez[oxm], eyn = Ey[oym], ezn = Ez[oym];  // at i - 1, at j - 1
        const T byx = step_b(By[oxm], Ex[xm + y0 + zp] - exm, ez - ezm);
        const T bxy = step_b(Bx[oym], ez - ezn, Ey[x0 + ym + zp] - eyn);
        if (l != 0) {
            const T exn = Ex[oym], eym = Ey[oxm], exz = Ex[ozm], eyz = Ey[ozm], ezz = Ez[ozm];
            const T bzx = step_b(Bz[oxm], ey - eym, Ex[xm + yp + z0] - exm);
            const T bzy = step_b(Bz[oym], Ey[xp + ym + z0] - eyn, ex - exn);
            const T bxz = step_b(Bx[ozm], Ez[x0 + yp + zm] - ezz, ey - eyz);
            const T byz = step_b(By[ozm], ex - exz, Ez[xp + y0 + zm] - ezz);
            nx = fma(dt, (bz - bzy) - (by - byz) - (T)jvalue<JT>(ix, P.finv), ex);
            ny = fma(dt, (bx - bxz) - (bz - bzx) - (T)jvalue<JT>(iy, P.finv), ey);
            if (l == 1 && !shift) {
                g.E[0][ozm] = fma(cm, nx - exz, ex);
                g.E[1][ozm] = fma(cm, ny - eyz, ey);
            }
            if (l == P.nz - 2 && front_mur) {
                g.E[0][x0 + y0 + zp] = fma(cm, nx - Ex[x0 + y0 + zp], ex);
                g.E[1][x0 + y0 + zp] = fma(cm, ny - Ey[x0 + y0 + zp], ey);
            }
        }
        const double jt = jvalue<JT>(iz, P.finv) + (jion ? jvalue<JT>(jion[l], P.finv) : 0.0);
        nz = fma(dt, (by - byx) - (bx - bxy) - (T)jt, ez);
    }
    if (l == 0 && shift) nx = ny = nz = bx = by = bz = T(0);  // the new front plane enters empty
    if (!(l == 0 && !shift) && !(top && front_mur)) {
        g.E[0][o] = nx;
        g.E[1][o] = ny;
    }
    g.E[2][o] = nz;
    g.B[0][o] = bx;
    g.B[1][o] = by;
    g.B[2][o] = bz;
}

void launch_fields32(const Params &P, int k0r, int shift, int front_mur, FieldsT<float> f, FieldsT<float> g,
                     long long *J[3], const long long *jion, float dt, hipStream_t st) {
    const int nbx = nblocks(P.plane, 256);
    const float cm = (dt - 1.0f) / (dt + 1.0f);
    hipLaunchKernelGGL((k_fields<float, long long>), dim3((unsigned)(nbx * P.nz)), dim3(256), 0, st, P, k0r, shift,
                       front_mur, nbx, f, g, J[0], J[1], J[2], jion, dt, cm);
}

template <typename T>
void launch_bhalf(const Params &P, int k0r, FieldsT<T> f, FieldsT<T> g, T h, T *profile, hipStream_t st) {
    hipLaunchKernelGGL(k_bhalf<T>, dim3(nblocks(P.plane, 256), P.nz), dim3(256), 0, st, P, k0r, f, g, h, profile);
}

template <typename T, typename JT>
void launch_eupdate(const Params &P, int k0r, int shift, int front_mur, FieldsT<T> f, JT *J[3], const JT *jion, T dt,
                    hipStream_t st) {
    const T cm = (dt - T(1)) / (dt + T(1));
    hipLaunchKernelGGL((k_eupdate<T, JT>), dim3(nblocks(P.plane, 256), P.nz), dim3(256), 0, st, P, k0r, shift,
                       front_mur, f, J[0], J[1], J[2], jion, dt, cm);
    if (shift) hipLaunchKernelGGL(k_shift<T>, dim3(nblocks(P.plane, 256)), dim3(256), 0, st, P, k0r, f);
}

template void launch_bhalf<double>(const Params &, int, FieldsT<double>, FieldsT<double>, double, double *, hipStream_t);
template void launch_bhalf<float>(const Params &, int, FieldsT<float>, FieldsT<float>, float, float *, hipStream_t);
template void launch_eupdate<double, double>(const Params &, int, int, int, FieldsT<double>, double *[3],
                                             const double *, double, hipStream_t);
template void launch_eupdate<float, long long>(const Params &, int, int, int, FieldsT<float>, long long *[3],
                                               const long long *, float, hipStream_t);

// ---------------------------------------------------------------- ion current
// Immobile lab ions: the plasma lattice drifting rigidly at -beta_R.  Summed
// over a transversely uniform lattice, their Esirkepov current is J_z(z) only:
// per sheet the running sum of -q w ppx ppy (S(z1 - k) - S(z0 - k)) / dt.
// One thread per sheet, contributions added into a logical-plane profile.
// w32: the FP32 mode's ions, which carry the FP32-rounded weight of their sheet's electrons
// (the weight the electrons are stored with), so that the cold lattice is exactly neutral
// and current-free in either mode
__device__ inline void ion_sheet_terms(const Params &P, int64_t l, double t0, double t1, int64_t k0, double out[4],
                                       int &lbase, bool w32) {
    double w = sheet_weight(P, l);
    if (w32) w = (double)(float)w;
    double z0 = sheet_z(l, P.ppz, P.bR, t0), z1 = sheet_z(l, P.ppz, P.bR, t1);
    int64_t b = (int64_t)floor(z0 + 0.5) - 2;
    double acc = 0.0, f = -w * (double)(P.ppx * P.ppy) / P.dt;
    for (int m = 0; m < 4; ++m) {
        acc += spline2<double>(z1 - (double)(b + m)) - spline2<double>(z0 - (double)(b + m));
        out[m] = f * acc;
    }
    lbase = (int)(b - k0);
}

__global__ void k_ion64(Params P, int64_t sh_lo, int64_t ns, double t0, double t1, int64_t k0, double *jion) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ns) return;
    double v[4];
    int lb;
    ion_sheet_terms(P, sh_lo + q, t0, t1, k0, v, lb, false);
    for (int m = 0; m < 4; ++m)
        if (v[m] != 0.0 && lb + m >= 0 && lb + m < P.nz) atomicAdd(&jion[lb + m], v[m]);
}

// FP32 mode; next: the profile of the following step, cleared
__global__ void k_ion_fixed(Params P, int64_t sh_lo, int64_t ns, double t0, double t1, int64_t k0, long long *jion,
                            long long *next, int32_t *flags) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < P.nz) next[q] = 0;
    if (q >= ns) return;
    double v[4];
    int lb;
    ion_sheet_terms(P, sh_lo + q, t0, t1, k0, v, lb, true);
    for (int m = 0; m < 4; ++m) {
        double s = v[m] * P.fscale;
        if (fabs(s) > 4.0e18) atomicOr(flags, DFLAG_FIXED_OVERFLOW);
        long long iv = (long long)rint(s);
        if (iv != 0 && lb + m >= 0 && lb + m < P.nz)
            atomicAdd((unsigned long long *)&jion[lb + m], (unsigned long long)iv);
    }
}

void launch_ion64(const Params &P, int64_t sh_lo, int64_t ns, double t0, double t1, int64_t k0, double *jion,
                  hipStream_t st) {
    if (ns <= 0) return;
    hipLaunchKernelGGL(k_ion64, dim3(nblocks(ns, 128)), dim3(128), 0, st, P, sh_lo, ns, t0, t1, k0, jion);
}

void launch_ion_fixed(const Params &P, int64_t sh_lo, int64_t ns, double t0, double t1, int64_t k0,
                      long long *jion, long long *next, int32_t *flags, hipStream_t st) {
    hipLaunchKernelGGL(k_ion_fixed, dim3(nblocks(std::max<int64_t>(ns, P.nz), 128)), dim3(128), 0, st, P, sh_lo, ns,
                       t0, t1, k0, jion, next, flags);
}

}  // namespace pic
