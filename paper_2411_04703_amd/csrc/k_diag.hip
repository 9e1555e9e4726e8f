// k_diag.hip -- diagnostics: beam moments and normalised emittances, bunching
// factor, energies and the Gauss-law residual div E - rho.
//
// The paper bases its analysis on quantities that do not depend on the
// frame change (transverse dynamics, charge; section 2) and reports the beam
// modulation at the boosted undulator period and half of it (section 3); the
// bunching factor |sum w exp(i k z')| / sum w is taken at fixed t' in the
// boosted frame.  All sums are FP64 with per-block partials, reduced on the
// device in a fixed order (k_reduce_rows), so a diagnostic of a given
// particle order is reproducible bit for bit.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "diag_dev.h"

namespace pic {

// FP64 particles: pass 1 and pass 2 of the beam, plasma count and kinetic energy
__global__ void __launch_bounds__(DT) k_mom1(Part64 p, int64_t n, double kb, double *out) {
    double v[13] = {0};
    int64_t a, b;
    row_range(n, a, b);
    for (int64_t q = a + threadIdx.x; q < b; q += DT)
        if (p.alive[q]) moment1_add(v, p.w[q], p.x[q], p.y[q], p.z[q], p.ux[q], p.uy[q], p.uz[q], kb);
    block_sums<13>(v, out + 13 * (int64_t)blockIdx.x);
}

__global__ void __launch_bounds__(DT) k_mom2(Part64 p, int64_t n, const double *m1, double *out) {
    double v[8] = {0};
    const Means M(m1);
    int64_t a, b;
    row_range(n, a, b);
    for (int64_t q = a + threadIdx.x; q < b; q += DT)
        if (p.alive[q]) moment2_add(v, M, p.w[q], p.x[q], p.y[q], p.z[q], p.ux[q], p.uy[q], p.uz[q]);
    block_sums<8>(v, out + 8 * (int64_t)blockIdx.x);
}

__global__ void __launch_bounds__(DT) k_kin(Part64 p, int64_t n, double mi, double *out) {
    double v[2] = {0};
    int64_t a, b;
    row_range(n, a, b);
    for (int64_t q = a + threadIdx.x; q < b; q += DT)
        if (p.alive[q]) kinetic_add(v, p.w[q], p.ux[q], p.uy[q], p.uz[q], mi);
    block_sums<2>(v, out + 2 * (int64_t)blockIdx.x);
}

template <typename T> __global__ void __launch_bounds__(DT) k_fenergy(FieldsT<T> f, int64_t nc, double *out) {
    double v[1] = {0};
    for (int64_t q = (int64_t)blockIdx.x * DT + threadIdx.x; q < nc; q += (int64_t)gridDim.x * DT)
        for (int c = 0; c < 3; ++c) {
            double e = f.E[c][q], b = f.B[c][q];
            v[0] += e * e + b * b;
        }
    block_sums<1>(v, out + blockIdx.x);
}

// ion charge profile (logical planes): sum over sheets of w ppx ppy S(k - z_l)
// w32: the FP32 mode's ions carry their electrons' FP32-rounded weight
__global__ void k_rho_ion(Params P, int64_t sh_lo, int64_t ns, double t, int64_t k0, double *prof, int w32) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ns) return;
    int64_t l = sh_lo + q;
    double w = sheet_weight(P, l);
    if (w32) w = (double)(float)w;
    w *= (double)(P.ppx * P.ppy);
    if (w == 0.0) return;
    double z = sheet_z(l, P.ppz, P.bR, t);
    double nn = floor(z + 0.5), ws[3];
    weights3<double>(z - nn, ws);
    for (int c = 0; c < 3; ++c) {
        int lp = (int)((int64_t)nn - 1 + c - k0);
        if (lp >= 0 && lp < P.nz) atomicAdd(&prof[lp], w * ws[c]);
    }
}

// r = div E - rho on nodes of the band [band, nz - band); max |r|, max |rho|, max |r - r_prev| where the
// previous call's residual covers the same absolute plane.  The residual is kept in ring order: a plane
// keeps its place while it is in the window, so that one pass reads the old value, stores the new one
// and clears the charge (the scratch is a current array, zero between steps).  In-plane indices in 32
// bits; a block takes its cells of every gridDim.y-th ring plane.  HBM: 64 us
// at 128x128x512 (44 bytes a cell) against 65 + 46 + 20 for residual, store and clearing apart.
template <typename T>
__global__ void __launch_bounds__(DT) k_gauss(Params P, int k0r, FieldsT<T> f, double *rho, const double *ion,
                                              double *rprev, int64_t dk, int have, int band, double *out) {
    __shared__ double s[3][DT / 64];
    double v[3] = {0, 0, 0};
    const int c = (int)blockIdx.x * DT + (int)threadIdx.x;
    if (c < P.plane) {
        const int j = c / P.nx, i = c - j * P.nx;
        const int64_t di = i == 0 ? P.nx - 1 : -1, dj = j == 0 ? (int64_t)P.nx * (P.ny - 1) : -(int64_t)P.nx;
        for (int p = (int)blockIdx.y; p < P.nz; p += (int)gridDim.y) {
            const int l = p < k0r ? p - k0r + P.nz : p - k0r, pm = p == 0 ? P.nz - 1 : p - 1;
            const int64_t o = (int64_t)p * P.plane + c;
            double rv = 0.0;
            if (l >= band && l < P.nz - band) {
                const double dv = ((double)f.E[0][o] - (double)f.E[0][o + di]) +
                                  ((double)f.E[1][o] - (double)f.E[1][o + dj]) +
                                  ((double)f.E[2][o] - (double)f.E[2][(int64_t)pm * P.plane + c]);
                const double rh = rho[o] + ion[l];
                rv = dv - rh;
                v[0] = v[0] < fabs(rv) ? fabs(rv) : v[0];
                v[1] = v[1] < fabs(rh) ? fabs(rh) : v[1];
                const int64_t lp = (int64_t)l + dk;  // same absolute plane in the previous call
                if (have && lp >= band && lp < P.nz - band) {
                    const double dr = fabs(rv - rprev[o]);
                    v[2] = v[2] < dr ? dr : v[2];
                }
            }
            rprev[o] = rv;
            rho[o] = 0.0;
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double t = v[k];
        for (int h = 32; h > 0; h >>= 1) {
            const double q = __shfl_down(t, h);
            t = t < q ? q : t;
        }
        if ((threadIdx.x & 63) == 0) s[k][threadIdx.x >> 6] = t;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = s[threadIdx.x][0];
        for (int w = 1; w < DT / 64; ++w) t = t < s[threadIdx.x][w] ? s[threadIdx.x][w] : t;
        out[3 * ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) + threadIdx.x] = t;
    }
}

// The nv <= 16 values of `rows` partials (part[row nv + k]) reduced to res[0 .. nv) in a fixed order by
// one workgroup: wave k takes value k, its lanes the rows lane, lane + 64, ..., then a fixed tree.  OP 0
// sums, OP 1 takes the maximum with 0.
template <int OP> __global__ void __launch_bounds__(1024) k_reduce_rows(const double *part, int64_t rows, int nv,
                                                                        double *res) {
    const int k = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (k >= nv) return;
    double t = 0.0;
    for (int64_t r = lane; r < rows; r += 64) {
        const double v = part[r * nv + k];
        t = OP == 0 ? t + v : (t < v ? v : t);
    }
    for (int h = 32; h > 0; h >>= 1) {
        const double v = __shfl_down(t, h);
        t = OP == 0 ? t + v : (t < v ? v : t);
    }
    if (lane == 0) res[k] = t;
}

static void reduce_rows(Ctx &c, const double *part, int64_t rows, int nv, int op, double *res) {
    if (op == 0)
        hipLaunchKernelGGL(k_reduce_rows<0>, dim3(1), dim3(64 * nv), 0, c.st, part, rows, nv, res);
    else
        hipLaunchKernelGGL(k_reduce_rows<1>, dim3(1), dim3(64 * nv), 0, c.st, part, rows, nv, res);
}

// lab-frame probe over the live FP64 beam slots: each block's five sums added to acc
__global__ void __launch_bounds__(DT) k_probe64(Params P, Part64 p, int64_t n, double t1, double T, double k,
                                                double *acc) {
    __shared__ double s[5][DT];
    double v[5] = {0, 0, 0, 0, 0};
    for (int64_t q = (int64_t)blockIdx.x * DT + threadIdx.x; q < n; q += (int64_t)gridDim.x * DT)
        if (p.alive[q]) probe_particle(P, p.z[q], p.ux[q], p.uy[q], p.uz[q], p.w[q], t1, T, k, v);
    for (int j = 0; j < 5; ++j) s[j][threadIdx.x] = v[j];
    __syncthreads();
    for (int h = DT / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h)
            for (int j = 0; j < 5; ++j) s[j][threadIdx.x] += s[j][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int j = 0; j < 5; ++j) atomicAdd(&acc[j], s[j][0]);
}

// ---------------------------------------------------------------- lab frame (section 2)
__global__ void __launch_bounds__(DT) k_lab64(Params P, Part64 p, int64_t n, double t, double *out) {
    const int64_t q = (int64_t)blockIdx.x * DT + threadIdx.x;
    if (q >= n) return;
    double L[8];
    lab_of(P, t, p.x[q], p.y[q], p.z[q], p.ux[q], p.uy[q], p.uz[q], L);
    for (int k = 0; k < 8; ++k) out[(uint64_t)k * n + q] = L[k];
}

// FP32 mode: in place over the absolute FP64 phase space split_read wrote (rows x y z ux uy uz w)
__global__ void __launch_bounds__(DT) k_lab_inplace(Params P, double *a, int64_t n, double t) {
    const int64_t q = (int64_t)blockIdx.x * DT + threadIdx.x;
    if (q >= n) return;
    double L[8];
    lab_of(P, t, a[q], a[n + q], a[2 * n + q], a[3 * n + q], a[4 * n + q], a[5 * n + q], L);
    for (int k = 0; k < 8; ++k) a[(uint64_t)k * n + q] = L[k];
}

__global__ void k_lab_groups_init(double *out, int ng) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= LAB_GROUP_VALUES * ng) return;
    const int v = k % LAB_GROUP_VALUES;
    out[k] = v == 3 ? INFINITY : (v == 4 ? -INFINITY : 0.0);
}

__global__ void __launch_bounds__(DT) k_lab_groups64(Params P, LabGroupSpec G, Part64 p, int64_t n, double t,
                                                     double *out) {
    __shared__ double tab[LAB_GROUP_VALUES * LAB_GROUPS_MAX];
    const int ng = G.nz * G.nu;
    lab_table_clear(tab, ng);
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * DT; base < n; base += (int64_t)gridDim.x * DT) {
        const int64_t q = std::min<int64_t>(base + threadIdx.x, n - 1);
        const bool in = base + threadIdx.x < n && p.alive[q];
        lab_group_add_wave(tab, G, P, t, in, p.x[q], p.y[q], p.z[q], p.ux[q], p.uy[q], p.uz[q], p.w[q]);
    }
    __syncthreads();
    lab_table_flush(tab, ng, out);
}

void lab_groups_clear(double *out, int ng, hipStream_t st) {
    hipLaunchKernelGGL(k_lab_groups_init, dim3(nblocks(LAB_GROUP_VALUES * ng, DT)), dim3(DT), 0, st, out, ng);
}

pic_status lab_groups(Ctx &c, const LabGroupSpec &G, double *out) {
    const int ng = G.nz * G.nu;
    const double t = (double)c.step * c.P.dt;
    if (c.precision == PIC_FP64_PLAIN) {
        lab_groups_clear(out, ng, c.st);
        if (c.nb_slots)
            hipLaunchKernelGGL(k_lab_groups64, dim3(std::min(nblocks(c.nb_slots, DT), 1024)), dim3(DT), 0, c.st, c.P,
                               G, c.b64, c.nb_slots, t, out);
    } else {
        split_lab_groups(c, G, t, out);
    }
    PIC_HIP(c, hipStreamSynchronize(c.st));
    return PIC_OK;
}

pic_status lab_beam(Ctx &c, double *out, int64_t *n) {
    const double t = (double)c.step * c.P.dt;
    if (c.precision == PIC_FP64_PLAIN) {
        *n = c.nb_slots;
        if (out && c.nb_slots)
            hipLaunchKernelGGL(k_lab64, dim3(nblocks(c.nb_slots, DT)), dim3(DT), 0, c.st, c.P, c.b64, c.nb_slots, t,
                               out);
    } else {
        split_read(c, 0, nullptr, nullptr, n);
        if (out && *n) {
            split_read(c, 0, out, nullptr, n);
            hipLaunchKernelGGL(k_lab_inplace, dim3(nblocks(*n, DT)), dim3(DT), 0, c.st, c.P, out, *n, t);
        }
    }
    PIC_HIP(c, hipStreamSynchronize(c.st));
    return PIC_OK;
}

// after a step (c.step, c.k0 already advanced): sample the beam particles whose lab time passed the probe's
void probe_step(Ctx &c) {
    const double t1 = (double)c.step * c.P.dt;
    if (c.precision == PIC_FP64_PLAIN) {
        if (c.nb_slots > 0) {
            const int nblk = (int)std::min<int64_t>(nblocks(c.nb_slots, DT), 1024);
            hipLaunchKernelGGL(k_probe64, dim3(nblk), dim3(DT), 0, c.st, c.P, c.b64, c.nb_slots, t1, c.probe_t,
                               c.probe_k, c.probe_acc);
        }
    } else {
        split_probe(c, c.probe_acc);
    }
}

// beam charge on the nodes (ring order), added into rho
void beam_rho(Ctx &c, double *rho) {
    if (c.precision == PIC_FP64_PLAIN)
        rho64(c, rho, 1);
    else
        split_rho(c, rho, 1);
}

// what the caller's reduction buffer has to hold (doubles), by the documented rule of one row of partials
// per 256 particles, FP32 bins or cells; run_diag's sums need far fewer rows
int64_t diag_partials(const Ctx &c, uint32_t mask) {
    const Params &P = c.P;
    const int64_t nb = c.precision == PIC_FP64_PLAIN ? c.nb_slots : c.beam.n_macro;
    int64_t need = 13 * (int64_t)nblocks(std::max<int64_t>(nb, 1), DT);
    if (mask & PIC_DIAG_ENERGY) need = std::max<int64_t>(need, 1024);
    if (P.has_plasma)
        need = std::max<int64_t>(need, 2 * (c.precision == PIC_FP64_PLAIN
                                                ? (int64_t)nblocks(std::max<int64_t>(c.np_slots, 1), DT)
                                                : (int64_t)P.nbins + 1));
    if (mask & PIC_DIAG_GAUSS) need = std::max<int64_t>(need, 3 * (int64_t)nblocks(P.nc, DT));
    return need;
}

pic_status run_diag(Ctx &c, uint32_t mask, double kb, pic_diag_out *o, double *red, int64_t red_cap) {
    memset(o, 0, sizeof *o);
    const Params &P = c.P;
    if (diag_partials(c, mask) > red_cap) {
        c.err = "diagnostics: more partial sums than the reduction buffer holds";
        return PIC_ERANGE;
    }
    o->t = (double)c.step * P.dt;
    o->step = (double)c.step;
    o->k0 = (double)c.k0;
    o->window_beta = c.bw;
    o->window_x = c.win_x0 + c.bw * ((double)c.step * P.dt - c.win_t0);
    o->frac_bits = P.frac_bits;
    const int k0r = (int)(c.k0 % P.nz);
    const bool plain = c.precision == PIC_FP64_PLAIN;
    // every sum's results stay on the device (res) until all are there: one copy, one synchronisation
    enum { R_M1 = 0, R_M2 = 16, R_FIELD = 24, R_PLASMA = 26, R_GAUSS = 28, R_END = 31 };
    static_assert(R_END <= SUM_RESULTS, "results fit");
    double *const res = red, *const part = red + SUM_RESULTS;
    PIC_HIP(c, hipMemsetAsync(res, 0, 8 * SUM_RESULTS, c.st));
    const bool beam = plain ? c.nb_slots > 0 : c.beam.n_macro > 0;
    if (beam) {
        int rows = plain ? sum_rows(c.nb_slots) : 0;
        if (plain)
            hipLaunchKernelGGL(k_mom1, dim3(rows), dim3(DT), 0, c.st, c.b64, c.nb_slots, kb, part);
        else
            rows = split_moments1(c, kb, part);
        reduce_rows(c, part, rows, 13, 0, res + R_M1);
        if (mask & PIC_DIAG_MOMENTS) {
            if (plain)
                hipLaunchKernelGGL(k_mom2, dim3(rows), dim3(DT), 0, c.st, c.b64, c.nb_slots, res + R_M1, part);
            else
                rows = split_moments2(c, res + R_M1, part);
            reduce_rows(c, part, rows, 8, 0, res + R_M2);
        }
    }
    FieldsT<double> f64;
    FieldsT<float> f32;
    for (int k = 0; k < 3; ++k) {
        f64.E[k] = c.E64[k];
        f64.B[k] = c.B64[k];
        f32.E[k] = c.E32[k];
        f32.B[k] = c.B32[k];
    }
    if (mask & PIC_DIAG_ENERGY) {
        const int rows = sum_rows(P.nc);
        if (plain)
            hipLaunchKernelGGL(k_fenergy<double>, dim3(rows), dim3(DT), 0, c.st, f64, P.nc, part);
        else
            hipLaunchKernelGGL(k_fenergy<float>, dim3(rows), dim3(DT), 0, c.st, f32, P.nc, part);
        reduce_rows(c, part, rows, 1, 0, res + R_FIELD);
    }
    if (P.has_plasma && (!plain || c.np_slots > 0)) {  // plasma counts and kinetic energy
        int rows = plain ? sum_rows(c.np_slots) : 0;
        if (plain)
            hipLaunchKernelGGL(k_kin, dim3(rows), dim3(DT), 0, c.st, c.p64, c.np_slots, P.mi, part);
        else
            rows = split_plasma_kinetic(c, part);
        reduce_rows(c, part, rows, 2, 0, res + R_PLASMA);
    }
    if (mask & PIC_DIAG_GAUSS) {
        const int band = 8;
        // scratch: rho in J_x (zero between steps), ion profile in the ion-current buffer (FP32: zero too;
        // FP64: cleared when a step begins)
        double *rho = plain ? c.J64[0] : (double *)c.Ji[0];
        double *ion = plain ? c.jion64 : (double *)c.jioni;
        if (plain)
            rho64(c, rho, 3);
        else
            split_rho(c, rho, 3);
        if (plain) PIC_HIP(c, hipMemsetAsync(ion, 0, 8 * P.nz, c.st));
        if (P.ions && c.sh_hi > c.sh_lo)
            hipLaunchKernelGGL(k_rho_ion, dim3(nblocks(c.sh_hi - c.sh_lo, 128)), dim3(128), 0, c.st, P, c.sh_lo,
                               c.sh_hi - c.sh_lo, o->t, c.k0, ion, !plain);
        launch_neutraliser_rho(c, rho);
        // about 2048 workgroups, never more rows than the buffer of diag_partials() holds
        const int nbx = nblocks(P.plane, DT);
        const int64_t most = std::min<int64_t>(2048, 8 * (int64_t)nblocks(P.nc, DT));
        const dim3 grid(nbx, (unsigned)std::min<int64_t>(P.nz, std::max<int64_t>(1, most / nbx)));
        const int64_t dk = c.k0 - c.rprev_k0;
        if (plain)
            hipLaunchKernelGGL(k_gauss<double>, grid, dim3(DT), 0, c.st, P, k0r, f64, rho, ion, c.rprev, dk,
                               c.have_rprev, band, part);
        else
            hipLaunchKernelGGL(k_gauss<float>, grid, dim3(DT), 0, c.st, P, k0r, f32, rho, ion, c.rprev, dk,
                               c.have_rprev, band, part);
        PIC_HIP(c, hipMemsetAsync(ion, 0, 8 * P.nz, c.st));
        reduce_rows(c, part, (int64_t)grid.x * grid.y, 3, 1, res + R_GAUSS);
    }
    double h[R_END];
    int32_t fl = 0;
    PIC_HIP(c, hipMemcpyAsync(h, res, sizeof h, hipMemcpyDeviceToHost, c.st));
    PIC_HIP(c, hipMemcpyAsync(&fl, c.dflags, 4, hipMemcpyDeviceToHost, c.st));
    hipError_t e = hipStreamSynchronize(c.st);
    if (e != hipSuccess) return hip_check(c, e, "diag");
    o->error_flags = fl;
    const double *m1 = h + R_M1, *m2 = h + R_M2, W = m1[1];
    o->n_beam = m1[0];
    o->beam_lost = (double)c.beam.n_macro - m1[0];
    o->wsum = W;
    if (W > 0) {
        for (int k = 0; k < 3; ++k) {
            o->mean[k] = m1[2 + k] / W;
            o->umean[k] = m1[5 + k] / W;
        }
        o->b1_re = m1[8] / W;
        o->b1_im = m1[9] / W;
        o->b2_re = m1[10] / W;
        o->b2_im = m1[11] / W;
        o->b1_abs = sqrt(m1[8] * m1[8] + m1[9] * m1[9]) / W;
        o->b2_abs = sqrt(m1[10] * m1[10] + m1[11] * m1[11]) / W;
        o->kin_beam = m1[12];
        if (mask & PIC_DIAG_MOMENTS) {
            for (int k = 0; k < 3; ++k) {
                o->sigma[k] = sqrt(m2[k] / W);
                o->usigma[k] = sqrt(m2[3 + k] / W);
            }
            for (int k = 0; k < 2; ++k) {
                double a = m2[k] / W, b = m2[3 + k] / W, x = m2[6 + k] / W;
                o->emit[k] = sqrt(std::max(0.0, a * b - x * x));
            }
        }
    }
    if (mask & PIC_DIAG_ENERGY) o->field_energy = 0.5 * h[R_FIELD];
    o->n_plasma = h[R_PLASMA];
    o->kin_plasma = h[R_PLASMA + 1];
    if (mask & PIC_DIAG_GAUSS) {
        o->gauss_max = h[R_GAUSS];
        o->rho_max = h[R_GAUSS + 1];
        o->gauss_drift = c.have_rprev ? h[R_GAUSS + 2] : -1.0;
        c.have_rprev = 1;
        c.rprev_k0 = c.k0;
    }
    return PIC_OK;
}

// ---------------------------------------------------------------- allocation-free diagnostics
// The reduction buffer of pic_diag_static: a file-scope device array, one per
// GPU the library runs on, held until the process ends.  Host code reaches it
// only through the address hipGetSymbolAddress returns for each device.
static __device__ __align__(256) double scratch[DIAG_STATIC_DOUBLES];
static std::mutex g_scratch_mu;
static double *g_scratch[64];

pic_status static_scratch_setup(Ctx &c) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (c.device < 0 || c.device >= 64) {
        c.err = "static scratch: device ordinal beyond 63";
        return PIC_EDEVICE;
    }
    if (g_scratch[c.device]) return PIC_OK;
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_check(c, e != hipSuccess ? e : hipErrorInvalidSymbol, "static scratch");
    g_scratch[c.device] = (double *)p;
    return PIC_OK;
}

double *static_scratch(int device) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return device >= 0 && device < 64 ? g_scratch[device] : nullptr;
}

}  // namespace pic
