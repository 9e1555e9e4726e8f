// k_plain64.hip -- FP64 particles: beam sampling, plasma lattice sheets and
// compaction.  Absolute FP64 positions in slots; the step works on them tile by
// tile (k_tiles64.hip).
#include "pic_internal.h"

namespace pic {

// ---------------------------------------------------------------- beam init
// Lab-frame Gaussian at lab time 0 around the box axis (section 3: beam defined
// in the lab), per-particle Lorentz transform of the event and the momentum
// (Eq. Lor1, Lor2), then a straight drift to t' = 0 (the event of particle j
// happens at t'_j = -gR bR z_j).  FP64 throughout.
__global__ void k_beam_init64(Params P, const double *g, int64_t n, double sx, double sy, double szl, double sux,
                              double suy, double gB, double es, Part64 p, double *part) {
    __shared__ double red[2][256];
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double cnt = 0.0, vzs = 0.0;
    if (q < n) {
        double x = 0.5 * P.nx + sx * g[q];
        double y = 0.5 * P.ny + sy * g[n + q];
        double zl = szl * g[2 * n + q];
        double ux = sux * g[3 * n + q], uy = suy * g[4 * n + q];
        double gam = gB * (1.0 + es * g[5 * n + q]);
        double uz = sqrt(gam * gam - 1.0 - ux * ux - uy * uy);
        double glab = sqrt(1.0 + ux * ux + uy * uy + uz * uz);
        double zb = P.gR * zl;
        double tb = -P.gR * P.bR * zl;
        double uzb = P.gR * (uz - P.bR * glab);
        double gb = sqrt(1.0 + ux * ux + uy * uy + uzb * uzb);
        double drift = -tb;
        x = x + ux / gb * drift;
        y = y + uy / gb * drift;
        double z = zb + uzb / gb * drift + P.zoff;
        x = fmod(x, (double)P.nx);
        if (x < 0) x += P.nx;
        y = fmod(y, (double)P.ny);
        if (y < 0) y += P.ny;
        p.x[q] = x;
        p.y[q] = y;
        p.z[q] = z;
        p.ux[q] = ux;
        p.uy[q] = uy;
        p.uz[q] = uzb;
        p.w[q] = P.wbeam;
        int al = (z >= 3.0 && z < (double)(P.nz - 4));
        p.alive[q] = al;
        if (al) {
            cnt = 1.0;
            vzs = uzb / gb;
        }
    }
    red[0][threadIdx.x] = cnt;
    red[1][threadIdx.x] = vzs;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = red[0][0];
        part[2 * blockIdx.x + 1] = red[1][0];
    }
}

void launch_beam_init64(const Params &P, const double *normals, int64_t n, const double sig[5], double gB, double es,
                        Part64 p, double *partials, int nblk, hipStream_t st) {
    hipLaunchKernelGGL(k_beam_init64, dim3(nblk), dim3(256), 0, st, P, normals, n, sig[0], sig[1], sig[2], sig[3],
                       sig[4], gB, es, p, partials);
}

// ---------------------------------------------------------------- plasma sheets
// Cold lattice electrons at rest in the lab: boosted u = -gR bR zhat, boosted
// density gR n (Eq. Nnormi).  Sheet l holds nx ny ppx ppy particles in the
// order (j, b, i, a), x = i + (a + 1/2)/ppx, y = j + (b + 1/2)/ppy; with
// mobile ions, as many ions follow in the same order, with the same velocity
// and the weight negated (the charge sign: the deposit and the charge density
// take -w, and the push selects q/m = +1/M by it).
__global__ void k_inject64(Params P, int64_t l0, int64_t total, double t, Part64 p, int64_t slot0) {
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= total) return;
    const int64_t per = sheet_particles(P), pe = (int64_t)P.plane * P.ppx * P.ppy;
    int64_t l = l0 + q / per;
    int64_t r = q % per;
    const bool ion = r >= pe;
    if (ion) r -= pe;
    int a = (int)(r % P.ppx);
    r /= P.ppx;
    int i = (int)(r % P.nx);
    r /= P.nx;
    int b = (int)(r % P.ppy);
    int j = (int)(r / P.ppy);
    int64_t s = slot0 + q;
    p.x[s] = i + (a + 0.5) / P.ppx;
    p.y[s] = j + (b + 0.5) / P.ppy;
    p.z[s] = sheet_z(l, P.ppz, P.bR, t);
    p.ux[s] = 0.0;
    p.uy[s] = 0.0;
    p.uz[s] = -P.uR;
    p.w[s] = ion ? -sheet_weight(P, l) : sheet_weight(P, l);
    p.alive[s] = 1;
}

void launch_inject64(const Params &P, int64_t l0, int64_t nsheets, double t, Part64 p, int64_t slot0,
                     hipStream_t st) {
    int64_t total = nsheets * sheet_particles(P);
    if (total <= 0) return;
    hipLaunchKernelGGL(k_inject64, dim3(nblocks(total, 256)), dim3(256), 0, st, P, l0, total, t, p, slot0);
}

// ---------------------------------------------------------------- compaction
// Stable removal of dead slots (forward mode only): block-local ranks plus a
// host-side exclusive scan of the block counts, then a scatter.
__global__ void k_count_alive(const int32_t *alive, int64_t n, int32_t *bc) {
    __shared__ int32_t s[256];
    int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    s[threadIdx.x] = (q < n && alive[q]) ? 1 : 0;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) bc[blockIdx.x] = s[0];
}

__global__ void k_scatter_alive(Part64 src, Part64 dst, int64_t n, const int64_t *boff) {
    __shared__ int32_t s[256];
    int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int al = (q < n && src.alive[q]) ? 1 : 0;
    s[threadIdx.x] = al;
    __syncthreads();
    // inclusive scan (Hillis-Steele) inside the block
    for (int k = 1; k < 256; k <<= 1) {
        int v = (int)threadIdx.x >= k ? s[threadIdx.x - k] : 0;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    if (!al) return;
    int64_t o = boff[blockIdx.x] + s[threadIdx.x] - 1;
    dst.x[o] = src.x[q];
    dst.y[o] = src.y[q];
    dst.z[o] = src.z[q];
    dst.ux[o] = src.ux[q];
    dst.uy[o] = src.uy[q];
    dst.uz[o] = src.uz[q];
    dst.w[o] = src.w[q];
    dst.alive[o] = 1;
}

int64_t compact64(Ctx &c, Part64 src, Part64 dst, int64_t n) {
    if (n <= 0) return 0;
    int nb = nblocks(n, 256);
    int32_t *bc = (int32_t *)c.i64scratch;  // reuse: nb int32 then nb+1 int64 offsets
    int64_t *boff = c.i64scratch + (nb + 1) / 2 + 1;
    hipLaunchKernelGGL(k_count_alive, dim3(nb), dim3(256), 0, c.st, src.alive, n, bc);
    std::string tmp;
    int32_t *h = (int32_t *)malloc(sizeof(int32_t) * nb);
    int64_t *ho = (int64_t *)malloc(sizeof(int64_t) * (nb + 1));
    (void)hipMemcpyAsync(h, bc, sizeof(int32_t) * nb, hipMemcpyDeviceToHost, c.st);
    (void)hipStreamSynchronize(c.st);
    ho[0] = 0;
    for (int b = 0; b < nb; ++b) ho[b + 1] = ho[b] + h[b];
    (void)hipMemcpyAsync(boff, ho, sizeof(int64_t) * (nb + 1), hipMemcpyHostToDevice, c.st);
    hipLaunchKernelGGL(k_scatter_alive, dim3(nb), dim3(256), 0, c.st, src, dst, n, boff);
    (void)hipStreamSynchronize(c.st);
    int64_t tot = ho[nb];
    free(h);
    free(ho);
    return tot;
}

}  // namespace pic
