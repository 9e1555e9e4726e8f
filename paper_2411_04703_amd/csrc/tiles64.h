// tiles64.h -- cell tiles of the FP64 particle kernels: per-call lists of the
// live particles of each tile, and the geometry of a tile's LDS boxes.
//
// FP64 particles keep their slots (the adjoint follows them, output is in slot
// order), so a kernel that works tile by tile reads its particles through a
// list of slot numbers.  The list is built afresh for every use (count, scan,
// scatter: 0.34 ms for 21 M particles against 2.1 ms for the step that uses it);
// nothing of it is kept from one call to the next.
#pragma once
#include "pic_internal.h"

namespace pic {

constexpr int QPAD64 = 64;  // int32 stride of the queue counters: a 256-byte block each

// one species as the tile kernels address it: arrays d = 0..6 (x y z ux uy uz w) of `cap` doubles
// from `x` on, then the alive flags (carve64)
struct Species64 {
    double *x;
    int64_t cap, n;
    __host__ __device__ int32_t *alive() const { return (int32_t *)(x + 7 * cap); }
};

constexpr uint32_t NO_BIN = 0xffffffffu;

// Tile edges.  8 x 8 x 4: fields (41 KB) and currents (33 KB) of two workgroups fit a CU's LDS,
// which 8 x 8 x 8 would fill with one; 8 x 1 x 16 on two-dimensional x-z grids, where 8 rows along y would all be row 0.
template <int TX_, int TY_, int TZ_> struct Geom64 {
    static constexpr int TX = TX_, TY = TY_, TZ = TZ_;
    // component k of E (0-2) or B (3-5): half-integer sites along these axes
    static constexpr bool half(int k, int d) { return k < 3 ? k == d : k - 3 != d; }
    // field boxes, one per component: (half-)nodes -1 .. T + 1 along every axis
    static constexpr int FX = TX + 3, FY = TY + 3, FZ = TZ + 3, NB = FX * FY * FZ, NF = 6 * NB;
    // current box of component k: nodes -2 .. T + 1 along its axis, -2 .. T + 2 across
    static constexpr int jx(int k) { return TX + (k == 0 ? 4 : 5); }
    static constexpr int jy(int k) { return TY + (k == 1 ? 4 : 5); }
    static constexpr int jz(int k) { return TZ + (k == 2 ? 4 : 5); }
    static constexpr int jsize(int k) { return jx(k) * jy(k) * jz(k); }
    static constexpr int jofs(int k) { return k == 0 ? 0 : jofs(k - 1) + jsize(k - 1); }
    static constexpr int NJ = jofs(2) + jsize(2);
};
using Geom3D = Geom64<8, 8, 4>;
using Geom2D = Geom64<8, 1, 16>;

// one work item as a kernel sees it (wave-uniform)
struct Item64 {
    uint32_t begin, end;
    int t0x, t0y, t0z;
};

// The item queues: eight contiguous ranges of the item list, one per XCD (workgroups are dispatched
// round-robin over the XCDs), so that neighbouring tiles share an L2.  A workgroup's first item is
// its own by number (no counter: on small grids it is the only one), the following ones come from
// its range's counter, then from the other ranges'.  Used by one thread of the workgroup: claim()
// starts the counter's round trip, resolve() returns the item, -1 when all are taken.  Before it
// takes from another range it reads all eight counters at once, rather than visit eight empty
// queues one atomic after the other.
struct ItemQueue64 {
    int q, got;
    __device__ static int lo(int n, int q) { return (int)((int64_t)n * q / 8); }
    __device__ int first(const TileList &T) {
        q = (int)(blockIdx.x & 7);
        got = (int)(blockIdx.x >> 3);
        return resolve(T);
    }
    __device__ void claim(const TileList &T) { got = atomicAdd(&T.qnext[q * QPAD64], 1); }
    __device__ int resolve(const TileList &T) {
        const int n = *T.nitems;
        for (;;) {
            const int k = lo(n, q) + got;
            if (k < lo(n, q + 1)) return k;
            int next[8], at = -1;
#pragma unroll
            for (int i = 0; i < 8; ++i)
                next[i] = __hip_atomic_load(&T.qnext[i * QPAD64], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int i = 7; i >= 0; --i) {  // the next range with something left, from this one on
                const int c = (q + i) & 7;
                int left = 0;
#pragma unroll
                for (int m = 0; m < 8; ++m) left = m == c ? lo(n, m + 1) - lo(n, m) - next[m] : left;
                if (left > 0) at = c;
            }
            if (at < 0) return -1;
            q = at;  // a failed claim leaves that counter past its range's end: it is not chosen again
            claim(T);
        }
    }
};

__device__ inline Item64 item64(const TileList &T, int item, int tx, int ty, int tz) {
    Item64 I;
    const int4 it = T.items[item];
    const int bin = __builtin_amdgcn_readfirstlane(it.x);
    I.begin = (uint32_t)__builtin_amdgcn_readfirstlane(it.y);
    I.end = (uint32_t)__builtin_amdgcn_readfirstlane(it.z);
    I.t0x = (bin % T.ntx) * tx;
    I.t0y = ((bin / T.ntx) % T.nty) * ty;
    I.t0z = (bin / (T.ntx * T.nty)) * tz;
    return I;
}

// linear index of node (i, j) of ring plane p; tile boxes reach a few nodes beyond the grid, on the
// smallest grids more than a period
__device__ inline int64_t cell_near(const Params &P, int i, int j, int p) {
    i = i < 0 ? i + P.nx : (i >= P.nx ? i - P.nx : i);
    j = j < 0 ? j + P.ny : (j >= P.ny ? j - P.ny : j);
    if ((unsigned)i >= (unsigned)P.nx) i = wrapi(i, P.nx);
    if ((unsigned)j >= (unsigned)P.ny) j = wrapi(j, P.ny);
    return (int64_t)i + (int64_t)P.nx * ((int64_t)j + (int64_t)P.ny * p);
}

// Window and grid bounds as doubles.  Kernel arguments, so that they stay in scalar registers:
// converted in the kernel they are vector registers, kept (or spilled) across its loops.
struct Bounds64 {
    double k0, nx, ny, nz;  // window origin and extents
    double lo, hi;          // active band after the step's shift: [k0n + 3, k0n + nz - 4)
    __host__ Bounds64(const Params &P, int64_t k0_, int64_t k0n)
        : k0((double)k0_), nx(P.nx), ny(P.ny), nz(P.nz), lo((double)(k0n + 3)), hi((double)(k0n + P.nz - 4)) {}
};

// cell (i, j in the grid, l logical) of an absolute position; false outside the window or not finite
__device__ inline bool locate64(const Params &P, const Bounds64 &W, double x, double y, double z, int &i, int &j,
                                int &l) {
    const double zl = floor(z) - W.k0;
    if (!(zl >= 0.0 && zl < W.nz) || !isfinite(x) || !isfinite(y)) return false;
    l = (int)zl;
    i = (int)floor(x);
    j = (int)floor(y);
    if (i < 0 || i >= P.nx) i = wrapi(i, P.nx);
    if (j < 0 || j >= P.ny) j = wrapi(j, P.ny);
    return true;
}

// The same for a listed particle, whose place the list kernel has checked: relative to its tile, and
// without a branch (the coordinate wraps on the way out of a step, so it lies in the grid but for
// positions a caller wrote).
__device__ inline void cell_in_tile64(const Params &P, const Bounds64 &W, const Item64 &I, const double fl[3],
                                      int c0[3]) {
    int i = (int)fl[0], j = (int)fl[1];
    if (__any((unsigned)i >= (unsigned)P.nx || (unsigned)j >= (unsigned)P.ny)) {
        i = wrapi(i, P.nx);
        j = wrapi(j, P.ny);
    }
    c0[0] = i - I.t0x;
    c0[1] = j - I.t0y;
    c0[2] = (int)(fl[2] - W.k0) - I.t0z;
}

// Weights of the three integer nodes around a coordinate: n the nearest node's distance above the
// cell's lower node (0 or 1), w the weights of n - 1, n, n + 1.
__device__ inline int near_int(double x, double fl, double w[3]) {
    const double n = floor(x + 0.5);
    weights3<double>(x - n, w);
    return (int)(n - fl);
}

// derivatives of weights3 with respect to the offset d
__device__ inline void dweights3(double d, double w[3]) {
    w[0] = d - 0.5;
    w[1] = -2.0 * d;
    w[2] = d + 0.5;
}

// three weights in a four-node window, one node up where `up`
__device__ inline void window4(const double w[3], bool up, double o[4]) {
    o[0] = up ? 0.0 : w[0];
    o[1] = up ? w[0] : w[1];
    o[2] = up ? w[1] : w[2];
    o[3] = up ? w[2] : 0.0;
}

// one component at a particle from its tile's box
template <class G, int K> __device__ inline double gather_lds(const double *F, const double wi[3][3],
                                                              const double wh[3][3], const int bi[3], const int bh[3]) {
    constexpr bool hx = G::half(K, 0), hy = G::half(K, 1), hz = G::half(K, 2);
    const double *wx = hx ? wh[0] : wi[0], *wy = hy ? wh[1] : wi[1], *wz = hz ? wh[2] : wi[2];
    constexpr int SY = G::FX, SZ = G::FX * G::FY;
    const double *f = F + K * G::NB + (hx ? bh[0] : bi[0]) + SY * (hy ? bh[1] : bi[1]) + SZ * (hz ? bh[2] : bi[2]);
    double v = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double py = 0.0;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const double *r = f + SY * b + SZ * c;
            py = fma(wy[b], fma(wx[2], r[2], fma(wx[1], r[1], wx[0] * r[0])), py);
        }
        v = fma(wz[c], py, v);
    }
    // the sum is taken here: left to itself the compiler sinks the arithmetic of all six components
    // below their 162 reads and spills what they returned
    asm volatile("" : "+v"(v));
    __builtin_amdgcn_sched_barrier(0);
    return v;
}

// Hides v's value from the optimiser, so that what is computed from it is not hoisted out of the
// work-item loop and kept live (or spilled) across it.
__device__ inline void opaque64(int &v) { asm volatile("" : "+v"(v)); }

// The six fields of the tile into LDS (nodes outside the window: 0, never gathered with a nonzero
// weight).  A thread takes whole nodes: one address for six loads.  load() leaves all of a thread's
// loads in flight together, store() writes what came.
template <class G, int NT> struct Stage64 {
    static constexpr int R = (G::NB + NT - 1) / NT;
    double v[R][6];
    __device__ void load(const Params &P, int k0r, const Item64 &I, const FieldsT<double> &f) {
        const double *src[6] = {f.E[0], f.E[1], f.E[2], f.B[0], f.B[1], f.B[2]};
        int e0 = threadIdx.x;
        opaque64(e0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = e0 + r * NT, y = e / G::FX, a = e - y * G::FX, c = y / G::FY, b = y - c * G::FY;
            const int l = I.t0z - 1 + c;
            const bool in = e < G::NB && l >= 0 && l < P.nz;
            const int64_t o = in ? cell_near(P, I.t0x - 1 + a, I.t0y - 1 + b, ring_plane(l, k0r, P.nz)) : 0;
#pragma unroll
            for (int k = 0; k < 6; ++k) v[r][k] = in ? src[k][o] : 0.0;
        }
    }
    __device__ void store(double *F) const {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int e = threadIdx.x + r * NT;
            if (e < G::NB)
#pragma unroll
                for (int k = 0; k < 6; ++k) F[k * G::NB + e] = v[r][k];
        }
    }
};

// a particle as loaded, and its number in the list
struct Raw64 {
    double X[3], U[3], w;
    uint32_t id;
};

// where a particle's x is (the other arrays follow `cap` doubles apart), and its alive flag
__device__ inline double *slot64(const Species64 &sb, const Species64 &sp, uint32_t id, int64_t &cap, int32_t *&alive) {
    const bool beam = id < (uint32_t)sb.n;
    const uint32_t s = beam ? id : id - (uint32_t)sb.n;
    double *const x0 = beam ? sb.x : sp.x;
    cap = beam ? sb.cap : sp.cap;
    alive = (int32_t *)(x0 + 7 * cap) + s;
    return x0 + s;
}

__device__ inline Raw64 load_raw64(const Species64 &sb, const Species64 &sp, uint32_t id) {
    Raw64 r;
    int64_t cap;
    int32_t *alive;
    const double *at = slot64(sb, sp, id, cap, alive);
    r.id = id;
    for (int d = 0; d < 3; ++d) {
        r.X[d] = at[d * cap];
        r.U[d] = at[(3 + d) * cap];
    }
    r.w = at[6 * cap];
    return r;
}

// host side (k_tiles64.hip)
bool tiles64_flat(const Params &P);  // two-dimensional tiles?
// lists of the live particles of beam and plasma (either may be empty) for the window of c.k0
// and for a kernel of `grid` workgroups (a multiple of 8) that takes their items from ItemQueue64;
// take_out: live particles that no tile can hold are marked dead (the step), else only left out
void tiles64_build(Ctx &c, Species64 b, Species64 p, int grid, bool take_out);

}  // namespace pic
