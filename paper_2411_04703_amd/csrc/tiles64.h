// tiles64.h -- cell tiles of the FP64 particle kernels: per-call lists of the
// live particles of each tile, and the geometry of a tile's LDS boxes.
//
// FP64 particles keep their slots (the adjoint follows them, output is in slot
// order), so a kernel that works tile by tile reads its particles through a
// list of slot numbers.  The list is built afresh for every use (count, scan,
// scatter: 0.37 ms for 21 M particles against 2.1 ms for the step that uses it);
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

// host side (k_tiles64.hip)
bool tiles64_flat(const Params &P);  // two-dimensional tiles?
// lists of the live particles of beam and plasma (either may be empty) for the window of c.k0
// and for a kernel of `grid` workgroups (a multiple of 8) that takes their items from ItemQueue64
void tiles64_build(Ctx &c, Species64 b, Species64 p, int grid);

}  // namespace pic
