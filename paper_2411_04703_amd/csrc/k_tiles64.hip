// k_tiles64.hip -- FP64 particle step on cell tiles: per-call particle lists of
// every tile, then gather, push, move and deposit with the tile's fields and
// currents in LDS.  FP64 throughout (absolute positions, FP64 sums).
#include <algorithm>

#include "tiles64.h"

namespace pic {

constexpr int LT = 256;   // threads of the list kernels
constexpr int ST64 = 512; // threads of the step kernel

// ---------------------------------------------------------------- lists
bool tiles64_flat(const Params &P) { return P.ny == 1; }

void tiles64_dims(const Params &P, int &ntx, int &nty, int &ntz) {
    const bool flat = tiles64_flat(P);
    const int tx = flat ? Geom2D::TX : Geom3D::TX, ty = flat ? Geom2D::TY : Geom3D::TY,
              tz = flat ? Geom2D::TZ : Geom3D::TZ;
    ntx = (P.nx + tx - 1) / tx;
    nty = (P.ny + ty - 1) / ty;
    ntz = (P.nz + tz - 1) / tz;
}

// Particles per item: few flushes of a crowded tile in large runs, half a workgroup in small ones,
// where the items would leave compute units idle (110 k particles: 43 us a step at 256, 48 at 512).
constexpr int CHUNK_MIN = ST64 / 2;
static int chunk_of(int64_t slots) {
    return slots >= (int64_t)1 << 22 ? 4 * ST64 : (slots >= (int64_t)1 << 18 ? ST64 : CHUNK_MIN);
}

// bins that a block of the scan takes at a time, and how many one block goes through alone (k_tile_scan)
constexpr int SCAN_V = 4, SCAN_BINS = 1024 * SCAN_V, FEW_BINS = 4 * SCAN_BINS;

static uint64_t al(uint64_t v) { return (v + 255) & ~(uint64_t)255; }

static int64_t bins_of(const Params &P) {
    int a, b, c;
    tiles64_dims(P, a, b, c);
    return (int64_t)a * b * c;
}

uint64_t tiles64_bytes(const Params &P, int64_t slots) {
    const uint64_t nb = (uint64_t)bins_of(P), n = (uint64_t)std::max<int64_t>(slots, 1);
    return al(4 * nb) + al(16 * (nb + n / CHUNK_MIN + 16)) + al(8 * (nb / SCAN_BINS + 1)) + 256 * 9;
}

uint64_t tiles64_count_bytes(const Params &P) { return 4 * (uint64_t)bins_of(P); }

uint64_t tiles64_list_bytes(int64_t slots) { return 3 * al(4 * (uint64_t)std::max<int64_t>(slots, 1)); }

// the arrays with an entry per slot, in `room`
static void place_lists(TileList &T, char *room, int64_t slots) {
    const uint64_t n = al(4 * (uint64_t)std::max<int64_t>(slots, 1));
    T.key = (uint32_t *)room;
    T.rank = (uint32_t *)(room + n);
    T.list = (uint32_t *)(room + 2 * n);
}

// Bin of every live particle and its place there.  A block counts its particles in an LDS hash
// table of bins and adds each bin's count to the global one once: a beam's particles come in no
// order and crowd a few hundred bins, whose counters took 0.60 ms for 4.2 M particles when every
// wave added to them (0.07 ms with the table).  A particle that finds no slot in 16 probes counts
// globally.  A live particle that is not finite or outside the window (positions a caller wrote) is not
// listed; the step, which passes its flags, takes it out, the other users leave the state as it is.
constexpr int CT = 1024, HB = 13;
template <int PPT>
__global__ void __launch_bounds__(CT) k_tile_count(Params P, Bounds64 W, Species64 b, Species64 p, int lgx, int lgy,
                                                   int lgz, TileList T, int32_t *flags) {
    __shared__ uint32_t hkey[1 << HB], hcnt[1 << HB];
    for (int e = threadIdx.x; e < 1 << HB; e += CT) {
        hkey[e] = NO_BIN;
        hcnt[e] = 0;
    }
    __syncthreads();
    const int64_t q0 = (int64_t)blockIdx.x * (CT * PPT) + threadIdx.x;
    uint32_t key[PPT], place[PPT];
    int slot[PPT];
#pragma unroll
    for (int v = 0; v < PPT; ++v) {
        const int64_t q = q0 + v * CT;
        const bool beam = q < b.n;
        const int64_t s = beam ? q : q - b.n;
        const Species64 S = beam ? b : p;
        key[v] = NO_BIN;
        if (q < b.n + p.n && S.alive()[s]) {
            const double x = S.x[s], y = S.x[S.cap + s], z = S.x[2 * S.cap + s];
            int i, j, l;
            if (locate64(P, W, x, y, z, i, j, l)) {
                key[v] = (uint32_t)((i >> lgx) + T.ntx * ((j >> lgy) + T.nty * (l >> lgz)));
            } else if (flags) {
                S.alive()[s] = 0;
                if (!(isfinite(x) && isfinite(y) && isfinite(z))) atomicOr(flags, DFLAG_NONFINITE);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < PPT; ++v) {
        slot[v] = -1;
        place[v] = 0;
        if (key[v] == NO_BIN) continue;
        uint32_t h = (key[v] * 2654435761u) >> (32 - HB);
        for (int probe = 0; probe < 16; ++probe, h = (h + 1) & ((1 << HB) - 1)) {
            uint32_t have = hkey[h];
            if (have == NO_BIN) have = atomicCAS(&hkey[h], NO_BIN, key[v]);
            if (have == NO_BIN || have == key[v]) {
                slot[v] = (int)h;
                break;
            }
        }
        place[v] = slot[v] >= 0 ? atomicAdd(&hcnt[slot[v]], 1u) : atomicAdd(&T.cnt[key[v]], 1u);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 1 << HB; e += CT) {
        const uint32_t n = hcnt[e];
        if (n) hcnt[e] = atomicAdd(&T.cnt[hkey[e]], n);
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < PPT; ++v) {
        const int64_t q = q0 + v * CT;
        if (q >= b.n + p.n) continue;
        T.key[q] = key[v];
        T.rank[q] = place[v] + (slot[v] >= 0 ? hcnt[slot[v]] : 0u);
    }
}

// First list entry of every bin and the work items; clears the counts.  A block takes SCAN_BINS bins at a
// time.  Up to FEW_BINS bins one block goes through them all; more (a grid of four million cells on, however
// few its particles) get a block each, which starts from the totals that k_tile_totals has left of those
// before it (a step of 256 x 256 x 1024 with 1000 particles: 3.59 ms by one block, 3.39 so).
__global__ void __launch_bounds__(1024) k_tile_totals(TileList T) {
    __shared__ uint32_t sn[16], si[16];
    uint32_t n = 0, it = 0;
    for (int v = 0; v < SCAN_V; ++v) {
        const int bin = (int)blockIdx.x * SCAN_BINS + v * 1024 + (int)threadIdx.x;
        const uint32_t k = bin < T.nbins ? T.cnt[bin] : 0u;
        n += k;
        it += (k + T.chunk - 1) / T.chunk;
    }
    for (int h = 32; h > 0; h >>= 1) {
        n += __shfl_down(n, h);
        it += __shfl_down(it, h);
    }
    if ((threadIdx.x & 63) == 0) {
        sn[threadIdx.x >> 6] = n;
        si[threadIdx.x >> 6] = it;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) {
            n += sn[w];
            it += si[w];
        }
        T.totals[blockIdx.x] = make_uint2(n, it);
    }
}

__global__ void __launch_bounds__(1024) k_tile_scan(TileList T, int per_queue) {
    constexpr int V = SCAN_V;
    __shared__ uint32_t wn[16], wi[16];
    __shared__ uint32_t run_n, run_i;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const bool alone = gridDim.x == 1;
    if (t == 0) run_n = run_i = 0;
    if (t < 8 && blockIdx.x == 0) T.qnext[t * QPAD64] = per_queue;  // the workgroups' first items are taken by number
    __syncthreads();
    if (!alone) {  // what the blocks before this one have
        uint32_t n = 0, it = 0;
        for (int b = t; b < (int)blockIdx.x; b += 1024) {
            const uint2 k = T.totals[b];
            n += k.x;
            it += k.y;
        }
        for (int h = 32; h > 0; h >>= 1) {
            n += __shfl_down(n, h);
            it += __shfl_down(it, h);
        }
        if (lane == 0) {
            atomicAdd(&run_n, n);
            atomicAdd(&run_i, it);
        }
        __syncthreads();
    }
    const int end = alone ? T.nbins : min(T.nbins, ((int)blockIdx.x + 1) * SCAN_BINS);
    for (int base = (int)blockIdx.x * SCAN_BINS; base < end; base += SCAN_BINS) {
        uint32_t n[V], it[V], sn = 0, si = 0;
        for (int v = 0; v < V; ++v) {
            const int bin = base + t * V + v;
            n[v] = bin < T.nbins ? T.cnt[bin] : 0u;
            it[v] = (n[v] + T.chunk - 1) / T.chunk;
            sn += n[v];
            si += it[v];
        }
        uint32_t an = sn, ai = si;  // inclusive scans over the wave, then over the waves
        for (int k = 1; k < 64; k <<= 1) {
            const uint32_t un = __shfl_up(an, k), ui = __shfl_up(ai, k);
            if (lane >= k) {
                an += un;
                ai += ui;
            }
        }
        if (lane == 63) {
            wn[wave] = an;
            wi[wave] = ai;
        }
        __syncthreads();
        uint32_t pn = run_n, pi = run_i;
        for (int w = 0; w < wave; ++w) {
            pn += wn[w];
            pi += wi[w];
        }
        pn += an - sn;
        pi += ai - si;
        for (int v = 0; v < V; ++v) {
            const int bin = base + t * V + v;
            if (bin < T.nbins) {
                T.off[bin] = pn;
                T.cnt[bin] = 0;
                for (uint32_t k = 0; k < it[v]; ++k)
                    T.items[pi + k] = make_int4(bin, (int)(pn + k * T.chunk),
                                                (int)(pn + min(n[v], (k + 1) * (uint32_t)T.chunk)), 0);
            }
            pn += n[v];
            pi += it[v];
        }
        __syncthreads();
        if (t == 1023) {
            run_n = pn;
            run_i = pi;
        }
        __syncthreads();
    }
    if (t == 0 && end == T.nbins) *T.nitems = (int)run_i;
}

__global__ void __launch_bounds__(LT) k_tile_scatter(int64_t n, TileList T) {
    const int64_t q = (int64_t)blockIdx.x * LT + threadIdx.x;
    if (q >= n) return;
    const uint32_t key = T.key[q];
    if (key != NO_BIN) T.list[T.off[key] + T.rank[q]] = (uint32_t)q;
}

void tiles64_build(Ctx &c, Species64 b, Species64 p, int grid, bool take_out) {
    int32_t *const flags = take_out ? c.dflags : nullptr;
    const int64_t n = b.n + p.n;
    const bool flat = tiles64_flat(c.P);
    c.tiles.chunk = chunk_of(n);
    // the compaction's buffer, whichever of the two it is now
    if (!c.tiles.room) place_lists(c.tiles, (char *)c.p64alt.x, c.cap_b + c.cap_p);
    const Bounds64 W(c.P, c.k0, c.k0);
    const int lgx = 3, lgy = flat ? 0 : 3, lgz = flat ? 4 : 2;
    if (n >= (int64_t)1 << 21)  // many particles a thread where there are blocks enough all the same
        hipLaunchKernelGGL(k_tile_count<8>, dim3(nblocks(n, 8 * CT)), dim3(CT), 0, c.st, c.P, W, b, p, lgx, lgy,
                           lgz, c.tiles, flags);
    else if (n > 0)
        hipLaunchKernelGGL(k_tile_count<1>, dim3(nblocks(n, CT)), dim3(CT), 0, c.st, c.P, W, b, p, lgx, lgy, lgz,
                           c.tiles, flags);
    const int blocks = c.tiles.nbins <= FEW_BINS ? 1 : nblocks(c.tiles.nbins, SCAN_BINS);
    if (blocks > 1) hipLaunchKernelGGL(k_tile_totals, dim3(blocks), dim3(1024), 0, c.st, c.tiles);
    hipLaunchKernelGGL(k_tile_scan, dim3(blocks), dim3(1024), 0, c.st, c.tiles, grid / 8);
    if (n > 0) hipLaunchKernelGGL(k_tile_scatter, dim3(nblocks(n, LT)), dim3(LT), 0, c.st, n, c.tiles);
}

// ---------------------------------------------------------------- the step
// current box of component K to the grid, cleared
template <class G, int K> __device__ inline void flush_lds(const Params &P, int k0r, const Item64 &I, double *Js,
                                                           double *J) {
    constexpr int X = G::jx(K), Y = G::jy(K), N = G::jsize(K);
    int e = threadIdx.x;
    opaque64(e);
    for (; e < N; e += ST64) {
        const double v = Js[G::jofs(K) + e];
        if (v == 0.0) continue;
        Js[G::jofs(K) + e] = 0.0;
        const int r = e / X, a = e - r * X, c = r / Y, b = r - c * Y;
        const int l = I.t0z - 2 + c;
        if (l >= 0 && l < P.nz) atomicAdd(&J[cell_near(P, I.t0x - 2 + a, I.t0y - 2 + b, ring_plane(l, k0r, P.nz))], v);
    }
}

// One component of the Esirkepov current (the scheme is described at esk_component in k_split32.hip:
// the same factorisation J_c(m, a, b) = f P_c[m] A_c[a][b], here in FP64): a component only where some
// lane of the wave moves along it, a window's last node only where some lane crosses a half cell, and
// there only by the lanes that do (27 x 33 x 70, a step: 41 -> 36 us; 128 x 128 x 512: the same).
template <class G, int C> __device__ inline void deposit_lds(double *Js, const int jb[3], const double S0[3][4],
                                                             const double DS[3][4], const bool cross[3], double f) {
    constexpr int CA = (C + 1) % 3, CB = (C + 2) % 3;
    constexpr int ST[3] = {1, G::jx(C), G::jx(C) * G::jy(C)};
    double P[3];
    P[0] = DS[C][0] * f;
    P[1] = (DS[C][0] + DS[C][1]) * f;
    P[2] = (DS[C][0] + DS[C][1] + DS[C][2]) * f;  // the running sum, rounded as the rigid ions' is
    if (!__any(P[0] != 0.0 || P[1] != 0.0 || P[2] != 0.0)) return;
    double *o = Js + G::jofs(C) + jb[0] + ST[1] * jb[1] + ST[2] * jb[2];
    const bool m2 = __any(cross[C]), a3 = __any(cross[CA]), b3 = __any(cross[CB]);
    double ub[4], vb[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        ub[b] = fma(0.5, DS[CB][b], S0[CB][b]);
        vb[b] = fma(1.0 / 3.0, DS[CB][b], 0.5 * S0[CB][b]);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (a == 3 && !a3) break;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            if (b == 3 && !b3) break;
            if ((a == 3 && !cross[CA]) || (b == 3 && !cross[CB])) continue;
            const double A = fma(S0[CA][a], ub[b], DS[CA][a] * vb[b]);
            double *e = o + ST[CA] * a + ST[CB] * b;
            atomicAdd(e, A * P[0]);
            atomicAdd(e + ST[C], A * P[1]);
            if (m2 && cross[C]) atomicAdd(e + 2 * ST[C], A * P[2]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Per item: stage the tile's E and B (B^n, already advanced), then per particle gather, push, move
// and deposit into the LDS current boxes, which are added to the grid at the end.  One thread per
// particle over the grid (fields from global memory, every contribution a global FP64 atomic) took
// 25.5 ms for the 128x128x512 run's 4.2 M beam and 16.5 M plasma particles; this takes 2.1 ms and
// its lists 0.34.  Bound: the plasma's 1.2 ms by VALU (1430 instructions a wave, 55 % busy) and LDS
// (162 reads and 27 to 144 FP64 adds of 8 clocks a wave), the beam's 0.9 ms by its slots, which are
// in no order (a 64-byte line for every 8 bytes read or written; 0.4 ms were they in tile order).
// Two 512-thread workgroups share a CU, so that one's rounds run under the other's staging and
// flush; 512 is the particles of a tile at 2 per cell (384 threads: 2.9 ms, 256: 2.2 ms).  Of
// its 128 VGPRs 16 are spilled (14 on x-z tiles).  The next item is claimed when the current
// one starts; loading its fields and particles across the flush as well took 10 to 40 % longer
// (spills).
template <class G>
__global__ void __launch_bounds__(ST64) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_step64(Params P, StepCtx S, Bounds64 W, Species64 sb, Species64 sp, TileList T, FieldsT<double> f, double *Jx, double *Jy,
         double *Jz, int32_t *flags) {
    extern __shared__ __align__(16) double sm64[];
    __shared__ int s_item;
    double *F = sm64, *Js = sm64 + G::NF;
    for (int e = threadIdx.x; e < G::NJ; e += ST64) Js[e] = 0.0;
    const uint32_t tid = threadIdx.x;
    ItemQueue64 Q;
    if (tid == 0) s_item = Q.first(T);
    __syncthreads();
    int cur = __builtin_amdgcn_readfirstlane(s_item);
    while (cur >= 0) {
        const Item64 I = item64(T, cur, G::TX, G::TY, G::TZ);
        Stage64<G, ST64> st;
        st.load(P, S.k0r, I, f);
        Raw64 r = load_raw64(sb, sp, T.list[min(I.begin + tid, I.end - 1)]);
        st.store(F);
        __syncthreads();  // fields staged, boxes clear, s_item read
        if (tid == 0) Q.claim(T);
        for (uint32_t base = I.begin; base < I.end; base += ST64) {
            if (base > I.begin) r = load_raw64(sb, sp, T.list[min(base + tid, I.end - 1)]);
            if (base + tid >= I.end) continue;
            double X1[3], Un[3], wi[3][3], fl[3];
            int c0[3], bi[3];
            for (int d = 0; d < 3; ++d) fl[d] = floor(r.X[d]);
            cell_in_tile64(P, W, I, fl, c0);
            double wh[3][3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                bi[d] = c0[d] + near_int(r.X[d], fl[d], wi[d]);
                weights3<double>(r.X[d] - 0.5 - fl[d], wh[d]);
            }
            double E[3], B[3], Ee[3], Be[3], dEe[3], dBe[3];
            E[0] = gather_lds<G, 0>(F, wi, wh, bi, c0);
            E[1] = gather_lds<G, 1>(F, wi, wh, bi, c0);
            E[2] = gather_lds<G, 2>(F, wi, wh, bi, c0);
            B[0] = gather_lds<G, 3>(F, wi, wh, bi, c0);
            B[1] = gather_lds<G, 4>(F, wi, wh, bi, c0);
            B[2] = gather_lds<G, 5>(F, wi, wh, bi, c0);
            ext_field64(P, r.X[2], S.t, Ee, Be, dEe, dBe);
            for (int d = 0; d < 3; ++d) {
                E[d] += Ee[d];
                B[d] += Be[d];
            }
            push<double>(P.pusher, r.w < 0.0 ? P.ahi : -0.5 * P.dt, r.U, E, B, Un);
            const double g = sqrt(1.0 + dot3(Un, Un));
            for (int d = 0; d < 3; ++d) X1[d] = r.X[d] + P.dt * Un[d] / g;
            int64_t cap;
            int32_t *alive;
            double *const at = slot64(sb, sp, r.id, cap, alive);
            if (!(isfinite(X1[0]) && isfinite(X1[1]) && isfinite(X1[2]) && isfinite(g))) {
                // never let a non-finite position reach the index arithmetic: drop the particle
                atomicOr(flags, DFLAG_NONFINITE);
                *alive = 0;
                continue;
            }
            double S0[3][4], DS[3][4];
            int jb[3];
            bool cross[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int n0 = bi[d] - c0[d];
                double w1[3];
                const int n1 = near_int(X1[d], fl[d], w1), lo = n0 < n1 ? n0 : n1;
                const bool h0 = n0 > lo, h1 = n1 > lo;
                cross[d] = n0 != n1;
                jb[d] = c0[d] + lo + 1;  // box node of offset lo - 1, origin -2
                window4(wi[d], h0, S0[d]);
                window4(w1, h1, DS[d]);
                for (int m = 0; m < 4; ++m) DS[d][m] -= S0[d][m];
            }
            if (X1[0] < 0) X1[0] += W.nx;
            if (X1[0] >= W.nx) X1[0] -= W.nx;
            if (X1[1] < 0) X1[1] += W.ny;
            if (X1[1] >= W.ny) X1[1] -= W.ny;
            for (int d = 0; d < 3; ++d) {
                at[d * cap] = X1[d];
                at[(3 + d) * cap] = Un[d];
            }
            // window after this step's shift: active band [k0n + 3, k0n + nz - 4)
            if (X1[2] < W.lo || X1[2] >= W.hi) *alive = 0;
            const double fq = r.w / P.dt;  // -q w / dt
            deposit_lds<G, 0>(Js, jb, S0, DS, cross, fq);
            deposit_lds<G, 1>(Js, jb, S0, DS, cross, fq);
            deposit_lds<G, 2>(Js, jb, S0, DS, cross, fq);
        }
        if (tid == 0) s_item = Q.resolve(T);
        __syncthreads();  // every deposit is in the boxes
        cur = __builtin_amdgcn_readfirstlane(s_item);
        flush_lds<G, 0>(P, S.k0r, I, Js, Jx);
        flush_lds<G, 1>(P, S.k0r, I, Js, Jy);
        flush_lds<G, 2>(P, S.k0r, I, Js, Jz);
    }
}

template <class G> static constexpr int step_lds() { return 8 * (G::NF + G::NJ); }

pic_status tiles64_carve(Ctx &c, char *cnt, char *base, char *room, int64_t slots) {
    const uint64_t nb = (uint64_t)bins_of(c.P), n = (uint64_t)std::max<int64_t>(slots, 1);
    TileList &T = c.tiles;
    tiles64_dims(c.P, T.ntx, T.nty, T.ntz);
    T.nbins = (int)nb;
    auto take = [&](uint64_t bytes) {
        char *r = base;
        base += al(bytes);
        return r;
    };
    T.cnt = (uint32_t *)cnt;
    T.off = (uint32_t *)take(4 * nb);
    T.room = room;
    if (room) place_lists(T, room, slots);
    T.items = (int4 *)take(16 * (nb + n / CHUNK_MIN + 16));
    T.totals = (uint2 *)take(8 * (nb / SCAN_BINS + 1));
    T.qnext = (int32_t *)take(256 * 8);
    T.nitems = (int32_t *)take(256);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, c.device) == hipSuccess && prop.multiProcessorCount > 0)
        c.ncu = (prop.multiProcessorCount + 7) / 8 * 8;
    const bool flat = tiles64_flat(c.P);
    PIC_HIP(c, hipFuncSetAttribute(flat ? (const void *)k_step64<Geom2D> : (const void *)k_step64<Geom3D>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   flat ? step_lds<Geom2D>() : step_lds<Geom3D>()));
    return PIC_OK;
}

template <class G>
static void launch_step(Ctx &c, const StepCtx &S, Species64 b, Species64 p, FieldsT<double> f, int grid) {
    constexpr int lds = step_lds<G>();
    static_assert(2 * lds + 512 <= 160 * 1024, "two workgroups per CU");
    hipLaunchKernelGGL(k_step64<G>, dim3(grid), dim3(ST64), lds, c.st, c.P, S, Bounds64(c.P, S.k0, S.k0n), b, p, c.tiles, f, c.J64[0],
                       c.J64[1], c.J64[2], c.dflags);
}

void step64_particles(Ctx &c, const StepCtx &S, FieldsT<double> f) {
    const Species64 b{c.b64.x, std::max<int64_t>(c.cap_b, 1), c.nb_slots},
        p{c.p64.x, std::max<int64_t>(c.cap_p, 1), c.np_slots};
    if (b.n + p.n <= 0) return;
    const int grid = 2 * c.ncu;
    tiles64_build(c, b, p, grid, true);
    if (tiles64_flat(c.P))
        launch_step<Geom2D>(c, S, b, p, f, grid);
    else
        launch_step<Geom3D>(c, S, b, p, f, grid);
}

// ---------------------------------------------------------------- charge
// Charge -w of the listed particles on the nodes (mobile ions carry w < 0), summed in an LDS box of the
// tile's nodes -1 .. T + 1 and added into rho (ring order).  With one thread per particle and 27 global
// FP64 atomics each, the 1 M particles of the 64x64x256 workload's beam took 3.2 ms.
template <class G>
__global__ void __launch_bounds__(ST64) k_rho64(Params P, int k0r, Bounds64 W, Species64 sb, Species64 sp, TileList T,
                                                double *rho) {
    __shared__ double box[G::NB];
    __shared__ int s_item;
    const uint32_t tid = threadIdx.x;
    for (int e = tid; e < G::NB; e += ST64) box[e] = 0.0;
    ItemQueue64 Q;
    if (tid == 0) s_item = Q.first(T);
    __syncthreads();
    int cur = __builtin_amdgcn_readfirstlane(s_item);
    while (cur >= 0) {
        const Item64 I = item64(T, cur, G::TX, G::TY, G::TZ);
        __syncthreads();  // s_item read, box clear
        if (tid == 0) Q.claim(T);
        for (uint32_t e = I.begin + tid; e < I.end; e += ST64) {
            int64_t cap;
            int32_t *alive;
            const double *at = slot64(sb, sp, T.list[e], cap, alive);
            const double X[3] = {at[0], at[cap], at[2 * cap]};
            double fl[3], w[3][3];
            int c0[3];
            for (int d = 0; d < 3; ++d) fl[d] = floor(X[d]);
            cell_in_tile64(P, W, I, fl, c0);
            for (int d = 0; d < 3; ++d) c0[d] += near_int(X[d], fl[d], w[d]);
            const double qw = -at[6 * cap];
            double *o = box + c0[0] + G::FX * (c0[1] + G::FY * c0[2]);
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int b = 0; b < 3; ++b)
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        atomicAdd(o + a + G::FX * (b + G::FY * c), qw * w[0][a] * w[1][b] * w[2][c]);
        }
        if (tid == 0) s_item = Q.resolve(T);
        __syncthreads();
        cur = __builtin_amdgcn_readfirstlane(s_item);
        for (int e = tid; e < G::NB; e += ST64) {
            const double v = box[e];
            if (v == 0.0) continue;
            box[e] = 0.0;
            const int y = e / G::FX, a = e - y * G::FX, c = y / G::FY, b = y - c * G::FY, l = I.t0z - 1 + c;
            if (l >= 0 && l < P.nz)
                atomicAdd(&rho[cell_near(P, I.t0x - 1 + a, I.t0y - 1 + b, ring_plane(l, k0r, P.nz))], v);
        }
    }
}

void rho64(Ctx &c, double *rho, int mask) {
    const Params &P = c.P;
    const Species64 b{c.b64.x, std::max<int64_t>(c.cap_b, 1), mask & 1 ? c.nb_slots : 0},
        p{c.p64.x, std::max<int64_t>(c.cap_p, 1), mask & 2 ? c.np_slots : 0};
    if (b.n + p.n <= 0) return;
    const int grid = 4 * c.ncu;  // four workgroups of 512 fill a compute unit
    tiles64_build(c, b, p, grid, false);
    const Bounds64 W(P, c.k0, c.k0);
    const int k0r = (int)(c.k0 % P.nz);
    if (tiles64_flat(P))
        hipLaunchKernelGGL(k_rho64<Geom2D>, dim3(grid), dim3(ST64), 0, c.st, P, k0r, W, b, p, c.tiles, rho);
    else
        hipLaunchKernelGGL(k_rho64<Geom3D>, dim3(grid), dim3(ST64), 0, c.st, P, k0r, W, b, p, c.tiles, rho);
}

}  // namespace pic
