// Red-black SOR with the pressure system resident on the chip (uniform grids).
//
// One launch runs a whole solve (or a long stretch of it): every compute unit
// holds one tile of the grid in its registers, pd and r0 of every cell of the
// tile, and the blocks exchange only the values on their tiles' faces.  Memory
// is touched when a launch begins and ends and when a check needs the float64
// operator, so an iteration is bound by its arithmetic and, below about a
// million cells, by the time a face value takes from one compute unit to
// another (about 1 us per half-sweep), where the sweep launches are bound by
// the launches (3 us each) and, from some million cells, by the 24 bytes per
// cell and half-sweep that they move.  Per iteration, checks and folds included,
// against the best sweep launches, MI355X: 64x64x32 with a check every 64: 2.7
// us (8.0), every 4: 3.7 (7.2); 150x150x90, every 64: 5.2 (10.6), every 4: 6.9
// (13.2) and, in the first 512 iterations with their fold every 8, 11.0 (15.9);
// 300x300x90, every 64: 11.4 (15.7), every 4: 13.8 (18.7).
//
// Same per-cell arithmetic as the sweep launches (sor_nb / sor_relax, the
// fold's TwoSum, the float64 operator), same schedule of folds, bounds and
// checks: the iterates are theirs bit for bit.
//
// Tile.  A block is 8 wavefronts; a wavefront covers 64 half-cells of a row
// and a patch of RY rows x RZ planes, so a thread holds RY x RZ pairs of cells:
// E (even i) and O (odd i).  RY and RZ are even, so in the half-sweep of colour
// F the cell of pair (r, z) that is updated is E where F + r + z is even and O
// elsewhere.  East / west neighbours: the pair's other cell and one adjacent
// lane (DPP wave shift).  North / south / up / down: registers inside the
// patch, LDS between the patches of a block, and between blocks 64-bit words
// {value, tag} written and read with relaxed agent-scope atomics: a word is
// its own flag (the tag numbers the publication), so one store-to-load trip is
// all a face costs and no fence is needed.
//
// Rows of more than 64 half-cells are split between tiles.  The lanes before a
// tile's first and after its last cell are ghosts: they hold the neighbours'
// cells and are relaxed like the tile's own, with the same values, as far as
// their surroundings reach: one column fewer per half-sweep and side.  g ghost
// columns (2 g cells) last g iterations and are then renewed by a copy, which
// takes a flag and two trips but only every g-th iteration (4 <= g <= 15).
//
// A patch's inner cells are updated first, while the last borders travel; its
// border cells follow and are published at once.
//
// All blocks of a launch wait for each other, so they have to be on the chip
// together.  The host keeps a compute unit for each of them (ChipShare): other
// kernels wait for nobody and drain, so the blocks come to be resident together
// whatever runs beside them.  Cooperative launches would give the same for the
// price of running one at a time, whatever part of the chip they need (the
// runtime has one queue for them): four threads with a 64x64x32 solve of 400
// iterations each took 8.0 ms that way and take 2.3 ms side by side, 2.1 ms for
// one; a solve alone is 20 us shorter as well.
//
// What the host does not know of (another process' launch of this kind) can
// still hold units for good, so a launch begins with a roll call: unless all
// blocks come within some milliseconds, all leave again, those that come later
// too, and nothing has changed (ctl->lost = kNoRoom).  Once all have come, only
// a suspended queue could keep one from the others; every later wait is bounded
// all the same.  A wavefront that waits in vain goes on without waiting to the
// end of its check interval, on borders that may be old and publishing what it
// makes of them; there its block raises ctl->lost, stores its cells and leaves.
// Blocks that wait for it follow within their next interval, so all but the last
// two intervals of a lost launch are sound (the host goes on with sweep launches).
#include "les_bodies.h"

namespace les {
namespace {

typedef unsigned long long u64;
constexpr int kResWaves = 8;
constexpr int kResThreads = 64 * kResWaves;
constexpr int kResSlots = 4;          // publications kept: a slot is rewritten four tags later
constexpr int kResPad = 16;           // flags 64 bytes apart

struct ResArgs {
    Geo g;
    PBufs P;
    Ctl* ctl;
    u64* xch;        // [kResSlots][blocks][face words]
    u64* gsum;       // [2][4][blocks]
    u64* xw;         // [2][blocks][west, east][wavefronts][pairs][g]: ghost columns
    unsigned* xflag; // [blocks][wavefronts][kResPad]: the patch's last event
    unsigned* gate;  // blocks that have come, launches so far times blocks
    u64* verdict;    // (tag0 << 1 | all came) of the last launch
    unsigned came;   // gate once all blocks of this launch have come
    int nbx, nby, w, gc;   // gc: ghost columns per side
    float omega;
    double omega_d;
    int K, R, cap;
    int spin, gate_spin;   // polls of one wait, and of the wait for all blocks to come
    unsigned tag0;
};

// Patches above kResBig pairs do not fit the registers with all of r0: the r0
// of their first cells stays in LDS (one conflict-free read per update), and
// the rows around the patches are kept once instead of by tag parity, at the
// price of a second barrier per half-sweep.
constexpr int kResBig = 32, kResLds = 51;

template <int RY, int RZ, int GY>
struct ResSmem {
    static constexpr bool kBig = RY * RZ > kResBig;
    static constexpr int kSets = kBig ? 1 : 2;
    // the rows south and north of each patch (RZ each) and the planes below and
    // above it (RY each): written by the neighbouring patch's wavefront, or
    // fetched from the neighbouring tile; zeros at the edge of the grid
    float halo[kSets][kResWaves][2 * RZ + 2 * RY][64];
    float r0[kBig ? kResLds : 1][kResThreads];
    double red[4][kResWaves];
};

__device__ __forceinline__ float from_left(float v) {    // lane l takes lane l - 1's v (lane 0: 0)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float v) {   // lane l takes lane l + 1's v (lane 63: 0)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
// Selection by value (a conditional between two lvalues would select an
// address and keep the patch state in memory).
template <class T>
__device__ __forceinline__ T pick(bool c, T x, T y) {
    return c ? x : y;
}
// A scalar the compiler may not trace back: what is computed from it stays
// where it is used (hoisted out of the solve's loops, the addresses and
// coefficients of the rare phases would crowd out the tile's registers).
__device__ __forceinline__ int opaque(int v) {
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ int opaque_lane(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ void put(u64* p, unsigned tag, float v) {
    __hip_atomic_store(p, ((u64)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Element of a row of a colour array: the row's address is uniform, the
// lane adds its half-index.
__device__ __forceinline__ float* at(float* row, unsigned i) {
    return (float*)((char*)row + 4u * i);
}
__device__ __forceinline__ float peek(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void poke(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int RY, int RZ, int GY>
struct Resident {
    typedef ResSmem<RY, RZ, GY> Smem;
    static_assert(RY % 2 == 0 && RZ % 2 == 0, "patch origins have even j + k, so a pair's phase is its colour");
    static constexpr int NP = RY * RZ, GZ = kResWaves / GY;
    static constexpr bool kBig = Smem::kBig;
    static constexpr int TY = GY * RY, TZ = GZ * RZ;          // rows and planes of a tile
    static constexpr int kWords = 128 * (TY + TZ);   // face words of a block
    typedef float Patch[RY][RZ];
    const ResArgs& a;
    Smem& sm;
    int lane, wv, gyi, gzi, ii, j0, k0;
    int first, last;                  // first and last own lane
    bool west, east, south, north, below, above;   // neighbouring tiles this wavefront exchanges with
    bool own, own_o, live, inside;    // the lane has cells of the tile (O cells), or ghosts of a neighbour's too
    unsigned t, nb, ymask, yok, zmask, zok;
    float om, cx, cy, cz;
    float inv[2][2][2];               // cn1 of E / O cells, [edge row][edge plane]
    bool dead = false;

    __device__ __forceinline__ Resident(const ResArgs& a_, Smem& s_) : a(a_), sm(s_) {
        const Geo& g = a.g;
        lane = threadIdx.x & 63;
        wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        nb = gridDim.x;
        auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };   // integer division leaves the scalar unit
        t = (unsigned)uni((int)xcd_block(blockIdx.x, nb));
        const int bx = uni(t % a.nbx), by = uni((t / a.nbx) % a.nby), bz = uni(t / (a.nbx * a.nby));
        gyi = uni(wv % GY);
        gzi = uni(wv / GY);
        const int x0 = bx * a.w, wc = min(a.w, g.H - x0);
        first = a.gc;
        last = first + wc - 1;
        west = bx > 0;
        east = bx < a.nbx - 1;
        ii = x0 + lane - first;
        j0 = by * TY + gyi * RY;
        k0 = bz * TZ + gzi * RZ;
        const unsigned plane = (unsigned)(a.nbx * a.nby);
        south = gyi == 0 && by > 0;
        north = gyi == GY - 1 && by < a.nby - 1;
        below = gzi == 0 && bz > 0;
        above = gzi == GZ - 1 && t + plane < nb;
        own = lane >= first && lane <= last;
        own_o = own && 2 * ii + 1 < g.nx;
        live = ii >= 0 && ii < g.H && lane <= last + first;
        const bool live_o = live && 2 * ii + 1 < g.nx;
        ymask = yok = zmask = zok = 0;
        for (int r = 0; r < RY; ++r) {
            const int j = j0 + r;
            ymask |= (j == 0 || j == g.ny - 1) ? 1u << r : 0u;
            yok |= j < g.ny ? 1u << r : 0u;
        }
        for (int z = 0; z < RZ; ++z) {
            const int k = k0 + z;
            zmask |= (k == 0 || k == g.nz - 1) ? 1u << z : 0u;
            zok |= k < g.nz ? 1u << z : 0u;
        }
        inside = !ymask && !zmask && yok == (1u << RY) - 1 && zok == (1u << RZ) - 1;
        om = live ? a.omega : 0.f;
        cx = g.cx;
        cy = g.cy;
        cz = g.cz;
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int ye = 0; ye < 2; ++ye)
#pragma unroll
                for (int ze = 0; ze < 2; ++ze) {
                    const float dxy = diag_x(g, 2 * ii + o) + (ye ? diag_y(g, 0) : g.cy + g.cy);
                    inv[o][ye][ze] = pick(o != 0, live_o, live) ? 1.0f / (dxy + (ze ? diag_z(g, 0) : g.cz + g.cz)) : 0.f;
                }
    }

    // ------------------------------------------------------- tile <-> memory
    // The two colour arrays q0, q1 into (or out of) the patch's cells; lanes
    // of `in` and rows and planes inside the grid.
    template <class F>
    __device__ __forceinline__ void each(bool in, float* q0, float* q1, F&& f) const {
        const Geo& g = a.g;
        const int i = opaque_lane(ii), j = opaque(j0), k = opaque(k0), yk = opaque(yok), zk = opaque(zok);
        const bool in_o = in && 2 * i + 1 < g.nx;   // an odd row has no last O cell
#pragma unroll
        for (int r = 0; r < RY; ++r)
#pragma unroll
            for (int z = 0; z < RZ; ++z) {
                const bool ok = ((yk >> r) & (zk >> z) & 1) != 0;
                const long long e = g.col(0, j + r, k + z);
                float* pe = ((r + z) & 1) ? q1 : q0;
                float* po = ((r + z) & 1) ? q0 : q1;
                f(r, z, at(pe + e, (unsigned)i), in && ok, at(po + e, (unsigned)i), in_o && ok);
            }
    }
    template <bool COHERENT = false>
    __device__ __forceinline__ void load(bool in, float* const q[2], Patch& E, Patch& O) const {
        each(in, q[0], q[1], [&](int r, int z, const float* pe, bool oke, const float* po, bool oko) {
            E[r][z] = oke ? (COHERENT ? peek(pe) : *pe) : 0.f;
            O[r][z] = oko ? (COHERENT ? peek(po) : *po) : 0.f;
        });
    }
    // (the tile's own cells are in the registers)
    __device__ __forceinline__ void load_ghosts(float* const q[2], Patch& E, Patch& O) const {
        if (live && !own)
            each(true, q[0], q[1], [&](int r, int z, const float* pe, bool oke, const float* po, bool oko) {
                if (oke) E[r][z] = peek(pe);
                if (oko) O[r][z] = peek(po);
            });
    }
    template <bool COHERENT = false>
    __device__ __forceinline__ void store(float* const (&q)[2], const Patch& E, const Patch& O) const {
        each(own, q[0], q[1], [&](int r, int z, float* pe, bool oke, float* po, bool oko) {
            if (oke) COHERENT ? poke(pe, E[r][z]) : (void)(*pe = E[r][z]);
            if (oko) COHERENT ? poke(po, O[r][z]) : (void)(*po = O[r][z]);
        });
    }

    // --------------------------------------------------------- face exchange
    __device__ __forceinline__ u64* area(unsigned tag, unsigned tile) const {
        return a.xch + ((size_t)(tag % kResSlots) * nb + tile) * kWords;
    }
    // Where the four borders of a patch begin in its halo and in a tile's face words.
    static constexpr int kS = 0, kN = RZ, kB = 2 * RZ, kT = 2 * RZ + RY;
    __device__ __forceinline__ int word_s() const { return gzi * RZ; }
    __device__ __forceinline__ int word_n() const { return TZ + gzi * RZ; }
    __device__ __forceinline__ int word_b() const { return 2 * TZ + gyi * RY; }
    __device__ __forceinline__ int word_t() const { return 2 * TZ + TY + gyi * RY; }
    // Publish the cells of phase F on the patch's rows and planes to the
    // neighbouring tiles ...
    template <int F>
    __device__ __forceinline__ void publish(unsigned tag, const Patch& E, const Patch& O) {
        auto val = [&](int r, int z) { return ((F + r + z) & 1) ? O[r][z] : E[r][z]; };
        u64* out = area(tag, t) + lane;
        if (live) {
            if (south)
#pragma unroll
                for (int z = 0; z < RZ; ++z) put(out + (word_s() + z) * 64, tag, val(0, z));
            if (north)
#pragma unroll
                for (int z = 0; z < RZ; ++z) put(out + (word_n() + z) * 64, tag, val(RY - 1, z));
            if (below)
#pragma unroll
                for (int r = 0; r < RY; ++r) put(out + (word_b() + r) * 64, tag, val(r, 0));
            if (above)
#pragma unroll
                for (int r = 0; r < RY; ++r) put(out + (word_t() + r) * 64, tag, val(r, RZ - 1));
        }
    }
    // ... and to the halos of the neighbouring patches of the block.
    template <int F>
    __device__ __forceinline__ void pass(unsigned tag, const Patch& E, const Patch& O) {
        auto& halo = sm.halo[tag & (Smem::kSets - 1)];
        auto val = [&](int r, int z) { return ((F + r + z) & 1) ? O[r][z] : E[r][z]; };
        // (from one address per publication: hoisted, a register per row)
        float* mine = &halo[0][0][0] + opaque_lane(wv * (2 * RZ + 2 * RY) * 64 + lane);
        constexpr int kPatch = (2 * RZ + 2 * RY) * 64;
        if (gyi > 0)
#pragma unroll
            for (int z = 0; z < RZ; ++z) mine[-kPatch + (kN + z) * 64] = val(0, z);
        if (gyi < GY - 1)
#pragma unroll
            for (int z = 0; z < RZ; ++z) mine[kPatch + (kS + z) * 64] = val(RY - 1, z);
        if (gzi > 0)
#pragma unroll
            for (int r = 0; r < RY; ++r) mine[-GY * kPatch + (kT + r) * 64] = val(r, 0);
        if (gzi < GZ - 1)
#pragma unroll
            for (int r = 0; r < RY; ++r) mine[GY * kPatch + (kB + r) * 64] = val(r, RZ - 1);
    }
    static __device__ __forceinline__ constexpr bool border(int r, int z) { return r == 0 || r == RY - 1 || z == 0 || z == RZ - 1; }
    static __device__ __forceinline__ u64 get(const u64* p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Renew the ghost columns (event number n): a tile's first and last g
    // columns, both colours, go to its x neighbours; the event's flag follows the
    // columns once they are at the point of coherence.  Patches pair one to one,
    // so two sets of words suffice.
    __device__ __forceinline__ void refresh(unsigned n, Patch& E, Patch& O) {
        const int g = first;
        auto column = [&](unsigned tile, int side, int l) {
            return a.xw + ((((size_t)(n & 1) * nb + tile) * 2 + side) * kResWaves + wv) * (NP * g) + l;
        };
        const bool tw = west && lane >= g && lane < 2 * g, te = east && lane >= a.w && lane < a.w + g;
        if (tw || te) {
            u64* p = column(t, te ? 1 : 0, te ? lane - a.w : lane - g);
#pragma unroll
            for (int q = 0; q < NP; ++q)
                __hip_atomic_store(p + q * g, ((u64)__float_as_uint(O[q / RZ][q % RZ]) << 32) | __float_as_uint(E[q / RZ][q % RZ]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        reach(n);
        meet(n);
        const bool gw = west && lane < g, ge = east && lane > last && lane <= last + g;
        if (gw || ge) {
            const u64* p = column(gw ? t - 1 : t + 1, gw ? 1 : 0, gw ? lane : lane - last - 1);
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                if (q % 8 == 0) asm volatile("" ::: "memory");   // eight columns in flight: the registers hold the tile
                const u64 v = get(p + q * g);
                E[q / RZ][q % RZ] = __uint_as_float((unsigned)v);
                O[q / RZ][q % RZ] = __uint_as_float((unsigned)(v >> 32));
            }
        }
    }
    // Event n of this patch, for its x neighbours: its columns are out, or it has
    // read its ghosts from memory.  Every load and store before it is done.
    __device__ __forceinline__ void reach(unsigned n) const {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0)
            __hip_atomic_store(a.xflag + (t * kResWaves + wv) * kResPad, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Both x neighbours have reached event n too.  One may be an event ahead, no
    // more (the next needs this patch), so only n and n + 1 count: a flag left by
    // an earlier launch, however old, or a cleared one is neither.
    __device__ __forceinline__ void meet(unsigned n) {
        const bool see = (lane == 0 && west) || (lane == 1 && east);
        const unsigned* flag = a.xflag + ((lane ? t + 1 : t - 1) * kResWaves + wv) * kResPad;
#pragma unroll 1
        for (int spin = 0;; ++spin) {
            bool ok = true;
            if (see) ok = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - n <= 1u;
            if (__builtin_expect(dead || __all(ok), 1)) break;
            if (spin >= a.spin) dead = true;
        }
        asm volatile("" ::: "memory");   // nothing that follows comes before the flags
    }
    // Fetch the neighbouring tiles' rows and planes of publication `tag` into
    // the halo: one wait for all words of the wavefront (a patch touches at most
    // one tile in y and one in z).  A wavefront reads back from LDS only what it
    // fetched itself, or what its block passed before the last barrier.
    __device__ __forceinline__ void halos(unsigned tag) {
        static_assert(GY >= 2 && GZ >= 2, "one tile boundary per axis");
        const int plane = a.nbx * a.nby;
        const bool iny = south || north, inz = below || above;
        const u64* py = area(tag, t + (south ? -a.nbx : a.nbx)) + (south ? word_n() : word_s()) * 64 + lane;
        const u64* pz = area(tag, t + (below ? -plane : plane)) + (below ? word_t() : word_b()) * 64 + lane;
        u64 vy[RZ] = {}, vz[RY] = {};   // lanes without a cell: 0
        if (iny || inz) {
#pragma unroll 1
            for (int spin = 0;; ++spin) {
                bool ok = true;
                if (live) {
                    if (iny)
#pragma unroll
                        for (int z = 0; z < RZ; ++z) vy[z] = get(py + z * 64);
                    if (inz)
#pragma unroll
                        for (int r = 0; r < RY; ++r) vz[r] = get(pz + r * 64);
                    if (iny)
#pragma unroll
                        for (int z = 0; z < RZ; ++z) ok = ok && (unsigned)(vy[z] >> 32) == tag;
                    if (inz)
#pragma unroll
                        for (int r = 0; r < RY; ++r) ok = ok && (unsigned)(vz[r] >> 32) == tag;
                }
                if (__builtin_expect(dead || __all(ok), 1)) break;
                if (spin >= a.spin) dead = true;
            }
        }
        auto& h = sm.halo[tag & (Smem::kSets - 1)][wv];
        if (iny) {
            float(*dst)[64] = &h[south ? kS : kN];
#pragma unroll
            for (int z = 0; z < RZ; ++z) dst[z][lane] = __uint_as_float((unsigned)vy[z]);
        }
        if (inz) {
            float(*dst)[64] = &h[below ? kB : kT];
#pragma unroll
            for (int r = 0; r < RY; ++r) dst[r][lane] = __uint_as_float((unsigned)vz[r]);
        }
    }
    // r0 of cell o of the pair (r, z)
    __device__ __forceinline__ float r0_of(const Patch& rE, const Patch& rO, int o, int r, int z, int tid) const {
        const int n = 2 * (r * RZ + z) + o;
        if (kBig && n < kResLds) return sm.r0[kBig && n < kResLds ? n : 0][tid];
        return o ? rO[r][z] : rE[r][z];
    }
    __device__ __forceinline__ void load_r0(Patch& rE, Patch& rO) {
        load<true>(live, a.P.r0, rE, rO);
        if constexpr (kBig)
#pragma unroll
            for (int n = 0; n < kResLds; ++n)
                sm.r0[n][threadIdx.x] = (n & 1) ? rO[n / 2 / RZ][n / 2 % RZ] : rE[n / 2 / RZ][n / 2 % RZ];
    }

    // ------------------------------------------------------------ half-sweep
    // The phase-F cells on the patch's border, or inside it.
    template <int F, bool ACC, bool BORDER, bool EDGE>
    __device__ __forceinline__ void relax_as(Patch& E, Patch& O, const Patch& rE, const Patch& rO, unsigned seen, double& r2,
                                          double& d2) {
        const auto& h = sm.halo[seen & (Smem::kSets - 1)][wv];   // publication `seen` around the patch
        const int ia = ACC ? opaque_lane(ii) : 0;   // the sums' diagonals are formed where they are used
        const int tid = opaque_lane((int)threadIdx.x);   // r0 is read from LDS where it is used
        // cn1: the grid's first and last rows and planes have their own, cells
        // past its end have 0 (and stay 0)
        const int ym = EDGE ? opaque(ymask) : 0, zm = EDGE ? opaque(zmask) : 0, yk = EDGE ? opaque(yok) : -1, zk = EDGE ? opaque(zok) : -1;
#pragma unroll
        for (int z = 0; z < RZ; ++z) {
            const bool ze = (zm >> z) & 1, zv = (zk >> z) & 1;
            float cz_[2][2];
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int e = 0; e < 2; ++e) cz_[o][e] = pick(zv, pick(ze, inv[o][e][1], inv[o][e][0]), 0.f);
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                if (border(r, z) != BORDER) continue;
                const int o = (F + r + z) & 1;
                Patch& X = o ? O : E;
                const float in_pair = o ? E[r][z] : O[r][z];
                const float beside = o ? from_right(E[r][z]) : from_left(O[r][z]);
                const float ps = r > 0 ? X[r > 0 ? r - 1 : 0][z] : h[kS + z][lane];
                const float pn = r < RY - 1 ? X[r < RY - 1 ? r + 1 : r][z] : h[kN + z][lane];
                const float pb = z > 0 ? X[r][z > 0 ? z - 1 : 0] : h[kB + r][lane];
                const float pt = z < RZ - 1 ? X[r][z < RZ - 1 ? z + 1 : z] : h[kT + r][lane];
                const bool ye = (ym >> r) & 1;
                const float c = pick(((yk >> r) & 1) != 0, pick(ye, cz_[o][1], cz_[o][0]), 0.f);
                float rt;
                X[r][z] = sor_relax(sor_nb(in_pair, beside, ps, pn, pb, pt, cx, cy, cz), c,
                                    r0_of(rE, rO, o, r, z, tid), X[r][z], om, rt);
                if constexpr (ACC) {
                    const Geo& g = a.g;
                    const float dxy = diag_x(g, 2 * ia + o) + (ye ? diag_y(g, 0) : g.cy + g.cy);
                    const float diag = dxy + (ze ? diag_z(g, 0) : g.cz + g.cz);
                    const double rd = (double)(own ? rt : 0.f);
                    r2 += rd * rd;
                    const double dd = (double)diag * rd;
                    d2 += dd * dd;
                }
            }
        }
    }
    template <int F, bool BORDER>
    __device__ __forceinline__ void relax(bool acc, Patch& E, Patch& O, const Patch& rE, const Patch& rO, unsigned seen, double& r2, double& d2) {
        if (acc) relax_as<F, true, BORDER, true>(E, O, rE, rO, seen, r2, d2);
        else if (inside) relax_as<F, false, BORDER, false>(E, O, rE, rO, seen, r2, d2);
        else relax_as<F, false, BORDER, true>(E, O, rE, rO, seen, r2, d2);
    }
    // One half-sweep.  The cells inside the patch need nothing of the last
    // publication from elsewhere and go first, while it travels; the border's
    // words leave before the block's own exchange.
    // Ghost columns lose one cell per half-sweep, so g columns last g
    // iterations; they are renewed before the last half-sweep's borders leave,
    // which then carry them.
    struct Step {
        unsigned tag, event;   // last publication, last event among x neighbours
        int age;
    };
    template <int F>
    __device__ __forceinline__ void half(bool acc, Step& st, Patch& E, Patch& O, const Patch& rE, const Patch& rO, double& r2, double& d2) {
        relax<F, false>(acc, E, O, rE, rO, st.tag, r2, d2);
        __syncthreads();   // the block's own borders are in the halos
        halos(st.tag);
        relax<F, true>(acc, E, O, rE, rO, st.tag, r2, d2);
        if (F == 1 && a.nbx > 1 && ++st.age == first) {
            refresh(++st.event, E, O);
            st.age = 0;
        }
        ++st.tag;
        publish<F>(st.tag, E, O);
        if (kBig) __syncthreads();   // the halos just read are overwritten
        pass<F>(st.tag, E, O);
    }
    // n iterations; the sums of the last one: reltmp^2 of both colours,
    // (diag reltmp)^2 of colour 1
    __device__ __forceinline__ void sweeps(int n, Step& st, Patch& E, Patch& O, const Patch& rE, const Patch& rO, double& r2, double& d2) {
        r2 = 0.0;
#pragma unroll 1
        for (int it = 0; it < n; ++it) {
            const bool acc = it == n - 1;
            half<0>(acc, st, E, O, rE, rO, r2, d2);
            d2 = 0.0;
            half<1>(acc, st, E, O, rE, rO, r2, d2);
        }
    }

    // ------------------------------------------- float64 residual, fold, rebase
    // These run once in many iterations, through memory: the blocks leave pd
    // (and the folded ph) there with agent-coherent stores, meet, and read
    // their cells' surroundings back with agent-coherent loads, so that the
    // sweeps keep the registers.
    // pd to memory; with FOLD, ph <- fl(ph + pd) and pd <- the exact rest
    // (TwoSum) on the way, a row of the patch per trip: 30 us at 300x300x90, 12
    // bytes per cell (all of ph at once did not fit the registers: 46 us).
    template <bool FOLD>
    __device__ __forceinline__ void leave(Patch& E, Patch& O) const {
        const Geo& g = a.g;
        const int i = opaque_lane(ii), j = opaque(j0), k = opaque(k0), yk = opaque(yok), zk = opaque(zok);
        const bool odd_last = 2 * i + 1 >= g.nx;   // an odd row has no last O cell
        if (own) {
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                const long long e = g.col(0, j + r, k);
                float be[RZ], bo[RZ], xe[RZ], xo[RZ];
                if constexpr (FOLD)
#pragma unroll
                    for (int z = 0; z < RZ; ++z) {   // (outside the grid: its first cell's, unused)
                        const long long ez = ((yk >> r) & (zk >> z) & 1) ? e + z * g.SP : g.col(0, 0, 0);
                        xe[z] = *at(a.P.ph[(r + z) & 1] + ez, (unsigned)i);
                        xo[z] = *at(a.P.ph[1 - ((r + z) & 1)] + ez, (unsigned)i);
                    }
#pragma unroll
                for (int z = 0; z < RZ; ++z) {
                    be[z] = E[r][z];
                    bo[z] = O[r][z];
                    if constexpr (FOLD) {
                        two_sum(xe[z], be[z]);
                        two_sum(xo[z], bo[z]);
                        E[r][z] = be[z];
                        O[r][z] = bo[z];
                    }
                }
#pragma unroll
                for (int z = 0; z < RZ; ++z) {
                    if (!((yk >> r) & (zk >> z) & 1)) continue;
                    const long long ez = e + z * g.SP;
                    const int c = (r + z) & 1;
                    poke(at(a.P.pd[c] + ez, (unsigned)i), be[z]);
                    if constexpr (FOLD) poke(at(a.P.ph[c] + ez, (unsigned)i), xe[z]);
                    if (odd_last) continue;
                    poke(at(a.P.pd[1 - c] + ez, (unsigned)i), bo[z]);
                    if constexpr (FOLD) poke(at(a.P.ph[1 - c] + ez, (unsigned)i), xo[z]);
                }
                asm volatile("" ::: "memory");   // a row at a time: the registers hold the tile
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // at the point of coherence before the blocks meet
    }
    // x <- fl(x + b), b <- the exact rest
    static __device__ __forceinline__ void two_sum(float& x, float& b) {
        const float f = x + b, bb = f - x;
        b = (x - (f - bb)) + (b - bb);
        x = f;
    }
    // Sum of squares over the tile of r = b - A x (float64), b = r0, x = pd; or,
    // with REBASE, of rhs - A (ph + pd), storing r0 = rhs - A ph.  Two planes of
    // a row at a time: their loads travel together, and few enough registers are
    // taken to leave the sweeps theirs (whole rows, and marches that read each
    // value once, made the compiler spill the tile in the sweeps: 12 -> 16 us per
    // iteration at 300x300x90).  It is bound by its loads, about 40 bytes per cell
    // that pass the caches by: 50 us at 300x300x90, 15 us at 150x150x90, of a fold
    // and rebase of 130 and 45 us (156 and 60 with one plane at a time).
    template <bool REBASE>
    __device__ __forceinline__ double residual() const {
        constexpr int kSlab = 2;
        const Geo& g = a.g;
        double s = 0.0;
        const int i = opaque_lane(ii), jb = opaque(j0), kb = opaque(k0);
        const unsigned il = live ? (unsigned)i : 0u;
        struct Column {
            float e[kSlab + 2], o[kSlab + 2];   // planes k - 1 .. k + kSlab
        };
        // kSlab planes of row j from k (and those around them) of a field; past the
        // grid's outer row or plane: those again, not used
        auto column = [&](float* const (&q)[2], int j, int k, bool around, Column& x) {
            j = min(j, g.ny);
            const bool odd = ((j + k) & 1) != 0;
            float* q0 = pick(odd, q[0], q[1]) + g.col(0, j, k - 1);   // E's at the first plane
            float* q1 = pick(odd, q[1], q[0]) + g.col(0, j, k - 1);
#pragma unroll
            for (int p = 0; p < kSlab + 2; ++p) {
                if (around || (p != 0 && p != kSlab + 1)) {
                    x.e[p] = peek(at((p & 1) ? q1 : q0, il));
                    x.o[p] = peek(at((p & 1) ? q0 : q1, il));
                }
                const long long up = k + p <= g.nz ? g.SP : 0;
                q0 += up;
                q1 += up;
            }
        };
        auto mask = [&](Column& x) {   // lanes without a cell: 0
#pragma unroll
            for (int p = 0; p < kSlab + 2; ++p) {
                x.e[p] = live ? x.e[p] : 0.f;
                x.o[p] = live ? x.o[p] : 0.f;
            }
        };
        float* const base[2] = {REBASE ? a.P.rhs[0] : a.P.r0[0], REBASE ? a.P.rhs[1] : a.P.r0[1]};
        const double dxe = (2 * i > 0 ? g.cxd : 0.0) + (2 * i < g.nx - 1 ? g.cxd : (g.outflow ? 2.0 * g.cxd : 0.0));
        const double dxo = g.cxd + (2 * i + 1 < g.nx - 1 ? g.cxd : (g.outflow ? 2.0 * g.cxd : 0.0));
#pragma unroll 1
        for (int q = 0; q < NP / kSlab; ++q) {
            const int j = jb + q / (RZ / kSlab), kz = kb + q % (RZ / kSlab) * kSlab;
            if (j >= g.ny || kz >= g.nz) continue;
            Column dc, ds, dn, hc, hs, hn, bc;
            column(a.P.pd, j, kz, true, dc);
            column(a.P.pd, j - 1, kz, false, ds);
            column(a.P.pd, j + 1, kz, false, dn);
            if constexpr (REBASE) {
                column(a.P.ph, j, kz, true, hc);
                column(a.P.ph, j - 1, kz, false, hs);
                column(a.P.ph, j + 1, kz, false, hn);
            }
            column(base, j, kz, false, bc);
            mask(dc);
            if constexpr (REBASE) mask(hc);
            const double dy = (j > 0 ? g.cyd : 0.0) + (j < g.ny - 1 ? g.cyd : 0.0);
#pragma unroll
            for (int z = 0; z < kSlab; ++z) {
                const int k = kz + z, p = z + 1;
                const bool ok = k < g.nz, odd = ((j + k) & 1) != 0;
                const double dz = (k > 0 ? g.czd : 0.0) + (k < g.nz - 1 ? g.czd : 0.0);
                const double de = dxe + dy + dz, dd = dxo + dy + dz;   // diag64
                double be = (double)bc.e[p], bo = (double)bc.o[p];
                if constexpr (REBASE) {
                    be -= op64(g, hc.o[p], from_left(hc.o[p]), hs.e[p], hn.e[p], hc.e[p - 1], hc.e[p + 1], de, hc.e[p]);
                    bo -= op64(g, hc.e[p], from_right(hc.e[p]), hs.o[p], hn.o[p], hc.o[p - 1], hc.o[p + 1], dd, hc.o[p]);
                    const long long e = g.col(0, j, k);
                    if (own && ok) poke(at(pick(odd, a.P.r0[1], a.P.r0[0]) + e, il), (float)be);
                    if (own_o && ok) poke(at(pick(odd, a.P.r0[0], a.P.r0[1]) + e, il), (float)bo);
                }
                const double te = be - op64(g, dc.o[p], from_left(dc.o[p]), ds.e[p], dn.e[p], dc.e[p - 1], dc.e[p + 1], de, dc.e[p]);
                const double to = bo - op64(g, dc.e[p], from_right(dc.e[p]), ds.o[p], dn.o[p], dc.o[p - 1], dc.o[p + 1], dd, dc.o[p]);
                if (own && ok) s += te * te;
                if (own_o && ok) s += to * to;
            }
        }
        if (REBASE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // r0 is out before the blocks meet: ghosts read it
        return s;
    }

    // Sums of v0 and v1 over all blocks, in one fixed order for every block
    // (all take the same decisions from them).
    __device__ __forceinline__ void gather(unsigned gtag, double& v0, double& v1) {
        const double x0 = wave_sum(v0), x1 = wave_sum(v1);
        __syncthreads();
        if (lane == 0) {
            sm.red[0][wv] = x0;
            sm.red[1][wv] = x1;
        }
        __syncthreads();
        u64* gs = a.gsum + (size_t)(gtag & 1) * 4 * nb;
        if (threadIdx.x < 2) {
            double s = 0.0;
            for (int q = 0; q < kResWaves; ++q) s += sm.red[threadIdx.x][q];
            const u64 bits = (u64)__double_as_longlong(s);
            u64* p = gs + 2 * threadIdx.x * nb + t;
            __hip_atomic_store(p, ((u64)gtag << 32) | (bits & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(p + nb, ((u64)gtag << 32) | (bits >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        double y[2] = {0.0, 0.0};
        if (wv * 64 < (int)nb) {
            const bool need = threadIdx.x < nb;
            u64 v[4] = {0, 0, 0, 0};
#pragma unroll 1
            for (int spin = 0;; ++spin) {
                bool ok = true;
                if (need)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        v[q] = __hip_atomic_load(gs + q * nb + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        ok = ok && (unsigned)(v[q] >> 32) == gtag;
                    }
                if (__builtin_expect(dead || __all(ok), 1)) break;
                if (spin >= a.spin) dead = true;
            }
            if (need)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    y[q] = __longlong_as_double((long long)((v[2 * q] & 0xffffffffull) | (v[2 * q + 1] << 32)));
        }
        const double y0 = wave_sum(y[0]), y1 = wave_sum(y[1]);
        if (lane == 0) {
            sm.red[2][wv] = y0;
            sm.red[3][wv] = y1;
        }
        __syncthreads();
        v0 = v1 = 0.0;
        for (int q = 0; q < kResWaves; ++q) {
            v0 += sm.red[2][q];
            v1 += sm.red[3][q];
        }
    }
};

// Whether all blocks of the launch are on the chip.  The block that completes the
// count says yes, one that has waited long enough says no; the first word stands.
__device__ __forceinline__ bool roll_call(const ResArgs& a) {
    bool go = false;
    if (threadIdx.x < 64) {
        auto say = [&](bool yes) {
            u64 v = __hip_atomic_load(a.verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const u64 mine = (u64)a.tag0 << 1 | (yes ? 1 : 0);
            if (v >> 1 != a.tag0 && __hip_atomic_compare_exchange_strong(a.verdict, &v, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                                         __HIP_MEMORY_SCOPE_AGENT) && !yes)
                a.ctl->lost = kNoRoom;
        };
        if (threadIdx.x == 0 && __hip_atomic_fetch_add(a.gate, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == a.came) say(true);
#pragma unroll 1
        for (int spin = 0;; ++spin) {
            const u64 v = __hip_atomic_load(a.verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            go = v & 1;
            if (__all(v >> 1 == a.tag0)) break;
            if (spin == a.gate_spin && threadIdx.x == 0) say(false);
        }
    }
    return __syncthreads_or(go);
}

template <int RY, int RZ, int GY>
__global__ __launch_bounds__(kResThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_resident(ResArgs a) {
    __shared__ ResSmem<RY, RZ, GY> sm;
    Ctl* ctl = a.ctl;
    if (!roll_call(a)) return;
    if (ctl->done) return;   // written by block 0 alone, at its end, after every block has passed here
    typedef Resident<RY, RZ, GY> Res;
    Res w(a, sm);
    typename Res::Patch E, O, rE, rO;
    w.load(w.live, a.P.pd, E, O);
    w.load_r0(rE, rO);
    for (int q = threadIdx.x; q < (int)(sizeof sm.halo / sizeof(float)); q += kResThreads) (&sm.halo[0][0][0][0])[q] = 0.f;
    __syncthreads();
    typename Res::Step st{a.tag0, a.tag0, 0};
    if (a.nbx > 1) w.reach(++st.event);   // the ghosts are read
    const int K = a.K, max_iter = ctl->max_iter;
    const double tol = ctl->tol, rhs2 = ctl->rhs2;
    int m = ctl->m, left = a.cap, done = 0;
    long long cidx = m / K;
    double R = ctl->resid, reltmp2 = 0.0;
    unsigned gtag = a.tag0;
    auto finish = [&](bool lost) {
        if (lost && threadIdx.x == 0) ctl->lost = 1;
        if (w.t != 0 || threadIdx.x != 0) return;
        ctl->m = m;
        ctl->skip = 0;
        ctl->resid = R;
        ctl->reltmp2 = reltmp2;
        ctl->done = done;
    };
    auto publish1 = [&]() {   // colour 1's borders as they stand
        w.template publish<1>(st.tag, E, O);
        w.template pass<1>(st.tag, E, O);
    };
    publish1();
    while (true) {
        const int n = min(K, max_iter - m);
        double r2 = 0.0, d2 = 0.0;
        w.sweeps(n, st, E, O, rE, rO, r2, d2);
        ++cidx;
        m += n;
        left -= n;
        const bool due = rebase_due_at(cidx, K, a.R);
        bool check = true;
        if (!due) {
            // the residual's lower bound from the sums of the last iteration
            // (finalize_body, FIN_BOUND): a check that cannot succeed is skipped
            w.gather(++gtag, d2, r2);
            reltmp2 = r2;
            const double lbd = fabs(a.omega_d - 1.0) / a.omega_d * sqrt(d2) / sqrt(rhs2);
            check = !(m < max_iter && lbd > 1.5 * tol);
        }
        if (check) {
            // pd in memory may still be read as ghosts: the other intervals have
            // met over the bound's sums since, a fold waits for its x neighbours
            if (due) {
                if (a.nbx > 1) w.meet(st.event);
                w.template leave<true>(E, O);
            } else {
                w.template leave<false>(E, O);
            }
            double meet = 0.0;
            if (due) {
                w.gather(++gtag, meet, r2);
                reltmp2 = r2;
            } else {
                w.gather(++gtag, meet, d2);
            }
            double s = due ? w.template residual<true>() : w.template residual<false>(), none = 0.0;
            w.gather(++gtag, s, none);
            R = sqrt(s) / sqrt(rhs2);
            done = !isfinite(R) ? 3 : (R <= tol ? 1 : (m >= max_iter ? 2 : 0));
            // (a stop leaves here: pd is in memory, and the tile's registers are
            // free in the residual)
            if (done) return finish(__syncthreads_or(w.dead));
            if (a.nbx > 1) {
                w.load_ghosts(a.P.pd, E, O);
                w.reach(++st.event);
            }
            w.load_r0(rE, rO);
            ++st.tag;
            st.age = 0;   // the ghosts came along
            __syncthreads();
            publish1();
        }
        const bool lost = __syncthreads_or(w.dead);
        if (left <= 0 || lost) {
            w.store(a.P.pd, E, O);
            return finish(lost);
        }
    }
}

template <int RY, int RZ, int GY>
hipError_t start(const ResArgs& a, unsigned blocks, hipStream_t st) {
    ResArgs args = a;
    void* p[] = {&args};
    return hipLaunchKernel(reinterpret_cast<const void*>(k_resident<RY, RZ, GY>), dim3(blocks), dim3(kResThreads), p, 0, st);
}

struct Shape {
    int ry, rz, gy;
    hipError_t (*start)(const ResArgs&, unsigned, hipStream_t);
};
#define LES_RES_SHAPE(RY, RZ, GY) {RY, RZ, GY, start<RY, RZ, GY>}
const Shape kShapes[] = {LES_RES_SHAPE(2, 2, 4), LES_RES_SHAPE(4, 4, 4), LES_RES_SHAPE(4, 6, 4), LES_RES_SHAPE(6, 8, 4)};
constexpr int kNumShapes = sizeof kShapes / sizeof kShapes[0];

}  // namespace

// The shape for a grid: its tiles have to fit the compute units, one block
// each (registers: 2 waves per SIMD; LDS: all of it for the largest).  Among
// those that fit, time goes as the pairs per thread plus the exchange between
// tiles: per iteration, with a check every 64, 2.7 us at 4 pairs (64x64x32), 4.8
// at 16 (300x300x16), 5.8 at 24 (124x300x120), 11.4 at 48 (300x300x90; some
// registers spilled).  Grids of at most
// 64 half-cells per row and one tile run without the exchange.  Larger grids,
// up to the 256 x 8 x 48 x 56 pairs that the chip holds, are refused.
ResPlan resident_plan(const Geo& g, int cus) {
    ResPlan best{};
    best.shape = -1;
    if (g.stretched) return best;
    double best_cost = 0.0;
    for (int q = 0; q < kNumShapes; ++q) {
        const Shape& s = kShapes[q];
        ResPlan p{};
        const int ty = s.gy * s.ry, tz = kResWaves / s.gy * s.rz;
        p.shape = q;
        // rows beyond 64 half-cells are split, with ghost columns in the lanes
        // that are left (at least four on each side)
        p.nbx = g.H <= 64 ? 1 : (g.H + 55) / 56;
        p.w = (g.H + p.nbx - 1) / p.nbx;
        p.g = p.nbx == 1 ? 0 : (64 - p.w) / 2;
        p.nby = (g.ny + ty - 1) / ty;
        p.nbz = (g.nz + tz - 1) / tz;
        const long long nb = (long long)p.nbx * p.nby * p.nbz;
        if (nb > cus) continue;
        p.blocks = (unsigned)nb;
        p.words = 128LL * (ty + tz);
        p.xwords = 2LL * kResWaves * s.ry * s.rz * p.g;
        const double cost = 0.04 * s.ry * s.rz + (nb > 1 ? 1.0 : 0.0);
        if (best.shape < 0 || cost < best_cost) {
            best = p;
            best_cost = cost;
        }
    }
    return best;
}

size_t resident_bytes(const ResPlan& p) {
    return ((size_t)kResSlots * p.words + 2 * 4 + 2 * (size_t)p.xwords) * p.blocks * sizeof(u64) +
           (size_t)p.blocks * kResWaves * kResPad * sizeof(unsigned) + 2 * 128;
}

// tags one launch of `iters` iterations may use: two publications each, and at
// most three sums and one publication per check interval
unsigned resident_tags(int iters, int K) { return 2u * (unsigned)iters + 4u * (unsigned)(iters / K + 2) + 8u; }

hipError_t launch_resident(const Geo& g, hipStream_t st, const ResPlan& p, const PBufs& P, Ctl* ctl, void* mem, double omega,
                           int K, int R, int iters, unsigned tag, unsigned launch, int spin, int gate_spin) {
    if (spin < 0) return hipErrorInvalidValue;
    ResArgs a{};
    a.g = g;
    a.P = P;
    a.ctl = ctl;
    a.xch = (u64*)mem;
    a.gsum = a.xch + (size_t)kResSlots * p.words * p.blocks;
    a.xw = a.gsum + 2 * 4 * (size_t)p.blocks;
    a.xflag = (unsigned*)(a.xw + 2 * (size_t)p.xwords * p.blocks);
    a.gate = a.xflag + (size_t)p.blocks * kResWaves * kResPad;
    a.verdict = (u64*)(a.gate + 32);
    a.came = (launch + 1) * p.blocks + (gate_spin == 0 ? 1 : 0);   // 0: out of reach, for tests
    a.nbx = p.nbx;
    a.nby = p.nby;
    a.w = p.w;
    a.gc = p.g;
    a.omega = (float)omega;
    a.omega_d = omega;
    a.K = K;
    a.R = R;
    a.cap = iters;
    a.spin = spin;
    a.gate_spin = gate_spin;
    a.tag0 = tag;
    return kShapes[p.shape].start(a, p.blocks, st);
}

}  // namespace les
