// Twinned double-buffer relaxation (section 2.6): the paper's GPU
// alternative to the red-black scheme, built here as a measured comparison
// solver beside the red-black SOR of the time step.
//
// p is held as a pair (p_0, p_1) per cell.  The first half of an iteration
// sets every cell's p_1 from the p_0 values (own and six neighbours, 0 outside
// the grid), the second half p_0 from p_1, each with the SOR point formula
// (sor_nb, sor_relax: the same rounding as the red-black sweeps).  Every
// neighbour therefore comes from the previous half: a relaxed Jacobi
// iteration, not red-black SOR.
//
// One kernel per iteration: p_1 lives in registers only, and p_0 goes from one
// array to another, so an iteration moves 12 bytes per cell at best (p_0 and
// rhs read, p_0 written).  See k_twin_iter.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "les_bodies.h"

using namespace les;

namespace {

constexpr int kTwRows = 2;                  // rows of a wavefront
constexpr int kTwWaves = kBlock / 64;
constexpr int kTwSpan = 2 * 62;             // cells of a row per wavefront: 64 lanes x 2, one lane a side recomputed
constexpr int kTwPlanesMax = 15;
constexpr long long kTwMinWaves = 1536;

// Two cells of a row, 4-byte aligned (rows of odd length).
struct __attribute__((packed, aligned(4))) TwPair {
    float x, y;
};
__device__ __forceinline__ float tw_left(float v) {    // lane l takes lane l - 1's v (lane 0: 0)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float tw_right(float v) {   // lane l takes lane l + 1's v (lane 63: 0)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

// One iteration, src -> dst (both halves).  A wavefront holds two cells per
// lane of kTwRows rows and marches up its planes: with p_0 of three planes and
// kTwRows + 4 rows in registers it forms p_1 one plane ahead on kTwRows + 2
// rows, and from three planes of that the new p_0.  Rows, planes and the one
// lane on either side that a neighbouring wavefront owns are computed twice,
// so that wavefronts need nothing of each other; x neighbours come from the
// lanes.  The next plane is loaded while one is computed.
// An iteration of 300x300x90 takes 32 us (two sweeps over interleaved pairs,
// 28 to 40 bytes per cell with the half-written lines: 98 us), of 150x150x90 14
// us, of 64x64x32 5.5 us.  12 bytes per cell take 12 us at 300x300x90 at the
// rate of a copy that stays in the Infinity Cache; the rest is the
// chain of a march, 1.8 us per step, with 17 steps to 15 planes.  Four rows per
// wavefront read less twice but leave fewer wavefronts: 31, 18 and 6.7 us;
// six: 49, 23 and 7.8.
template <bool ODD>
__global__ __launch_bounds__(kBlock) void k_twin_iter(Geo g, const float* __restrict__ src, const float* __restrict__ rhs,
                                                      float* __restrict__ dst, float omega, int nseg, int span, int nyb, int kt) {
    constexpr int RY = kTwRows, R0 = RY + 4, R1 = RY + 2;   // rows of p_0, p_1
    const int lane = (int)(threadIdx.x & 63);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lb = (int)xcd_block(blockIdx.x, gridDim.x);
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int seg = uni(lb % nseg), yb = uni((lb / nseg) % nyb), zb = uni(lb / (nseg * nyb));
    const int j0 = (yb * kTwWaves + wv) * RY;
    if (j0 >= g.ny) return;   // a whole wavefront
    const int kb = zb * kt, ke = min(g.nz, kb + kt);
    const int i = seg * span - 2 + 2 * lane;   // the lane's cells: i, i + 1
    const bool in_e = i >= 0 && i < g.nx, in_o = i + 1 >= 0 && i + 1 < g.nx;
    const bool last = i == g.nx - 1;           // the row's last cell, alone
    const int ic = min(max(i, 0), g.nx - 2);
    const bool own = lane > 0 && 2 * (lane - 1) < span && in_e;
    const long long sx = g.nx, sp = sx * g.ny;
    // 1 / diagonal of the lane's cells: [inside or on the grid's outer rows]
    struct Inv {
        float e[2], o[2];
    };
    Inv inner, outer;   // on inner and outer planes
#pragma unroll
    for (int ye = 0; ye < 2; ++ye) {
        const float dy = ye ? diag_y(g, 0) : g.cy + g.cy;
        const float de = diag_x(g, i) + dy, dd = diag_x(g, i + 1) + dy;
        inner.e[ye] = 1.0f / (de + (g.cz + g.cz));
        inner.o[ye] = 1.0f / (dd + (g.cz + g.cz));
        outer.e[ye] = 1.0f / (de + diag_z(g, 0));
        outer.o[ye] = 1.0f / (dd + diag_z(g, 0));
    }
    auto pick = [](bool c, float x, float y) { return c ? x : y; };
    struct Plane0 {
        float e[R0], o[R0];
    };
    struct Plane1 {
        float e[R1], o[R1];
    };
    // n rows of plane k from row j, as loaded (outside the grid its nearest row
    // and plane); trim() then clears what is outside
    auto fetch = [&](const float* q, int j, int k, auto& p, int n) {
        k = min(max(k, 0), g.nz - 1);
#pragma unroll
        for (int r = 0; r < n; ++r) {
            const TwPair v = *(const TwPair*)(q + (k * sp + min(max(j + r, 0), g.ny - 1) * sx) + ic);
            p.e[r] = v.x;
            p.o[r] = v.y;
        }
    };
    auto trim = [&](int j, int k, auto& p, int n) {
        const bool ok = k >= 0 && k < g.nz;
#pragma unroll
        for (int r = 0; r < n; ++r) {
            const bool row = ok && j + r >= 0 && j + r < g.ny;
            p.e[r] = in_e && row ? (ODD && last ? p.o[r] : p.e[r]) : 0.f;
            p.o[r] = in_o && row ? p.o[r] : 0.f;
        }
    };
    // one half at a pair of row j from the values around it
    auto half = [&](int j, const Inv& d, float e, float o, float se, float so, float ne, float no, float be, float bo, float te,
                    float to, float re, float ro, float& xe, float& xo) {
        const bool ye = j == 0 || j == g.ny - 1;
        float rt;
        xe = sor_relax(sor_nb(tw_left(o), o, se, ne, be, te, g.cx, g.cy, g.cz), pick(ye, d.e[1], d.e[0]), re, e, omega, rt);
        xo = sor_relax(sor_nb(e, tw_right(e), so, no, bo, to, g.cx, g.cy, g.cz), pick(ye, d.o[1], d.o[0]), ro, o, omega, rt);
    };
    auto inv_of = [&](int k) {
        const bool ze = k == 0 || k == g.nz - 1;
        Inv d;
#pragma unroll
        for (int ye = 0; ye < 2; ++ye) {
            d.e[ye] = pick(ze, outer.e[ye], inner.e[ye]);
            d.o[ye] = pick(ze, outer.o[ye], inner.o[ye]);
        }
        return d;
    };
    // Step k: p_1 on plane k + 1 (b2) from p_0 on k .. k + 2 (a0 .. a2), then the
    // new p_0 on plane k from p_1 on k - 1 .. k + 1; a3 and f2 come in meanwhile.
    auto step = [&](int k, const Plane0& a0, const Plane0& a1, const Plane0& a2, Plane0& a3, const Plane1& b0, const Plane1& b1,
                    Plane1& b2, const Plane1& f0, const Plane1& f1, Plane1& f2) {
        fetch(src, j0 - 2, k + 3, a3, R0);
        fetch(rhs, j0 - 1, k + 2, f2, R1);
        const Inv d1 = inv_of(k + 1), d0 = inv_of(k);
#pragma unroll
        for (int r = 0; r < R1; ++r) {
            const int j = j0 - 1 + r;
            float e, o;
            half(j, d1, a1.e[r + 1], a1.o[r + 1], a1.e[r], a1.o[r], a1.e[r + 2], a1.o[r + 2], a0.e[r + 1], a0.o[r + 1],
                 a2.e[r + 1], a2.o[r + 1], f1.e[r], f1.o[r], e, o);
            const bool row = k + 1 >= 0 && k + 1 < g.nz && j >= 0 && j < g.ny;
            b2.e[r] = in_e && row ? e : 0.f;
            b2.o[r] = in_o && row ? o : 0.f;
        }
        if (k >= kb) {
            TwPair v[RY];
#pragma unroll
            for (int r = 1; r <= RY; ++r)
                half(j0 - 1 + r, d0, b1.e[r], b1.o[r], b1.e[r - 1], b1.o[r - 1], b1.e[r + 1], b1.o[r + 1], b0.e[r], b0.o[r],
                     b2.e[r], b2.o[r], f0.e[r], f0.o[r], v[r - 1].x, v[r - 1].y);
            float* q = dst + (k * sp + j0 * sx) + i;
#pragma unroll
            for (int r = 0; r < RY; ++r)
                if (j0 + r < g.ny) {
                    if (own && in_o) *(TwPair*)(q + r * sx) = v[r];
                    else if (ODD && own) q[r * sx] = v[r].x;
                }
        }
        trim(j0 - 2, k + 3, a3, R0);
        trim(j0 - 1, k + 2, f2, R1);
    };
    Plane0 a0, a1, a2, a3;
    Plane1 b0{}, b1{}, b2, b3, f0{}, f1, f2, f3;
    fetch(src, j0 - 2, kb - 2, a0, R0);
    fetch(src, j0 - 2, kb - 1, a1, R0);
    fetch(src, j0 - 2, kb, a2, R0);
    fetch(rhs, j0 - 1, kb - 1, f1, R1);
    trim(j0 - 2, kb - 2, a0, R0);
    trim(j0 - 2, kb - 1, a1, R0);
    trim(j0 - 2, kb, a2, R0);
    trim(j0 - 1, kb - 1, f1, R1);
    // four steps a turn, so that the planes stay in their registers
#pragma unroll 1
    for (int k = kb - 2;; k += 4) {
        step(k, a0, a1, a2, a3, b0, b1, b2, f0, f1, f2);
        if (k + 1 >= ke) break;
        step(k + 1, a1, a2, a3, a0, b1, b2, b3, f1, f2, f3);
        if (k + 2 >= ke) break;
        step(k + 2, a2, a3, a0, a1, b2, b3, b0, f2, f3, f0);
        if (k + 3 >= ke) break;
        step(k + 3, a3, a0, a1, a2, b3, b0, b1, f3, f0, f1);
        if (k + 4 >= ke) break;
    }
}

__global__ __launch_bounds__(kBlock) void k_twin_copy(const float* __restrict__ src, float* __restrict__ dst, long long n) {
    for (long long e = (long long)blockIdx.x * kBlock + threadIdx.x; e < n; e += (long long)gridDim.x * kBlock) dst[e] = src[e];
}

// Per-block float64 partials of sum (rhs - A p_0)^2 and sum rhs^2, A p =
// sum_nb cn_nb p_nb - diag p, elementwise in float64 from the float32
// values; fixed order within the block.  A thread marches up 16 planes of its
// column (one cell per thread left tens of thousands of partials to copy and
// add on the host).
constexpr int kTwResidPlanes = 16;
__global__ __launch_bounds__(kBlock) void k_twin_resid(Geo g, const float* __restrict__ p,
                                                       const float* __restrict__ rhs,
                                                       double* __restrict__ part) {
    const int i0 = (int)blockIdx.x * 64 + (int)(threadIdx.x & 63);
    const int j0 = (int)blockIdx.y * kTwWaves + (int)(threadIdx.x >> 6);
    const int kb = (int)blockIdx.z * kTwResidPlanes, ke = min(g.nz, kb + kTwResidPlanes);
    double r2 = 0.0, b2 = 0.0;
    if (i0 < g.nx && j0 < g.ny) {
        const long long X = g.nx, P = X * g.ny;
        for (int k0 = kb; k0 < ke; ++k0) {
            const long long e = k0 * P + j0 * X + i0;
            auto at = [&](bool in, long long d) { return in ? (double)p[e + d] : 0.0; };
            const double nb = (double)g.cx * (at(i0 > 0, -1) + at(i0 < g.nx - 1, 1)) +
                              (double)g.cy * (at(j0 > 0, -X) + at(j0 < g.ny - 1, X)) +
                              (double)g.cz * (at(k0 > 0, -P) + at(k0 < g.nz - 1, P));
            const double ap = nb - (double)diag_of(g, i0, j0, k0) * (double)p[e];
            const double b = (double)rhs[e];
            r2 += (b - ap) * (b - ap);
            b2 += b * b;
        }
    }
    const long long lb = ((long long)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const double s = block_sum(r2);
    if (threadIdx.x == 0) part[2 * lb] = s;
    const double t = block_sum(b2);
    if (threadIdx.x == 0) part[2 * lb + 1] = t;
}

int tw_err(les_handle* h, int code, const char* what, hipError_t e = hipSuccess) {
    char buf[512];
    if (e != hipSuccess)
        std::snprintf(buf, sizeof buf, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
    else
        std::snprintf(buf, sizeof buf, "%s", what);
    h->err = buf;
    return code;
}

}  // namespace

namespace les {
void twinned_free(les_handle* h) {
    if (h->tw_q) (void)hipFree(h->tw_q);
    if (h->tw_part) (void)hipFree(h->tw_part);
    h->tw_q = nullptr;
    h->tw_part = nullptr;
}
}  // namespace les

extern "C" int les_pressure_solve_twinned(les_handle* h, const float* d_rhs, float* d_p, double omega,
                                          int32_t iters, les_solve_stats* st, double* ms,
                                          void* stream) {
    if (!h) return LES_EINVAL;
    if (!d_rhs || !d_p) return tw_err(h, LES_EINVAL, "NULL rhs or p");
    if (iters < 0) return tw_err(h, LES_EINVAL, "iters < 0");
    if (!(omega > 0.0 && omega <= 1.0)) return tw_err(h, LES_EINVAL, "omega outside (0, 1]");
    if (h->g.stretched) return tw_err(h, LES_EINVAL, "uniform grids only");
    const Geo& g = h->g;
    const long long n = (long long)g.nx * g.ny * g.nz;
    const dim3 grid((unsigned)((g.nx + 63) / 64), (unsigned)((g.ny + kTwWaves - 1) / kTwWaves),
                    (unsigned)((g.nz + kTwResidPlanes - 1) / kTwResidPlanes));
    const size_t nblocks = (size_t)grid.x * grid.y * grid.z;
    hipStream_t s = stream ? (hipStream_t)stream : h->stream;
    if (!h->tw_q) {
        // installed in the handle only once both buffers exist
        void* qa = nullptr;
        void* pa = nullptr;
        hipError_t e = hipMalloc(&qa, 2 * n * sizeof(float));
        if (e == hipSuccess) e = hipMalloc(&pa, 2 * nblocks * sizeof(double));
        if (e != hipSuccess) {
            if (qa) (void)hipFree(qa);
            if (pa) (void)hipFree(pa);
            return tw_err(h, e == hipErrorOutOfMemory ? LES_ENOMEM : LES_EDEVICE, "twinned workspace", e);
        }
        h->tw_q = qa;
        h->tw_part = (double*)pa;
    }
    float* q[2] = {(float*)h->tw_q, (float*)h->tw_q + n};
    double* part = h->tw_part;
    const dim3 block(kBlock);
    // rows in as few spans as cover them, even and as long as each other
    const int nseg = (g.nx + kTwSpan - 1) / kTwSpan, span = ((g.nx + nseg - 1) / nseg + 1) & ~1;
    const int nyb = (g.ny + kTwWaves * kTwRows - 1) / (kTwWaves * kTwRows);
    // Planes of a wavefront: a march reads four planes beyond its own, so the
    // longest one that leaves 1536 wavefronts (1.5 per SIMD), and at most 15:
    // 150x150x90 took 14.1 us this way, 17.9 with 1024 wavefronts, 19.0 with
    // 4096; 300x300x90 31.6 us with 15 planes, 35.4 with 8, 33.7 with 30.
    const long long columns = (long long)nseg * nyb * kTwWaves;
    const int kt = (int)std::min<long long>(kTwPlanesMax, std::max<long long>(1, g.nz * columns / kTwMinWaves));
    const dim3 iter_grid((unsigned)(nseg * nyb) * (unsigned)((g.nz + kt - 1) / kt));
    hipEvent_t ev[2] = {nullptr, nullptr};
    auto fin = [&](int rc) {
        for (auto& e : ev)
            if (e) (void)hipEventDestroy(e);
        return rc;
    };
    for (auto& e : ev)
        if (hipEventCreate(&e) != hipSuccess) return fin(tw_err(h, LES_EDEVICE, "hipEventCreate"));
    if (hipEventRecord(ev[0], s) != hipSuccess) return fin(tw_err(h, LES_EDEVICE, "event"));
    const float om = (float)omega;
    // d_p -> q[0] -> q[1] -> ... -> d_p; the last into q where d_p is still
    // read by it (one iteration) or is (part of) the right-hand side
    const bool apart = d_p + n <= d_rhs || d_rhs + n <= d_p;
    const auto iter = (g.nx & 1) ? k_twin_iter<true> : k_twin_iter<false>;
    const float* from = d_p;
    for (int m = 0; m < iters; ++m) {
        float* to = m > 0 && m == iters - 1 && apart ? d_p : q[m & 1];
        hipLaunchKernelGGL(iter, iter_grid, block, 0, s, g, from, d_rhs, to, om, nseg, span, nyb, kt);
        from = to;
    }
    if (hipGetLastError() != hipSuccess) return fin(tw_err(h, LES_EDEVICE, "k_twin_iter"));
    if (hipEventRecord(ev[1], s) != hipSuccess) return fin(tw_err(h, LES_EDEVICE, "event"));
    if (from != d_p) hipLaunchKernelGGL(k_twin_copy, dim3(1024), block, 0, s, from, d_p, n);
    hipLaunchKernelGGL(k_twin_resid, grid, block, 0, s, g, d_p, d_rhs, part);
    if (hipGetLastError() != hipSuccess) return fin(tw_err(h, LES_EDEVICE, "k_twin_resid"));
    std::vector<double> hp(2 * nblocks);
    hipError_t e = hipMemcpyAsync(hp.data(), part, hp.size() * sizeof(double), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fin(tw_err(h, LES_EDEVICE, "twinned solve", e));
    double r2 = 0.0, b2 = 0.0;
    for (size_t b = 0; b < nblocks; ++b) {
        r2 += hp[2 * b];
        b2 += hp[2 * b + 1];
    }
    float dt_ms = 0.f;
    if (hipEventElapsedTime(&dt_ms, ev[0], ev[1]) != hipSuccess) dt_ms = -1.f;
    if (ms) *ms = dt_ms;
    if (st) {
        st->iters = iters;
        st->rhs_norm = std::sqrt(b2);
        st->resid = b2 > 0.0 ? std::sqrt(r2 / b2) : 0.0;
        st->converged = st->resid <= h->prm.tol ? 1 : 0;
        st->reltmp2 = 0.0;
    }
    if (!std::isfinite(r2)) return fin(tw_err(h, LES_ENONFINITE, "non-finite residual"));
    return fin(LES_OK);
}
