// The resident solver's kernel (csrc/resident.hip) run on the host, one block
// after the other: every thread is a fibre, a wavefront's collective operations
// (__all, lane shifts, shuffles) and a block's barriers wait for all of it, and
// a block hands the processor on when it waits for another.  The order in which
// blocks run is the caller's: one block (the victim) can be held back, so that
// it moves by one collective operation only when all others wait.  What the
// kernel computes must not depend on it.
//
//   resident_host nx ny nz K R max_iter tag0 tol spin gate victim...
//
// victim -1: blocks run in turn; spin, gate: polls of one wait and of the roll
// call (0: the kernel's own bounds; with a bound for the roll call the victim
// comes later than that).  Prints, for each victim, a line with the control block
// and checksums of ph, pd and r0 of both colours.
#include <hip/hip_runtime.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

using std::isfinite;
using std::max;
using std::min;

namespace host {

enum Op { RUN, ALL, DPP, XOR, BARRIER, OR, DONE };

struct Fibre {
    ucontext_t ctx;
    std::unique_ptr<char[]> stack;
    Op op = RUN;
    long long in = 0, out = 0;   // value of a collective, and its result
    int arg = 0;
};

struct Grid;
struct Block {
    Grid* grid;
    unsigned id;
    std::vector<Fibre> f;
    ucontext_t sched;
    int at = 0;                  // the running fibre
};
thread_local Block* blk;

struct Grid {
    unsigned n;
    int victim, turn = 0, late = 0;   // late: rounds of polls before the victim starts
    std::function<void()> body;
    std::vector<char> done, waits;
    std::mutex m;
    std::condition_variable cv;

    // The next block after `b` yields; `waiting`: it made no progress.
    int next(int b, bool waiting) {
        waits[b] = waiting;
        if (!waiting && b != victim)
            return b;
        if (b == victim) std::fill(waits.begin(), waits.end(), 0);   // it may have let others go on
        for (unsigned q = 1; q <= n; ++q) {
            const int c = (int)((b + q) % n);
            if (!done[c] && !waits[c] && c != victim) return c;
        }
        const bool first = victim >= 0 && late > 0 && n > 1;   // the victim has yet to start, and is late
        if (victim >= 0 && !done[victim] && !first) return victim;
        if (first) --late;
        std::fill(waits.begin(), waits.end(), 0);
        for (unsigned q = 1; q <= n; ++q) {
            const int c = (int)((b + q) % n);
            if (!done[c] && (c != victim || !first)) return c;
        }
        return first ? victim : b;
    }
    void yield(int b, bool waiting) {
        std::unique_lock<std::mutex> l(m);
        if (!waiting && victim < 0) return;
        if (!waiting) std::fill(waits.begin(), waits.end(), 0);
        turn = next(b, waiting);
        cv.notify_all();
        cv.wait(l, [&] { return turn == b; });
    }
    void end(int b) {
        std::unique_lock<std::mutex> l(m);
        done[b] = 1;
        std::fill(waits.begin(), waits.end(), 0);
        turn = next(b, true);
        cv.notify_all();
    }
};

long long collective(Op op, long long v, int arg = 0) {
    Block* b = blk;
    Fibre& f = b->f[b->at];
    f.op = op;
    f.in = v;
    f.arg = arg;
    swapcontext(&f.ctx, &b->sched);
    return f.out;
}

void fibre_main() {
    blk->grid->body();
    blk->f[blk->at].op = DONE;
    swapcontext(&blk->f[blk->at].ctx, &blk->sched);
}

void run_block(Grid* grid, unsigned id, unsigned threads) {
    Block me;
    me.grid = grid;
    me.id = id;
    me.f.resize(threads);
    blk = &me;
    {
        std::unique_lock<std::mutex> l(grid->m);
        grid->cv.wait(l, [&] { return grid->turn == (int)id; });
    }
    constexpr size_t kStack = 128 << 10;
    for (Fibre& f : me.f) {
        f.stack.reset(new char[kStack]);
        getcontext(&f.ctx);
        f.ctx.uc_stack.ss_sp = f.stack.get();
        f.ctx.uc_stack.ss_size = kStack;
        f.ctx.uc_link = nullptr;
        makecontext(&f.ctx, fibre_main, 0);
    }
    const unsigned waves = threads / 64;
    while (true) {
        bool progress = false;
        unsigned barred = 0, ended = 0;
        for (unsigned w = 0; w < waves; ++w) {
            Fibre* f = &me.f[64 * w];
            for (int l = 0; l < 64; ++l)
                if (f[l].op == RUN) {
                    me.at = (int)(64 * w) + l;
                    swapcontext(&me.sched, &f[l].ctx);
                }
            const Op op = f[0].op;
            for (int l = 1; l < 64; ++l)
                if (f[l].op != op) {
                    std::printf("block %u wavefront %u: lanes at different operations\n", id, w);
                    std::exit(3);
                }
            if (op == DONE) {
                ++ended;
                continue;
            }
            if (op == BARRIER || op == OR) {
                ++barred;
                continue;
            }
            if (op == ALL) {
                long long ok = 1;
                for (int l = 0; l < 64; ++l) ok &= f[l].in;
                for (int l = 0; l < 64; ++l) f[l].out = ok;
                progress |= ok != 0;
            } else {
                for (int l = 0; l < 64; ++l) {
                    const int s = op == XOR ? l ^ f[l].arg : (f[l].arg == 0x138 ? l - 1 : l + 1);
                    f[l].out = s >= 0 && s < 64 ? f[s].in : 0;
                }
                progress = true;
            }
            for (int l = 0; l < 64; ++l) f[l].op = RUN;
            if ((int)id == grid->victim && progress) {   // one operation, then the others
                grid->yield((int)id, false);
                blk = &me;
            }
        }
        if (ended == waves) break;
        if (barred + ended == waves) {
            long long any = 0;
            for (Fibre& f : me.f)
                if (f.op == OR) any |= f.in;
            for (Fibre& f : me.f)
                if (f.op != DONE) {
                    f.out = any;
                    f.op = RUN;
                }
            progress = true;
            if ((int)id == grid->victim) grid->yield((int)id, false);
        }
        if (!progress) grid->yield((int)id, true);
    }
    grid->end((int)id);
}

struct Idx {
    unsigned x;
};
Idx tid() { return {(unsigned)blk->at}; }
Idx bid() { return {blk->id}; }
Idx dim() { return {blk->grid->n}; }
template <class T>
T move(Op op, T v, int arg) {
    long long b = 0;
    std::memcpy(&b, &v, sizeof v);
    b = collective(op, b, arg);
    std::memcpy(&v, &b, sizeof v);
    return v;
}
template <class T, class S>
T add(T* p, S v) {
    const T old = *p;
    *p += v;
    return old;
}
template <class T>
bool swap(T* p, T* old, T v) {
    if (*p != *old) {
        *old = *p;
        return false;
    }
    *p = v;
    return true;
}
template <class T>
T zero() {   // an operation no host run reaches
    std::abort();
    return T();
}
int g_victim = -1, g_late = 0;

}  // namespace host

#define threadIdx host::tid()
#define blockIdx host::bid()
#define gridDim host::dim()
#define __shared__ static thread_local
#define __launch_bounds__(...)
#define asm
#define volatile(...) ((void)0)
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, a, b, c) host::move(host::DPP, (int)(v), ctrl)
#define __shfl_xor(v, o, w) host::move(host::XOR, v, o)
#define __shfl_up(v, o, w) (host::zero<decltype(v)>())
#define __shfl_down(v, o, w) (host::zero<decltype(v)>())
#define __builtin_amdgcn_make_buffer_rsrc(...) (host::zero<__amdgpu_buffer_rsrc_t>())
#define __builtin_amdgcn_ds_bpermute(...) (host::zero<int>())
#define __all(v) ((int)host::collective(host::ALL, (v) ? 1 : 0))
#define __syncthreads() ((void)host::collective(host::BARRIER, 0))
#define __syncthreads_or(v) ((int)host::collective(host::OR, (v) ? 1 : 0))
#define __hip_atomic_load(p, ...) (*(p))
#define __hip_atomic_store(p, v, ...) ((void)(*(p) = (v)))
#define __hip_atomic_fetch_add(p, v, ...) (host::add(p, v))
#define __hip_atomic_compare_exchange_strong(p, old, v, ...) (host::swap(p, old, v))
#define __longlong_as_double(v) host::bits<double>(v)
#define __double_as_longlong(v) host::bits<long long>(v)
#define __int_as_float(v) host::bits<float>(v)
#define __uint_as_float(v) host::bits<float>(v)
#define __float_as_int(v) host::bits<int>(v)
#define __float_as_uint(v) host::bits<unsigned>(v)
namespace host {
template <class T, class S>
T bits(S s) {
    T t;
    static_assert(sizeof t == sizeof s, "");
    std::memcpy(&t, &s, sizeof t);
    return t;
}
}  // namespace host
struct __amdgpu_buffer_rsrc_t {};
#define __builtin_amdgcn_raw_buffer_load_b32(...) (host::zero<int>())
#define __builtin_amdgcn_raw_buffer_store_b32(...) (host::zero<int>())

#ifndef RESIDENT_SOURCE
#define RESIDENT_SOURCE "../paper_1504_02264_amd/csrc/resident.hip"
#endif
#include RESIDENT_SOURCE

#undef volatile
extern "C" hipError_t hipLaunchKernel(const void* f, dim3 blocks, dim3 threads, void** args, size_t, hipStream_t) {
    host::Grid grid;
    grid.n = blocks.x;
    grid.victim = host::g_victim;
    grid.late = host::g_late;
    grid.done.assign(grid.n, 0);
    grid.waits.assign(grid.n, 0);
    grid.turn = grid.victim == 0 && grid.n > 1 ? 1 : 0;
    const auto k = (void (*)(les::ResArgs))f;
    const les::ResArgs a = *(les::ResArgs*)args[0];
    grid.body = [=] { k(a); };
    std::vector<std::thread> t;
    for (unsigned b = 0; b < grid.n; ++b) t.emplace_back(host::run_block, &grid, b, threads.x);
    for (auto& x : t) x.join();
    return hipSuccess;
}

int main(int argc, char** argv) {
    if (argc < 12) return 2;
    auto num = [&](int q) { return std::atoll(argv[q]); };
    les::Geo g{};
    g.nx = (int)num(1);
    g.ny = (int)num(2);
    g.nz = (int)num(3);
    const int K = (int)num(4), R = (int)num(5), max_iter = (int)num(6);
    g.H = (g.nx + 1) / 2;
    g.S = (g.H + 1 + 31) / 32 * 32;
    g.SP = (long long)g.S * (g.ny + 2);
    g.ctot = 2LL * g.S + g.SP * (g.nz + 2);
    g.cx = 0.25f;
    g.cy = 0.11f;
    g.cz = 0.44f;
    g.cxd = g.cx;
    g.cyd = g.cy;
    g.czd = g.cz;
    g.outflow = 1;
    const les::ResPlan p = les::resident_plan(g, 256);
    if (p.shape < 0) return 4;
    for (int arg = 11; arg < argc; ++arg) {
        host::g_victim = (int)num(arg);
        host::g_late = num(10) ? 4 * (int)num(10) : 0;
        std::vector<float> mem[8];
        for (auto& v : mem) v.assign(g.ctot, 0.f);
        les::PBufs P{};
        for (int c = 0; c < 2; ++c) {
            P.ph[c] = mem[c].data();
            P.pd[c] = mem[2 + c].data();
            P.r0[c] = mem[4 + c].data();
            P.rhs[c] = mem[6 + c].data();
        }
        unsigned s = 12345;
        auto rnd = [&] {
            s = s * 1664525u + 1013904223u;
            return (float)(s >> 8) / (1 << 23) - 1.f;
        };
        double rhs2 = 0.0;
        for (int k = 0; k < g.nz; ++k)
            for (int j = 0; j < g.ny; ++j)
                for (int i = 0; i < g.nx; ++i) {
                    const long long e = g.col(i >> 1, j, k);
                    const int c = (i + j + k) & 1;
                    P.pd[c][e] = 0.1f * rnd();
                    P.rhs[c][e] = P.r0[c][e] = rnd();   // of ph = 0
                    rhs2 += (double)P.rhs[c][e] * P.rhs[c][e];
                }
        les::Ctl ctl{};
        ctl.K = K;
        ctl.max_iter = max_iter;
        ctl.tol = std::atof(argv[8]);
        ctl.rhs2 = rhs2;
        std::vector<unsigned long long> x(les::resident_bytes(p) / 8 + 1, 0);
        les::launch_resident(g, nullptr, p, P, &ctl, x.data(), 1.8, K, R, max_iter, (unsigned)num(7), 0,
                             num(9) ? (int)num(9) : les::kResSpin, num(10) ? (int)num(10) : 1 << 30);
        std::printf("blocks %u ghosts %d m %d done %d lost %u resid %.17g", p.blocks, p.g, ctl.m, ctl.done, ctl.lost, ctl.resid);
        for (int q = 0; q < 6; ++q) {
            unsigned long long h = 1469598103934665603ull;
            for (float v : mem[q]) {
                unsigned b;
                std::memcpy(&b, &v, 4);
                h = (h ^ b) * 1099511628211ull;
            }
            std::printf(" %016llx", h);
        }
        bool finite = true;
        for (int q = 0; q < 6; ++q)
            for (float v : mem[q]) finite = finite && isfinite(v);
        std::printf(" finite %d\n", finite);
        std::fflush(stdout);
    }
    return 0;
}
