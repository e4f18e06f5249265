// The kernels of the coarse BiCGStab on the CPU, one fiber per thread, in an order of waves
// that the caller picks: workgroup 1 of an RHS starts with its first `early` waves, workgroup
// 0 then runs to its end, and the rest of workgroup 1 follows.  Every order must give the
// same bits, and no wave may leave a workgroup whose other waves wait at a barrier.
// KERNELS names a file with the kernels' source, cut out of the library by the test.
// Prints the number of things that went wrong.
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

#define __global__
#define __device__
#define __forceinline__ inline
#define __launch_bounds__(n)
#define __shared__ static thread_local   // a workgroup has an OS thread of its own
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))

struct double2 {
    double x, y;
};
static double2 make_double2(double x, double y) { return {x, y}; }
struct Dim3 {
    int x = 0, y = 0;
};
static thread_local Dim3 threadIdx, blockIdx, gridDim;
using std::min;

constexpr int kWave = 64;
static int g_bad = 0;

enum { kReady, kShuffle, kBarrier, kDone };

// The threads of one workgroup.
struct Group {
    struct Fiber {
        ucontext_t ctx;
        std::vector<char> stack = std::vector<char>(1 << 16);
        int state = kReady;
    };
    int block, grid, n, cur = 0;
    std::function<void()> body;
    std::vector<std::unique_ptr<Fiber>> f;
    std::vector<double> lanes;   // values a wave's shuffle exchanges
    ucontext_t home;
    static thread_local Group *self;

    Group(int block_, int grid_, int threads, std::function<void()> b)
        : block(block_), grid(grid_), n(threads), body(b), lanes(threads) {}
    static void enter() {
        Group *g = self;
        g->body();
        g->f[g->cur]->state = kDone;
        swapcontext(&g->f[g->cur]->ctx, &g->home);
    }
    void start() {
        self = this;
        for (int i = 0; i < n; ++i) {
            f.emplace_back(new Fiber);
            getcontext(&f[i]->ctx);
            f[i]->ctx.uc_stack.ss_sp = f[i]->stack.data();
            f[i]->ctx.uc_stack.ss_size = f[i]->stack.size();
            f[i]->ctx.uc_link = nullptr;
            makecontext(&f[i]->ctx, enter, 0);
        }
    }
    void wait(int state) {
        f[cur]->state = state;
        swapcontext(&f[cur]->ctx, &home);
    }
    // all lanes of wave w are in `state`
    bool all(int w, int state) const {
        for (int i = w * kWave; i < (w + 1) * kWave; ++i)
            if (f[i]->state != state) return false;
        return true;
    }
    // wave w up to a barrier or its end
    void wave(int w) {
        for (;;) {
            for (int i = w * kWave; i < (w + 1) * kWave; ++i) {
                if (f[i]->state != kReady) continue;
                cur = i;
                threadIdx.x = i;
                blockIdx.x = block;
                gridDim.x = grid;
                swapcontext(&home, &f[i]->ctx);
            }
            if (!all(w, kShuffle)) break;
            for (int i = w * kWave; i < (w + 1) * kWave; ++i) f[i]->state = kReady;
        }
        if (!all(w, kBarrier) && !all(w, kDone)) throw "lanes of a wave apart";
    }
    // waves [0, last) up to their end (last == all) or to the first barrier
    void run(int first, int last, bool to_end) {
        for (int w = first; w < last; ++w) wave(w);
        while (to_end) {
            int done = 0;
            for (int w = 0; w < n / kWave; ++w) done += all(w, kDone);
            if (done == n / kWave) return;
            if (done) throw "a wave left while others wait at a barrier";
            for (auto &x : f) x->state = kReady;
            for (int w = 0; w < n / kWave; ++w) wave(w);
        }
    }
};
thread_local Group *Group::self = nullptr;

static void __syncthreads() { Group::self->wait(kBarrier); }
static double __shfl_xor(double v, int off, int) {
    Group &g = *Group::self;
    const int i = g.cur;
    g.lanes[i] = v;
    g.wait(kShuffle);
    const double r = g.lanes[i ^ off];
    g.wait(kShuffle);   // the slot is free when every lane has read
    return r;
}

#include KERNELS

// Runs fn as workgroups 0 and 1 of a grid of 2, workgroup 1's first `early` waves ahead.
static void launch(int early, const std::function<void()> &fn) {
    std::mutex m;
    std::condition_variable cv;
    int turn = 0;
    auto step = [&](int mine, const std::function<void()> &work) {
        std::unique_lock<std::mutex> l(m);
        cv.wait(l, [&] { return turn == mine; });
        try {
            work();
        } catch (const char *what) {
            std::fprintf(stderr, "early %d: %s\n", early, what);
            ++g_bad;
        }
        ++turn;
        cv.notify_all();
    };
    Group g0(0, 2, kMB, fn), g1(1, 2, kMB, fn);
    const int nw = kMB / kWave;
    std::thread t1([&] {
        step(0, [&] {
            g1.start();
            g1.run(0, early, false);
        });
        step(2, [&] { g1.run(early, nw, true); });
    });
    std::thread t0([&] {
        step(1, [&] {
            g0.start();
            g0.run(0, nw, true);
        });
    });
    t0.join();
    t1.join();
}

struct Solve {
    static constexpr int kLen = 700, kNp = 5;
    std::vector<double2> v[8];
    CgState st;
    double part[6], sums[3 * kNp];
    double2 &at(int k, int i) { return v[k][i]; }
};

// One RHS through the solve's kernels.  end: 0 the p update of iteration 1 finds |r| small, 1 the
// s update of iteration 1 finds <r^, v> = 0, 2 b = 0.
static Solve solve(int end, int early) {
    Solve s;
    std::memset(&s.st, 0, sizeof s.st);
    for (int k = 0; k < 8; ++k) {
        s.v[k].resize(Solve::kLen);
        for (int i = 0; i < Solve::kLen; ++i)
            s.at(k, i) = end == 2 && k == 7 ? make_double2(0, 0) : make_double2(std::sin(i + 7 * k), std::cos(3 * i + k));
    }
    const CgVec f{s.v[0].data(), s.v[1].data(), s.v[2].data(), s.v[3].data(),
                  s.v[4].data(), s.v[5].data(), s.v[6].data(), s.v[7].data()};
    // the products' sums, one per site
    auto sums = [&](double re, double im, double n2) {
        for (int i = 0; i < Solve::kNp; ++i) {
            s.sums[i] = re * (i + 1);
            s.sums[Solve::kNp + i] = im * (i + 1);
            s.sums[2 * Solve::kNp + i] = n2 * (i + 1);
        }
    };
    auto product = [&](int out, int in) {
        for (int i = 0; i < Solve::kLen; ++i) s.at(out, i) = make_double2(2 * s.at(in, i).x + 0.1, 2 * s.at(in, i).y);
    };
    std::vector<double2> x;
    launch(early, [&] { mg_cinit_kernel(&s.st, Solve::kLen, f, s.part); });
    for (int it = 0; it < 4; ++it) {
        const bool over = end == 2 || it > 1 || (it == 1 && end == 0);
        launch(early, [&] { mg_cp_kernel(&s.st, it, Solve::kLen, f, s.part, 2, end == 0 ? 1e3 : 1e-3); });
        product(4, 3);
        if (end == 1 && it == 1) sums(0, 0, 0);
        else sums(40 + it, 3, 0);
        launch(early, [&] { mg_cs_kernel(&s.st, it, Solve::kLen, f, s.sums, Solve::kNp); });
        product(6, 5);
        sums(30, 2 - it, 90);
        x = s.v[0];
        launch(early, [&] { mg_cxr_kernel(&s.st, Solve::kLen, f, s.sums, Solve::kNp, s.part); });
        const bool same = !std::memcmp(x.data(), s.v[0].data(), x.size() * sizeof(double2));
        if (same != (over || (end == 1 && it == 1))) {
            std::fprintf(stderr, "end %d early %d: iteration %d %s x\n", end, early, it, same ? "kept" : "changed");
            ++g_bad;
        }
    }
    return s;
}

int main() {
    for (int end = 0; end < 3; ++end) {
        Solve ref = solve(end, 0);
        for (int early = 1; early <= kMB / kWave; ++early) {
            Solve s = solve(end, early);
            for (int k = 0; k < 8; ++k)
                if (std::memcmp(ref.v[k].data(), s.v[k].data(), Solve::kLen * sizeof(double2))) {
                    std::fprintf(stderr, "end %d early %d: vector %d differs\n", end, early, k);
                    ++g_bad;
                }
        }
    }
    std::printf("%d\n", g_bad);
    return 0;
}
