#include "emulated_gpu.hpp"

#include <ucontext.h>

#include <algorithm>
#include <cstdlib>
#include <vector>

namespace emulated {
enum State { READY, AT_WAVE, AT_WG, DONE };
struct Fiber {
    Lane id;
    State state;
    int site;
    ucontext_t context;
    std::vector<unsigned char> stack;
};

dim3 block, block_dim, grid_dim;
unsigned long long exchange[16 * 64], votes[16];
static std::vector<Fiber> fibers;
static Fiber* running;
static ucontext_t scheduler;
static const std::function<void()>* kernel;

const Lane& self() { return running->id; }

static void wait(State s)
{
    running->state = s;
    swapcontext(&running->context, &scheduler);
}

void wg_sync() { wait(AT_WG); }

void wave_sync(int site)
{
    running->site = site;
    wait(AT_WAVE);
}

unsigned long long ballot(bool p, int site)
{
    unsigned long long& v = votes[running->id.wave];
    if (p) v |= 1ull << running->id.lane;
    wave_sync(site);
    const unsigned long long r = v;
    wave_sync(site + 1);
    v = 0;
    wave_sync(site + 2);
    return r;
}

static void body()
{
    (*kernel)();
    wait(DONE);
}

// Runs the lanes [begin, end) of a wave until all of them wait for the workgroup or are done.
static void run_wave(Fiber* begin, Fiber* end)
{
    for (;;) {
        for (Fiber* f = begin; f != end; ++f)
            if (f->state == READY) {
                running = f;
                swapcontext(&scheduler, &f->context);
            }
        int site = 0;
        bool waiting = false;
        for (Fiber* f = begin; f != end; ++f)
            if (f->state == AT_WAVE && (!waiting || f->site < site)) {
                site = f->site;
                waiting = true;
            }
        if (!waiting) return;
        for (Fiber* f = begin; f != end; ++f)
            if (f->state == AT_WAVE && f->site == site) f->state = READY;
    }
}

void run(dim3 grid, dim3 bl, const std::function<void()>& k)
{
    const int threads = (int)(bl.x * bl.y * bl.z);
    if (threads < 1 || threads > 1024) std::abort();
    fibers.resize(1024);
    block_dim = bl;
    grid_dim = grid;
    kernel = &k;
    for (unsigned y = 0; y < grid.y; ++y)
        for (unsigned x = 0; x < grid.x; ++x) {
            block = dim3(x, y, 0);
            for (int i = 0; i < threads; ++i) {
                Fiber& f = fibers[(size_t)i];
                f.id = {dim3((unsigned)i), i & 63, i >> 6};
                f.state = READY;
                f.stack.resize(64 * 1024);
                getcontext(&f.context);
                f.context.uc_stack.ss_sp = f.stack.data();
                f.context.uc_stack.ss_size = f.stack.size();
                f.context.uc_link = &scheduler;
                makecontext(&f.context, body, 0);
            }
            for (bool waiting = true; waiting;) {
                for (int w = 0; w < threads; w += 64)
                    run_wave(&fibers[(size_t)w], &fibers[0] + std::min(threads, w + 64));
                waiting = false;
                for (int i = 0; i < threads; ++i)
                    if (fibers[(size_t)i].state == AT_WG) {
                        fibers[(size_t)i].state = READY;
                        waiting = true;
                    }
            }
        }
}
}  // namespace emulated
