// Runs the blocks of a launch one after another, their threads as fibers.
#include <ucontext.h>

#include "hip/hip_runtime.h"

extern char __start_lds, __stop_lds;

namespace emu {
Idx tid, bid, bdim, gdim;
uint64_t wave_buf[16][64];
bool backwards = false;
std::function<void(const char *, uint32_t, uint32_t)> start;

namespace {
enum State { kRun, kBlockWait, kWaveWait, kDone };
struct Fiber {
    ucontext_t c;
    State state;
    std::vector<char> stack = std::vector<char>(64 << 10);
};
std::vector<Fiber *> fibers;
ucontext_t main_c;
Fiber *cur;
const std::function<void()> *body;
constexpr uint64_t kMaxTurns = 20'000'000;  // of one block: the build's largest takes some 100 000

void entry() {
    (*body)();
    cur->state = kDone;
    swapcontext(&cur->c, &main_c);
}
void wait(State s) {
    cur->state = s;
    Fiber *f = cur;
    swapcontext(&f->c, &main_c);
}
[[noreturn]] void stop(const char *what, const char *name, uint32_t block) {
    printf("%s: %s block %u\n", what, name, block);
    fflush(stdout);
    _Exit(3);
}
}  // namespace

void block_sync() { wait(kBlockWait); }
void wave_sync() { wait(kWaveWait); }

void launch(dim3 g, dim3 b, const std::function<void()> &f, const char *name) {
    if (g.x == 0 || b.x == 0) stop("empty grid", name, 0);
    body = &f;
    gdim = {g.x, g.y, g.z};
    bdim = {b.x, 1, 1};
    while (fibers.size() < b.x) fibers.push_back(new Fiber);
    for (uint32_t block = 0; block < g.x; ++block) {
        bid = {block, 0, 0};
        memset(&__start_lds, 0, (size_t)(&__stop_lds - &__start_lds));
        std::vector<char> begun(b.x, 0);
        for (uint32_t t = 0; t < b.x; ++t) {
            Fiber &x = *fibers[t];
            getcontext(&x.c);
            x.c.uc_stack.ss_sp = x.stack.data();
            x.c.uc_stack.ss_size = x.stack.size();
            x.c.uc_link = &main_c;
            makecontext(&x.c, entry, 0);
            x.state = kRun;
        }
        uint64_t turns = 0;
        for (;;) {
            bool ran = false;
            uint32_t done = 0, waiting = 0;
            for (uint32_t i = 0; i < b.x; ++i) {
                const uint32_t t = backwards ? b.x - 1 - i : i;
                Fiber &x = *fibers[t];
                if (x.state == kRun) {
                    if (!begun[t] && start) start(name, block, t);
                    begun[t] = 1;
                    if (++turns > kMaxTurns) stop("endless", name, block);
                    cur = &x;
                    tid = {t, 0, 0};
                    swapcontext(&main_c, &x.c);
                    ran = true;
                }
                done += x.state == kDone;
                waiting += x.state == kBlockWait;
            }
            if (done == b.x) break;
            for (uint32_t w = 0; w * 64 < b.x; ++w) {  // a wavefront goes on when all its threads are there
                const uint32_t n = std::min(64u, b.x - w * 64);
                uint32_t here = 0;
                for (uint32_t i = 0; i < n; ++i)
                    here += fibers[w * 64 + i]->state == kWaveWait || fibers[w * 64 + i]->state == kDone;
                for (uint32_t i = 0; i < n && here == n; ++i)
                    if (fibers[w * 64 + i]->state == kWaveWait) {
                        fibers[w * 64 + i]->state = kRun;
                        ran = true;
                    }
            }
            if (waiting && waiting + done == b.x) {  // ended threads don't hold up a barrier
                for (uint32_t t = 0; t < b.x; ++t)
                    if (fibers[t]->state == kBlockWait) fibers[t]->state = kRun;
                ran = true;
            }
            if (!ran) stop("deadlock", name, block);
        }
    }
}
}  // namespace emu
