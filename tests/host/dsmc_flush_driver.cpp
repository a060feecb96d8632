// Steps the threads of one workgroup through dsmc_flush_new, one after another
// between barriers, in several orders.  A thread that leaves is counted out of
// the later barriers, as on the GPU.
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <vector>

static struct { unsigned x; } threadIdx;
static void __syncthreads();
template <typename X, typename Y>
static X atomicAdd(X *p, Y v)
{
    const X o = *p;
    *p += (X)v;
    return o;
}
static void atomicOr(int *p, int v) { *p |= v; }
#define PIC_DSMC_FN static inline
#include "pic_dsmc_new.hpp"

struct Flags { int sticky_state; };
struct Args {
    void *v_new;
    int64_t cap;
    uint32_t *pid_new;
    int32_t *cell_new;
    unsigned long long *count;
    Flags *dflags;
};

static Args args;
static DsmcNew<float> nw;
static ucontext_t sched, ctx[DSMC_T];
static bool done[DSMC_T];
static unsigned cur;

static void __syncthreads()
{
    swapcontext(&ctx[cur], &sched);
    threadIdx.x = cur;
}

static void body()
{
    dsmc_flush_new<float>(args, nw);
    done[cur] = true;
    swapcontext(&ctx[cur], &sched);
}

// order: 0 first thread first, 1 last thread first, 2 from the middle on
static void run(int order, std::vector<char> &stacks, size_t ss)
{
    for (int t = 0; t < DSMC_T; ++t) {
        done[t] = false;
        getcontext(&ctx[t]);
        ctx[t].uc_stack.ss_sp = stacks.data() + t * ss;
        ctx[t].uc_stack.ss_size = ss;
        ctx[t].uc_link = nullptr;
        makecontext(&ctx[t], body, 0);
    }
    for (bool live = true; live;) {   // one round: every live thread to its next barrier
        live = false;
        for (int q = 0; q < DSMC_T; ++q) {
            const int t = order == 0 ? q : order == 1 ? DSMC_T - 1 - q : (q + DSMC_T / 2) % DSMC_T;
            if (done[t]) continue;
            live = true;
            cur = threadIdx.x = (unsigned)t;
            swapcontext(&sched, &ctx[t]);
        }
    }
}

int main()
{
    const size_t ss = 64 * 1024;
    std::vector<char> stacks(ss * DSMC_T);
    const uint32_t sizes[] = {0, 1, 63, 64, 65, 255, 256, 257, 511, 512};
    for (int order = 0; order < 3; ++order)
        for (uint32_t m : sizes)
            for (int64_t room : {(int64_t)600, (int64_t)m, (int64_t)(m / 2)}) {
                const int64_t first = 7, cap = first + room;
                std::vector<float> v(3 * cap, -1.0f);
                std::vector<uint32_t> pid(cap, 0xffffffffu);
                std::vector<int32_t> cell(cap, -1);
                unsigned long long count = first;
                Flags fl = {0};
                args = {v.data(), cap, pid.data(), cell.data(), &count, &fl};
                for (uint32_t i = 0; i < m; ++i) {
                    nw.x[i] = 1.0f + i;
                    nw.y[i] = 2.0f + i;
                    nw.z[i] = 3.0f + i;
                    nw.pid[i] = 100 + i;
                    nw.cell[i] = 5 + (int)i;
                }
                nw.n = m;
                run(order, stacks, ss);
                long bad = 0;
                for (uint32_t i = 0; i < m && i < room; ++i) {
                    const int64_t k = first + i;
                    bad += v[k] != 1.0f + i || v[cap + k] != 2.0f + i || v[2 * cap + k] != 3.0f + i ||
                           pid[k] != 100 + i || cell[k] != 5 + (int)i;
                }
                if (bad || nw.n != 0 || count != first + m || fl.sticky_state != (m > room)) {
                    printf("order %d, %u waiting, room %ld: %ld not written, n %u, count %llu, state %d\n", order,
                           m, (long)room, bad, nw.n, count, fl.sticky_state);
                    return 1;
                }
            }
    printf("dsmc flush ok\n");
    return 0;
}
