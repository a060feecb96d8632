// pic_dsmc_new.hpp -- the new electrons of the DSMC step, held in LDS until
// they are written out together.  Included behind the HIP runtime; a file of its
// own so that a host build can step a workgroup's threads through it in any order.
#pragma once

#include <stdint.h>

#ifndef PIC_DSMC_FN
#define PIC_DSMC_FN __device__ __forceinline__
#endif

constexpr int DSMC_T = 256;

// New electrons wait in LDS and take their slots from the shared counter
// together: with one addition per wave that ionizes, 16,000 for 40.96M
// particles, the contended counter alone took 200 us.
constexpr int DSMC_NEW = 2 * DSMC_T;
template <typename R>
struct DsmcNew {
    R x[DSMC_NEW], y[DSMC_NEW], z[DSMC_NEW];
    uint32_t pid[DSMC_NEW];
    int32_t cell[DSMC_NEW];
    uint32_t n;
    unsigned long long base;
};

// Writes the waiting new electrons out.  Every thread of the workgroup takes
// part, after a barrier behind the last addition; contains the barriers.  The
// number is read here, by every thread, before the barrier that lets thread 0
// set it back: a wave that read it behind that would leave its part unwritten.
template <typename R, typename Args>
PIC_DSMC_FN void dsmc_flush_new(const Args &a, DsmcNew<R> &nw)
{
    const uint32_t m = nw.n;
    __syncthreads();
    if (m == 0u) return;
    R *nx = (R *)a.v_new, *ny = nx + a.cap, *nz = ny + a.cap;
    if (threadIdx.x == 0) {
        nw.base = atomicAdd(a.count, (unsigned long long)m);
        nw.n = 0u;
    }
    __syncthreads();
    const unsigned long long base = nw.base;
    for (uint32_t i = threadIdx.x; i < m; i += DSMC_T) {
        const unsigned long long k = base + i;
        if (k < (unsigned long long)a.cap) {
            nx[k] = nw.x[i];
            ny[k] = nw.y[i];
            nz[k] = nw.z[i];
            a.pid_new[k] = nw.pid[i];
            a.cell_new[k] = nw.cell[i];
        } else {
            atomicOr(&a.dflags->sticky_state, 1);
        }
    }
    __syncthreads();
}
