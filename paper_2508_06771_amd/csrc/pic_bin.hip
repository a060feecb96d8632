// pic_bin.hip -- binning of particles into cells (Coulombic collision steps
// CCS1-CCS3): order check, cell starts, and a stable LSD counting sort by
// cell id that moves the particle data itself.
//
// The paper builds an index list with one atomic increment per particle and
// notes that those atomics cost up to 40% of its Coulomb kernel.  Here the
// storage is kept in cell order between steps, so the steady state is a
// single streaming check of cell_of (4 B per particle); only unsorted input
// runs the sort passes, which rank elements inside a wave with ballots
// instead of atomics, so the result is stable and deterministic.
#include <string.h>

#include "pic_internal.hpp"

#define HIP_OK(x) do { if ((x) != hipSuccess) return PIC_ERR_HIP; } while (0)

namespace {

constexpr int RS_T = 1024;                    // threads of the sort's kernels
constexpr int RS_K = 4;                       // elements per thread and tile
constexpr int RS_TILE = RS_T * RS_K;
constexpr int RS_WAVES = RS_T / PIC_WAVE;
constexpr int RS_PER_WAVE = RS_TILE / RS_WAVES;
constexpr int RS_DIGITS = 256;                // largest radix
constexpr int RS_MAX_BLOCKS = 512;            // two workgroups per CU
static_assert(RS_K * PIC_WAVE * RS_WAVES == RS_TILE, "tile split");

__global__ void k_reset_flags(DevFlags *f)
{
    if (threadIdx.x == 0) {
        f->unsorted = 0;
        f->range_err = 0;
        f->seg_fallback = 0;
        for (int k = 0; k < 4; ++k) f->sort_done[k] = 0;
        f->seg_done = 0;
    }
    if (threadIdx.x < 8) f->count[threadIdx.x] = 0;
    for (unsigned q = threadIdx.x; q < 8 * QUEUE_SPLIT; q += blockDim.x) f->head[q * QUEUE_LINE] = 0;
}

// Any non-finite component of v latches PIC_ERR_NONFINITE (a debug check:
// one streaming read of the velocities).
template <typename R>
__global__ void k_check_finite(const R *__restrict__ v, int64_t m, DevFlags *f)
{
    bool bad = false;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m;
         i += (int64_t)gridDim.x * blockDim.x)
        bad |= !isfinite(v[i]);
    if (__ballot(bad) && (threadIdx.x & (PIC_WAVE - 1)) == 0) atomicOr(&f->sticky_nonfinite, 1);
}

// Latches PIC_ERR_STATE when work list `list` holds any cell.
__global__ void k_reject_list(DevFlags *f, int list)
{
    if (threadIdx.x == 0 && f->count[list] != 0u) f->sticky_state = 1;
}

__global__ void k_set_step(uint64_t *s, uint64_t v)
{
    if (threadIdx.x == 0) *s = v;
}

__global__ void k_step_inc(uint64_t *s)
{
    if (threadIdx.x == 0) *s += 1;
}

// Position i in [0, n] is the boundary between element i-1 and i: every cell
// id j in (cell_of[i-1], cell_of[i]] starts at i, so with sorted input each
// entry of cell_start is written exactly once (empty cells included).  Each
// thread takes four consecutive positions (one 16-byte load when aligned) and
// reads the id before them too, from a line it shares (passed up from the lane
// below it took 42.9 us on 40.96M sorted ids, now 41.0: 4.0 TB/s).  A workgroup reports at most once, and only
// what is not reported yet: with one atomic per wave on the same word a check
// of 16M ids out of order took 350 us, most of it waiting for that word; now 20.
constexpr int BC_T = 256;

__global__ __launch_bounds__(BC_T) void k_bin_check(const int32_t *__restrict__ cell_of, int64_t n,
                                                    int32_t n_cells, int32_t *__restrict__ cell_start,
                                                    DevFlags *f, int set_unsorted, const int *gate)
{
    __shared__ int s_bad[BC_T / PIC_WAVE], s_uns[BC_T / PIC_WAVE];
    if (gate && *gate == 0) return;
    const int lane = threadIdx.x & (PIC_WAVE - 1), wid = threadIdx.x / PIC_WAVE;
    int bad = 0, uns = 0;
    const int64_t nq = n / 4 + 1;
    const bool vec = ((uintptr_t)cell_of & 15u) == 0;
    const int64_t stride = (int64_t)gridDim.x * BC_T;
    // whole waves take part in every round (the ballot below)
    for (int64_t q0 = blockIdx.x * (int64_t)BC_T + wid * PIC_WAVE; q0 < nq; q0 += stride) {
        const int64_t i0 = (q0 + lane) * 4;
        int32_t c[5];
        c[0] = i0 > 0 && i0 <= n ? cell_of[i0 - 1] : -1;
        if (vec && i0 + 4 <= n) {
            const int4 x = *(const int4 *)(cell_of + i0);
            c[1] = x.x;
            c[2] = x.y;
            c[3] = x.z;
            c[4] = x.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) c[1 + j] = i0 + j < n ? cell_of[i0 + j] : n_cells;
        }
        bool out[4], desc = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = i0 + j;
            out[j] = i < n && (c[1 + j] < 0 || c[1 + j] >= n_cells);
            desc |= i > 0 && i < n && c[1 + j] < c[j];
            bad |= out[j];
        }
        uns |= desc;
        // A wave whose elements are out of order writes no starts: the input
        // is unsorted, gets sorted, and the starts are written by the check
        // that follows the sort.  Without this, shuffled input would cost a
        // write per cell for every ascending neighbour pair.
        if (set_unsorted && __ballot(desc) != 0) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = i0 + j;
            if (i > n || out[j]) continue;
            const int32_t cur = c[1 + j];
            const int32_t lo = c[j] + 1 < 0 ? 0 : c[j] + 1;
            for (int32_t k = lo; k <= cur && k <= n_cells; ++k) cell_start[k] = (int32_t)i;
        }
    }
    const uint64_t wb = __ballot(bad), wu = __ballot(uns);
    if (lane == 0) {
        s_bad[wid] = wb != 0;
        s_uns[wid] = wu != 0;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    int any_bad = 0, any_uns = 0;
    for (int w = 0; w < BC_T / PIC_WAVE; ++w) {
        any_bad |= s_bad[w];
        any_uns |= s_uns[w];
    }
    if (any_bad) {
        atomicOr(&f->range_err, 1);
        atomicOr(&f->sticky_range, 1);
    }
    if (any_uns && set_unsorted &&
        __hip_atomic_load(&f->unsorted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
        if (set_unsorted == 2) atomicOr(&f->sticky_state, 1);
        atomicOr(&f->unsorted, 1);
    }
}

__device__ __forceinline__ uint32_t digit_of(int32_t key, int shift, int bits)
{
    return ((uint32_t)key >> shift) & ((1u << bits) - 1u);
}

// Re-binning: one least-significant-digit pass is two launches.  The tiles of
// RS_TILE elements are split into contiguous runs, one per workgroup (at most
// two workgroups per CU), so the digit counts to scan are few (digits x
// workgroups, not digits x tiles) and the last workgroup to finish counting
// scans them: no scan launches, and no launch of one workgroup per tile.  That
// matters most when the storage is in order and all of these kernels leave at
// once: the sort's empty launches took 41 us of a 40.96M-electron step with
// ten launches of full grids, and take 12 us now.
// Two passes of 16M binary32 electrons, 5% of them moved to a neighbouring
// cell: 740 -> 345 us; of 40.96M shuffled ones: 1,690 -> 1,110 us.

// One more element of digit d, counted in LDS.  In nearly sorted storage a
// wave's elements share a digit or two: these are added by one lane each
// (64 lanes adding to one LDS word serialise).
__device__ __forceinline__ void count_digit(uint32_t *h, uint32_t d, bool valid)
{
    const int lane = threadIdx.x & (PIC_WAVE - 1);
#pragma unroll
    for (int peel = 0; peel < 2; ++peel) {
        const uint64_t m = __ballot(valid);
        if (!m) return;
        const int leader = __ffsll((unsigned long long)m) - 1;
        const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, leader);
        const uint64_t same = __ballot(valid && d == d0);
        if (lane == leader) atomicAdd(&h[d0], (uint32_t)__popcll(same));
        valid = valid && d != d0;
    }
    if (valid) atomicAdd(&h[d], 1u);
}

// Digit counts of each workgroup's run of tiles, hist[d * gridDim.x + block];
// the last workgroup turns every digit's row into an exclusive scan over the
// workgroups and writes the digits' starts behind the rows.
// The hand-over between the workgroups is outside the language's memory model
// (a relaxed counter orders nothing) and stands on this GPU's: stores and loads
// of device scope pass by the XCDs' L2s, each wave waits until its stores have
// been acknowledged (s_waitcnt, which the compiler does not take for an ordering;
// the __syncthreads behind it is one) before thread 0 counts the workgroup's
// arrival, and the last workgroup's loads are issued behind a __syncthreads that
// follows the arrival it has seen.  A release there instead would write back a
// whole L2 per workgroup (25 us; 150 us when every wave issued one).
constexpr int RC_T = 1024;
constexpr int RC_WAIT_VM = 0x0F70;   // s_waitcnt operand: vector memory only

__global__ __launch_bounds__(RC_T) void k_radix_count(const int32_t *__restrict__ key_in, int64_t n, int shift,
                                                      int bits, int tiles_per_block, uint32_t *__restrict__ hist,
                                                      unsigned int *done, const int *gate)
{
    if (gate && *gate == 0) return;
    __shared__ uint32_t h[RS_DIGITS];
    __shared__ int s_last;
    const int R = 1 << bits;
    const int lane = threadIdx.x & (PIC_WAVE - 1), wid = threadIdx.x / PIC_WAVE;
    if (threadIdx.x < RS_DIGITS) h[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t beg = (int64_t)blockIdx.x * tiles_per_block * RS_TILE;
    int64_t end = beg + (int64_t)tiles_per_block * RS_TILE;
    end = end < n ? end : n;
    const bool vec = ((uintptr_t)key_in & 15u) == 0;
    for (int64_t base = beg; base < end; base += 4 * RC_T) {
        const int64_t e = base + 4 * (int64_t)threadIdx.x;
        int32_t k[4];
        if (vec && e + 4 <= end) {
            const int4 x = *(const int4 *)(key_in + e);
            k[0] = x.x;
            k[1] = x.y;
            k[2] = x.z;
            k[3] = x.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) k[j] = e + j < end ? key_in[e + j] : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) count_digit(h, digit_of(k[j], shift, bits), e + j < end);
    }
    __syncthreads();
    const int G = gridDim.x;
    if ((int)threadIdx.x < R)
        __hip_atomic_store(&hist[(int64_t)threadIdx.x * G + blockIdx.x], h[threadIdx.x], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(RC_WAIT_VM);   // the counts are visible to the device
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(done, 1u) == (unsigned)(G - 1);
    __syncthreads();
    if (!s_last) return;
    // one wave per digit row: all of the row's loads in flight together
    constexpr int RU = RS_MAX_BLOCKS / PIC_WAVE;
    for (int d = wid; d < R; d += RC_T / PIC_WAVE) {
        uint32_t *row = hist + (int64_t)d * G;
        uint32_t v[RU], carry = 0;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int g = u * PIC_WAVE + lane;
            v[u] = g < G ? __hip_atomic_load(&row[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int g = u * PIC_WAVE + lane;
            const uint32_t inc = wave_incl_scan_dpp(v[u]);
            if (g < G) row[g] = carry + inc - v[u];
            carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, PIC_WAVE - 1);
        }
        if (lane == 0) h[d] = carry;
    }
    __syncthreads();
    if (wid == 0) {
        uint32_t carry = 0;
        for (int d0 = 0; d0 < R; d0 += PIC_WAVE) {
            const int d = d0 + lane;
            const uint32_t c = d < R ? h[d] : 0u;
            const uint32_t inc = wave_incl_scan_dpp(c);
            if (d < R) hist[(int64_t)R * G + d] = carry + inc - c;
            carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, PIC_WAVE - 1);
        }
    }
}

// Stable placement of the workgroup's tiles, one after another.  Wave w holds
// elements [w * 256, w * 256 + 256) of the tile in four rounds of 64 (keys and
// payload in registers, every load in flight before the first use); an
// element's rank among equal digits of its wave comes from ballots over the
// digit bits and a per-wave running count in LDS (no block barrier while
// ranking).  The waves' counts then give each (wave, digit) its start inside
// the tile.  The arrays pass through LDS one at a time: every element goes to
// its place in the digit-sorted tile and the tile is written out in slot
// order, so consecutive slots of one digit go to consecutive addresses.
// Bound by the memory: 40 bytes per binary32 electron at 4.6 TB/s when few
// digits meet in a tile, 3.3 TB/s when 64 digits do (runs of 64 elements).
// Staging one array at a time (two buffers of RS_TILE entries instead of a
// whole tile of every array) and loading the payload with the keys leaves one
// memory round trip per tile; tiles of 2,048 on 512 threads, three workgroups
// per CU, have runs half as long: 590 against 490 us per pass of 40.96M
// shuffled electrons.
template <int N32, int N64, bool IOTA>
__global__ __launch_bounds__(RS_T) void k_radix_place(RadixPass p, int tiles_per_block,
                                                      const uint32_t *__restrict__ hist)
{
    if (p.gate && *p.gate == 0) return;
    constexpr int ES = N64 > 0 ? 8 : 4;
    __shared__ __align__(16) unsigned char buf[2][(size_t)RS_TILE * ES];
    __shared__ uint16_t wc[RS_WAVES * RS_DIGITS];   // per-wave digit counts, then starts in the tile
    __shared__ uint32_t goff[RS_DIGITS];            // next output slot of each digit
    __shared__ uint32_t tst[RS_DIGITS];             // digit starts inside the tile
    __shared__ uint32_t dlt[RS_DIGITS];             // output slot minus slot in the tile
    __shared__ uint32_t wsum[RS_DIGITS / PIC_WAVE];
    const int R = 1 << p.bits, G = gridDim.x;
    const int lane = threadIdx.x & (PIC_WAVE - 1), wid = threadIdx.x / PIC_WAVE;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (PIC_WAVE - lane));
    if ((int)threadIdx.x < R)
        goff[threadIdx.x] = hist[(int64_t)R * G + threadIdx.x] + hist[(int64_t)threadIdx.x * G + blockIdx.x];
    uint16_t *wrun = wc + wid * RS_DIGITS;
    const int64_t ntiles = (p.n + RS_TILE - 1) / RS_TILE;
    int64_t t_end = ((int64_t)blockIdx.x + 1) * tiles_per_block;
    t_end = t_end < ntiles ? t_end : ntiles;
    for (int64_t t = (int64_t)blockIdx.x * tiles_per_block; t < t_end; ++t) {
        const int64_t tile = t * RS_TILE;
        const int tn = (int)(p.n - tile < RS_TILE ? p.n - tile : RS_TILE);   // elements in this tile
        int32_t key[RS_K];
        uint32_t x32[N32][RS_K];
        uint64_t x64[N64 > 0 ? N64 : 1][RS_K];
        // elements past the end reload the tile's last one (not placed)
#pragma unroll
        for (int r = 0; r < RS_K; ++r) {
            const int le = wid * RS_PER_WAVE + r * PIC_WAVE + lane;
            key[r] = ld_at(p.key_in + tile, (uint32_t)(le < tn ? le : tn - 1));
        }
#pragma unroll
        for (int s = 0; s < N32; ++s)
#pragma unroll
            for (int r = 0; r < RS_K; ++r) {
                const int le = wid * RS_PER_WAVE + r * PIC_WAVE + lane;
                const uint32_t i = (uint32_t)(le < tn ? le : tn - 1);
                if constexpr (IOTA) x32[s][r] = (uint32_t)tile + i;   // one array: the element's index
                else x32[s][r] = ld_at(p.p32_in[s] + tile, i);
            }
#pragma unroll
        for (int s = 0; s < N64; ++s)
#pragma unroll
            for (int r = 0; r < RS_K; ++r) {
                const int le = wid * RS_PER_WAVE + r * PIC_WAVE + lane;
                x64[s][r] = ld_at(p.p64_in[s] + tile, (uint32_t)(le < tn ? le : tn - 1));
            }
#pragma unroll
        for (int q = 0; q < RS_WAVES * RS_DIGITS / 2 / RS_T; ++q) ((uint32_t *)wc)[threadIdx.x + q * RS_T] = 0u;
        lds_barrier();
        uint32_t pos[RS_K];   // rank in the wave, then slot in the tile
#pragma unroll
        for (int r = 0; r < RS_K; ++r) {
            const bool valid = wid * RS_PER_WAVE + r * PIC_WAVE + lane < tn;
            const uint32_t d = digit_of(key[r], p.shift, p.bits);
            uint64_t peers = __ballot(valid);
            for (int b = 0; b < p.bits; ++b) {
                const uint64_t m = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? m : ~m;
            }
            const uint32_t before = valid ? wrun[d] : 0u;
            pos[r] = before + __popcll(peers & lt);
            // the group's first lane advances the wave's count (same wave: LDS
            // operations stay in order)
            if (valid && (peers & lt) == 0ull) wrun[d] = (uint16_t)(before + __popcll(peers));
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the count is in LDS
            __builtin_amdgcn_wave_barrier();
        }
        lds_barrier();
        // wave starts per digit, then the digits' starts in the tile
        uint32_t tot = 0, inc = 0;
        if (threadIdx.x < RS_DIGITS) {
            if ((int)threadIdx.x < R) {
#pragma unroll
                for (int w = 0; w < RS_WAVES; ++w) {
                    const uint32_t c = wc[w * RS_DIGITS + threadIdx.x];
                    wc[w * RS_DIGITS + threadIdx.x] = (uint16_t)tot;
                    tot += c;
                }
            }
            inc = wave_incl_scan(tot);
            if (lane == PIC_WAVE - 1) wsum[wid] = inc;
        }
        lds_barrier();
        if ((int)threadIdx.x < R) {
            uint32_t off = inc - tot;
            for (int w = 0; w < wid; ++w) off += wsum[w];
            tst[threadIdx.x] = off;
            dlt[threadIdx.x] = goff[threadIdx.x] - off;
            goff[threadIdx.x] += tot;
        }
        lds_barrier();
        uint32_t *k0 = (uint32_t *)buf[0];
#pragma unroll
        for (int r = 0; r < RS_K; ++r) {
            const uint32_t d = digit_of(key[r], p.shift, p.bits);
            pos[r] += tst[d] + wrun[d];
            if (wid * RS_PER_WAVE + r * PIC_WAVE + lane < tn) k0[pos[r]] = (uint32_t)key[r];
        }
        lds_barrier();
        uint32_t dst[RS_K];   // output slots of tile slots threadIdx.x + r * RS_T
#pragma unroll
        for (int r = 0; r < RS_K; ++r) {
            const int q = threadIdx.x + r * RS_T;
            dst[r] = 0u;
            if (q < tn) {
                const uint32_t k = k0[q];
                dst[r] = dlt[digit_of((int32_t)k, p.shift, p.bits)] + (uint32_t)q;
                p.key_out[dst[r]] = (int32_t)k;
            }
        }
#pragma unroll
        for (int s = 0; s < N32; ++s) {
            uint32_t *st = (uint32_t *)buf[(s + 1) & 1];
#pragma unroll
            for (int r = 0; r < RS_K; ++r)
                if (wid * RS_PER_WAVE + r * PIC_WAVE + lane < tn) st[pos[r]] = x32[s][r];
            lds_barrier();
#pragma unroll
            for (int r = 0; r < RS_K; ++r) {
                const int q = threadIdx.x + r * RS_T;
                if (q < tn) p.p32_out[s][dst[r]] = st[q];
            }
        }
#pragma unroll
        for (int s = 0; s < N64; ++s) {
            uint64_t *st = (uint64_t *)buf[(N32 + s + 1) & 1];
#pragma unroll
            for (int r = 0; r < RS_K; ++r)
                if (wid * RS_PER_WAVE + r * PIC_WAVE + lane < tn) st[pos[r]] = x64[s][r];
            lds_barrier();
#pragma unroll
            for (int r = 0; r < RS_K; ++r) {
                const int q = threadIdx.x + r * RS_T;
                if (q < tn) p.p64_out[s][dst[r]] = st[q];
            }
        }
    }
}

// Cells by size class.  lists[c * n_cells + k] = k-th cell of class c; the
// class lengths go to flags->count[c].  Within a class the order is
// arbitrary: cells are independent and their random numbers depend only on
// (seed, step, pid), so processing order never changes results.  Cells the
// gate defers go to the deferred list when they still need a visit.
// A workgroup of 1,024 cells reserves its places with one atomic per list (and
// one for its segments and work items): these counters are contended by the
// whole device at about 12 ns an addition, so with one addition per wave and
// list 200,000 cells took 40 us, 16,384 cells of log-normal size 23 us.
constexpr int QB_T = 1024;
constexpr int QB_W = QB_T / PIC_WAVE;

// Segment plan of cell h of the multi-workgroup list with cnt members: S
// segments (equal key ranges) from table entry sb, and the counting work items
// from cb.
__device__ void plan_segments(const SegScratch &ss, int h, uint32_t S, uint32_t nch, uint32_t sb, uint32_t cb)
{
    ss.hc_fb[h] = 0;
    ss.hc_S[h] = S;
    ss.hc_seg[h] = (int32_t)sb;
    ss.hc_chunk[h] = (int32_t)cb;
    for (uint32_t q = 0; q < S; ++q) {
        ss.sg_cell[sb + q] = h;
        ss.sg_cnt[sb + q] = 0;
        ss.bnd_head[sb + q] = -1;
        ss.bnd_tail[sb + q] = -1;
    }
    for (uint32_t q = 0; q < nch; ++q) ss.ch_owner[cb + q] = h;
}

__global__ __launch_bounds__(QB_T) void k_build_queue(const int32_t *__restrict__ cell_start, int32_t n_cells,
                                                      ClassCaps caps, int32_t *__restrict__ lists, DevFlags *f,
                                                      const uint8_t *__restrict__ skip, int visit,
                                                      SegScratch ss, int plan, int seg_target)
{
    __shared__ uint32_t wcnt[QUEUE_LISTS][QB_W];   // cells per list and wave, then the wave's first place
    __shared__ uint32_t wtot[QB_W];
    __shared__ uint32_t s_base[2];                 // first segment, first work item
    const int lane = threadIdx.x & (PIC_WAVE - 1), wid = threadIdx.x / PIC_WAVE;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (PIC_WAVE - lane));
    for (int64_t j0 = blockIdx.x * (int64_t)QB_T; j0 < n_cells; j0 += (int64_t)gridDim.x * QB_T) {
        const int64_t j = j0 + threadIdx.x;
        int cls = -1;
        int32_t cnt = 0;
        if (j < n_cells) {
            // every cell is visited: cells with fewer than two members still
            // need the null-collision step and their moment sums
            cnt = cell_start[j + 1] - cell_start[j];
            cls = caps.ncls;
            for (int c = caps.ncls - 1; c >= 0; --c)
                if (cnt <= caps.cap[c]) cls = c;
            if (skip && skip[j]) cls = visit ? LIST_DEFERRED : -1;
        }
        uint32_t mine = 0;   // place among the wave's cells of the same list
#pragma unroll
        for (int c = 0; c < QUEUE_LISTS; ++c) {
            const uint64_t m = __ballot(cls == c);
            if (cls == c) mine = (uint32_t)__popcll(m & lt);
            if (lane == 0) wcnt[c][wid] = (uint32_t)__popcll(m);
        }
        __syncthreads();
        if (threadIdx.x < QUEUE_LISTS) {
            uint32_t tot = 0;
            for (int w = 0; w < QB_W; ++w) tot += wcnt[threadIdx.x][w];
            uint32_t b = tot ? atomicAdd(&f->count[threadIdx.x], tot) : 0u;
            for (int w = 0; w < QB_W; ++w) {
                const uint32_t c = wcnt[threadIdx.x][w];
                wcnt[threadIdx.x][w] = b;
                b += c;
            }
        }
        const bool seg = plan && cls == caps.ncls;
        const bool any_seg = __syncthreads_or(seg ? 1 : 0) != 0;   // also: the places above are set
        uint32_t h = 0;
        if (cls >= 0) {
            h = wcnt[cls][wid] + mine;
            lists[(int64_t)cls * n_cells + h] = (int32_t)j;
        }
        if (any_seg) {
            const int64_t want = ((int64_t)cnt + seg_target - 1) / seg_target;
            const bool fb = seg && want > SEG_MAX;
            const uint32_t S = seg && !fb ? (want > 0 ? (uint32_t)want : 1u) : 0u;
            const uint32_t nch = S ? (uint32_t)(((int64_t)cnt + SEG_CHUNK - 1) / SEG_CHUNK) : 0u;
            const uint32_t so = block_excl(S, wtot), co = block_excl(nch, wtot);
            if (threadIdx.x == QB_T - 1) {
                s_base[0] = so + S ? atomicAdd(&f->count[SEG_SLOT], so + S) : 0u;
                s_base[1] = co + nch ? atomicAdd(&f->count[CHUNK_SLOT], co + nch) : 0u;
            }
            __syncthreads();
            if (S) plan_segments(ss, (int)h, S, nch, s_base[0] + so, s_base[1] + co);
            if (fb) {
                ss.hc_fb[h] = 1;
                ss.hc_S[h] = 0;
                f->seg_fallback = 1;
            }
        }
        __syncthreads();   // the shared places are rewritten by the next round
    }
}

int grid_for(int64_t n, int threads, int cap)
{
    int64_t g = (n + threads - 1) / threads;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

}  // namespace

int launch_reset_flags(DevFlags *flags, hipStream_t st)
{
    hipLaunchKernelGGL(k_reset_flags, dim3(1), dim3(8 * QUEUE_SPLIT), 0, st, flags);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

int launch_check_finite(int dtype, const void *v, int64_t n, DevFlags *flags, hipStream_t st)
{
    if (n <= 0) return PIC_OK;
    const int g = grid_for(3 * n, 256, 4096);
    if (dtype == PIC_F32)
        hipLaunchKernelGGL(k_check_finite<float>, dim3(g), dim3(256), 0, st, (const float *)v, 3 * n, flags);
    else
        hipLaunchKernelGGL(k_check_finite<double>, dim3(g), dim3(256), 0, st, (const double *)v, 3 * n, flags);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

int launch_reject_list(DevFlags *flags, int list, hipStream_t st)
{
    hipLaunchKernelGGL(k_reject_list, dim3(1), dim3(64), 0, st, flags, list);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

int launch_set_step(uint64_t *step_dev, uint64_t value, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_step, dim3(1), dim3(64), 0, st, step_dev, value);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

int launch_step_inc(uint64_t *step_dev, hipStream_t st)
{
    hipLaunchKernelGGL(k_step_inc, dim3(1), dim3(64), 0, st, step_dev);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

int launch_bin_check(const int32_t *cell_of, int64_t n, int32_t n_cells, int32_t *cell_start,
                     DevFlags *flags, int set_unsorted, const int *gate, hipStream_t st)
{
    hipLaunchKernelGGL(k_bin_check, dim3(grid_for(n / 4 + 1, BC_T, 2048)), dim3(BC_T), 0, st, cell_of, n,
                       n_cells, cell_start, flags, set_unsorted, gate);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

// Scratch of a pass: a count per digit and workgroup (at most one workgroup per
// tile, and RS_MAX_BLOCKS), the digits' starts behind them, and alignment.
size_t radix_scratch_bytes(int64_t n)
{
    const int64_t tiles = (n + RS_TILE - 1) / RS_TILE;
    const int64_t groups = tiles < RS_MAX_BLOCKS ? tiles : RS_MAX_BLOCKS;
    return (size_t)(RS_DIGITS * (groups + 1)) * sizeof(uint32_t) + 512;
}

namespace {
template <int N32, int N64, bool IOTA>
void place_pass(const RadixPass &p, int G, int tpb, const uint32_t *hist, hipStream_t st)
{
    hipLaunchKernelGGL((k_radix_place<N32, N64, IOTA>), dim3(G), dim3(RS_T), 0, st, p, tpb, hist);
}
}  // namespace

int radix_pass(const RadixPass &p, const BinScratch &s, hipStream_t st)
{
    if (p.n <= 0) return PIC_OK;
    const int64_t tiles = (p.n + RS_TILE - 1) / RS_TILE;
    const int tpb = (int)((tiles + RS_MAX_BLOCKS - 1) / RS_MAX_BLOCKS);
    const int G = (int)((tiles + tpb - 1) / tpb);
    hipLaunchKernelGGL(k_radix_count, dim3(G), dim3(RC_T), 0, st, p.key_in, p.n, p.shift, p.bits, tpb, s.hist,
                       p.done, p.gate);
    const bool iota = p.iota_slot == 0;
    if (p.n32 == 4 && p.n64 == 0 && !iota) place_pass<4, 0, false>(p, G, tpb, s.hist, st);
    else if (p.n32 == 1 && p.n64 == 3 && !iota) place_pass<1, 3, false>(p, G, tpb, s.hist, st);
    else if (p.n32 == 1 && p.n64 == 0 && iota) place_pass<1, 0, true>(p, G, tpb, s.hist, st);
    else if (p.n32 == 1 && p.n64 == 0 && !iota) place_pass<1, 0, false>(p, G, tpb, s.hist, st);
    else return PIC_ERR_ARG;   // no caller sorts other payloads
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

int launch_build_queue(const int32_t *cell_start, int32_t n_cells, const ClassCaps &caps,
                       int32_t *lists, DevFlags *flags, const uint8_t *skip, int visit,
                       const SegScratch *seg, int seg_target, hipStream_t st)
{
    SegScratch ss;
    memset(&ss, 0, sizeof(ss));
    if (seg) ss = *seg;
    hipLaunchKernelGGL(k_build_queue, dim3(grid_for(n_cells, QB_T, 512)), dim3(QB_T), 0, st,
                       cell_start, n_cells, caps, lists, flags, skip, visit, ss, seg ? 1 : 0,
                       seg_target);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}
