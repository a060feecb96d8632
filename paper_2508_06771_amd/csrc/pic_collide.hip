// pic_collide.hip -- the per-cell Coulomb collision pass (Table "Coulombic
// Collision Steps", CCS3-CCS5) with the null-collision step, the per-cell
// FP64 conservation sums and the moment sums fused into the same pass.
//
// The paper keeps particles unsorted, builds index lists and then gathers
// velocities at random addresses for every pair ("6 reads and 6 writes" per
// pair, non-coalesced, the bulk of its Coulomb time).  Here storage is in
// cell order, so one workgroup owns a cell's contiguous range: velocities and
// ids are streamed in and out coalesced exactly once, the random pairing is a
// sort of the cell's keys in LDS, and partners meet through LDS.  The random
// numbers come from Philox in registers (no pre-generated arrays).
//
// Per cell (n members, all in registers: K per thread):
//   1. load pid, v; one Philox4x32-10 call per particle (domain 0):
//      word0 pairing key, word1 null-collision candidate, words 2-3 for the pair
//   2. sort by (key, pid) with an LDS bucket sort: bucket = (key * nb) >> 32
//      is monotone in key, so buckets in order and (key, pid) order inside a
//      bucket (expected 2 members) give the full order
//   3. pairs (2i, 2i+1): second members post (v, word2) in LDS, first members
//      apply the Takizuka & Abe rotation and post the half change back
//   4. optional FP64 momentum/energy correction, null-collision scattering of
//      candidates, optional moment sums; store v.
//
// Cells larger than the biggest LDS class take the "huge" path below, the same
// algorithm with its per-cell arrays in global scratch indexed by slot.
#include <float.h>

#include <algorithm>
#include <type_traits>

#include "pic_internal.hpp"

#define HIP_OK(x) do { if ((x) != hipSuccess) return PIC_ERR_HIP; } while (0)

namespace {

constexpr double PI_D = 3.14159265358979323846;

// Half of the Takizuka & Abe velocity change of the pair (a, b) with
// relative velocity u = v_a - v_b.  C = 8 pi n lnL dt (so s^2 = C / |u|^3);
// U1, U2 (words 2, 3 of a) give z by Box-Muller, U3 (word 2 of b) the
// azimuth.  The rotation keeps |u|: u' = u cos T + |u| sin T (cos P e1 + sin P e2).
// The standard normal deviate of the pair from words 2, 3 of its first member
// (Box-Muller, cosine branch; the hardware log is base 2 and the cosine takes
// revolutions; the hardware square root, within 1 ulp, where the correctly
// rounded one costs about 16 more instructions).
__device__ __forceinline__ float ta_z(uint32_t wa2, uint32_t wa3)
{
    return __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u01f(wa2))) *
           __builtin_amdgcn_cosf(u01f(wa3));
}

// The same from the deviate z already drawn.
__device__ __forceinline__ void ta_half_z(float ux, float uy, float uz, float C, float z,
                                          uint32_t wb2, float &hx, float &hy, float &hz)
{
    const float uu = ux * ux + uy * uy + uz * uz;
    hx = hy = hz = 0.0f;
    if (!(uu >= FLT_MIN)) return;   // u = 0 (or below the normal range): no change
    const float rinv = __builtin_amdgcn_rsqf(uu);     // 1 / |u|
    const float um = uu * rinv;                        // |u|
    const float s = __builtin_amdgcn_sqrtf(C * rinv * rinv * rinv);
    const float d = s * z;
    // sin T = 2d / (1 + d^2), 1 - cos T = 2 d^2 / (1 + d^2); for |d| > 1 the
    // same ratios in t = 1/d avoid overflow of d^2.
    float sin_t, omc;
    if (fabsf(d) <= 1.0f) {
        const float inv = __builtin_amdgcn_rcpf(1.0f + d * d);
        sin_t = 2.0f * d * inv;
        omc = 2.0f * d * d * inv;
    } else {
        const float t = __builtin_amdgcn_rcpf(d);
        const float inv = __builtin_amdgcn_rcpf(1.0f + t * t);
        sin_t = 2.0f * t * inv;
        omc = 2.0f * inv;
    }
    const float u3 = u01f(wb2);
    const float cp = __builtin_amdgcn_cosf(u3), sp = __builtin_amdgcn_sinf(u3);  // revolutions
    const float up2 = ux * ux + uy * uy;
    float dx, dy, dz;
    if (up2 > 0.0f) {
        const float upinv = __builtin_amdgcn_rsqf(up2);
        const float up = up2 * upinv;
        const float a = uz * sin_t * cp;
        const float b = um * sin_t * sp;
        dx = (ux * upinv) * a - (uy * upinv) * b - ux * omc;
        dy = (uy * upinv) * a + (ux * upinv) * b - uy * omc;
        dz = -up * sin_t * cp - uz * omc;
    } else {
        dx = um * sin_t * cp;
        dy = um * sin_t * sp;
        dz = -uz * omc;
    }
    hx = 0.5f * dx;
    hy = 0.5f * dy;
    hz = 0.5f * dz;
}

template <bool MEM = false>
__device__ __forceinline__ void ta_half(float ux, float uy, float uz, float C, uint32_t wa2,
                                        uint32_t wa3, uint32_t wb2, float &hx, float &hy,
                                        float &hz)
{
    ta_half_z(ux, uy, uz, C, ta_z(wa2, wa3), wb2, hx, hy, hz);
}

template <bool MEM = false>   // see m64_ta_half
__device__ __forceinline__ void ta_half(double ux, double uy, double uz, double C, uint32_t wa2,
                                        uint32_t wa3, uint32_t wb2, double &hx, double &hy,
                                        double &hz)
{
    m64_ta_half<MEM>(ux, uy, uz, C, u01d(wa2), u01d(wa3), u01d(wb2), hx, hy, hz);
}

template <typename R, bool MEM = false>
__device__ __forceinline__ void mcc_scatter(R &vx, R &vy, R &vz, uint32_t pid, uint64_t seed,
                                            uint32_t step, double mass_ratio)
{
    scatter_dir<MEM>(vx, vy, vz, draw4(seed, pid, step, 1u, 0u), mass_ratio);
}

// The same with CALL out of line in binary64, for the kernel of all classes: its
// one workgroup a CU waits for every spilled register of a scatter in line.  6M
// electrons in cells of 300, four steps: 5,379 us with it in line, 2,758 so, 2,434
// without null collisions (of 1,000: 2,336, 1,250, 1,114).
struct Velocity {
    double x, y, z;
};
__device__ __noinline__ Velocity scatter_call(double x, double y, double z, W4 w, double mass_ratio)
{
    scatter_dir<false>(x, y, z, w, mass_ratio);
    return {x, y, z};
}
template <typename R, bool CALL, bool MEM = false>
__device__ __forceinline__ void mcc_scatter_as(R &vx, R &vy, R &vz, uint32_t pid, uint64_t seed, uint32_t step,
                                               double mass_ratio)
{
    if constexpr (CALL && std::is_same<R, double>::value) {
        const Velocity v = scatter_call(vx, vy, vz, draw4(seed, pid, step, 1u, 0u), mass_ratio);
        vx = v.x;
        vy = v.y;
        vz = v.z;
    } else {
        mcc_scatter<R, MEM>(vx, vy, vz, pid, seed, step, mass_ratio);
    }
}

__device__ __forceinline__ uint64_t read_step(const CollideArgs &a)
{
    return a.step_dev ? *a.step_dev : a.step;
}

__device__ __forceinline__ double cell_C(const CollideArgs &a, int cell)
{
    const double dens = a.density ? a.density[cell] : 1.0;
    const double dts = a.dt_scale ? a.dt_scale[cell] : 1.0;
    return 8.0 * PI_D * dens * a.lnL * a.dt * dts;
}

__device__ __forceinline__ bool gated_off(const CollideArgs &a)
{
    if (a.dflags->range_err) return true;
    if ((a.flags & PIC_ASSUME_SORTED) && a.dflags->unsorted) return true;
    return false;
}

// Variants compiled per kernel: which optional parts of the pass exist.
enum { F_MCC = 1, F_CONS = 2, F_MOM = 4, F_PAIRS = 8, F_WT = 16, F_NANBU = 32, F_TRIP = 64, F_CALL = 128 };

// Variable-weight rule for the pair (a, b) with half change h (a += h,
// b -= h in the uniform step): the member of smaller weight always takes its
// half, the other one iff U4 * w_heavy < w_light in binary64, U4 = U(word 3 of
// b's domain-0 draw).  Equal weights: both take it.
template <typename R>
__device__ __forceinline__ void weight_rule(R wa, R wb, uint32_t w3b, bool &take_a, bool &take_b)
{
    take_a = take_b = true;
    if (wa != wb) {
        const double U4 = u01d(w3b);
        if (wa > wb) take_a = U4 * (double)wa < (double)wb;
        else take_b = U4 * (double)wb < (double)wa;
    }
}

// Pair-major exchange records.  In each round the members whose sorted
// position falls in the round post their velocity and word 2 at that
// position (first members also word 3, at the pair index); one thread per
// pair applies the Takizuka & Abe rotation and writes both new velocities
// back in place; each member then reads its own record.
template <typename R> struct Rec;
template <> struct __align__(16) Rec<float> { float x, y, z; uint32_t w2; };
template <> struct __align__(16) Rec<double> { double x, y, z; uint32_t w2, pad; };

// Dynamic LDS a cell pass may use (the static part is below 4 KB).
constexpr size_t LDS_DYN_LIMIT = 152 * 1024;

// Layout of one exchange round of P positions: P + 2 records (two beyond P
// for an odd cell's triplet that straddles the end of the round), the first
// members' word 3 per pair, and with weights the second members' word 3 and
// the weight per position, with Nanbu's operator or the triplet the member
// index per position.
template <typename R, int F>
struct ExchLayout {
    static constexpr bool WT = (F & F_WT) != 0;
    static constexpr bool SLOT = (F & (F_NANBU | F_TRIP)) != 0;
    __host__ __device__ static constexpr size_t bytes(uint32_t P)
    {
        size_t b = ((size_t)P + 2) * sizeof(Rec<R>) + ((size_t)P / 2 + 1) * 4;
        if (WT) b += ((size_t)P / 2 + 1) * 4 + ((size_t)P + 2) * sizeof(R);
        if (SLOT) b += ((size_t)P + 2) * 2;
        return (b + 15) & ~(size_t)15;
    }
};

// Positions per exchange round: the whole cell when its records fit.
template <typename R, int F = 0>
__host__ __device__ constexpr uint32_t round_positions(int cap)
{
    const uint32_t want = (uint32_t)(((size_t)cap + 1) & ~(size_t)1);
    uint32_t P = want;
    while (P > 64 && ExchLayout<R, F>::bytes(P) > LDS_DYN_LIMIT) P -= 64;
    return P;
}

template <typename R, int F = 0>
__host__ __device__ constexpr size_t lds_bytes(int cap)
{
    const size_t ex = ExchLayout<R, F>::bytes(round_positions<R, F>(cap));
    const size_t s = sort_bytes(cap);
    return s > ex ? s : ex;
}

// Nanbu's deflection of the pair (a, b), a the member in the lower storage
// slot: 1 - cos chi from Nanbu's distribution with U = U(word 2 of a) and
// A(s), s twice the Takizuka & Abe variance (C / |u|^3, C = 8 pi n lnL dt);
// azimuth 2 pi U(word 2 of b); rotation and halves as in Takizuka & Abe.
// Binary64 computes the oracle's steps; binary32 its own (see nb_A).
template <typename R>
__device__ __forceinline__ void nanbu_half(R ux, R uy, R uz, R C, uint32_t wa2, uint32_t wb2, R &hx,
                                           R &hy, R &hz)
{
#pragma clang fp contract(off)
    const double PI = 3.14159265358979323846;
    hx = hy = hz = (R)0;
    const R uu = ux * ux + uy * uy + uz * uz;
    if (uu == (R)0) return;
    const R um = sqrt(uu), uperp = sqrt(ux * ux + uy * uy);
    const R s = (R)2 * nb_div(C, um * um * um);
    const R U = sizeof(R) == 4 ? (R)u01f(wa2) : (R)u01d(wa2);
    const R omc = nb_omc(nb_A(s), U);
    const R sin_t = sqrt(omc * ((R)2 - omc));
    const R phi = (R)(2.0 * PI) * (sizeof(R) == 4 ? (R)u01f(wb2) : (R)u01d(wb2));
    const R cphi = cos(phi), sphi = sin(phi);
    R dx, dy, dz;
    if (uperp > (R)0) {
        const R ex = nb_div(ux, uperp), ey = nb_div(uy, uperp);
        dx = ex * uz * sin_t * cphi - ey * um * sin_t * sphi - ux * omc;
        dy = ey * uz * sin_t * cphi + ex * um * sin_t * sphi - uy * omc;
        dz = -uperp * sin_t * cphi - uz * omc;
    } else {
        dx = um * sin_t * cphi;
        dy = um * sin_t * sphi;
        dz = -uz * omc;
    }
    hx = (R)0.5 * dx;
    hy = (R)0.5 * dy;
    hz = (R)0.5 * dz;
}

// Takizuka & Abe's triplet for an odd cell: the members p0 p1 p2 (the last
// three in pairing order) collide pairwise at dt/2 in the order (p0, p1),
// (p1, p2), (p2, p0), each on the velocities the previous one left, with the
// uniforms of Philox domains 0, 4 and 5.  In place on x, y, z.
template <typename R>
__device__ __forceinline__ void triplet_collide(R (&x)[3], R (&y)[3], R (&z)[3], const uint32_t (&pd)[3],
                                                R Ch, uint64_t seed, uint32_t step)
{
    const uint32_t dom[3] = {0u, 4u, 5u};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int i = c, k = (c + 1) % 3;
        const W4 wa = draw4(seed, pd[i], step, dom[c], 0u);
        const W4 wb = draw4(seed, pd[k], step, dom[c], 0u);
        R hx, hy, hz;
        ta_half(x[i] - x[k], y[i] - y[k], z[i] - z[k], Ch, wa.z, wa.w, wb.z, hx, hy, hz);
        x[i] += hx;
        y[i] += hy;
        z[i] += hz;
        x[k] -= hx;
        y[k] -= hy;
        z[k] -= hz;
    }
}

// ------------------------------------------------------------ LDS-class pass
// Adds the 14 moment terms of v to m[0..13] (layout of pic_cell_moments:
// count, sum v, the second-order products, sum |v|^2 v, sum |v|^4).
__device__ __forceinline__ void moment_terms(double (&m)[16], double x, double y, double z)
{
    const double q2 = x * x + y * y + z * z;
    m[0] += 1.0;
    m[1] += x; m[2] += y; m[3] += z;
    m[4] += x * x; m[5] += y * y; m[6] += z * z;
    m[7] += x * y; m[8] += x * z; m[9] += y * z;
    m[10] += q2 * x; m[11] += q2 * y; m[12] += q2 * z;
    m[13] += q2 * q2;
}

// The 14 moment sums of the pass's members (layout of pic_cell_moments): four
// wave reduce-scatters of 4 values (so at most 4 accumulators are live), each
// into its own quarter of red, then one cross-wave pass.  The count is n.
// red: 16 doubles per wave.  Contains the barriers; threads 0..13 write.
template <typename R, int T, int K>
__device__ __forceinline__ void cell_moments_out(double *out, const R (&vx)[K], const R (&vy)[K],
                                                 const R (&vz)[K], int n, double *red)
{
    constexpr int NW = T / PIC_WAVE;
#pragma unroll
    for (int part = 0; part < 4; ++part) {
        double h[4] = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (threadIdx.x + k * T < n) {
                const double x = vx[k], y = vy[k], z = vz[k];
                if (part == 0) {
                    h[0] += x; h[1] += y; h[2] += z; h[3] += x * x;
                } else if (part == 1) {
                    h[0] += y * y; h[1] += z * z; h[2] += x * y; h[3] += x * z;
                } else {
                    const double q2 = x * x + y * y + z * z;
                    if (part == 2) {
                        h[0] += y * z; h[1] += q2 * x; h[2] += q2 * y; h[3] += q2 * z;
                    } else {
                        h[0] += q2 * q2;
                    }
                }
            }
        }
        wave_scatter_to<4>(h, red + part * 4 * NW);
    }
    __syncthreads();
    if (threadIdx.x < 13) {
        const double *r = red + (threadIdx.x >> 2) * 4 * NW + (threadIdx.x & 3);
        double t = 0.0;
        for (int w = 0; w < NW; ++w) t += r[w * 4];
        out[1 + threadIdx.x] = t;
    } else if (threadIdx.x == 13) {
        out[0] = (double)n;
    }
    __syncthreads();
}

// Adds the thread's members to s: sum v, sum |v|^2.
template <typename R, int T, int K>
__device__ __forceinline__ void add_sums(double *s, int n, const R (&vx)[K], const R (&vy)[K], const R (&vz)[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < n) {
            const double x = vx[k], y = vy[k], z = vz[k];
            s[0] += x;
            s[1] += y;
            s[2] += z;
            s[3] += x * x + y * y + z * z;
        }
    }
}

// The conservation correction of a cell of n members whose velocities sit in
// registers: before and after are its sums around the step, debt (four
// doubles, nullable) what earlier steps left unmet; what the output rounding
// leaves goes to debt_out (nullable).  Contains barriers.
template <typename R, int T, int K>
__device__ __forceinline__ void conserve_regs(int n, R (&vx)[K], R (&vy)[K], R (&vz)[K], const double *before,
                                              const double *after, const double *debt, double *debt_out,
                                              double *red)
{
    const Correction cr = make_correction((double)n, before, after, debt);
    if (cr.ok) {
        double real[4] = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = threadIdx.x + k * T;
            if (i < n) {
                vx[k] = (R)(cr.Vt[0] + cr.al * ((double)vx[k] - cr.Vn[0]));
                vy[k] = (R)(cr.Vt[1] + cr.al * ((double)vy[k] - cr.Vn[1]));
                vz[k] = (R)(cr.Vt[2] + cr.al * ((double)vz[k] - cr.Vn[2]));
            }
        }
        add_sums<R, T, K>(real, n, vx, vy, vz);
        const double t = block_sum_scatter<4>(real, red);
        if (debt_out) store_debt_lane(debt_out, cr, t);
    }
}

// Null collisions of the thread's candidate members (bits of cand) on their
// registers, one candidate at a time per lane.
template <typename R, int T, int K, bool CALL = false>
__device__ __forceinline__ void scatter_regs(const CollideArgs &a, uint32_t cand, R (&vx)[K], R (&vy)[K],
                                             R (&vz)[K], const uint32_t *pid_c, uint32_t step)
{
    uint32_t left = cand;
    while (__ballot(left != 0u) != 0ull) {
        if (left) {
            const int kk = __builtin_ctz(left);
            left &= left - 1u;
            // selected and put back without a branch (a conditional access is
            // turned into an indexed one, and the arrays into scratch memory)
            R x = vx[0], y = vy[0], z = vz[0];
#pragma unroll
            for (int k = 1; k < K; ++k) {
                const R ax = vx[k], ay = vy[k], az = vz[k];
                x = kk == k ? ax : x;
                y = kk == k ? ay : y;
                z = kk == k ? az : z;
            }
            mcc_scatter_as<R, CALL, (T >= 1024)>(x, y, z, pid_c[threadIdx.x + kk * T], a.seed, step, a.mass_ratio);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const R ax = vx[k], ay = vy[k], az = vz[k];
                vx[k] = kk == k ? x : ax;
                vy[k] = kk == k ? y : ay;
                vz[k] = kk == k ? z : az;
            }
        }
    }
}

template <typename R, int T, int K, int F>
__device__ __forceinline__ void cell_pass(const CollideArgs &a, int cell, unsigned char *smem, double *red,
                          uint32_t *wtot, double *s_before)
{
    constexpr bool PAIRS = (F & F_PAIRS) != 0;
    constexpr bool MCC = (F & F_MCC) != 0;
    constexpr bool CONS = (F & F_CONS) != 0;
    constexpr bool MOM = (F & F_MOM) != 0;
    constexpr bool WT = (F & F_WT) != 0;
    constexpr bool NANBU = (F & F_NANBU) != 0;
    constexpr bool TRIP = (F & F_TRIP) != 0;
    constexpr int CAP = T * K;
    const int lo = a.cell_start[cell];
    const int n = a.cell_start[cell + 1] - lo;
    const uint32_t step = (uint32_t)read_step(a);
    const bool coul = n >= 2;
    R *vx_g = (R *)a.v + lo;
    R *vy_g = (R *)a.v + a.n + lo;
    R *vz_g = (R *)a.v + 2 * a.n + lo;
    const uint32_t *pid_c = a.pid + lo;

    const SortLDS<T, CAP> L(smem);

    R vx[K], vy[K], vz[K];
    uint32_t w2[K], w3[K], pos[K];
    uint32_t cand = 0;

    const uint32_t bits = sort_bits(n);
    // every load of the thread is issued before any is used, so they are in
    // flight together and overlap the clearing of the counters (pos holds
    // the pid until the key is counted)
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < n) {
            pos[k] = pid_c[i];
            if (!PAIRS) {
                vx[k] = vx_g[i];
                vy[k] = vy_g[i];
                vz[k] = vz_g[i];
            }
        }
    }
    L.clear();
    __syncthreads();
    {
        // one Philox call per particle, and the bucket count of its key with
        // its arrival rank
        double before[4] = {0, 0, 0, 0};   // sum v, sum |v|^2
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = threadIdx.x + k * T;
            if (i < n) {
                const W4 w = draw4(a.seed, pos[k], step, 0u, 0u);
                w2[k] = w.z;
                w3[k] = w.w;
                if (MCC && (uint64_t)w.y < a.mcc_thr) cand |= 1u << k;
                pos[k] = L.count(i, w.x, bits);
                if (CONS) {
                    const double x = vx[k], y = vy[k], z = vz[k];
                    before[0] += x;
                    before[1] += y;
                    before[2] += z;
                    before[3] += x * x + y * y + z * z;
                }
            }
        }
        if constexpr (CONS) {
            const double t = block_sum_scatter<4>(before, red);   // contains the barriers
            if (threadIdx.x < 4) s_before[threadIdx.x] = t;
        }
    }
    __syncthreads();

    if (coul || PAIRS) rank_in_lds<T, K, CAP>(pos, n, bits, L, pid_c, wtot);

    if (PAIRS) {
        // sorted[] and partner[] for the test export
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = threadIdx.x + k * T;
            if (i < n) {
                L.lst[pos[k]] = (uint16_t)i;
                a.sorted_out[lo + pos[k]] = lo + i;
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int i = threadIdx.x + k * T;
            if (i < n) {
                const uint32_t q = pos[k] ^ 1u;
                a.partner_out[lo + i] = (q < (uint32_t)n) ? lo + (int)L.lst[q] : -1;
            }
        }
        __syncthreads();
        return;
    }

    if (coul) {
        const R C = (R)cell_C(a, cell);
        const uint32_t np2 = (uint32_t)n & ~1u;     // positions with a partner
        // with the triplet, an odd cell's last three positions form it
        const uint32_t tstart = (TRIP && (n & 1) && n >= 3) ? (uint32_t)n - 3u : np2;
        const uint32_t npost = tstart < np2 ? (uint32_t)n : np2;   // positions with records
        constexpr uint32_t P = round_positions<R, F>(CAP);
        Rec<R> *rec = (Rec<R> *)smem;
        uint32_t *w3s = (uint32_t *)(rec + P + 2);
        // with weights: the second member's word 3 per pair, the weight per position
        uint32_t *w3b = w3s + P / 2 + 1;
        R *wts = (R *)(w3b + (WT ? P / 2 + 1 : 0));
        // with Nanbu's operator or the triplet: the member index per position
        uint16_t *slt = (uint16_t *)(wts + (WT ? P + 2 : 0));
        const R *w_c = (const R *)a.w + lo;
        for (uint32_t base = 0; base < npost; base += P) {
            // a member posts in the round of its position; the triplet's three
            // in the round holding its start
            const bool tri_here = tstart < npost && tstart >= base && tstart - base < P;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int i = threadIdx.x + k * T;
                const uint32_t q = pos[k] - base;
                const bool mine = pos[k] < tstart ? q < P : (pos[k] < npost && tri_here);
                if (i < n && mine) {
                    Rec<R> e;
                    e.x = vx[k];
                    e.y = vy[k];
                    e.z = vz[k];
                    e.w2 = w2[k];
                    rec[q] = e;
                    if (!(q & 1u)) w3s[q >> 1] = w3[k];
                    if constexpr (WT) {
                        if (q & 1u) w3b[q >> 1] = w3[k];
                        wts[q] = w_c[i];
                    }
                    if constexpr (NANBU || TRIP) slt[q] = (uint16_t)i;
                }
            }
            __syncthreads();
            const uint32_t lim = min(base + P, tstart);
            const uint32_t m = lim > base ? (lim - base) / 2 : 0u;
            for (uint32_t j = threadIdx.x; j < m; j += T) {
                Rec<R> A = rec[2 * j], B = rec[2 * j + 1];
                R hx, hy, hz;
                bool ta = true, tb = true;
                if constexpr (NANBU) {
                    // the member in the lower storage slot is the operator's first
                    if (slt[2 * j] < slt[2 * j + 1]) {
                        nanbu_half<R>(A.x - B.x, A.y - B.y, A.z - B.z, C, A.w2, B.w2, hx, hy, hz);
                    } else {
                        nanbu_half<R>(B.x - A.x, B.y - A.y, B.z - A.z, C, B.w2, A.w2, hx, hy, hz);
                        hx = -hx;
                        hy = -hy;
                        hz = -hz;
                    }
                } else {
                    ta_half<(T >= 1024)>(A.x - B.x, A.y - B.y, A.z - B.z, C, A.w2, w3s[j], B.w2, hx, hy, hz);
                    if constexpr (WT) weight_rule<R>(wts[2 * j], wts[2 * j + 1], w3b[j], ta, tb);
                }
                if (ta) {
                    A.x += hx;
                    A.y += hy;
                    A.z += hz;
                }
                if (tb) {
                    B.x -= hx;
                    B.y -= hy;
                    B.z -= hz;
                }
                rec[2 * j] = A;
                rec[2 * j + 1] = B;
            }
            if constexpr (TRIP) {
                if (tri_here && threadIdx.x == 0) {
                    const uint32_t q0 = tstart - base;
                    R x[3], y[3], z[3];
                    uint32_t pd[3];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const Rec<R> e = rec[q0 + c];
                        x[c] = e.x;
                        y[c] = e.y;
                        z[c] = e.z;
                        pd[c] = pid_c[slt[q0 + c]];
                    }
                    const double dens = a.density ? a.density[cell] : 1.0;
                    triplet_collide<R>(x, y, z, pd, (R)(8.0 * PI_D * dens * a.lnL * (0.5 * a.dt)),
                                       a.seed, step);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        Rec<R> e = rec[q0 + c];
                        e.x = x[c];
                        e.y = y[c];
                        e.z = z[c];
                        rec[q0 + c] = e;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int i = threadIdx.x + k * T;
                const uint32_t q = pos[k] - base;
                const bool mine = pos[k] < tstart ? q < P : (pos[k] < npost && tri_here);
                if (i < n && mine) {
                    const Rec<R> e = rec[q];
                    vx[k] = e.x;
                    vy[k] = e.y;
                    vz[k] = e.z;
                }
            }
            if (base + P < npost) __syncthreads();
        }

        if constexpr (CONS) {
            double after[4] = {0, 0, 0, 0};
            add_sums<R, T, K>(after, n, vx, vy, vz);
            block_sum_bcast<4>(after, red);
            double *debt = a.debt ? a.debt + (int64_t)cell * 4 : nullptr;
            conserve_regs<R, T, K>(n, vx, vy, vz, s_before, after, debt, debt, red);
        }
    }

    // null collisions: about 1% of the particles are candidates, so each lane
    // takes its candidates one at a time (selected out of its register slots)
    // instead of branching per slot, which would run the scattering for every
    // slot holding a candidate in any lane of the wave
    if constexpr (MCC) scatter_regs<R, T, K, (F & F_CALL) != 0>(a, cand, vx, vy, vz, pid_c, step);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < n) {
            vx_g[i] = vx[k];
            vy_g[i] = vy[k];
            vz_g[i] = vz[k];
        }
    }
    if constexpr (MOM) cell_moments_out<R, T, K>(a.moments + (int64_t)cell * 14, vx, vy, vz, n, red);
    // every thread leaves the pass together: the caller's loop starts with a
    // thread-0 work fetch, and a thread-0 block just before it must not be
    // merged with it or moved out of the loop
    __syncthreads();
}

template <typename R, int T, int K, int F>
__global__ __launch_bounds__(T) void k_collide(CollideArgs a, const int32_t *__restrict__ list,
                                               int cls)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[16 * (T / PIC_WAVE)];
    __shared__ double s_before[4];
    __shared__ uint32_t wtot[T / PIC_WAVE];
    __shared__ int s_item;
    if (gated_off(a)) return;
    const uint32_t count = a.dflags->count[cls];
    if (blockIdx.x >= count) return;   // no work for this workgroup (nor a queue atomic)
    if constexpr (T >= 1024 && std::is_same<R, float>::value) {
        // large cells: one counter, for the first items too (with 16 queues cells
        // of 8,000 with the correction take 888 us instead of 836, by index first 844)
        // (a uniform item, or one by index where the workgroups cover the list, made
        // the pass slower: cells of 8,000 858 and 867 us)
        for (;;) {
            if (threadIdx.x == 0) s_item = (int)list_take(a.dflags, cls);
            __syncthreads();
            const int item = s_item;
            __syncthreads();
            if (item >= (int)count) return;
            cell_pass<R, T, K, F>(a, list[item], smem, red, wtot, s_before);
        }
    }
    for (uint32_t item = blockIdx.x; item < count;) {
        if (threadIdx.x == 0) s_item = (int)queue_take(a.dflags, cls, queue_of(blockIdx.x, gridDim.x), gridDim.x);   // read after the pass's barriers
        cell_pass<R, T, K, F>(a, list[item], smem, red, wtot, s_before);
        item = (uint32_t)s_item;
        __syncthreads();
    }
}

// ------------------------------------------------------------ lean pass
// The binary32 pass for cells of up to T*K members, written for few VALU
// instructions and few LDS operations per member:
//   * bucket counters are whole words (no 16-bit packing), nb = 2^bits >= n
//     buckets, so a bucket holds 0.5..1 members on average;
//   * after the scan only members that share their bucket write their key
//     and index to LDS, and only they compare keys to rank themselves
//     (about half the members are alone in their bucket);
//   * the first member of each pair draws its Box-Muller deviate before the
//     exchange, so a record is 16 bytes (velocity and one word) and a cell of
//     up to LeanExch::P members exchanges in one round;
//   * pair threads write both new velocities back in place; members read
//     their record.
// The pairs, the rotation (ta_half_z) and the null collisions are those of
// cell_pass, so the two give identical velocities.

// One exchange round over P sorted positions: a record each; with weights the
// weight per position and the second members' word 3 per pair, with Nanbu's
// operator or the triplet the member index per position (the triplet may need
// two positions past the round).  P covers the whole cell where that fits.
template <int T, int K, int F>
struct LeanExch {
    static constexpr bool WT = (F & F_WT) != 0;
    static constexpr bool SLOT = (F & (F_NANBU | F_TRIP)) != 0;
    static constexpr uint32_t EXTRA = (F & F_TRIP) ? 2u : 0u;
    static constexpr size_t LIMIT = T >= 1024 ? LEAN_LDS_LIMIT - ((F & (F_CONS | F_MOM)) ? 2560 : 0)
                                              : 80 * 1024 - ((F & (F_CONS | F_MOM)) ? 2048 : 512);
    static constexpr size_t bytes(uint32_t P)
    {
        size_t b = ((size_t)P + EXTRA) * sizeof(Rec<float>);
        if (WT) b += (size_t)P * 4 + (size_t)P / 2 * 4;
        if (SLOT) b += ((size_t)P + EXTRA) * 2;
        return (b + 15) & ~(size_t)15;
    }
    static constexpr uint32_t fit()
    {
        const uint32_t want = ((uint32_t)(T * K) + 1u) & ~1u;
        uint32_t P = (want + 63u) & ~63u;
        while (P > 64 && bytes(P) > LIMIT) P -= 64;
        return P < want ? P : want;
    }
    static constexpr uint32_t P = fit();
};

template <int T, int K, int F>
__host__ __device__ constexpr size_t lean_lds_bytes()
{
    const size_t ex = LeanExch<T, K, F>::bytes(LeanExch<T, K, F>::P);
    const size_t s = LeanGeom<T, K>::SORT_BYTES;
    return s > ex ? s : ex;
}

// One exchange round over the sorted positions [base, base + P): members post
// (velocity, word) at their position (the unpaired last one too), one thread
// per pair rotates, null-collision candidates scatter their records (with the
// conservation correction, which comes first, they wait for lean_pass), members
// read their record back.  Contains the barriers.
template <int T, int K, int F>
__device__ __forceinline__ void lean_round(uint32_t base, uint32_t np2, int n, float C, unsigned char *smem,
                                           float (&vx)[K], float (&vy)[K], float (&vz)[K],
                                           const uint32_t (&w2)[K], const uint32_t (&w3)[K],
                                           const float (&wt)[(F & F_WT) ? K : 1], const uint32_t (&pos)[K],
                                           uint32_t &cand, int kf, uint32_t cpid, const uint32_t *pid_c,
                                           const CollideArgs &a, int cell, uint32_t step)
{
    typedef LeanExch<T, K, F> X;
    constexpr bool MCC = (F & F_MCC) != 0 && (F & F_CONS) == 0;
    constexpr bool WT = (F & F_WT) != 0, NANBU = (F & F_NANBU) != 0, TRIP = (F & F_TRIP) != 0;
    constexpr uint32_t P = X::P;
    Rec<float> *rec = (Rec<float> *)smem;
    float *wts = (float *)(rec + P + X::EXTRA);
    uint32_t *w3b = (uint32_t *)(wts + (WT ? P : 0));
    uint16_t *slt = (uint16_t *)(w3b + (WT ? P / 2 : 0));
    // with the triplet, an odd cell's last three positions form it, in the
    // round that holds its start
    const uint32_t tstart = (TRIP && (n & 1) && n >= 3) ? (uint32_t)n - 3u : np2;
    const bool tri_here = TRIP && tstart < np2 && tstart - base < P;
    auto mine = [&](uint32_t p) { return (!TRIP || tstart == np2 || p < tstart) ? p - base < P : tri_here; };
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        const uint32_t q = pos[k] - base;
        if (i < n && mine(pos[k])) {
            Rec<float> e;
            e.x = vx[k];
            e.y = vy[k];
            e.z = vz[k];
            if constexpr (NANBU) {
                e.w2 = w2[k];
            } else {
                // first members carry their deviate, second ones word 2
                const float z = ta_z(w2[k], w3[k]);
                e.w2 = (pos[k] & 1u) ? w2[k] : __float_as_uint(z);
            }
            rec[q] = e;
            if constexpr (WT) {
                wts[q] = wt[k];
                if (q & 1u) w3b[q >> 1] = w3[k];
            }
            if constexpr (X::SLOT) slt[q] = (uint16_t)i;
        }
    }
    lds_barrier();
    const uint32_t lim = min(base + P, tstart);
    const uint32_t m = lim > base ? (lim - base) / 2 : 0u;
    for (uint32_t j = threadIdx.x; j < m; j += T) {
        Rec<float> A = rec[2 * j], B = rec[2 * j + 1];
        float hx, hy, hz;
        bool ta = true, tb = true;
        if constexpr (NANBU) {
            // the member in the lower storage slot is the operator's first
            if (slt[2 * j] < slt[2 * j + 1]) {
                nanbu_half<float>(A.x - B.x, A.y - B.y, A.z - B.z, C, A.w2, B.w2, hx, hy, hz);
            } else {
                nanbu_half<float>(B.x - A.x, B.y - A.y, B.z - A.z, C, B.w2, A.w2, hx, hy, hz);
                hx = -hx;
                hy = -hy;
                hz = -hz;
            }
        } else {
            ta_half_z(A.x - B.x, A.y - B.y, A.z - B.z, C, __uint_as_float(A.w2), B.w2, hx, hy, hz);
            if constexpr (WT) weight_rule<float>(wts[2 * j], wts[2 * j + 1], w3b[j], ta, tb);
        }
        if (ta) {
            A.x += hx;
            A.y += hy;
            A.z += hz;
        }
        if (tb) {
            B.x -= hx;
            B.y -= hy;
            B.z -= hz;
        }
        rec[2 * j] = A;
        rec[2 * j + 1] = B;
    }
    if constexpr (TRIP) {
        if (tri_here && threadIdx.x == 0) {
            const uint32_t q0 = tstart - base;
            float x[3], y[3], z[3];
            uint32_t pd[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const Rec<float> e = rec[q0 + c];
                x[c] = e.x;
                y[c] = e.y;
                z[c] = e.z;
                pd[c] = pid_c[slt[q0 + c]];
            }
            const double dens = a.density ? a.density[cell] : 1.0;
            triplet_collide<float>(x, y, z, pd, (float)(8.0 * PI_D * dens * a.lnL * (0.5 * a.dt)), a.seed, step);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                Rec<float> e = rec[q0 + c];
                e.x = x[c];
                e.y = y[c];
                e.z = z[c];
                rec[q0 + c] = e;
            }
        }
    }
    lds_barrier();
    // null collisions of this round's candidates, on their own records (each
    // record is read back by its member's thread only, so no barrier), one
    // candidate at a time per lane; the pid of the thread's first candidate
    // (member kf) was kept from the sort
    if constexpr (MCC) {
        uint32_t left = cand, later = 0;
        while (__ballot(left != 0u) != 0ull) {
            if (left) {
                const int kk = __builtin_ctz(left);
                left &= left - 1u;
                uint32_t pk = pos[0];
#pragma unroll
                for (int k = 1; k < K; ++k)
                    if (kk == k) pk = pos[k];
                const uint32_t q = pk - base;
                if (q < P) {
                    uint32_t id = cpid;
                    if (kk != kf) {
                        // a later candidate (rare): its pid from memory, waited
                        // for here, so that the common path does not wait for
                        // the next cell's lines requested above
                        id = pid_c[threadIdx.x + kk * T];
                        asm volatile("" ::"v"(id));
                    }
                    Rec<float> e = rec[q];
                    mcc_scatter<float>(e.x, e.y, e.z, id, a.seed, step, a.mass_ratio);
                    rec[q] = e;
                } else {
                    later |= 1u << kk;
                }
            }
        }
        cand = later;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        const uint32_t q = pos[k] - base;
        if (i < n && mine(pos[k])) {
            const Rec<float> e = rec[q];
            vx[k] = e.x;
            vy[k] = e.y;
            vz[k] = e.z;
        }
    }
}

// s_waitcnt operand that waits for vector memory only: vmcnt (bits 3:0 and
// 15:14) 0, expcnt (6:4) and lgkmcnt (11:8) at their maxima.
constexpr int WAIT_VMCNT0 = 0x0F70;

// Segment of a key among S equal key ranges, and the key's position inside
// its range scaled to 32 bits (order-preserving within the segment).
__device__ __forceinline__ uint32_t seg_of(uint32_t key, uint32_t S)
{
    return (uint32_t)(((uint64_t)key * S) >> 32);
}
__device__ __forceinline__ uint32_t seg_key(uint32_t key, uint32_t S)
{
    return (uint32_t)((uint64_t)key * S);
}

// Counting sort of a cell's members by (key, pid) in LDS, shared by the lean
// passes (n >= 2): one Philox call per member (key, words 2 and 3, the
// null-collision candidate bit; cpid: the pid of the thread's first
// candidate), bucket counts (at least one bucket per
// member), scan, placement, rank inside the buckets.  On entry pos[k] holds
// member k's pid, on return its position in the cell's sorted order.
// Contains the barriers; the sort's memory is free after a further barrier.
// With SEG the members are those of one of a cell's S segments: the key is
// its position inside the segment's range (see seg_key).
template <int T, int K, bool MCC, bool CLEAR2 = false, bool SEG = false>
__device__ __forceinline__ void lean_sort(const CollideArgs &a, int n, uint32_t step,
                                          const uint32_t *pid_c, unsigned char *smem, uint32_t *wtot,
                                          uint32_t (&w2)[K], uint32_t (&w3)[K], uint32_t (&key)[K],
                                          uint32_t (&pos)[K], uint32_t &cand, uint32_t &cpid, uint32_t S = 1u)
{
    const uint32_t bits = sort_bits(n);
    uint32_t *cnt = (uint32_t *)smem;
    // (the binary64 pass measured slower with 8-byte writes)
    lean_clear<T, K, CLEAR2>(cnt, bits);
    lds_barrier();
    // one Philox call per particle; count its key's bucket
    const int n1 = opaque(n);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < n1) {
            const W4 w = draw4(a.seed, pos[k], step, 0u, 0u);
            key[k] = SEG ? seg_key(w.x, S) : w.x;
            w2[k] = w.z;
            w3[k] = w.w;
            if (MCC && (uint64_t)w.y < a.mcc_thr) {
                if (!cand) cpid = pos[k];
                cand |= 1u << k;
            }
            const uint32_t b = key[k] >> (32u - bits);
            pos[k] = atomicAdd(&cnt[b], 1u);   // arrival rank in the bucket
        }
    }
    lean_rank<T, K>(n, bits, pid_c, smem, wtot, key, pos);
}

// The next cell's lines of pid and v are requested while this cell is still
// being worked on, so that its loads find them in the caches (the last-level
// cache holds every workgroup's next cell).  The loads go to LDS (a 256-byte
// sink that nothing reads): they write no register, so nothing waits for them
// before the next cell's own loads.
struct LeanNext {
    int *slot;                 // LDS: [0] receives the next work item; [1] the queue, [2] the takers
    int cls;                   // the queue
    const int32_t *list;
    uint32_t count;
    float *sink;               // 64 words of LDS
};

// The next work item.  The cells of the 1,024-thread class take 10 us and more:
// one counter for the whole list is not contended and deals them evenly to the
// end.  Replayed steps of 12M electrons in cells of 9,000: 172 us (166 without
// null collisions) against 176 (172) from 16 queues, of 40.96M in cells of
// 10,000 449 us (437) against 451 (440); with two cells a workgroup or of 4,500
// up to 0.6% more.  The first items are taken by index: from the counter too,
// 256 workgroups begin 3 us late (100 cells of 9,000 56 us a step instead of 53).
template <int T>
__device__ __forceinline__ int lean_take(DevFlags *f, const LeanNext *nx)
{
    if constexpr (T >= 1024) return nx->slot[2] + (int)list_take(f, nx->cls);
    else return (int)queue_take(f, nx->cls, (unsigned)nx->slot[1], (unsigned)nx->slot[2]);
}

// n entries of pid and of `arrays` further arrays of dwords, stride apart.
template <int T>
__device__ __forceinline__ void prefetch_run(const uint32_t *pid, uint32_t arrays, const float *v, size_t stride,
                                             int n, float *sink)
{
    if (n <= 0) return;
    // 128-byte lines of each of the arrays (one more for a start inside a
    // line); one dword per line
    const uint32_t lines = ((uint32_t)n + 31u) / 32u + 1u;
    for (uint32_t t = threadIdx.x; t < (arrays + 1u) * lines; t += T) {
        const uint32_t arr = t / lines, l = t - arr * lines;
        const uint32_t idx = min(l * 32u, (uint32_t)n - 1u);
        const float *p = arr == 0 ? (const float *)(pid + idx) : v + (size_t)(arr - 1u) * stride + idx;
        __builtin_amdgcn_global_load_lds((const void *)p, (__attribute__((address_space(3))) void *)sink,
                                         4, 0, 0);
    }
}
template <int T>
__device__ __forceinline__ void prefetch_cell(const CollideArgs &a, int cell, float *sink)
{
    const int lo = a.cell_start[cell];
    prefetch_run<T>(a.pid + lo, 3u, (const float *)a.v + lo, (size_t)a.n, a.cell_start[cell + 1] - lo, sink);
}

// With nx, the pass also takes the next work item from the queue and
// returns it (every thread reads it after a barrier that follows its write
// and precedes the pass's end, so the next pass may overwrite the slot);
// without, it returns 0.
template <int T, int K, int F>
__device__ __forceinline__ int lean_pass(const CollideArgs &a, int cell, unsigned char *smem, uint32_t *wtot,
                                         const LeanNext *nx = nullptr, double *red = nullptr,
                                         double *s_debt = nullptr)
{
    constexpr bool MCC = (F & F_MCC) != 0, CONS = (F & F_CONS) != 0, MOM = (F & F_MOM) != 0;
    constexpr bool WT = (F & F_WT) != 0;
    constexpr uint32_t P = LeanExch<T, K, F>::P;
    const int lo = a.cell_start[cell];
    const int n = a.cell_start[cell + 1] - lo;
    const uint32_t step = (uint32_t)read_step(a);
    float *vx_g = (float *)a.v + lo;
    float *vy_g = (float *)a.v + a.n + lo;
    float *vz_g = (float *)a.v + 2 * a.n + lo;
    const uint32_t *pid_c = a.pid + lo;

    float vx[K], vy[K], vz[K];
    float wt[WT ? K : 1];
    uint32_t w2[K], w3[K], key[K], pos[K];
    uint32_t cand = 0;

    int next = 0;
    if (n == 0) {
        if constexpr (MOM)
            if (threadIdx.x < 14) a.moments[(int64_t)cell * 14 + threadIdx.x] = 0.0;
        if (nx && threadIdx.x == 0) *nx->slot = lean_take<T>(a.dflags, nx);
        lds_barrier();   // leave together (see the end of the pass)
        if (nx) next = *nx->slot;
        lds_barrier();
        return next;
    }
    // every load of the thread is in flight before the first is used, the
    // ids first (the Philox calls wait for them only).  Members past the end
    // load the last one instead (ignored): with no branch around the loads the
    // compiler waits for each load by count instead of for all of them.
    {
        uint32_t ic[K];
#pragma unroll
        for (int k = 0; k < K; ++k) ic[k] = (uint32_t)min((int)threadIdx.x + k * T, n - 1);
#pragma unroll
        for (int k = 0; k < K; ++k) pos[k] = ld_at(pid_c, ic[k]);
        asm volatile("" ::: "memory");   // keep the id loads ahead of the velocity loads
#pragma unroll
        for (int k = 0; k < K; ++k) {
            vx[k] = ld_at((const float *)vx_g, ic[k]);
            vy[k] = ld_at((const float *)vy_g, ic[k]);
            vz[k] = ld_at((const float *)vz_g, ic[k]);
        }
        if constexpr (WT && T < 1024) {
#pragma unroll
            for (int k = 0; k < K; ++k) wt[k] = ld_at((const float *)a.w + lo, ic[k]);
        }
    }
    // the cell's shortfall, read behind the other loads (and barriers later)
    if constexpr (CONS)
        if (a.debt && threadIdx.x < 4) s_debt[threadIdx.x] = a.debt[(int64_t)cell * 4 + threadIdx.x];
    // the next work item (issued behind this cell's loads, so waiting for it
    // costs nothing extra); read after a barrier below
    if (nx && threadIdx.x == 0) *nx->slot = lean_take<T>(a.dflags, nx);
    if (n >= 2) {
        uint32_t cpid = 0;
        lean_sort<T, K, MCC, true>(a, n, step, pid_c, smem, wtot, w2, w3, key, pos, cand, cpid);
        lds_barrier();   // the sort's memory becomes the exchange records
        if constexpr (WT && T >= 1024) {   // only now: the sort has no registers to spare
#pragma unroll
            for (int k = 0; k < K; ++k)
                wt[k] = ld_at((const float *)a.w + lo, (uint32_t)min((int)threadIdx.x + k * T, n - 1));
        }
        // the thread's part of the sums before the step waits in registers for
        // the sums after it: one reduction of eight values for both
        double sums[CONS ? 8 : 1] = {0};
        if constexpr (CONS) add_sums<float, T, K>(sums, n, vx, vy, vz);

        const float C = (float)cell_C(a, cell);
        // last global loads before the exchange: a later wait for a load (the
        // density above) would wait for these too, so C is complete first
        if (nx) {
            asm volatile("" ::"v"(C));
            const uint32_t nxt = (uint32_t)*nx->slot;
            if (nxt < nx->count) prefetch_cell<T>(a, nx->list[nxt], nx->sink);
        }
        const uint32_t np2 = (uint32_t)n & ~1u;     // positions with a partner
        const int kf = cand ? __builtin_ctz(cand) : K;
        for (uint32_t base = 0; base < (uint32_t)n; base += P) {
            if (base) lds_barrier();
            lean_round<T, K, F>(base, np2, opaque(n), C, smem, vx, vy, vz, w2, w3, wt, pos, cand, kf, cpid, pid_c,
                                a, cell, step);
        }
        if constexpr (CONS) {
            add_sums<float, T, K>(sums + 4, n, vx, vy, vz);
            block_sum_bcast<8>(sums, red);
            conserve_regs<float, T, K>(n, vx, vy, vz, sums, sums + 4, a.debt ? s_debt : nullptr,
                                       a.debt ? a.debt + (int64_t)cell * 4 : nullptr, red);
            if constexpr (MCC) {
                scatter_regs<float, T, K>(a, cand, vx, vy, vz, pid_c, step);
                cand = 0;
            }
        }
    } else if (MCC) {
        const W4 w = draw4(a.seed, pos[0], step, 0u, 0u);
        if (threadIdx.x == 0 && (uint64_t)w.y < a.mcc_thr) cand = 1u;
    }

    // null collision of a lone member (n = 1: thread 0's member 0, whose pid
    // is in pos[0]; the exchange rounds took every candidate of a larger cell)
    if (MCC && cand) mcc_scatter<float>(vx[0], vy[0], vz[0], pos[0], a.seed, step, a.mass_ratio);
    // one wait for every load still outstanding (the next cell's lines,
    // requested long before) ahead of the stores: the compiler would otherwise
    // wait before each member's stores, and each wait drains the stores
    // before it too
    if (nx) __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
    const int n3 = opaque(n);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < n3) {
            vx_g[i] = vx[k];
            vy_g[i] = vy[k];
            vz_g[i] = vz[k];
        }
    }
    if constexpr (MOM) cell_moments_out<float, T, K>(a.moments + (int64_t)cell * 14, vx, vy, vz, n, red);
    // the next item: written by thread 0 before at least one barrier of
    // this pass when n >= 2 (else one more barrier), read by everyone before
    // the last one (the next pass writes it only after that)
    if (nx) {
        if (n < 2) lds_barrier();
        next = *nx->slot;
    }
    // the next cell reuses the LDS; the stores stay in flight into it
    lds_barrier();
    return next;
}

// At most 128 registers for eight members a thread and cell sums: with one more (129
// to 147 with moments, and with the correction and null collisions) the second
// workgroup, for which the LDS leaves room, does not fit on the CU.  Cells of
// 3,000 with moments 220 us a step of 12M electrons without the bound, 160 with it.
template <int T, int K, int F>
__global__ __launch_bounds__(T, T < 1024 && K >= 8 && (F & (F_CONS | F_MOM)) ? 4 : 1) void k_collide_lean(CollideArgs a, const int32_t *__restrict__ list,
                                                    int cls)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t wtot[T / PIC_WAVE];
    __shared__ int s_next[3];
    __shared__ float sink[PIC_WAVE];
    if (gated_off(a)) return;
    const uint32_t count = a.dflags->count[cls];
    if (blockIdx.x >= count) return;   // no work for this workgroup (nor a queue atomic)
    if (threadIdx.x == 0) {   // kept in LDS (no registers held), read by thread 0 only
        s_next[1] = (int)queue_of(blockIdx.x, gridDim.x);
        s_next[2] = (int)gridDim.x;
    }
    int item = (int)blockIdx.x;
    const LeanNext nx{s_next, cls, list, count, sink};
    if constexpr ((F & (F_CONS | F_MOM)) != 0) {
        __shared__ double red[16 * (T / PIC_WAVE)];
        __shared__ double s_debt[4];
        while (item < (int)count) item = lean_pass<T, K, F>(a, list[item], smem, wtot, &nx, red, s_debt);
    } else {
        while (item < (int)count) item = lean_pass<T, K, F>(a, list[item], smem, wtot, &nx);
    }
}

// ------------------------------------------------------------ lean pass, binary64
// The plain binary64 step (optionally with the fused null collisions) for
// cells of up to T*K members on one workgroup: the lean pass's sort, then the
// exchange in rounds of Lean64Geom::P sorted positions (two for a
// 10,000-member cell): the round's members load their velocity and post it
// with their words 2 and 3 at their position, one thread per pair computes
// the binary64 half change (ta_half, the oracle's order of operations) and
// writes both members back, the round's members read their record, scatter
// if they are null-collision candidates, and store it.  No velocity is held
// in registers across a round, which leaves the register file to the
// binary64 rotation.  The pairs, the rotation and the null collisions are
// those of cell_pass.


template <int T, int K>
struct Lean64Geom {
    static constexpr int CAP = T * K;
    static constexpr uint32_t P = (uint32_t)((LEAN_LDS_LIMIT / sizeof(Rec<double>)) & ~(size_t)63);
    static constexpr size_t BYTES = (size_t)P * sizeof(Rec<double>);
};

template <int T, int K>
__host__ __device__ constexpr size_t lean64_lds_bytes()
{
    typedef Lean64Geom<T, K> G;
    const size_t s = LeanGeom<T, K>::SORT_BYTES;
    return s > G::BYTES ? s : G::BYTES;
}

template <int T, int K, bool MCC>
__device__ __forceinline__ void lean64_pass(const CollideArgs &a, int cell, unsigned char *smem,
                                            uint32_t *wtot, float *sink)
{
    typedef Lean64Geom<T, K> G;
    constexpr uint32_t P = G::P;
    const int lo = a.cell_start[cell];
    const int n = a.cell_start[cell + 1] - lo;
    const uint32_t step = (uint32_t)read_step(a);
    double *vx_g = (double *)a.v + lo;
    double *vy_g = (double *)a.v + a.n + lo;
    double *vz_g = (double *)a.v + 2 * a.n + lo;
    const uint32_t *pid_c = a.pid + lo;

    uint32_t pos[K];
    uint32_t cand = 0;
    if (n == 0) {
        lds_barrier();
        return;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) pos[k] = pid_c[min((int)threadIdx.x + k * T, n - 1)];
    // the cell's velocity lines are requested now (into an LDS sink, no
    // register written), so that the rounds' loads find them cached
    {
        const uint32_t lines = ((uint32_t)n + 15u) / 16u + 1u;   // 128-byte lines of doubles
        for (uint32_t t = threadIdx.x; t < 3u * lines; t += T) {
            const uint32_t arr = t / lines, l = t - arr * lines;
            const double *p = (const double *)a.v + (size_t)arr * (size_t)a.n + (uint32_t)lo +
                              min(l * 16u, (uint32_t)n - 1u);
            __builtin_amdgcn_global_load_lds((const void *)p, (__attribute__((address_space(3))) void *)sink,
                                             4, 0, 0);
        }
    }
    uint32_t np2 = 0;
    if (n >= 2) {
        uint32_t w2[K], w3[K];
        {
            uint32_t key[K], cpid = 0;
            lean_sort<T, K, MCC>(a, n, step, pid_c, smem, wtot, w2, w3, key, pos, cand, cpid);
        }
        lds_barrier();   // the sort's memory becomes the records
        Rec<double> *rec = (Rec<double> *)smem;
        const double C = cell_C(a, cell);
        np2 = (uint32_t)n & ~1u;
        for (uint32_t base = 0; base < np2; base += P) {
            if (base) lds_barrier();
            // the thread index as a per-round value the compiler cannot hoist:
            // each round recomputes its members' offsets instead of keeping
            // them all live from the kernel's start
            uint32_t tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            {
                // loads in two halves, each posted before the next is loaded
                // (all ten members' velocities at once would not fit beside
                // the rotation's constants)
                constexpr int H = (K + 1) / 2;
#pragma unroll
                for (int h = 0; h < K; h += H) {
                    const int n4 = opaque(n);
                    double x[H], y[H], z[H];
#pragma unroll
                    for (int kk = 0; kk < H; ++kk) {
                        const int k = h + kk;
                        if (k < K) {
                            const int i = (int)tid + k * T;
                            const uint32_t q = pos[k] - base;
                            if (i < n4 && q < P && pos[k] < np2) {
                                x[kk] = ld_at(vx_g, (uint32_t)i);
                                y[kk] = ld_at(vy_g, (uint32_t)i);
                                z[kk] = ld_at(vz_g, (uint32_t)i);
                            }
                        }
                    }
#pragma unroll
                    for (int kk = 0; kk < H; ++kk) {
                        const int k = h + kk;
                        if (k < K) {
                            const int i = (int)tid + k * T;
                            const uint32_t q = pos[k] - base;
                            if (i < n4 && q < P && pos[k] < np2) {
                                Rec<double> e;
                                e.x = x[kk];
                                e.y = y[kk];
                                e.z = z[kk];
                                e.w2 = w2[k];
                                e.pad = w3[k];
                                rec[q] = e;
                            }
                        }
                    }
                }
            }
            lds_barrier();
            const uint32_t m = min(P, np2 - base) / 2;
            for (uint32_t j = threadIdx.x; j < m; j += T) {
                Rec<double> A = rec[2 * j], B = rec[2 * j + 1];
                double hx, hy, hz;
                ta_half<(K > 4)>(A.x - B.x, A.y - B.y, A.z - B.z, C, A.w2, A.pad, B.w2, hx, hy, hz);
                A.x += hx;
                A.y += hy;
                A.z += hz;
                B.x -= hx;
                B.y -= hy;
                B.z -= hz;
                rec[2 * j] = A;
                rec[2 * j + 1] = B;
            }
            lds_barrier();
            // the round's members store their record (null-collision
            // candidates after their scattering, one at a time per lane); the
            // members' offsets and tests are recomputed, not kept from the posts
            const int n5 = opaque(n);
            asm volatile("" : "+v"(tid));
            uint32_t base5 = base;
            asm volatile("" : "+s"(base5));
            uint32_t left = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int i = (int)tid + k * T;
                const uint32_t q = pos[k] - base5;
                if (i < n5 && q < P && pos[k] < np2) {
                    if (MCC && ((cand >> k) & 1u)) {
                        left |= 1u << k;
                    } else {
                        const Rec<double> e = rec[q];
                        st_at(vx_g, (uint32_t)i, e.x);
                        st_at(vy_g, (uint32_t)i, e.y);
                        st_at(vz_g, (uint32_t)i, e.z);
                    }
                }
            }
            if constexpr (MCC) {
                while (__ballot(left != 0u) != 0ull) {
                    if (left) {
                        const int kk = __builtin_ctz(left);
                        left &= left - 1u;
                        uint32_t pk = pos[0];
#pragma unroll
                        for (int k = 1; k < K; ++k)
                            if (kk == k) pk = pos[k];
                        const int i = (int)tid + kk * T;
                        const Rec<double> e = rec[pk - base5];
                        double x = e.x, y = e.y, z = e.z;
                        mcc_scatter<double, (K > 4)>(x, y, z, pid_c[i], a.seed, step, a.mass_ratio);
                        st_at(vx_g, (uint32_t)i, x);
                        st_at(vy_g, (uint32_t)i, y);
                        st_at(vz_g, (uint32_t)i, z);
                    }
                }
            }
        }
    } else if (MCC) {
        const W4 w = draw4(a.seed, pos[0], step, 0u, 0u);
        if (threadIdx.x == 0 && (uint64_t)w.y < a.mcc_thr) cand = 1u;
    }
    // the member without a partner (odd n) keeps its velocity, apart from
    // its null collision
    if constexpr (MCC) {
        uint32_t left = 0;
        const int n6 = opaque(n);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if ((int)threadIdx.x + k * T < n6 && ((cand >> k) & 1u) && (n < 2 || pos[k] >= np2))
                left |= 1u << k;
        if (left) {
            const int kk = __builtin_ctz(left);   // at most one such member per cell
            const int i = threadIdx.x + kk * T;
            double x = ld_at(vx_g, (uint32_t)i), y = ld_at(vy_g, (uint32_t)i), z = ld_at(vz_g, (uint32_t)i);
            mcc_scatter<double, (K > 4)>(x, y, z, pid_c[i], a.seed, step, a.mass_ratio);
            st_at(vx_g, (uint32_t)i, x);
            st_at(vy_g, (uint32_t)i, y);
            st_at(vz_g, (uint32_t)i, z);
        }
    }
    lds_barrier();   // the next cell reuses the LDS
}

template <int T, int K, bool MCC>
__global__ __launch_bounds__(T) void k_collide_lean64(CollideArgs a, const int32_t *__restrict__ list,
                                                      int cls)
{
    // one cell per workgroup (not persistent: a loop over cells would let
    // the compiler hoist the rotation's constants and the members' offsets
    // to the kernel's start and keep them live through every cell)
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t wtot[T / PIC_WAVE];
    __shared__ float sink[PIC_WAVE];
    if (gated_off(a)) return;
    if (blockIdx.x >= a.dflags->count[cls]) return;
    lean64_pass<T, K, MCC>(a, list[blockIdx.x], smem, wtot, sink);
}

// After the segments (k_collide_huge): the pairs across segment edges.  The lower member (even position) is the
// last of the previous non-empty segment of the cell, the upper one the first
// of this segment; both are still unchanged.  Rotation, the null collisions of
// both, stores.
template <typename R>
__device__ __forceinline__ void seg_fixup(const CollideArgs &a, const int32_t *list, const SegScratch &ss)
{
    const uint32_t nseg = a.dflags->count[SEG_SLOT];
    const uint32_t step = (uint32_t)read_step(a);
    R *vx_g = (R *)a.v;
    R *vy_g = vx_g + a.n;
    R *vz_g = vy_g + a.n;
    for (uint32_t seg = blockIdx.x * blockDim.x + threadIdx.x; seg < nseg; seg += gridDim.x * blockDim.x) {
        const int32_t sb = ss.bnd_head[seg];
        if (sb < 0) continue;
        const int h = ss.sg_cell[seg];
        if (ss.hc_fb[h]) continue;
        int32_t sa = -1;
        for (int p = (int)seg - 1; p >= ss.hc_seg[h]; --p)
            if (ss.sg_cnt[p]) {
                sa = ss.bnd_tail[p];
                break;
            }
        if (sa < 0) continue;   // not reached: an odd offset follows a segment that ends on an even one
        const R C = (R)cell_C(a, list[h]);
        const uint32_t pa = ss.m_pid[sa], pb = ss.m_pid[sb];
        const W4 wa = draw4(a.seed, pa, step, 0u, 0u);
        const W4 wb = draw4(a.seed, pb, step, 0u, 0u);
        const int32_t ga = ss.m_orig[sa], gb = ss.m_orig[sb];
        R ax = vx_g[ga], ay = vy_g[ga], az = vz_g[ga];
        R bx = vx_g[gb], by = vy_g[gb], bz = vz_g[gb];
        R hx, hy, hz;
        ta_half(ax - bx, ay - by, az - bz, C, wa.z, wa.w, wb.z, hx, hy, hz);
        ax += hx;
        ay += hy;
        az += hz;
        bx -= hx;
        by -= hy;
        bz -= hz;
        if (a.mcc_thr && (uint64_t)wa.y < a.mcc_thr) mcc_scatter<R>(ax, ay, az, pa, a.seed, step, a.mass_ratio);
        if (a.mcc_thr && (uint64_t)wb.y < a.mcc_thr) mcc_scatter<R>(bx, by, bz, pb, a.seed, step, a.mass_ratio);
        vx_g[ga] = ax;
        vy_g[ga] = ay;
        vz_g[ga] = az;
        vx_g[gb] = bx;
        vy_g[gb] = by;
        vz_g[gb] = bz;
    }
}

// ------------------------------------------------------------ huge cells
// One workgroup per cell; per-particle state in global scratch indexed by the
// particle's slot, so scratch regions of different cells never overlap.
// What the kernel is built for.  A form without the others' code keeps its
// members' values in registers: with everything in one kernel the binary64 form
// spilled 98 registers (cells of 7,000 with weights 890 us for 6M electrons, with
// the correction 3,540 for four steps; 4 registers now, 833 and 3,255).
enum { HUGE_PAIRS, HUGE_SEG, HUGE_ONE, HUGE_NANBU };

// Nanbu's operator out of line in binary64: in line its constants are kept over
// the loop and spill (cells of 7,000, 6M electrons, 1,715 us; 1,040 now).
struct HalfChange {
    double x, y, z;
};
__device__ __noinline__ HalfChange nanbu_call(double ux, double uy, double uz, double C, uint32_t wa2, uint32_t wb2)
{
    HalfChange h;
    nanbu_half<double>(ux, uy, uz, C, wa2, wb2, h.x, h.y, h.z);
    return h;
}
template <typename R>
__device__ __forceinline__ void nanbu_huge(R ux, R uy, R uz, R C, uint32_t wa2, uint32_t wb2, R &hx, R &hy, R &hz)
{
    if constexpr (std::is_same<R, double>::value) {
        const HalfChange h = nanbu_call(ux, uy, uz, C, wa2, wb2);
        hx = h.x;
        hy = h.y;
        hz = h.z;
    } else {
        nanbu_half<R>(ux, uy, uz, C, wa2, wb2, hx, hy, hz);
    }
}

template <typename R, int MODE>
__global__ __launch_bounds__(1024) void k_collide_huge(CollideArgs a, const int32_t *__restrict__ list,
                                                       int cls, HugeScratch hs, SegScratch ss,
                                                       const uint8_t *__restrict__ only)
{
    __shared__ double red[16 * 16];
    __shared__ uint32_t wtot[16];
    __shared__ int s_item;
    if (gated_off(a)) return;
    constexpr bool PAIRS = MODE == HUGE_PAIRS;
    if constexpr (MODE == HUGE_SEG)
        if (only) seg_fixup<R>(a, list, ss);
    if (only && !a.dflags->seg_fallback) return;   // every cell went the segmented way
    const uint32_t count = a.dflags->count[cls];
    if (blockIdx.x >= count) return;   // no work for this workgroup (nor a queue atomic)
    const int T = blockDim.x;
    R *vx_g = (R *)a.v;
    R *vy_g = vx_g + a.n;
    R *vz_g = vy_g + a.n;
    Rec<R> *pb = (Rec<R> *)hs.pbuf;
    for (uint32_t item = blockIdx.x;; item = count) {
        // Up to one cell a workgroup: by index, so that in the next step the cell
        // comes to the same XCD, whose L2 may still hold it (20 cells of 20,000 with
        // weights 244 us, from the counter 274).  Else one counter for the list,
        // for the first items too: a cell takes 50 us to milliseconds.  (Log-normal
        // cells up to 134,000 members with the correction, mean of eight grids of
        // 900 to 1,600: from 16 queues the step took 3.2 ms, 8% more than from one;
        // equal cells of 30,000 4% more.)
        if (count > gridDim.x) {
            if (threadIdx.x == 0) s_item = (int)list_take(a.dflags, cls);
            __syncthreads();
            item = (uint32_t)s_item;
            __syncthreads();
        }
        if (item >= count) break;
        if (only && !only[item]) continue;   // taken by the segmented path
        const int cell = list[item];
        const int lo = a.cell_start[cell];
        const int n = a.cell_start[cell + 1] - lo;
        const uint32_t step = (uint32_t)read_step(a);
        const bool coul = n >= 2;
        double before[4] = {0, 0, 0, 0};   // sum v, sum |v|^2
        for (int i = threadIdx.x; i < n; i += T) {
            const W4 w = draw4(a.seed, a.pid[lo + i], step, 0u, 0u);
            hs.keys[lo + i] = w.x;
            hs.w23[2 * (int64_t)(lo + i)] = w.z;
            hs.w23[2 * (int64_t)(lo + i) + 1] = w.w;
            hs.cand[lo + i] = (uint64_t)w.y < a.mcc_thr;
            if (!PAIRS && (a.flags & PIC_CONSERVE_FIX)) {
                const double x = vx_g[lo + i], y = vy_g[lo + i], z = vz_g[lo + i];
                before[0] += x;
                before[1] += y;
                before[2] += z;
                before[3] += x * x + y * y + z * z;
            }
        }
        __syncthreads();
        if (coul || PAIRS) gsort_positions(hs, a.pid, lo, n, wtot);
        if (PAIRS) {
            for (int i = threadIdx.x; i < n; i += T) a.sorted_out[lo + hs.pos[lo + i]] = lo + i;
            for (int i = threadIdx.x; i < n; i += T) {
                const uint32_t q = hs.pos[lo + i] ^ 1u;
                a.partner_out[lo + i] = (q < (uint32_t)n) ? lo + (int)hs.lst[lo + q] : -1;
            }
            __syncthreads();
            continue;
        }
        if (coul) {
            const R C = (R)cell_C(a, cell);
            Rec<R> *pc = pb + lo / 2 + (lo & 1);   // disjoint per cell
            for (int i = threadIdx.x; i < n; i += T) {
                const uint32_t p = hs.pos[lo + i];
                if (p & 1u) {
                    Rec<R> &e = pc[p >> 1];
                    e.x = vx_g[lo + i];
                    e.y = vy_g[lo + i];
                    e.z = vz_g[lo + i];
                    e.w2 = hs.w23[2 * (int64_t)(lo + i)];
                }
            }
            __syncthreads();
            // with the triplet, an odd cell's last three positions form it
            const uint32_t tstart = (a.variant == VAR_TRIPLET && (n & 1) && n >= 3) ? (uint32_t)n - 3u
                                                                                 : (uint32_t)n & ~1u;
            for (int i = threadIdx.x; i < n; i += T) {
                const uint32_t p = hs.pos[lo + i];
                if (!(p & 1u) && p + 1 < tstart) {
                    Rec<R> &e = pc[p >> 1];
                    R x = vx_g[lo + i], y = vy_g[lo + i], z = vz_g[lo + i];
                    R hx, hy, hz;
                    if constexpr (MODE == HUGE_NANBU) {
                        // the member in the lower storage slot is the operator's first
                        const uint32_t j = hs.lst[lo + p + 1];
                        const uint32_t own = hs.w23[2 * (int64_t)(lo + i)];
                        if ((uint32_t)i < j) {
                            nanbu_huge<R>(x - e.x, y - e.y, z - e.z, C, own, e.w2, hx, hy, hz);
                        } else {
                            nanbu_huge<R>(e.x - x, e.y - y, e.z - z, C, e.w2, own, hx, hy, hz);
                            hx = -hx;
                            hy = -hy;
                            hz = -hz;
                        }
                    } else {
                        ta_half(x - e.x, y - e.y, z - e.z, C, hs.w23[2 * (int64_t)(lo + i)],
                                hs.w23[2 * (int64_t)(lo + i) + 1], e.w2, hx, hy, hz);
                    }
                    bool ta = true, tb = true;
                    if (a.w) {
                        // the partner: the member at the next position
                        const R *wg = (const R *)a.w + lo;
                        const uint32_t j = hs.lst[lo + p + 1];
                        weight_rule<R>(wg[i], wg[j], hs.w23[2 * (int64_t)(lo + j) + 1], ta, tb);
                    }
                    if (ta) {
                        vx_g[lo + i] = x + hx;
                        vy_g[lo + i] = y + hy;
                        vz_g[lo + i] = z + hz;
                    }
                    // the second member subtracts what is left here
                    e.x = tb ? hx : (R)0;
                    e.y = tb ? hy : (R)0;
                    e.z = tb ? hz : (R)0;
                }
            }
            __syncthreads();
            for (int i = threadIdx.x; i < n; i += T) {
                const uint32_t p = hs.pos[lo + i];
                if ((p & 1u) && p < tstart) {
                    const Rec<R> &e = pc[p >> 1];
                    vx_g[lo + i] -= e.x;
                    vy_g[lo + i] -= e.y;
                    vz_g[lo + i] -= e.z;
                }
            }
            __syncthreads();
            if (tstart + 3 == (uint32_t)n && (n & 1) && threadIdx.x == 0) {
                // the triplet: one thread, members read through the sorted list
                int64_t sl[3];
                R x[3], y[3], z[3];
                uint32_t pd[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    sl[c] = lo + (int64_t)hs.lst[lo + tstart + c];
                    x[c] = vx_g[sl[c]];
                    y[c] = vy_g[sl[c]];
                    z[c] = vz_g[sl[c]];
                    pd[c] = a.pid[sl[c]];
                }
                const double dens = a.density ? a.density[cell] : 1.0;
                triplet_collide<R>(x, y, z, pd, (R)(8.0 * PI_D * dens * a.lnL * (0.5 * a.dt)), a.seed,
                                   step);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    vx_g[sl[c]] = x[c];
                    vy_g[sl[c]] = y[c];
                    vz_g[sl[c]] = z[c];
                }
            }
            __syncthreads();
            if (a.flags & PIC_CONSERVE_FIX) {
                double after[4] = {0, 0, 0, 0};
                for (int i = threadIdx.x; i < n; i += T) {
                    const double x = vx_g[lo + i], y = vy_g[lo + i], z = vz_g[lo + i];
                    after[0] += x;
                    after[1] += y;
                    after[2] += z;
                    after[3] += x * x + y * y + z * z;
                }
                block_sum<4>(before, red);
                block_sum<4>(after, red);
                const Correction cr = make_correction((double)n, before, after,
                                                      a.debt ? a.debt + (int64_t)cell * 4 : nullptr);
                if (cr.ok) {
                    double real[4] = {0, 0, 0, 0};
                    for (int i = threadIdx.x; i < n; i += T) {
                        const R x = (R)(cr.Vt[0] + cr.al * ((double)vx_g[lo + i] - cr.Vn[0]));
                        const R y = (R)(cr.Vt[1] + cr.al * ((double)vy_g[lo + i] - cr.Vn[1]));
                        const R z = (R)(cr.Vt[2] + cr.al * ((double)vz_g[lo + i] - cr.Vn[2]));
                        vx_g[lo + i] = x;
                        vy_g[lo + i] = y;
                        vz_g[lo + i] = z;
                        real[0] += (double)x;
                        real[1] += (double)y;
                        real[2] += (double)z;
                        real[3] += (double)x * x + (double)y * y + (double)z * z;
                    }
                    block_sum<4>(real, red);
                    if (a.debt && threadIdx.x == 0) store_debt(a.debt + (int64_t)cell * 4, cr, real);
                }
                __syncthreads();
            }
        }
        double m[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) m[q] = 0.0;
        for (int i = threadIdx.x; i < n; i += T) {
            R x = vx_g[lo + i], y = vy_g[lo + i], z = vz_g[lo + i];
            if (a.mcc_thr && hs.cand[lo + i]) {
                mcc_scatter<R>(x, y, z, a.pid[lo + i], a.seed, step, a.mass_ratio);
                vx_g[lo + i] = x;
                vy_g[lo + i] = y;
                vz_g[lo + i] = z;
            }
            if (a.flags & PIC_MOMENTS) moment_terms(m, x, y, z);
        }
        if (a.flags & PIC_MOMENTS) {
            const double t = block_sum_scatter<16>(m, red);
            if (threadIdx.x < 14) a.moments[(int64_t)cell * 14 + threadIdx.x] = t;
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------ segmented cells
// Cells beyond the largest LDS class with several workgroups each (see
// SegScratch): count members per segment, scan, copy ids and slots segment-major,
// sort and pair each segment in LDS, then the pairs across segment edges.
// The counting and copying kernels: one work item's members are one batch of
// SEG_U per thread, all loads in flight together.
constexpr int SEG_CT = 1024;
constexpr int SEG_U = SEG_CHUNK / SEG_CT;
static_assert(SEG_U * SEG_CT == SEG_CHUNK, "a work item is one batch");

struct SegItem {
    int h, lo, b, e;
    uint32_t S;
};

// Cells of at most this many segments are not copied: their segments' passes
// gather the velocities by storage slot, which saves 24 bytes a member of the
// copy (in binary32).  A gather finds its neighbours' lines in the XCD's L2 as
// long as a line's members belong to segments worked on together (32 a XCD);
// with thousands of segments every load is a line of its own.  Copied against
// gathered, the whole path: 100 cells of 90,000 346 / 315 us, 1,000 of 12,000
// 357 / 324, one of 2,000,000 (224 segments) 210 / 193, one of 20,000,000
// (2,233) 2,234 / 2,390; binary64, 100 of 40,000 426 / 350.
constexpr uint32_t SEG_GATHER = 1024;

// Work item -> its cell h of the list, the cell's first slot and the item's
// member range [b, e) inside the cell.
__device__ __forceinline__ SegItem seg_item(const CollideArgs &a, const SegScratch &ss,
                                            const int32_t *list, uint32_t item)
{
    SegItem it;
    it.h = ss.ch_owner[item];
    const int cell = list[it.h];
    it.lo = a.cell_start[cell];
    const int n = a.cell_start[cell + 1] - it.lo;
    // equal parts of whole 128-byte lines of a binary32 array
    const int parts = (n + SEG_CHUNK - 1) / SEG_CHUNK;
    const int per = ((n + parts - 1) / parts + 31) & ~31;
    it.b = min(n, (int)(item - (uint32_t)ss.hc_chunk[it.h]) * per);
    it.e = min(n, it.b + per);
    it.S = ss.hc_S[it.h];
    return it;
}

// Each segment's run in the scratch (exclusive scan of the sizes in table
// order) and the copy cursors, by one workgroup; a cell with a segment beyond
// cap takes the one-workgroup path.
__device__ __forceinline__ void seg_scan(const CollideArgs &a, const SegScratch &ss, uint32_t cap, uint32_t *wtot,
                                         uint32_t *s_tot)
{
    const uint32_t nseg = a.dflags->count[SEG_SLOT];
    uint32_t base = 0;
    for (uint32_t j0 = 0; j0 < nseg; j0 += SEG_CT) {
        const uint32_t j = j0 + threadIdx.x;
        // written by the other workgroups of this launch: read past the caches
        const uint32_t c =
            j < nseg ? __hip_atomic_load(&ss.sg_cnt[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        const uint32_t off = block_excl(c, wtot);
        if (j < nseg) {
            ss.sg_start[j] = base + off;
            ss.sg_cur[j] = base + off;
            if (c > cap) {
                ss.hc_fb[ss.sg_cell[j]] = 1;
                a.dflags->seg_fallback = 1;
            }
        }
        if (threadIdx.x == SEG_CT - 1) *s_tot = off + c;
        __syncthreads();
        base += *s_tot;
        __syncthreads();
    }
}

// Segment sizes: an LDS histogram per work item, then one global add per
// non-empty segment.  The workgroup that ends last scans them: the adds are done
// where the device is coherent, each wave waits for its own (s_waitcnt vmcnt, with
// a __syncthreads behind it that also orders the compiler) before its workgroup
// reports, and the last one reads past the caches.  (A relaxed counter orders
// nothing in the language's memory model; see k_radix_count for the reasons it
// holds here.)  With the edge pairs done in k_collide_huge the
// path is four launches instead of six, about 2.7 us each where it has nothing
// to do.
__global__ __launch_bounds__(SEG_CT) void k_seg_count(CollideArgs a, const int32_t *__restrict__ list,
                                                      SegScratch ss, uint32_t cap)
{
    __shared__ uint32_t hist[SEG_MAX];
    __shared__ uint32_t wtot[SEG_CT / PIC_WAVE];
    __shared__ uint32_t s_tot;
    if (gated_off(a)) return;
    const uint32_t items = a.dflags->count[CHUNK_SLOT];
    if (blockIdx.x >= items) return;
    const uint32_t step = (uint32_t)read_step(a);
    for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
        const SegItem it = seg_item(a, ss, list, item);
        const uint32_t S = it.S;
        for (uint32_t q = threadIdx.x; q < S; q += SEG_CT) hist[q] = 0u;
        __syncthreads();
        uint32_t pv[SEG_U];
#pragma unroll
        for (int u = 0; u < SEG_U; ++u)
            pv[u] = ld_at(a.pid + it.lo, (uint32_t)min(it.b + (int)threadIdx.x + u * SEG_CT, it.e - 1));
#pragma unroll
        for (int u = 0; u < SEG_U; ++u)
            if (it.b + (int)threadIdx.x + u * SEG_CT < it.e)
                atomicAdd(&hist[seg_of(draw4(a.seed, pv[u], step, 0u, 0u).x, S)], 1u);
        __syncthreads();
        const int32_t sb = ss.hc_seg[it.h];
        for (uint32_t q = threadIdx.x; q < S; q += SEG_CT)
            if (hist[q]) atomicAdd(&ss.sg_cnt[sb + q], hist[q]);
        __syncthreads();
    }
    __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);   // this wave's adds have completed
    __syncthreads();
    if (threadIdx.x == 0)
        s_tot = __hip_atomic_fetch_add(&a.dflags->seg_done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const bool last = s_tot + 1u == min(gridDim.x, items);
    __syncthreads();
    if (last) seg_scan(a, ss, cap, wtot, &s_tot);
}

// Members to their segment's run: each member's arrival rank in its segment
// from an LDS counter, one global reservation per non-empty segment, then each
// member at its reservation plus its rank (the order inside a run is free: the
// segment pass sorts by key and pid).  Bound by its bytes (36 a member in
// binary32): one read of the members, ids and velocities together, with the
// ranks kept in registers, on 32 waves a CU (256 threads, two reads and two
// counts: 93 us for the cells beyond 10,240 members of a log-normal 40M
// electrons; copying ids and slots only, now 53).
template <typename R>
__global__ __launch_bounds__(SEG_CT) void k_seg_scatter(CollideArgs a, const int32_t *__restrict__ list,
                                                        SegScratch ss)
{
    __shared__ uint32_t hist[SEG_MAX];   // counts, then the first slots reserved
    if (gated_off(a)) return;
    const uint32_t items = a.dflags->count[CHUNK_SLOT];
    const uint32_t step = (uint32_t)read_step(a);
    for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
        const SegItem it = seg_item(a, ss, list, item);
        if (ss.hc_fb[it.h]) continue;   // the same for the whole workgroup
        // the cell's members and its run in the scratch (indices within a cell
        // fit the 32-bit offsets of ld_at and st_at)
        const int32_t sb = ss.hc_seg[it.h];
        const uint32_t run = ss.sg_start[sb];
        const R *v = (const R *)a.v + it.lo;
        R *mv = (R *)ss.m_v + run;
        const uint32_t S = it.S;
        uint32_t pv[SEG_U], q[SEG_U];
        R x[SEG_U], y[SEG_U], z[SEG_U];
        const bool copy = S > SEG_GATHER;
#pragma unroll
        for (int u = 0; u < SEG_U; ++u) {
            const uint32_t i = (uint32_t)min(it.b + (int)threadIdx.x + u * SEG_CT, it.e - 1);
            pv[u] = ld_at(a.pid + it.lo, i);
            if (copy) {
                x[u] = ld_at(v, i);
                y[u] = ld_at(v + a.n, i);
                z[u] = ld_at(v + 2 * a.n, i);
            }
        }
        for (uint32_t j = threadIdx.x; j < S; j += SEG_CT) hist[j] = 0u;
        lds_barrier();
#pragma unroll
        for (int u = 0; u < SEG_U; ++u) {
            q[u] = seg_of(draw4(a.seed, pv[u], step, 0u, 0u).x, S);
            // segment (12 bits) and arrival rank (below SEG_CHUNK)
            if (it.b + (int)threadIdx.x + u * SEG_CT < it.e) q[u] |= atomicAdd(&hist[q[u]], 1u) << 16;
        }
        lds_barrier();
        for (uint32_t j = threadIdx.x; j < S; j += SEG_CT)
            if (hist[j]) hist[j] = atomicAdd(&ss.sg_cur[sb + j], hist[j]) - run;
        lds_barrier();
#pragma unroll
        for (int u = 0; u < SEG_U; ++u) {
            const int i = it.b + (int)threadIdx.x + u * SEG_CT;
            if (i < it.e) {
                const uint32_t slot = hist[q[u] & 0xffffu] + (q[u] >> 16);
                st_at(ss.m_orig + run, slot, it.lo + i);
                st_at(ss.m_pid + run, slot, pv[u]);
                if (copy) {
                    st_at(mv, slot, x[u]);
                    st_at(mv + ss.m_stride, slot, y[u]);
                    st_at(mv + 2 * ss.m_stride, slot, z[u]);
                }
            }
        }
        lds_barrier();
    }
}
static_assert(SEG_MAX <= 1 << 16 && SEG_CHUNK <= 1 << 16, "segment and rank share a word");

// One segment: the members of run [start, start + n) sort by key (by their
// position inside the segment's key range, scaled to 32 bits, whose top bits
// bucket them) and pid; local
// position q is position off + q of the cell.  The cell's pairs (2i, 2i + 1)
// inside the segment collide here as in the cell pass; a member whose
// partner lies in a neighbouring segment is recorded for seg_fixup and left
// unchanged (its null collision too).
template <typename R, int T, int K, int F>
__device__ __forceinline__ void seg_pass(const CollideArgs &a, const int32_t *list, const SegScratch &ss, int seg,
                         unsigned char *smem, uint32_t *wtot)
{
    constexpr bool MCC = (F & F_MCC) != 0;
    constexpr int CAP = T * K;
    const int h = ss.sg_cell[seg];
    const uint32_t n = ss.sg_cnt[seg];
    if (ss.hc_fb[h] || n == 0) {
        __syncthreads();
        return;
    }
    const int cell = list[h];
    const int lo_c = a.cell_start[cell];
    const uint32_t n_c = (uint32_t)(a.cell_start[cell + 1] - lo_c);
    const uint32_t start = ss.sg_start[seg];
    const uint32_t off = start - ss.sg_start[ss.hc_seg[h]];
    const uint32_t S = ss.hc_S[h];
    const uint32_t step = (uint32_t)read_step(a);
    const R *mx = (const R *)ss.m_v + start;
    const R *my = mx + ss.m_stride;
    const R *mz = my + ss.m_stride;
    const uint32_t *pid_s = ss.m_pid + start;
    const int32_t *orig = ss.m_orig + start;
    R *vx_g = (R *)a.v;
    R *vy_g = vx_g + a.n;
    R *vz_g = vy_g + a.n;
    const SortLDS<T, CAP> L(smem);
    const bool gather = S <= SEG_GATHER;

    R vx[K], vy[K], vz[K];
    uint32_t w2[K], w3[K], pos[K];
    uint32_t cand = 0;
    const uint32_t bits = sort_bits((int)n);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < (int)n) {
            pos[k] = pid_s[i];
            if (gather) {
                const int32_t g = orig[i];
                vx[k] = vx_g[g];
                vy[k] = vy_g[g];
                vz[k] = vz_g[g];
            } else {
                vx[k] = mx[i];
                vy[k] = my[i];
                vz[k] = mz[i];
            }
        }
    }
    L.clear();
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < (int)n) {
            const W4 w = draw4(a.seed, pos[k], step, 0u, 0u);
            w2[k] = w.z;
            w3[k] = w.w;
            if (MCC && (uint64_t)w.y < a.mcc_thr) cand |= 1u << k;
            pos[k] = L.count(i, seg_key(w.x, S), bits);
        }
    }
    __syncthreads();
    rank_in_lds<T, K, CAP>(pos, (int)n, bits, L, pid_s, wtot);

    // local pairs cover positions [first, first + np2)
    const uint32_t first = off & 1u;
    const uint32_t np2 = (n - first) & ~1u;
    uint32_t edge = 0;   // bit k: the partner is in a neighbouring segment
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < (int)n) {
            if (first && pos[k] == 0u) {
                edge |= 1u << k;
                ss.bnd_head[seg] = (int32_t)(start + i);
            } else if (pos[k] == first + np2 && off + pos[k] + 1u < n_c) {
                edge |= 1u << k;
                ss.bnd_tail[seg] = (int32_t)(start + i);
            }
        }
    }
    {
        const R C = (R)cell_C(a, cell);
        constexpr uint32_t P = round_positions<R>(CAP);
        Rec<R> *rec = (Rec<R> *)smem;
        uint32_t *w3s = (uint32_t *)(rec + P);
        for (uint32_t base = 0; base < np2; base += P) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int i = threadIdx.x + k * T;
                const uint32_t pl = pos[k] - first;   // wraps for the lower edge member
                const uint32_t q = pl - base;
                if (i < (int)n && pl < np2 && q < P) {
                    Rec<R> e;
                    e.x = vx[k];
                    e.y = vy[k];
                    e.z = vz[k];
                    e.w2 = w2[k];
                    rec[q] = e;
                    if (!(q & 1u)) w3s[q >> 1] = w3[k];
                }
            }
            __syncthreads();
            const uint32_t m = min(P, np2 - base) / 2;
            for (uint32_t j = threadIdx.x; j < m; j += T) {
                Rec<R> A = rec[2 * j], B = rec[2 * j + 1];
                R hx, hy, hz;
                ta_half<true>(A.x - B.x, A.y - B.y, A.z - B.z, C, A.w2, w3s[j], B.w2, hx, hy, hz);
                A.x += hx;
                A.y += hy;
                A.z += hz;
                B.x -= hx;
                B.y -= hy;
                B.z -= hz;
                rec[2 * j] = A;
                rec[2 * j + 1] = B;
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int i = threadIdx.x + k * T;
                const uint32_t pl = pos[k] - first;
                const uint32_t q = pl - base;
                if (i < (int)n && pl < np2 && q < P) {
                    const Rec<R> e = rec[q];
                    vx[k] = e.x;
                    vy[k] = e.y;
                    vz[k] = e.z;
                }
            }
            if (base + P < np2) __syncthreads();
        }
    }
    if constexpr (MCC) {
        uint32_t left = cand & ~edge;
        while (__ballot(left != 0u) != 0ull) {
            if (left) {
                const int kk = __builtin_ctz(left);
                left &= left - 1u;
                R x = vx[0], y = vy[0], z = vz[0];
#pragma unroll
                for (int k = 1; k < K; ++k)
                    if (kk == k) {
                        x = vx[k];
                        y = vy[k];
                        z = vz[k];
                    }
                mcc_scatter_as<R, (F & F_CALL) != 0, true>(x, y, z, pid_s[threadIdx.x + kk * T], a.seed, step, a.mass_ratio);
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (kk == k) {
                        vx[k] = x;
                        vy[k] = y;
                        vz[k] = z;
                    }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        if (i < (int)n && !((edge >> k) & 1u)) {
            const int32_t g = orig[i];
            vx_g[g] = vx[k];
            vy_g[g] = vy[k];
            vz_g[g] = vz[k];
        }
    }
    // every thread leaves together (see cell_pass)
    __syncthreads();
}

// Work items in order of arrival -> segments such that the items of one
// remainder mod 8 (the workgroups of one XCD take them) are neighbouring
// segments: the scattered stores of a cell's segments then meet in one L2.
__device__ __forceinline__ uint32_t xcd_run(uint32_t item, uint32_t count)
{
    const uint32_t q = count / 8u, r = count % 8u, x = item % 8u;
    return x * q + min(x, r) + item / 8u;
}

// The same in binary32, on the lean pass's sort and exchange rounds: positions
// count from the first one paired inside the segment, so the member paired
// across the lower edge has position -1 and takes part in no round; the one
// paired across the upper edge is the round's unpaired last one.  With nx the
// next segment's members are requested meanwhile, and the next work item is
// returned (see lean_pass).  The large cells of a log-normal 40M electrons:
// 164 us (the class kernels' sort and exchange on copied members 180).
template <int T, int K, int F>
__device__ __forceinline__ int lean_seg_pass(const CollideArgs &a, const int32_t *list, const SegScratch &ss,
                                             uint32_t seg, unsigned char *smem, uint32_t *wtot,
                                             const LeanNext *nx = nullptr)
{
    constexpr bool MCC = (F & F_MCC) != 0;
    constexpr uint32_t P = LeanExch<T, K, F>::P;
    const int h = ss.sg_cell[seg];
    const int n = (int)ss.sg_cnt[seg];
    const uint32_t step = (uint32_t)read_step(a);
    if (ss.hc_fb[h] || n == 0) {
        if (nx && threadIdx.x == 0) *nx->slot = (int)queue_take(a.dflags, nx->cls, (unsigned)nx->slot[1], (unsigned)nx->slot[2]);
        lds_barrier();
        const int next = nx ? *nx->slot : 0;
        lds_barrier();
        return next;
    }
    const int cell = list[h];
    const int lo_c = a.cell_start[cell];
    const uint32_t n_c = (uint32_t)(a.cell_start[cell + 1] - lo_c);
    const uint32_t start = ss.sg_start[seg];
    const uint32_t off = start - ss.sg_start[ss.hc_seg[h]];
    const uint32_t S = ss.hc_S[h];
    const uint32_t *pid_s = ss.m_pid + start;

    float vx[K], vy[K], vz[K];
    float wt[1];
    uint32_t w2[K], w3[K], key[K], pos[K];
    uint32_t cand = 0, cpid = 0;
    {
        uint32_t ic[K];
#pragma unroll
        for (int k = 0; k < K; ++k) ic[k] = (uint32_t)min((int)threadIdx.x + k * T, n - 1);
#pragma unroll
        for (int k = 0; k < K; ++k) pos[k] = ld_at(pid_s, ic[k]);
        asm volatile("" ::: "memory");   // keep the id loads ahead of the velocity loads
        // the copy, or the members in their storage slots
        const float *mx = (const float *)ss.m_v + start;
        size_t stride = (size_t)ss.m_stride;
        if (S <= SEG_GATHER) {
            mx = (const float *)a.v + lo_c;
            stride = (size_t)a.n;
#pragma unroll
            for (int k = 0; k < K; ++k) ic[k] = (uint32_t)(ld_at(ss.m_orig + start, ic[k]) - lo_c);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            vx[k] = ld_at(mx, ic[k]);
            vy[k] = ld_at(mx + stride, ic[k]);
            vz[k] = ld_at(mx + 2 * stride, ic[k]);
        }
    }
    if (nx && threadIdx.x == 0) *nx->slot = (int)queue_take(a.dflags, nx->cls, (unsigned)nx->slot[1], (unsigned)nx->slot[2]);
    if (n >= 2) {
        lean_sort<T, K, MCC, true, true>(a, n, step, pid_s, smem, wtot, w2, w3, key, pos, cand, cpid, S);
    } else {
        // a lone member: only its null collision and its place are needed
        const W4 w = draw4(a.seed, pos[0], step, 0u, 0u);
        if (MCC && threadIdx.x == 0 && (uint64_t)w.y < a.mcc_thr) {
            cpid = pos[0];
            cand = 1u;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            w2[k] = w.z;
            w3[k] = w.w;
            pos[k] = 0u;
        }
    }
    lds_barrier();   // the sort's memory becomes the exchange records

    // pairs inside the segment cover local positions [first, first + np2)
    const uint32_t first = off & 1u;
    const uint32_t np2 = ((uint32_t)n - first) & ~1u;
    const bool tail = off + first + np2 + 1u < n_c;   // the position after them has its partner above
    const int kf = cand ? __builtin_ctz(cand) : K;
    uint32_t edge = 0;   // bit k: the partner is in a neighbouring segment
    const int n1 = opaque(n);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = threadIdx.x + k * T;
        pos[k] -= first;
        if (i < n1) {
            if (pos[k] == 0xffffffffu) {
                edge |= 1u << k;
                ss.bnd_head[seg] = (int32_t)(start + i);
            } else if (tail && pos[k] == np2) {
                edge |= 1u << k;
                ss.bnd_tail[seg] = (int32_t)(start + i);
            }
        }
    }
    if constexpr (MCC) cand &= ~edge;
    const float C = (float)cell_C(a, cell);
    if (nx) {
        asm volatile("" ::"v"(C));   // complete before the requests below
        const uint32_t nxt = (uint32_t)*nx->slot;
        if (nxt < nx->count) {
            const uint32_t s2 = xcd_run(nxt, nx->count);
            const uint32_t st = ss.sg_start[s2];
            const int n2 = (int)ss.sg_cnt[s2];
            prefetch_run<T>(ss.m_pid + st, 1u, (const float *)ss.m_orig + st, 0, n2, nx->sink);
            if (ss.hc_S[ss.sg_cell[s2]] > SEG_GATHER)
                prefetch_run<T>(ss.m_pid + st, 3u, (const float *)ss.m_v + st, (size_t)ss.m_stride, n2, nx->sink);
        }
    }
    for (uint32_t base = 0; base + first < (uint32_t)n; base += P) {
        if (base) lds_barrier();
        lean_round<T, K, F>(base, np2, opaque(n), C, smem, vx, vy, vz, w2, w3, wt, pos, cand, kf, cpid, pid_s, a,
                            cell, step);
    }
    if (nx) __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
    const int n3 = opaque(n);
    uint32_t g[K];
#pragma unroll
    for (int k = 0; k < K; ++k)
        g[k] = (uint32_t)(ld_at(ss.m_orig + start, (uint32_t)min((int)threadIdx.x + k * T, n3 - 1)) - lo_c);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if ((int)threadIdx.x + k * T < n3 && !((edge >> k) & 1u)) {
            st_at((float *)a.v + lo_c, g[k], vx[k]);
            st_at((float *)a.v + a.n + lo_c, g[k], vy[k]);
            st_at((float *)a.v + 2 * a.n + lo_c, g[k], vz[k]);
        }
    }
    const int next = nx ? *nx->slot : 0;
    lds_barrier();   // every thread leaves together; the stores stay in flight
    return next;
}

template <typename R, int T, int K, int F>
__global__ __launch_bounds__(T) void k_seg_collide(CollideArgs a, const int32_t *__restrict__ list,
                                                   SegScratch ss)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t wtot[T / PIC_WAVE];
    __shared__ int s_next[3];
    if (gated_off(a)) return;
    const uint32_t count = a.dflags->count[SEG_SLOT];
    if (blockIdx.x >= count) return;   // no work for this workgroup (nor a queue atomic)
    // a queue of the workgroup's own XCD (see xcd_run)
    const unsigned queue = blockIdx.x % QUEUE_SPLIT;
    if constexpr (std::is_same<R, float>::value) {
        __shared__ float sink[PIC_WAVE];
        if (threadIdx.x == 0) {
            s_next[1] = (int)queue;
            s_next[2] = (int)gridDim.x;
        }
        const LeanNext nx{s_next, SEG_SLOT, list, count, sink};
        for (uint32_t item = blockIdx.x; item < count;)
            item = (uint32_t)lean_seg_pass<T, K, F>(a, list, ss, xcd_run(item, count), smem, wtot, &nx);
    } else {
        for (uint32_t item = blockIdx.x; item < count;) {
            if (threadIdx.x == 0) s_next[0] = (int)queue_take(a.dflags, SEG_SLOT, queue, gridDim.x);   // read after the pass's barriers
            seg_pass<R, T, K, F>(a, list, ss, (int)xcd_run(item, count), smem, wtot);
            item = (uint32_t)s_next[0];
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------ deferred cells
// A cell the gate defers skips the Coulomb step and enters no class queue.
// When null collisions are on it is listed here for its candidates (about 1%
// of the members: one Philox word per member decides).  One workgroup per
// cell, cells dealt round-robin (no queue atomics).
constexpr int DEFER_T = 256;

template <typename R>
__global__ __launch_bounds__(DEFER_T) void k_deferred(CollideArgs a, const int32_t *__restrict__ list)
{
    if (gated_off(a)) return;
    const uint32_t count = a.dflags->count[LIST_DEFERRED];
    const uint32_t step = (uint32_t)read_step(a);
    for (uint32_t item = blockIdx.x; item < count; item += gridDim.x) {
        const int cell = list[item];
        const int lo = a.cell_start[cell];
        const int n = a.cell_start[cell + 1] - lo;
        R *vx_g = (R *)a.v + lo;
        R *vy_g = (R *)a.v + a.n + lo;
        R *vz_g = (R *)a.v + 2 * a.n + lo;
        const uint32_t *pid_c = a.pid + lo;
        for (int i = threadIdx.x; i < n; i += DEFER_T) {
            if ((uint64_t)draw4(a.seed, pid_c[i], step, 0u, 0u).y < a.mcc_thr) {
                R x = vx_g[i], y = vy_g[i], z = vz_g[i];
                mcc_scatter<R>(x, y, z, pid_c[i], a.seed, step, a.mass_ratio);
                vx_g[i] = x;
                vy_g[i] = y;
                vz_g[i] = z;
            }
        }
    }
}

// ------------------------------------------------------------ class table
// Class c handles cells with at most cap[c] members (T threads x K items).
template <typename R> struct Classes;
template <> struct Classes<float> {
    static constexpr int T0 = 256, K0 = 2;    // <= 512
    static constexpr int T1 = 512, K1 = 4;    // <= 2048
    // 512 x 8 rather than 1024 x 4: two workgroups (74 KB of LDS each) are
    // resident per CU, and one hides the other's latencies
    static constexpr int T2 = 512, K2 = 8;    // <= 4096
    static constexpr int T3 = 1024, K3 = 10;  // <= 10240
};
template <> struct Classes<double> {
    static constexpr int T0 = 256, K0 = 2;
    static constexpr int T1 = 512, K1 = 4;
    static constexpr int T2 = 1024, K2 = 4;
    static constexpr int T3 = 1024, K3 = 6;   // <= 6144
};
static_assert(Classes<float>::T3 * Classes<float>::K3 == PIC_NOALLOC_MAX_CELL_F32 &&
                  Classes<double>::T3 * Classes<double>::K3 == PIC_NOALLOC_MAX_CELL_F64,
              "the allocation-free step takes the cells of the LDS classes");

// The binary64 lean pass: 1,024 threads of ten members (cells of up to
// 10,240 members on one workgroup instead of the segmented path).
constexpr int LEAN64_T = 1024, LEAN64_K = 10;

// Workgroup geometry of one segment of the segmented path: the largest
// class's (segments of 2,560 members on two 512-thread workgroups per CU
// were slower: more segments, histograms and edge pairs).
template <typename R> struct SegGeom;
template <> struct SegGeom<float> {
    static constexpr int T = 1024, K = 10, PER_CU = 1;
};
template <> struct SegGeom<double> {
    static constexpr int T = 1024, K = 6, PER_CU = 1;
};

// ------------------------------------------------------------ one wave per cell
// Small cells on a single wave with its own slice of LDS: the same pairing,
// rotation and null collisions as the block passes, with wave-level
// synchronisation only (LDS operations of one wave complete in order), so the
// 16 waves of a workgroup work on 16 cells at once.
template <typename R> struct WaveGeom;
template <> struct WaveGeom<float> {
    static constexpr int KW = 8;       // cells of up to 512 members
};
template <> struct WaveGeom<double> {
    static constexpr int KW = 4;       // up to 256 (records of 32 bytes)
};
constexpr size_t WAVE_SLICE = 8 * 1024 + 512;   // LDS bytes per wave

__device__ __forceinline__ void wave_sync()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

template <typename R, bool MCC>
__device__ __forceinline__ void wave_pass(const CollideArgs &a, int cell, unsigned char *slice)
{
    constexpr int KW = WaveGeom<R>::KW;
    constexpr int CAP = PIC_WAVE * KW;
    const int lane = threadIdx.x & (PIC_WAVE - 1);
    const int lo = a.cell_start[cell];
    const int n = a.cell_start[cell + 1] - lo;
    if (n == 0) return;
    const uint32_t step = (uint32_t)read_step(a);
    R *vx_g = (R *)a.v + lo;
    R *vy_g = (R *)a.v + a.n + lo;
    R *vz_g = (R *)a.v + 2 * a.n + lo;
    const uint32_t *pid_c = a.pid + lo;
    R vx[KW], vy[KW], vz[KW];
    uint32_t w2[KW], w3[KW], key[KW], pos[KW];
    uint32_t cand = 0, multi = 0;
    {
        int ic[KW];
#pragma unroll
        for (int k = 0; k < KW; ++k) ic[k] = min(lane + k * PIC_WAVE, n - 1);
#pragma unroll
        for (int k = 0; k < KW; ++k) pos[k] = pid_c[ic[k]];
        asm volatile("" ::: "memory");   // keep the id loads ahead of the velocity loads
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            vx[k] = vx_g[ic[k]];
            vy[k] = vy_g[ic[k]];
            vz[k] = vz_g[ic[k]];
        }
    }
    if (n >= 2) {
        const uint32_t bits = sort_bits(n);
        const uint32_t nb = 1u << bits;
        uint32_t *cnt = (uint32_t *)slice;
        uint32_t *sk = cnt + CAP + 4;
        uint16_t *lst = (uint16_t *)(sk + CAP);
        for (uint32_t q = lane; q < nb; q += PIC_WAVE) cnt[q] = 0u;
        wave_sync();
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const int i = lane + k * PIC_WAVE;
            if (i < n) {
                const W4 w = draw4(a.seed, pos[k], step, 0u, 0u);
                key[k] = w.x;
                w2[k] = w.z;
                w3[k] = w.w;
                if (MCC && (uint64_t)w.y < a.mcc_thr) cand |= 1u << k;
                pos[k] = atomicAdd(&cnt[w.x >> (32u - bits)], 1u);
            }
        }
        wave_sync();
        {
            // bucket starts: rows of 64 counters with a running carry
            uint32_t carry = 0;
            for (uint32_t r0 = 0; r0 < nb; r0 += PIC_WAVE) {
                const uint32_t q = r0 + lane;
                const uint32_t v = q < nb ? cnt[q] : 0u;
                const uint32_t inc = wave_incl_scan_dpp(v);
                if (q < nb) cnt[q] = carry + inc - v;
                carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, PIC_WAVE - 1);
            }
            if (lane == 0) cnt[nb] = carry;
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const int i = lane + k * PIC_WAVE;
            if (i < n) {
                const uint32_t b = key[k] >> (32u - bits);
                const uint32_t st = cnt[b], en = cnt[b + 1];
                const uint32_t slot = st + pos[k];
                pos[k] = slot;
                if (en - st > 1u) {
                    multi |= 1u << k;
                    sk[slot] = key[k];
                    lst[slot] = (uint16_t)i;
                }
            }
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            if ((multi >> k) & 1u) {
                const int i = lane + k * PIC_WAVE;
                const uint32_t b = key[k] >> (32u - bits);
                const uint32_t st = cnt[b], en = cnt[b + 1];
                uint32_t r = 0, tie = 0;
                for (uint32_t j = st; j < en; ++j) {
                    const uint32_t kj = sk[j];
                    r += kj < key[k] ? 1u : 0u;
                    tie |= (kj == key[k] && j != pos[k]) ? 1u : 0u;
                }
                if (tie) {
                    const uint32_t pi = pid_c[i];
                    for (uint32_t j = st; j < en; ++j)
                        if (j != pos[k] && sk[j] == key[k] && pid_c[lst[j]] < pi) ++r;
                }
                pos[k] = st + r;
            }
        }
        wave_sync();   // the sort's slice becomes the exchange records
        const R C = (R)cell_C(a, cell);
        const uint32_t np2 = (uint32_t)n & ~1u;
        Rec<R> *rec = (Rec<R> *)slice;
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const int i = lane + k * PIC_WAVE;
            if (i < n && pos[k] < np2) {
                Rec<R> e;
                e.x = vx[k];
                e.y = vy[k];
                e.z = vz[k];
                if constexpr (std::is_same<R, float>::value) {
                    // first members carry their deviate, second ones word 2
                    e.w2 = (pos[k] & 1u) ? w2[k] : __float_as_uint(ta_z(w2[k], w3[k]));
                } else {
                    e.w2 = w2[k];
                    e.pad = w3[k];
                }
                rec[pos[k]] = e;
            }
        }
        wave_sync();
        for (uint32_t j = lane; j < np2 / 2; j += PIC_WAVE) {
            Rec<R> A = rec[2 * j], B = rec[2 * j + 1];
            R hx, hy, hz;
            if constexpr (std::is_same<R, float>::value)
                ta_half_z(A.x - B.x, A.y - B.y, A.z - B.z, C, __uint_as_float(A.w2), B.w2, hx, hy, hz);
            else
                ta_half(A.x - B.x, A.y - B.y, A.z - B.z, C, A.w2, A.pad, B.w2, hx, hy, hz);
            A.x += hx;
            A.y += hy;
            A.z += hz;
            B.x -= hx;
            B.y -= hy;
            B.z -= hz;
            rec[2 * j] = A;
            rec[2 * j + 1] = B;
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const int i = lane + k * PIC_WAVE;
            if (i < n && pos[k] < np2) {
                const Rec<R> e = rec[pos[k]];
                vx[k] = e.x;
                vy[k] = e.y;
                vz[k] = e.z;
            }
        }
    } else if (MCC) {
        const W4 w = draw4(a.seed, pos[0], step, 0u, 0u);
        if (lane == 0 && (uint64_t)w.y < a.mcc_thr) cand = 1u;
    }
    if constexpr (MCC) {
        uint32_t left = cand;
        while (__ballot(left != 0u) != 0ull) {
            if (left) {
                const int kk = __builtin_ctz(left);
                left &= left - 1u;
                R x = vx[0], y = vy[0], z = vz[0];
#pragma unroll
                for (int k = 1; k < KW; ++k)
                    if (kk == k) {
                        x = vx[k];
                        y = vy[k];
                        z = vz[k];
                    }
                mcc_scatter_as<R, true>(x, y, z, pid_c[lane + kk * PIC_WAVE], a.seed, step, a.mass_ratio);
#pragma unroll
                for (int k = 0; k < KW; ++k)
                    if (kk == k) {
                        vx[k] = x;
                        vy[k] = y;
                        vz[k] = z;
                    }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        const int i = lane + k * PIC_WAVE;
        if (i < n) {
            vx_g[i] = vx[k];
            vy_g[i] = vy[k];
            vz_g[i] = vz[k];
        }
    }
    wave_sync();   // the slice is free for the wave's next cell
}

// ------------------------------------------------------------ one launch per step
// The block cells of the step (every class that a whole workgroup takes, and
// with the wave schedule off also the smallest class) in one list ordered
// largest first: a counting sort of the cells by a size bucket that halves
// every four steps (sizes within a bucket differ by at most 19%).  One
// workgroup; order[] gets the cells, flags->pad[ORDER_TOTAL] their number.
constexpr int ORDER_BUCKETS = 72;
constexpr int ORDER_TOTAL = 0;   // index into DevFlags::pad

__device__ __forceinline__ int order_bucket(int32_t n)
{
    // 4 log2 n rounded down, from the leading bit and the two bits after it
    const uint32_t u = n > 1 ? (uint32_t)n : 1u;
    const int msb = 31 - __clz(u);
    const int frac = msb >= 2 ? (int)((u >> (msb - 2)) & 3u) : (int)((u << (2 - msb)) & 3u);
    const int key = 4 * msb + frac;                 // grows with n
    const int b = ORDER_BUCKETS - 1 - key;          // largest first
    return b < 0 ? 0 : b;
}

__global__ __launch_bounds__(1024) void k_order_queue(const int32_t *__restrict__ cs,
                                                      const int32_t *__restrict__ lists, int32_t M,
                                                      int first_cls, int last_cls, DevFlags *f,
                                                      int32_t *__restrict__ order)
{
    __shared__ uint32_t hist[ORDER_BUCKETS];
    __shared__ uint32_t cls_off[5];
    if (threadIdx.x < ORDER_BUCKETS) hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (int c = first_cls; c <= last_cls; ++c) {
            cls_off[c] = acc;
            acc += f->count[c];
        }
        cls_off[4] = acc;
        f->pad[ORDER_TOTAL] = acc;
    }
    __syncthreads();
    const uint32_t total = cls_off[4];
    // the cells of classes first..last, walked as one run
    auto cell_at = [&](uint32_t q) {
        int c = first_cls;
        while (c < last_cls && q >= cls_off[c + 1]) ++c;
        return lists[(int64_t)c * M + (q - cls_off[c])];
    };
    for (uint32_t q = threadIdx.x; q < total; q += 1024) {
        const int32_t cell = cell_at(q);
        atomicAdd(&hist[order_bucket(cs[cell + 1] - cs[cell])], 1u);
    }
    __syncthreads();
    if (threadIdx.x < PIC_WAVE) {
        uint32_t carry = 0;
        for (int b0 = 0; b0 < ORDER_BUCKETS; b0 += PIC_WAVE) {
            const int b = b0 + (int)threadIdx.x;
            const uint32_t v = b < ORDER_BUCKETS ? hist[b] : 0u;
            const uint32_t inc = wave_incl_scan(v);
            if (b < ORDER_BUCKETS) hist[b] = carry + inc - v;
            carry += __shfl(inc, PIC_WAVE - 1, PIC_WAVE);
        }
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < total; q += 1024) {
        const int32_t cell = cell_at(q);
        order[atomicAdd(&hist[order_bucket(cs[cell + 1] - cs[cell])], 1u)] = cell;
    }
}

// The whole collide pass of a step in one persistent launch: each workgroup
// takes items from one queue, the segments of the largest cells first, then
// the block cells largest first (their size picks the pass: 1024 threads with
// K members each), and when that queue is empty each of its waves takes cells
// of the smallest class one at a time.  Small cells thus fill the tail that
// the large ones leave, inside the same launch.
template <typename R, int F>
__global__ __launch_bounds__(1024) void k_collide_all(CollideArgs a, const int32_t *__restrict__ lists,
                                                      int32_t M, const int32_t *__restrict__ order,
                                                      SegScratch ss, ClassCaps caps, int use_seg,
                                                      int wave_cls)
{
    constexpr bool MCC = (F & F_MCC) != 0;
    typedef Classes<R> CL;
    typedef SegGeom<R> SG;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t wtot[16];
    __shared__ int s_item;
    if (gated_off(a)) return;
    const uint32_t nseg = use_seg ? a.dflags->count[SEG_SLOT] : 0u;
    const uint32_t nblk = nseg + a.dflags->pad[ORDER_TOTAL];
    const int32_t *l4 = lists + (int64_t)4 * M;
    for (uint32_t item = blockIdx.x, nxt; item < nblk; item = nxt) {
        if (threadIdx.x == 0) s_item = (int)queue_take(a.dflags, 0, queue_of(blockIdx.x, gridDim.x), gridDim.x);
        lds_barrier();   // the previous cell's stores stay in flight
        nxt = (uint32_t)s_item;
        lds_barrier();
        if (item < nseg) {
            if constexpr (std::is_same<R, float>::value) lean_seg_pass<SG::T, SG::K, F>(a, l4, ss, item, smem, wtot);
            else seg_pass<R, SG::T, SG::K, F | F_CALL>(a, l4, ss, (int)item, smem, wtot);
            continue;
        }
        const int cell = order[item - nseg];
        const int n = a.cell_start[cell + 1] - a.cell_start[cell];
        if constexpr (std::is_same<R, float>::value && (F & ~F_MCC) == 0) {
            // one geometry for every block cell (a second one in the same
            // kernel pushes the largest past the register file)
            (void)n;
            lean_pass<1024, CL::K3, F>(a, cell, smem, wtot);
        } else {
            __shared__ double red[16 * 16];
            __shared__ double s_before[4];
            if (n <= 2048) cell_pass<R, 1024, 2, F | F_CALL>(a, cell, smem, red, wtot, s_before);
            else if (n <= 4096) cell_pass<R, 1024, 4, F | F_CALL>(a, cell, smem, red, wtot, s_before);
            else cell_pass<R, 1024, CL::K3, F | F_CALL>(a, cell, smem, red, wtot, s_before);
        }
    }
    if (wave_cls < 0) return;
    // wave phase: one cell per wave, no workgroup barriers from here on
    const uint32_t nw = a.dflags->count[wave_cls];
    const int32_t *wl = lists + (int64_t)wave_cls * M;
    unsigned char *slice = smem + (threadIdx.x / PIC_WAVE) * WAVE_SLICE;
    const uint32_t taker = blockIdx.x + gridDim.x * (threadIdx.x / PIC_WAVE);
    const uint32_t takers = gridDim.x * (blockDim.x / PIC_WAVE);
    for (uint32_t item = taker; item < nw;) {
        wave_pass<R, MCC>(a, wl[item], slice);
        if ((threadIdx.x & (PIC_WAVE - 1)) == 0) item = queue_take(a.dflags, 1, queue_of(taker, takers), takers);
        item = (uint32_t)__builtin_amdgcn_readfirstlane((int)item);
    }
}

template <typename R, int T, int K, int F>
int launch_class(const CollideArgs &a, const int32_t *list, int cls, int blocks, hipStream_t st)
{
    const size_t lds = lds_bytes<R, F>(T * K);
    auto kern = k_collide<R, T, K, F>;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_OK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
        attr_done = true;
    }
    ktime_begin(KT_CLASS0 + cls, st);
    hipLaunchKernelGGL(kern, dim3(persistent_grid(blocks)), dim3(T), lds, st, a, list, cls);
    ktime_end(KT_CLASS0 + cls, st);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

// The lean pass for binary32 steps; cell_pass for the pairing export, and for
// the correction without null collisions in the largest class: there the lean
// pass spills 15 registers, cell_pass 5 (12M electrons, four steps: cells of
// 4,200 1,093 and 1,009 us, of 8,000 883 and 833, of 10,000 882 and 852).  With
// null collisions cell_pass spills more and the lean pass is twice as fast.  Where
// the list holds at most one cell a workgroup (few), the lean pass's shorter way
// through a cell counts: 100 cells of 9,000 220 us against 241.
template <typename R, int T, int K, int F>
int launch_class_best(const CollideArgs &a, const int32_t *list, int cls, int blocks, hipStream_t st,
                      bool few = false)
{
    if constexpr (std::is_same<R, float>::value && !(F & F_PAIRS)) {
        if (F != F_CONS || T < 1024 || few) {
            const size_t lds = lean_lds_bytes<T, K, F>();
            auto kern = k_collide_lean<T, K, F>;
            static bool attr_done = false;
            if (!attr_done) {
                HIP_OK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds));
                attr_done = true;
            }
            ktime_begin(KT_CLASS0 + cls, st);
            hipLaunchKernelGGL(kern, dim3(persistent_grid(blocks)), dim3(T), lds, st, a, list, cls);
            ktime_end(KT_CLASS0 + cls, st);
            HIP_OK(hipGetLastError());
            return PIC_OK;
        }
    }
    if constexpr (!std::is_same<R, float>::value || (F & F_PAIRS) || (F == F_CONS && T >= 1024))
        return launch_class<R, T, K, F>(a, list, cls, blocks, st);
    else
        return PIC_ERR_ARG;   // not reached
}

template <bool MCC, int K = LEAN64_K>
int launch_lean64(const CollideArgs &a, const int32_t *list, int cls, int blocks, hipStream_t st)
{
    constexpr int T = LEAN64_T;
    const size_t lds = lean64_lds_bytes<T, K>();
    auto kern = k_collide_lean64<T, K, MCC>;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_OK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        attr_done = true;
    }
    ktime_begin(KT_CLASS0 + cls, st);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(T), lds, st, a, list, cls);
    ktime_end(KT_CLASS0 + cls, st);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

SegScratch g_seg;   // set from the workspace before each step's launches

template <typename R, int T, int K, int F>
constexpr size_t seg_lds_bytes()
{
    if constexpr (std::is_same<R, float>::value) return lean_lds_bytes<T, K, F>();
    else return lds_bytes<R>(T * K);
}

template <typename R, int T, int K, int F>
int launch_seg_collide(const CollideArgs &a, const int32_t *list, const SegScratch &ss, int blocks,
                       hipStream_t st)
{
    const size_t lds = seg_lds_bytes<R, T, K, F>();
    auto kern = k_seg_collide<R, T, K, F>;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_OK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
        attr_done = true;
    }
    hipLaunchKernelGGL(kern, dim3(persistent_grid(blocks)), dim3(T), lds, st, a, list, ss);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

template <typename R, int F>
int launch_all(const CollideArgs &a, const int32_t *lists, int32_t n_cells, int num_cu,
               const HugeScratch &hs, const ClassCaps &caps, bool seg_path, uint32_t live,
               hipStream_t st)
{
    typedef Classes<R> C;
    constexpr bool PAIRS = (F & F_PAIRS) != 0;
    constexpr bool SEG_OK = !PAIRS && !(F & (F_CONS | F_MOM | F_WT | F_NANBU | F_TRIP));
    constexpr int HUGE = PAIRS ? HUGE_PAIRS : SEG_OK ? HUGE_SEG : (F & F_NANBU) ? HUGE_NANBU : HUGE_ONE;
    int rc;
    const int64_t M = n_cells;
    const int *bp = caps.blocks_per_cu;
    const int32_t *l4 = lists + 4 * M;
    // A list's cells have more members than the class below takes, so the
    // n members fill at most n / (cap + 1) of them: no more workgroups than
    // that, and no launch for a list that cannot hold a cell.  The binary64 lean
    // passes take one workgroup per cell: with one for each cell of the grid
    // their empty launches cost 40 us each on 40,000 small cells.
    auto most = [&](int c) { return c == 0 ? M : std::min(M, a.n / ((int64_t)caps.cap[c - 1] + 1)); };
    auto grid = [&](int c) { return (int)std::min<int64_t>(bp[c] * num_cu, most(c)); };
    for (int c = 1; c <= 4; ++c)
        if (most(c) == 0) live &= ~(1u << c);
    // largest cells first so the small ones fill the tail
    bool seg_done = !(live & (1u << 4));   // no cell beyond the LDS classes
    if (!seg_done) ktime_begin(KT_HUGE, st);
    if constexpr (SEG_OK) {
      if (!seg_done && seg_path) {
        seg_done = true;
        const SegScratch &ss = g_seg;
        typedef SegGeom<R> G;
        hipLaunchKernelGGL(k_seg_count, dim3(num_cu * 2), dim3(SEG_CT), 0, st, a, l4, ss, (uint32_t)(G::T * G::K));
        hipLaunchKernelGGL(k_seg_scatter<R>, dim3(num_cu * 2), dim3(SEG_CT), 0, st, a, l4, ss);
        HIP_OK(hipGetLastError());
        if ((rc = launch_seg_collide<R, G::T, G::K, F>(a, l4, ss, G::PER_CU * num_cu, st))) return rc;
        // cells the plan could not segment
        hipLaunchKernelGGL((k_collide_huge<R, HUGE>), dim3(persistent_grid(grid(4))), dim3(1024), 0, st, a, l4, 4,
                           hs, g_seg, (const uint8_t *)ss.hc_fb);
      }
    }
    if (!seg_done)
        hipLaunchKernelGGL((k_collide_huge<R, HUGE>), dim3(persistent_grid(grid(4))), dim3(1024), 0, st, a, l4, 4,
                           hs, g_seg, (const uint8_t *)nullptr);
    if (live & (1u << 4)) ktime_end(KT_HUGE, st);
    HIP_OK(hipGetLastError());
    if (live & (1u << 3)) {
        // binary64 plain steps whose caps widen the largest class: the lean pass
        bool done = false;
        if constexpr (std::is_same<R, double>::value && (F & ~F_MCC) == 0) {
            if (caps.cap[3] > C::T3 * C::K3) {
                // one workgroup per listed cell (the kernel is not persistent)
                if ((rc = launch_lean64<(F & F_MCC) != 0>(a, lists + 3 * M, 3, (int)most(3), st)))
                    return rc;
                done = true;
            }
        }
        if (!done && (rc = launch_class_best<R, C::T3, C::K3, F>(a, lists + 3 * M, 3, grid(3), st, most(3) <= num_cu)))
            return rc;
    }
    if (live & (1u << 2)) {
        bool done = false;
        if constexpr (std::is_same<R, double>::value && (F & ~F_MCC) == 0) {
            if (caps.cap[3] > C::T3 * C::K3) {   // the binary64 plain step's lean passes
                if ((rc = launch_lean64<(F & F_MCC) != 0, C::K2>(a, lists + 2 * M, 2, (int)most(2), st)))
                    return rc;
                done = true;
            }
        }
        if (!done && (rc = launch_class_best<R, C::T2, C::K2, F>(a, lists + 2 * M, 2, grid(2), st)))
            return rc;
    }
    if ((live & (1u << 1)) && (rc = launch_class_best<R, C::T1, C::K1, F>(a, lists + 1 * M, 1, grid(1), st)))
        return rc;
    if ((live & (1u << 0)) && (rc = launch_class<R, C::T0, C::K0, F>(a, lists + 0 * M, 0, grid(0), st)))
        return rc;
    return PIC_OK;
}

// Dynamic LDS of the one-launch pass: the largest of its block passes and the
// waves' slices.
template <typename R, int F>
constexpr size_t all_lds_bytes()
{
    typedef Classes<R> CL;
    size_t b = 16 * WAVE_SLICE;
    const size_t seg = seg_lds_bytes<R, SegGeom<R>::T, SegGeom<R>::K, F>();
    b = seg > b ? seg : b;
    if constexpr (std::is_same<R, float>::value && (F & ~F_MCC) == 0) {
        const size_t l = lean_lds_bytes<1024, CL::K3, F>();
        b = l > b ? l : b;
    } else {
        const size_t l = lds_bytes<R>(1024 * CL::K3);
        b = l > b ? l : b;
    }
    return b;
}

// The step's collide pass as one persistent launch (see k_collide_all): the
// segment pre-passes of the cells beyond the LDS classes, the largest-first
// order of the block cells, the launch, then the pairs across segment edges
// and the cells no segment plan could take.
template <typename R, int F>
int launch_unified(const CollideArgs &a, const int32_t *lists, int32_t n_cells, int num_cu,
                   const HugeScratch &hs, const ClassCaps &caps, bool seg_path, hipStream_t st)
{
    const int32_t *l4 = lists + 4 * (int64_t)n_cells;
    const SegScratch &ss = g_seg;
    if (seg_path) {
        ktime_begin(KT_HUGE, st);
        typedef SegGeom<R> G;
        hipLaunchKernelGGL(k_seg_count, dim3(num_cu * 2), dim3(SEG_CT), 0, st, a, l4, ss, (uint32_t)(G::T * G::K));
        hipLaunchKernelGGL(k_seg_scatter<R>, dim3(num_cu * 2), dim3(SEG_CT), 0, st, a, l4, ss);
        ktime_end(KT_HUGE, st);
    }
    const int wave_cls = caps.wave ? 0 : -1;
    ktime_begin(KT_QUEUE, st);
    hipLaunchKernelGGL(k_order_queue, dim3(1), dim3(1024), 0, st, a.cell_start, lists, n_cells,
                       caps.wave ? 1 : 0, caps.ncls - 1, a.dflags, a.order);
    ktime_end(KT_QUEUE, st);
    constexpr size_t lds = all_lds_bytes<R, F>();
    auto kern = k_collide_all<R, F>;
    static bool attr_done = false;
    if (!attr_done) {
        HIP_OK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)lds));
        attr_done = true;
    }
    ktime_begin(KT_ALL, st);
    hipLaunchKernelGGL(kern, dim3(persistent_grid(num_cu)), dim3(1024), lds, st, a, lists, n_cells,
                       (const int32_t *)a.order, ss, caps, seg_path ? 1 : 0, wave_cls);
    ktime_end(KT_ALL, st);
    HIP_OK(hipGetLastError());
    ktime_begin(KT_HUGE, st);
    if (seg_path) {
        hipLaunchKernelGGL((k_collide_huge<R, HUGE_SEG>), dim3(persistent_grid(num_cu)), dim3(1024), 0, st, a, l4, 4, hs, g_seg,
                           (const uint8_t *)ss.hc_fb);
    } else {
        hipLaunchKernelGGL((k_collide_huge<R, HUGE_SEG>), dim3(persistent_grid(num_cu)), dim3(1024), 0, st, a, l4, 4, hs, g_seg,
                           (const uint8_t *)nullptr);
    }
    ktime_end(KT_HUGE, st);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

template <typename R>
int launch_deferred_t(const CollideArgs &a, const int32_t *lists, int32_t n_cells, int num_cu,
                      hipStream_t st)
{
    const int g = n_cells < num_cu * 8 ? n_cells : num_cu * 8;
    hipLaunchKernelGGL(k_deferred<R>, dim3(g), dim3(DEFER_T), 0, st, a,
                       lists + (int64_t)LIST_DEFERRED * n_cells);
    HIP_OK(hipGetLastError());
    return PIC_OK;
}

template <typename R>
int launch_flags(const CollideArgs &a, const int32_t *lists, int32_t n_cells, int num_cu,
                 const HugeScratch &hs, const ClassCaps &cc, int pairs_only, bool sp, uint32_t lv,
                 hipStream_t st)
{
    if (pairs_only) return launch_all<R, F_PAIRS>(a, lists, n_cells, num_cu, hs, cc, false, ~0u, st);
    if (a.variant == VAR_NANBU) return launch_all<R, F_NANBU>(a, lists, n_cells, num_cu, hs, cc, false, lv, st);
    if (a.variant == VAR_TRIPLET) return launch_all<R, F_TRIP>(a, lists, n_cells, num_cu, hs, cc, false, lv, st);
    if (a.w) {
        // variable weights: the plain step (optionally with null collisions),
        // cells beyond the LDS classes on one workgroup each
        if (a.mcc_thr) return launch_all<R, F_WT | F_MCC>(a, lists, n_cells, num_cu, hs, cc, false, lv, st);
        return launch_all<R, F_WT>(a, lists, n_cells, num_cu, hs, cc, false, lv, st);
    }
    const int f = (a.mcc_thr ? F_MCC : 0) | ((a.flags & PIC_CONSERVE_FIX) ? F_CONS : 0) |
                  ((a.flags & PIC_MOMENTS) ? F_MOM : 0);
    // the plain step (with or without null collisions) as one launch
    if (cc.unified && a.order && (f & ~F_MCC) == 0)
        return f ? launch_unified<R, F_MCC>(a, lists, n_cells, num_cu, hs, cc, sp, st)
                 : launch_unified<R, 0>(a, lists, n_cells, num_cu, hs, cc, sp, st);
    switch (f) {
    case 0: return launch_all<R, 0>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    case 1: return launch_all<R, 1>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    case 2: return launch_all<R, 2>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    case 3: return launch_all<R, 3>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    case 4: return launch_all<R, 4>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    case 5: return launch_all<R, 5>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    case 6: return launch_all<R, 6>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    default: return launch_all<R, 7>(a, lists, n_cells, num_cu, hs, cc, sp, lv, st);
    }
}

HugeScratch g_huge;   // set by launch_collide from the workspace

}  // namespace

const HugeScratch &huge_scratch() { return g_huge; }

namespace {


}  // namespace

ClassCaps collide_caps(int dtype, size_t)
{
    ClassCaps c;
    c.ncls = 4;
    // one launch per size class by default: measured faster than the single
    // persistent launch on the uniform and the log-normal workloads (the
    // autotuner tries both)
    c.unified = 0;
    c.wave = 1;
    c.blocks_per_cu[0] = 8;
    c.blocks_per_cu[1] = 4;
    c.blocks_per_cu[2] = 2;
    c.blocks_per_cu[3] = 1;
    c.blocks_per_cu[4] = 1;
    if (dtype == PIC_F32) {
        typedef Classes<float> C;
        c.cap[0] = C::T0 * C::K0;
        c.cap[1] = C::T1 * C::K1;
        c.cap[2] = C::T2 * C::K2;
        c.cap[3] = C::T3 * C::K3;
    } else {
        typedef Classes<double> C;
        // the wave schedule takes cells of up to 256 members in binary64
        c.cap[0] = PIC_WAVE * WaveGeom<double>::KW;
        c.cap[1] = C::T1 * C::K1;
        c.cap[2] = C::T2 * C::K2;
        c.cap[3] = C::T3 * C::K3;
    }
    return c;
}



int lean64_cap()
{
    return LEAN64_T * LEAN64_K;
}

size_t huge_scratch_bytes(int dtype, int64_t n)
{
    const size_t rec = dtype == PIC_F32 ? 16 : 32;
    return (size_t)n * (4 * 4 + 8 + 1) + ((size_t)n / 2 + 2) * rec + 7 * 256;   // 7 aligned parts
}

void set_huge_scratch(int dtype, int64_t n, void *base)
{
    unsigned char *p = (unsigned char *)base;
    auto take = [&](size_t bytes) {
        unsigned char *r = p;
        p += (bytes + 255) & ~(size_t)255;
        return (void *)r;
    };
    g_huge.keys = (uint32_t *)take((size_t)n * 4);
    g_huge.cnt = (uint32_t *)take((size_t)n * 4);
    g_huge.lst = (uint32_t *)take((size_t)n * 4);
    g_huge.pos = (uint32_t *)take((size_t)n * 4);
    g_huge.w23 = (uint32_t *)take((size_t)n * 8);
    g_huge.cand = (uint8_t *)take((size_t)n);
    g_huge.pbuf = take(((size_t)n / 2 + 2) * (dtype == PIC_F32 ? 16 : 32));
}

int launch_collide(int dtype, const CollideArgs &a, const int32_t *lists, int32_t n_cells,
                   const ClassCaps &cc, int pairs_only, int num_cu, hipStream_t st, bool seg_path,
                   uint32_t live)
{
    if (dtype == PIC_F32)
        return launch_flags<float>(a, lists, n_cells, num_cu, g_huge, cc, pairs_only, seg_path, live, st);
    return launch_flags<double>(a, lists, n_cells, num_cu, g_huge, cc, pairs_only, seg_path, live, st);
}

const SegScratch &seg_scratch() { return g_seg; }

int seg_cap(int dtype)
{
    return dtype == PIC_F32 ? SegGeom<float>::T * SegGeom<float>::K
                            : SegGeom<double>::T * SegGeom<double>::K;
}

int seg_target(int dtype)
{
    return seg_cap(dtype) * 7 / 8;
}

static int64_t seg_max_for(int dtype, int64_t n, int32_t n_cells)
{
    // S = ceil(n_c / target) <= n_c / target + 1 per cell
    return n / seg_target(dtype) + n_cells + 2;
}

static int64_t chunk_max_for(int64_t n, int32_t n_cells)
{
    return n / SEG_CHUNK + n_cells + 1;
}

size_t seg_scratch_bytes(int dtype, int64_t n, int32_t n_cells)
{
    const size_t S = (size_t)seg_max_for(dtype, n, n_cells), Q = (size_t)chunk_max_for(n, n_cells);
    return (size_t)n_cells * (4 + 1 + 4 + 4) + S * 6 * 4 + Q * 4 + 11 * 256;   // 11 aligned parts
}

void set_seg_scratch(int dtype, int64_t n, int32_t n_cells, void *base, int32_t *m_orig,
                     uint32_t *m_pid, void *m_v)
{
    unsigned char *p = (unsigned char *)base;
    auto take = [&](size_t bytes) {
        unsigned char *r = p;
        p += (bytes + 255) & ~(size_t)255;
        return (void *)r;
    };
    const int64_t S = seg_max_for(dtype, n, n_cells), Q = chunk_max_for(n, n_cells);
    g_seg.hc_S = (uint32_t *)take((size_t)n_cells * 4);
    g_seg.hc_fb = (uint8_t *)take((size_t)n_cells);
    g_seg.hc_seg = (int32_t *)take((size_t)n_cells * 4);
    g_seg.hc_chunk = (int32_t *)take((size_t)n_cells * 4);
    g_seg.sg_cell = (int32_t *)take((size_t)S * 4);
    g_seg.sg_cnt = (uint32_t *)take((size_t)S * 4);
    g_seg.sg_start = (uint32_t *)take((size_t)S * 4);
    g_seg.sg_cur = (uint32_t *)take((size_t)S * 4);
    g_seg.bnd_head = (int32_t *)take((size_t)S * 4);
    g_seg.bnd_tail = (int32_t *)take((size_t)S * 4);
    g_seg.ch_owner = (int32_t *)take((size_t)Q * 4);
    g_seg.m_orig = m_orig;
    g_seg.m_pid = m_pid;
    g_seg.m_v = m_v;
    g_seg.m_stride = n;
    g_seg.seg_max = S;
    g_seg.chunk_max = Q;
}

int launch_deferred(int dtype, const CollideArgs &a, const int32_t *lists, int32_t n_cells,
                    int num_cu, hipStream_t st)
{
    if (dtype == PIC_F32) return launch_deferred_t<float>(a, lists, n_cells, num_cu, st);
    return launch_deferred_t<double>(a, lists, n_cells, num_cu, st);
}
