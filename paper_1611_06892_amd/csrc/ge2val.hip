// The two steps after the band reduction (the GE2VAL pipeline of Sections 2
// and 6.2): BND2BD, band to bidiagonal by bulge chasing, and BD2VAL,
// singular values of the bidiagonal, on gfx950.
//
// BND2BD.  An n x n upper band of bandwidth nb.
// Sweep k clears row k beyond its superdiagonal and chases the bulge this
// makes down the band, one block of nb columns per step.  Step t of sweep k
// works at column c = k + 1 + t nb:
//   * a reflector from the right clears row rr (rr = k for t = 0, else
//     c - nb, the row the previous step filled) beyond column c; it is
//     applied to rows rr+1 .. c+nb-1 of columns c .. c+nb-1;
//   * a reflector from the left clears column c below the diagonal; it is
//     applied to rows c .. c+nb-1 of columns c+1 .. c+2nb-1.
// Only the first row or column of a bulge is cleared; the rest is cleared
// by later sweeps.  Step t of sweep k+1 works one row and one column further
// down than step t of sweep k, on entries that steps t and t+1 of sweep k
// write, so it may start once sweep k has finished step t+1: two steps
// separate consecutive sweeps, and about n / (2 nb) sweeps run at once.
//
// Where the band fits in the registers of the chip, it is held there and the
// sweeps pass through it (hold_kernel); else, and when the compute units are
// not free for that, the sweeps pass over the band array (chase_kernel):
//
// the band is copied into a band work array with room for the fill of the
// chase (nb - 1 diagonals below the main one, 2 nb - 1 above), column-major by
// diagonal offset:
//     W[(i - j + 2 nb - 1) + j * 3 nb]  holds entry (i, j).
// One persistent launch: each group of workgroups takes the next sweep
// (tickets from an atomic counter, so a sweep is only ever waited for by a
// later one that running workgroups hold: no deadlock for any grid) and runs
// its steps in order, each after the previous sweep's progress counters allow
// it.  The
// band array is written and read with agent-scope stores and loads (past the
// XCD's L2, at the coherence point), so a counter is published once every
// wave has waited for its own memory operations, with no L2 write-back, and the loads that follow a counter's load see every
// store performed before it was written, with no L2 invalidation; a
// wall-clock watchdog bounds every wait.
//
// BD2VAL.  The singular values of the bidiagonal (d, e) are the positive
// eigenvalues of the 2n x 2n Golub-Kahan matrix, symmetric tridiagonal with
// a zero diagonal and off-diagonal d1, e1, d2, ..., dn; its pivots in pairs
// are those of B^T B - x^2 I.  A Sturm count (their signs, by a recurrence
// without divisions) gives the number of singular values below x; a group of lanes narrows the interval
// of one singular value by multisection, so all n are found at once (the
// bisection method of the paper's list of BD2VAL methods, chosen over the
// serial bidiagonal QR for its parallelism).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdint>

#include "bidiag.h"

namespace bbg {

constexpr int NT = 512;                 // threads of the chase kernel (8 waves)
constexpr int NW = NT / 64;
constexpr int BT = 256;                 // threads of a bisection workgroup
constexpr int MS_LANES = 1 << 16;       // lanes of the bisection: one wave a SIMD
constexpr int MAX_NB = 256;
constexpr int GROUP_MAX = 16;
constexpr int SLICE = 4096;             // entries of a member's slice of one quadrant
enum : int { G_ERROR = 1, G_MET = 2, G_RUNNING = 3, G_HEAD = 32, G_WORDS = 64 };

// Quadrant width the kernel is compiled for (64, 128, 256), rows of a
// member's slice and workgroups (members) per sweep.
inline int width_of(int nb) { return nb <= 64 ? 64 : nb <= 128 ? 128 : 256; }
inline int slice_rows(int nb) { return SLICE / width_of(nb); }
inline int group_of(int nb) { return (nb + slice_rows(nb) - 1) / slice_rows(nb); }

// Exchange areas: sweeps in progress span at most MAX_WG / group + 2 of them
// (a sweep cannot finish before the one ahead of it, and every workgroup
// holds one ticket), so sweep k uses area k % nareas.
constexpr int MAX_WG = 256;
inline int nareas_of(int group) { return MAX_WG / group + 2; }
// doubles of one area: two steps' parity, each the members' partial column
// products and row 0
inline int64_t area_doubles(int nb, int group) { return 2 * (int64_t)(group + 1) * 2 * width_of(nb); }

struct ChaseArgs {
    double* W;
    int64_t ldw;          // 3 nb
    int64_t n;
    int nb;
    int nsweeps;
    int32_t* ctrl;        // G_* words
    int32_t* prog;        // steps finished, per sweep and member
    int32_t* bar;         // exchange arrivals, per sweep
    double* xch;          // exchange areas (group > 1)
    int group;            // workgroups per sweep
    int nareas;
    int64_t watchdog_ticks;
    const int32_t* met;   // the meeting of hold_kernel before this launch, or null
};

__host__ __device__ inline int64_t nsteps(int64_t n, int nb, int64_t k) {
    return (n - 1 - k + nb - 1) / nb;
}

// Stores to the band array: agent-scope stores, performed past the XCD's L2
// at the device's coherence point, so no L2 line of the band array is ever
// dirty and a publication needs no L2 write-back, only each wave's wait for
// its own stores (the same protocol as the band reduction's scheduler).
__device__ __forceinline__ void st(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Loads from the band array: agent-scope loads, served at the coherence
// point, so they see every store that completed before the progress counter
// they follow was written, with no L2 invalidation.
__device__ __forceinline__ double ld(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int aload(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

enum : int { MET_GO = 1, MET_GIVE_UP = 2 };     // the word G_MET

// A barrier for LDS traffic only: it waits for this wave's LDS operations,
// not for its global accesses, so stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// This wave's loads and stores have completed.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Sum over the four rows of 16 lanes (equal lane % 16), in every lane: four
// 4 x 4 x 4 matrix products with ones, whose k index is the row.
__device__ __forceinline__ double sum_rows(double v) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, v, 0.0, 0, 0, 0);
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum over the lanes l, l + R, l + 2R, ... (64 / R of them; R = 16, 8, 4), or
// over the wave (R = 1), in each of them.
template <int R>
__device__ __forceinline__ double sum_parts(double v) {
    if (R <= 8) v += dpp<0x128>(v);     // row_ror:8
    if (R <= 4) v += dpp<0x124>(v);     // row_ror:4
    if (R <= 2) v += dpp<0x122>(v);     // row_ror:2
    if (R <= 1) v += dpp<0x121>(v);     // row_ror:1
    return sum_rows(v);
}

// Sum of a lane and lane ^ 32.
__device__ __forceinline__ double sum_halves(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
           __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

// Householder reflector of (al, x) with ss = x^T x: beta = -sign(al) nrm,
// tau = (beta - al) / beta, scale = 1 / (al - beta) (v = (1, scale x)); a
// zero tail gives the identity.  1 / nrm and scale take one step of third
// order from the hardware approximations.
struct Refl {
    double beta, tau, scale;
};
__device__ __forceinline__ Refl reflector(double al, double ss) {
    if (ss == 0.0) return {al, 0.0, 0.0};
    const double t = fma(al, al, ss), ts = copysign(t, al), r0 = __builtin_amdgcn_rsq(t);
    const double s0 = ts * r0, y0 = __builtin_amdgcn_rcp(al + s0);
    const double e0 = fma(-fabs(s0), r0, 1.0);
    const double r = fma(r0 * e0, fma(e0, 0.375, 0.5), r0);
    const double s1 = ts * r;
    const double e1 = fma(-(al + s1), y0, 1.0);
    return {-fma(fma(-s1, s1, t), copysign(0.5 * r, al), s1), fma(fabs(al), r, 1.0), fma(y0, fma(e1, e1, e1), y0)};
}

// Called by a whole wave: polls *p (each lane's own) until all have reached
// target; false when an error was reported or the watchdog fired.
__device__ __forceinline__ bool poll(const ChaseArgs& a, const int32_t* p, int target) {
    const uint64_t t0 = wall_clock64();
    for (;;) {
        const int v = aload(p);
        if (__builtin_amdgcn_ballot_w64(v < target) == 0) return true;
        if (__builtin_amdgcn_readfirstlane(aload(&a.ctrl[G_ERROR])) != 0) return false;
        if ((int64_t)(wall_clock64() - t0) > a.watchdog_ticks) {
            if (threadIdx.x % 64 == 0)
                __hip_atomic_store(&a.ctrl[G_ERROR], BB_ETIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// The chase.  A group of a.group workgroups runs a sweep; member m holds, in
// LDS, rows s = m S .. m S + S - 1 of each block row of the sweep's window
// (S = 4096 / NBP, so a quadrant's slice is 4096 entries for any nb): three
// quadrants, by step t with block column c:
//     U  rows c - nb + s, columns c .. c + nb - 1   (t >= 1),
//     D  rows c + s,      columns c .. c + nb - 1,
//     Q  rows c + s,      columns c + nb .. c + 2 nb - 1.
// Q of step t is U of step t + 1, with the same owner, and no other sweep
// touches it between the two: the buffers rotate, a step loads D and Q and
// stores U and D.
//   * Right reflector (row rr, cleared): every member knows the row, from
//     the step before, and applies the reflector to its rows alone.
//   * Left reflector (column c): with x the column below its first entry,
//     v = (1, scale x), so v^T M = M(0, :) + scale (x^T M): one exchange of
//     the members' partial products x^T M (its first entry is x^T x) and of row 0 gives
//     every member the norm, the reflector, the products it applies to its
//     rows, and the new row 0 of Q -- the row the next step clears.
// So a step has one exchange between members (none for nb <= 64, a group of
// one) and one wait for the sweep ahead.  Members' sums are added in the
// order of the members, so all members compute the same values.
//
// What bounds it: the chain of steps.  A sweep follows the one ahead at a
// distance of two steps, so the chase is about 2 n steps one after the other
// plus, per step, the round trips to the coherence point: the poll of the
// sweep ahead, the loads, for groups the exchange (store, counter, poll,
// loads), and the publication, which is taken off the chain: a step's stores
// complete while the next step's wait is polled, and the last wave whose
// stores have completed publishes.
// Why this split: a right update needs whole rows and a left update whole
// columns, and slices by rows make the first local and leave the second one
// exchange of sums; shares of rows and of columns by turns, as before, moved
// every quadrant through memory between the two and met at two group
// barriers a step.  Measured, before and now: 2000 at nb = 64 70.7 and
// 24.7 ms (6.2 us a step), 8192 at nb = 256 477 and 232 ms (14.1 us), 16384
// at nb = 128 982 and 333 ms (10.2 us); 9000 at nb = 16 217 and 100 ms.
template <int NBP>
__global__ __launch_bounds__(NT) void chase_kernel(ChaseArgs a) {
    constexpr int S = SLICE / NBP;          // rows of a slice: 64, 32, 16
    constexpr int PR = NBP / 16, R = 64 / PR;   // right update: lanes per row, rows per wave
    constexpr int PL = S / 16, C = 64 / PL;     // left update: lanes per column, columns per wave
    constexpr int ST = S + PL;              // LDS column stride: columns and rows spread over the banks
    static_assert(NW * R == 2 * S && NW * C == 2 * NBP, "one pass");
    constexpr bool GROUPED = NBP > 64;
    __shared__ double quad[3][NBP * ST];
    __shared__ double vr[NBP], xr[NBP];     // the right reflector; the row it comes from
    __shared__ double srefl[2];             // its beta, tau
    __shared__ int sk, flag, stored;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = a.nb, G = GROUPED ? a.group : 1;
    const int64_t cs = a.ldw - 1;           // from entry (i, j) to (i, j + 1)
    // right update: row (U for waves 0-3, D for waves 4-7), columns rp + PR u
    const int rrow = (w % (NW / 2)) * R + lane % R, rp = lane / R;
    // left update: column (D for waves 0-3, Q for waves 4-7), rows lp + PL u
    const int lcol = (w % (NW / 2)) * C + lane % C, lp = lane / C;
    const bool low = w < NW / 2;
    if (tid == 0) stored = 0;
    if (a.met && aload(a.met) == MET_GO) return;

    for (;;) {
        // ticket = sweep * G + member: a group's members are consecutive
        // tickets, all taken by running workgroups before any of them can
        // be needed by a later sweep (grid >= G)
        if (tid == 0) sk = __hip_atomic_fetch_add(&a.ctrl[G_HEAD], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int ticket = __builtin_amdgcn_readfirstlane(sk);
        __syncthreads();
        const int64_t k = ticket / G;
        const int m = ticket - (int)k * G;
        if (k >= a.nsweeps) return;
        const int T = (int)nsteps(a.n, nb, k);
        const int Tp = k > 0 ? (int)nsteps(a.n, nb, k - 1) : 0;
        double* area = GROUPED ? a.xch + (k % a.nareas) * (2 * (int64_t)(G + 1) * 2 * NBP) : nullptr;
        int32_t* prog = a.prog + k * G;

        // The reflector that clears row (i, j .. j + len - 1) held in xr, by
        // this wave: vr and srefl; the owner of the row stores it cleared
        // (row k later, when every member has read it).
        auto right_reflector = [&](int64_t i, int64_t j, int len) {
            double x[NBP / 64], ss = 0.0;
#pragma unroll
            for (int h = 0; h < NBP / 64; ++h) {
                x[h] = xr[lane + 64 * h];
                if (lane + 64 * h > 0) ss = fma(x[h], x[h], ss);
            }
            const Refl f = reflector(xr[0], sum_parts<1>(ss));
#pragma unroll
            for (int h = 0; h < NBP / 64; ++h) {
                const int q = lane + 64 * h;
                vr[q] = q == 0 ? 1.0 : f.scale * x[h];
                if (i > k && m == 0 && q < len)
                    st(a.W + (i - j + 2 * nb - 1) + j * a.ldw + q * cs, q == 0 ? f.beta : 0.0);
            }
            if (lane == 0) {
                srefl[0] = f.beta;
                srefl[1] = f.tau;
            }
        };

        for (int t = 0; t < T; ++t) {
            const int64_t c = k + 1 + (int64_t)t * nb;
            const int L = (int)(a.n - c < nb ? a.n - c : nb);
            const int64_t nq = a.n - (c + nb);
            const int Lq = nq <= 0 ? 0 : (int)(nq < nb ? nq : nb);
            double* U = quad[(2 * t) % 3];          // Q of step t is U of step t + 1
            double* D = quad[(2 * t + 1) % 3];
            double* Q = quad[(2 * t + 2) % 3];
            double* w0 = a.W + (2 * nb - 1) + c * a.ldw;    // entry (c, c)

            // The sweep ahead has finished step t + 1 (and with it stored the
            // row its step t + 2 clears): this member's rows, one further down than
            // there, belong to members m and m + 1 of it (the last one to
            // member 0, in the next block); row k, which every member reads
            // at the first step, to member 0.
            const bool waits = k > 0 && w == 0;
            const int32_t* ahead = a.prog + (k - 1) * G + (lane == 0 ? m : lane == 1 ? (m + 1 < G ? m + 1 : 0)
                                                                                           : (t > 0 ? m : 0));
            const int target = t + 2 < Tp ? t + 2 : Tp;
            const int seen = waits ? aload(ahead) : 0;      // beside the stores still in flight
            // the previous step's stores: published by the wave whose stores
            // complete last
            if (t > 0) {
                wait_memory();
                if (lane == 0 && __hip_atomic_fetch_add(&stored, 1, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP) % NW == NW - 1)
                    __hip_atomic_store(&prog[m], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (waits) {
                const bool ok = __builtin_amdgcn_ballot_w64(seen < target) == 0 || poll(a, ahead, target);
                if (lane == 0) flag = ok;
            }
            lds_barrier();
            if (k > 0 && __builtin_amdgcn_readfirstlane(flag) == 0) return;
            {
                double xd[SLICE / NT], xq[SLICE / NT], xk = 0.0;
#pragma unroll
                for (int h = 0; h < SLICE / NT; ++h) {
                    const int e = tid + NT * h, i = e % S, q = e / S, s = m * S + i;
                    xd[h] = s < L && q < L ? ld(w0 + s + q * cs) : 0.0;
                    xq[h] = s < L && q < Lq ? ld(w0 + s + (q + nb) * cs) : 0.0;
                }
                if (t == 0 && tid < L) xk = ld(w0 - 1 + tid * cs);       // row k
#pragma unroll
                for (int h = 0; h < SLICE / NT; ++h) {
                    const int e = tid + NT * h, i = e % S, q = e / S;
                    D[i + q * ST] = xd[h];
                    Q[i + q * ST] = xq[h];
                }
                if (t == 0 && tid < NBP) xr[tid] = xk;
            }
            lds_barrier();
            if (t == 0) {
                if (w == NW - 1) right_reflector(k, c, L);
                lds_barrier();
            }

            // right update M -= tau (M v) v^T of rows rr + 1 .. c + L - 1
            if (!low || t > 0) {
                double* M = (low ? U : D) + rrow + rp * ST;
                const double tau = srefl[1];
                double x[16], v[16], p[2] = {0.0, 0.0};
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    x[u] = M[u * PR * ST];
                    v[u] = vr[rp + PR * u];
                }
#pragma unroll
                for (int u = 0; u < 16; ++u) p[u & 1] = fma(x[u], v[u], p[u & 1]);
                const double wt = tau * sum_parts<R>(p[0] + p[1]);
#pragma unroll
                for (int u = 0; u < 16; ++u) x[u] = fma(-wt, v[u], x[u]);
                if (low) {
                    // U is final; its row 0 is rr, stored cleared already
                    const int s = m * S + rrow;
                    if (s > 0 && s < nb) {
#pragma unroll
                        for (int u = 0; u < 16; ++u)
                            if (rp + PR * u < L) st(w0 - nb + s + (rp + PR * u) * cs, x[u]);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < 16; ++u) M[u * PR * ST] = x[u];
                }
            }
            lds_barrier();

            // left update M -= tau v (v^T M) of columns c + 1 .. c + nb + Lq - 1,
            // x_0 taken as zero; column c itself becomes (beta_l, 0, ..), but
            // stays as it is in LDS, where every wave reads x
            double beta_l;
            {
                double* M = (low ? D : Q) + lcol * ST + lp;
                const bool top = m == 0 && lp == 0;             // element 0 is row 0
                double x[16], y[16], p[2] = {0.0, 0.0};
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    y[u] = M[u * PL];
                    x[u] = D[lp + PL * u];
                }
                if (top) x[0] = 0.0;
#pragma unroll
                for (int u = 0; u < 16; ++u) p[u & 1] = fma(x[u], y[u], p[u & 1]);
                double dot = p[0] + p[1], ss, row0, al;
                if (PL == 4) dot = sum_rows(dot);
                if (PL == 2) dot = sum_halves(dot);
                if constexpr (!GROUPED) {
                    row0 = (low ? D : Q)[lcol * ST];
                    al = D[0];
                    const double xi = lane > 0 ? D[lane] : 0.0;
                    ss = sum_parts<1>(xi * xi);
                } else {
                    double* slot = area + (t & 1) * (int64_t)(G + 1) * 2 * NBP;
                    const int q = (low ? 0 : NBP) + lcol;
                    if (lp == 0) {
                        st(slot + m * 2 * NBP + q, dot);
                        if (m == 0) st(slot + G * 2 * NBP + q, y[0]);
                    }
                    wait_memory();
                    lds_barrier();
                    if (w == 0) {
                        if (lane == 0)
                            __hip_atomic_fetch_add(&a.bar[k], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const bool ok = poll(a, &a.bar[k], (t + 1) * G);
                        if (lane == 0) flag = ok;
                    }
                    lds_barrier();
                    if (__builtin_amdgcn_readfirstlane(flag) == 0) return;
                    double pd[GROUP_MAX], ps[GROUP_MAX];
#pragma unroll
                    for (int h = 0; h < GROUP_MAX; ++h) {
                        pd[h] = h < G ? ld(slot + h * 2 * NBP + q) : 0.0;
                        ps[h] = h < G ? ld(slot + h * 2 * NBP) : 0.0;
                    }
                    row0 = ld(slot + G * 2 * NBP + q);
                    al = ld(slot + G * 2 * NBP);
                    dot = ss = 0.0;
#pragma unroll
                    for (int h = 0; h < GROUP_MAX; ++h) {
                        dot += pd[h];
                        ss += ps[h];
                    }
                }
                const Refl f = reflector(al, ss);
                const double wt = f.tau * fma(f.scale, dot, row0);
                const double ws = wt * f.scale;
                beta_l = f.beta;
                // row k, which every member has read by now, is stored cleared
                if (low && t == 0 && m == 0 && tid < L) st(w0 - 1 + tid * cs, tid == 0 ? srefl[0] : 0.0);
                if (!low || lcol > 0) {
                    if (top) y[0] -= wt;
#pragma unroll
                    for (int u = 0; u < 16; ++u) M[u * PL] = fma(-ws, x[u], y[u]);  // (x_0 is zero)
                }
                if (!low && lp == 0) xr[lcol] = row0 - wt;      // the row the next step clears
            }
            lds_barrier();

            // D is final: whole columns of the slice; the last wave first
            // forms the next right reflector
            if (w == NW - 1 && Lq > 0) right_reflector(c, c + nb, Lq);
#pragma unroll
            for (int h = 0; h < SLICE / NT; ++h) {
                const int e = tid + NT * h, i = e % S, q = e / S, s = m * S + i;
                const double v = q > 0 ? D[i + q * ST] : s == 0 ? beta_l : 0.0;
                if (s < L && q < L) st(w0 + s + q * cs, v);
            }
        }
        // the whole sweep
        wait_memory();
        __syncthreads();
        if (tid == 0) {
            stored = 0;
            __hip_atomic_store(&prog[m], T, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---- the chase with the band held in registers -----------------------------
//
// When every block row of the window has workgroups of its own, nothing of
// the band has to move: block b keeps, through all sweeps, the nb rows below
// row c = k + 1 + b nb and in them the columns c .. c + nb - 1 (D) and
// c + nb .. c + 2 nb - 1 (Q), in registers, and sweeps pass through the
// blocks.  In sweep k block b
//   * receives from block b - 1 the row that the right reflector clears
//     (its columns are D's), forms the reflector and applies it to D;
//   * forms the left reflector of D's first column and applies it to D and Q;
//   * sends the new first row of Q to block b + 1, as the row to be cleared
//     there, and applies its reflector to its own other rows of Q;
//   * moves its window one row and one column on: its first row, finished for
//     this block, goes to block b - 1 as that one's new last row (from block
//     0 it is the row the next sweep clears), the last row comes from b + 1.
// Rows and columns are held in rings of nb: row or column c + i of sweep k,
// of D and of Q, is in slot (k + i) mod nb, so the window moves without moving
// anything but one column of Q, which becomes D's in the same lanes, and the
// messages, indexed by slot, need no rotation.  Rows and columns past the
// matrix are zeros and stay zeros; a zero column or row gives the identity.
//
// Lane l holds the columns of slots l + 64 h, wave w and register i row slot
// 8 i + w (+ 8 RW m for member m of a group, nb > 128).  Row sums go over the
// lanes of a wave; column sums over a wave's registers, then the waves (LDS)
// and, in a group, the members.
//
// A message is its values: an inbox word holds MARK, a NaN no arithmetic
// gives (and senders replace), until the value comes; the receiver polls the
// words it needs and sets them back.  Two inboxes by parity are enough: what
// a receiver reads in sweep k is set back before it leaves sweep k + 1, and
// no value of sweep k + 2 can be sent to it before that.
//
// What bounds it: the chain of 2 n steps, a message (about 1.3 us from the
// store to the polling load that sees it) and the step's own chain (reflector,
// row sums, column sums over the waves, reflector) each; the rest of a step's
// work falls into the time the block waits anyway, as a block works in every
// other step only.  A step takes 1.8 us (nb = 32), 2.1 (64), 2.9 (128) and 4.6
// (256, with the exchange between four members).  Against the chase by sweeps
// below: 2000 at nb = 64 24.7 -> 8.0 ms, 8192 at nb = 256 232 -> 76.5 ms, 16384
// at nb = 128 333 -> 96.4 ms, 9000 at nb = 16 99 -> 40 ms.
//
// All workgroups have to run at once, so they meet first; if they have not
// met within MEET_SECONDS (other work holds compute units) the launch ends
// without having done anything, and the chase by sweeps, which needs no more
// than one running group, does the work.
constexpr uint64_t MARK = 0x7FF4B1D1A60CA11Eull;
constexpr double MEET_SECONDS = 2e-3;

struct HoldArgs {
    const double* B;
    int64_t rs, cs, n;
    int nb;
    int group;            // workgroups per block
    int32_t* ctrl;
    double* box;          // inboxes, per workgroup
    double* d;
    double* e;
    int64_t watchdog_ticks, meet_ticks;
};

// An inbox: two rows to clear, two last rows (and a diagonal entry behind
// each), for groups two sets of the members' column sums and of row 0.
constexpr int box_row(int ch) { return 64 * ch; }
constexpr int box_last(int ch) { return 64 * ch + 8; }
constexpr int box_sums(int ch, int group) { return ch <= 2 ? 0 : (group + 1) * 128 * ch; }
constexpr int box_doubles(int ch, int group) { return 2 * (box_row(ch) + box_last(ch) + box_sums(ch, group)); }

__device__ __forceinline__ bool marked(double v) { return __builtin_bit_cast(uint64_t, v) == MARK; }
__device__ __forceinline__ void send(double* p, double v) {
    st(p, v != v ? __builtin_bit_cast(double, 0x7FF8000000000000ull) : v);
}
__device__ __forceinline__ void set_back(double* p) { st(p, __builtin_bit_cast(double, MARK)); }

// Called by a whole wave: v[h] = p[h * stride] where use, once none of them
// is MARK; false when an error was reported or the watchdog fired.
template <int N>
__device__ __forceinline__ bool await(const HoldArgs& a, const double* p, int stride, const bool (&use)[N],
                                      double (&v)[N]) {
    uint64_t t0 = 0;
    for (int tries = 0;; ++tries) {
        bool missing = false;
#pragma unroll
        for (int h = 0; h < N; ++h) {
            v[h] = use[h] ? ld(p + h * stride) : 0.0;
        }
#pragma unroll
        for (int h = 0; h < N; ++h) missing = missing || marked(v[h]);
        if (__builtin_amdgcn_ballot_w64(missing) == 0) return true;
        if (tries % 32 == 0) {
            const uint64_t now = wall_clock64();
            if (tries == 0) t0 = now;
            if (tries > 0 && __builtin_amdgcn_readfirstlane(aload(&a.ctrl[G_ERROR])) != 0) return false;
            if ((int64_t)(now - t0) >= a.watchdog_ticks) {
                if (threadIdx.x % 64 == 0)
                    __hip_atomic_store(&a.ctrl[G_ERROR], BB_ETIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return false;
            }
        }
    }
}

// One thread of each workgroup: whether all of them are running.
__device__ __forceinline__ bool meet(const HoldArgs& a) {
    const uint64_t t0 = wall_clock64();
    int none = 0;
    if (__hip_atomic_fetch_add(&a.ctrl[G_RUNNING], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
        (int)gridDim.x - 1)
        __hip_atomic_compare_exchange_strong(&a.ctrl[G_MET], &none, (int)MET_GO, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        const int met = aload(&a.ctrl[G_MET]);
        if (met != 0) return met == MET_GO;
        if ((int64_t)(wall_clock64() - t0) > a.meet_ticks) {
            none = 0;
            __hip_atomic_compare_exchange_strong(&a.ctrl[G_MET], &none, (int)MET_GIVE_UP, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_s_sleep(4);
    }
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Lanes < 32: a summed over l, l ^ 32, the others b (WIDE); by rows of 16
// lanes: even a, odd b, summed over l, l ^ 16.
template <bool WIDE>
__device__ __forceinline__ double fold(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    uint64_t p, q;
    if constexpr (WIDE) {
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
        p = (uint64_t)hi[0] << 32 | lo[0], q = (uint64_t)hi[1] << 32 | lo[1];
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
        p = (uint64_t)hi[0] << 32 | lo[0], q = (uint64_t)hi[1] << 32 | lo[1];
    }
    return __builtin_bit_cast(double, p) + __builtin_bit_cast(double, q);
}

// Sums over the wave of RW = 4, 8 or 16 values a lane, each made uniform:
// values are paired off while lanes are folded, so half as many are left at
// each of the first levels.
template <int RW>
__device__ __forceinline__ void wave_sums(double (&p)[RW]) {
    const int lane = threadIdx.x & 63;
    double q[RW / 4];
#pragma unroll
    for (int i = 0; i < RW / 4; ++i)
        q[i] = fold<false>(fold<true>(p[i], p[i + RW / 2]), fold<true>(p[i + RW / 4], p[i + 3 * RW / 4]));
    if constexpr (RW == 16) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const bool up = lane & 8;
            q[i] = (up ? q[i + 2] : q[i]) + dpp<0x128>(up ? q[i] : q[i + 2]);   // row_ror:8
        }
        const bool up = lane & 4;
        q[0] = (up ? q[1] : q[0]) + dpp<0x141>(up ? q[0] : q[1]);               // row_half_mirror
    } else if constexpr (RW == 8) {
        const bool up = lane & 8;
        q[0] = (up ? q[1] : q[0]) + dpp<0x128>(up ? q[0] : q[1]);
        q[0] += dpp<0x141>(q[0]);
    } else {
        q[0] += dpp<0x128>(q[0]);
        q[0] += dpp<0x141>(q[0]);
    }
    q[0] += dpp<0x4E>(q[0]);            // quad_perm:[2,3,0,1]
    q[0] += dpp<0xB1>(q[0]);            // quad_perm:[1,0,3,2]
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int half = i / (RW / 2), r = i % (RW / 2), row = r / (RW / 4), s = r % (RW / 4);
        const int lane_of = 32 * half + 16 * row + (RW == 16 ? 8 * (s / 2) + 4 * (s % 2) : RW == 8 ? 8 * s : 0);
        p[i] = lane_value(q[0], lane_of);
    }
}

template <int CH, int RW>
__global__ __launch_bounds__(NT) void hold_kernel(HoldArgs a) {
    constexpr int NBP = 64 * CH;
    constexpr int PARTS = NW * CH / 4;          // waves' sums a lane adds: 2, 4, 8
    constexpr bool GROUPED = CH == 4;
    __shared__ double part[NW][2 * NBP];        // column sums of each wave
    __shared__ double total[2 * NBP];           // of the block
    __shared__ double row0[2][2 * NBP];         // the first row, by parity of the sweep
    __shared__ int fail[2], go;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) {
        fail[0] = fail[1] = 0;
        go = meet(a) && aload(&a.ctrl[G_ERROR]) == 0;   // (an error reported before stops the chase)
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(go) == 0) return;
    const int nb = a.nb, G = GROUPED ? a.group : 1;
    const int b = (int)blockIdx.x / G, m = (int)blockIdx.x % G;
    const int size = box_doubles(CH, G);
    double* box = a.box + (int64_t)blockIdx.x * size;
    double* box_l = box + 2 * box_row(CH);
    double* box_x = box_l + 2 * box_last(CH);
    const int64_t K = a.n - 1 - (int64_t)b * nb, Kn = K - nb;   // sweeps of this block, of the next
    bool use[CH];
    double D[RW][CH], Q[RW][CH];
#pragma unroll
    for (int h = 0; h < CH; ++h) {
        use[h] = lane + 64 * h < nb;
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = 8 * (RW * m + i) + w, q = lane + 64 * h;
            const int64_t row = 1 + (int64_t)b * nb + r, col = 1 + (int64_t)b * nb + q;
            const bool in = r < nb && use[h] && row < a.n;
            D[i][h] = in && col >= row && col < a.n ? a.B[row * a.rs + col * a.cs] : 0.0;
            Q[i][h] = in && col <= row && col + nb < a.n ? a.B[row * a.rs + (col + nb) * a.cs] : 0.0;
        }
    }
    if (blockIdx.x == 0 && tid == 0) a.d[0] = a.B[0];

    int i0 = 0, ip = 0;                         // slots of the first row and column: of this sweep, of the last
    for (int64_t k = 0; k < K; ++k) {
        const int par = (int)(k & 1);
        bool ok = true;
        // the last row, which was the first one of the next block
        const bool takes = k > 0 && k <= Kn && w == ip % 8 && (!GROUPED || m == ip / (8 * RW));
        if (takes) {
            double x[CH], diag[1];
            const bool one[1] = {true};
            ok = await(a, box_l + (par ^ 1) * box_last(CH) + lane, 64, use, x);
            ok = ok && await(a, box_l + (par ^ 1) * box_last(CH) + NBP, 0, one, diag);
            const int reg = ip / 8 % RW;
#pragma unroll
            for (int i = 0; i < RW; ++i)
                if (i == reg) {
#pragma unroll
                    for (int h = 0; h < CH; ++h) {
                        D[i][h] = lane + 64 * h == ip ? diag[0] : 0.0;
                        Q[i][h] = x[h];
                        asm volatile("" : "+v"(D[i][h]), "+v"(Q[i][h]));
                    }
                }
        }
        // the row to clear, its reflector and D (I - tau v v^T)
        const int l0 = i0 % 64, h0 = i0 / 64;
        double v[CH];
        if (b > 0 || k > 0) {
            ok = await(a, box + par * box_row(CH) + lane, 64, use, v) && ok;
        } else {
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                const int64_t col = 1 + lane + 64 * h;
                v[h] = use[h] && col < a.n ? a.B[col * a.cs] : 0.0;
            }
        }
        auto first = [&](const double (&x)[CH]) {       // entry of slot i0, uniform
            double y = x[0];
#pragma unroll
            for (int h = 1; h < CH; ++h) {
                double z = x[h];
                asm("" : "+v"(z));              // a value, not an address to choose
                y = h == h0 ? z : y;
            }
            return lane_value(y, l0);
        };
        auto clear = [&](double (&x)[CH]) {             // row x becomes the reflector's v
            double ss = 0.0;
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                const double y = lane + 64 * h == i0 ? 0.0 : x[h];
                ss = fma(y, y, ss);
            }
            const Refl f = reflector(first(x), sum_parts<1>(ss));
#pragma unroll
            for (int h = 0; h < CH; ++h) x[h] = lane + 64 * h == i0 ? 1.0 : f.scale * x[h];
            return f;
        };
        auto from_right = [&](double (&M)[RW][CH], const double (&x)[CH], double tau) {
            double p[RW];
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                p[i] = M[i][0] * x[0];
#pragma unroll
                for (int h = 1; h < CH; ++h) p[i] = fma(M[i][h], x[h], p[i]);
            }
            wave_sums<RW>(p);
            double tx[CH];
#pragma unroll
            for (int h = 0; h < CH; ++h) tx[h] = -tau * x[h];
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int h = 0; h < CH; ++h) M[i][h] = fma(p[i], tx[h], M[i][h]);
        };
        const Refl fr = clear(v);
        from_right(D, v, fr.tau);
        if (b == 0 && m == 0 && tid == 0) a.e[k] = fr.beta;

        // the first row leaves the registers
        const bool gives = w == i0 % 8 && (!GROUPED || m == i0 / (8 * RW));
        if (gives) {
            const int reg = i0 / 8 % RW;
#pragma unroll
            for (int i = 0; i < RW; ++i)
                if (i == reg) {
#pragma unroll
                    for (int h = 0; h < CH; ++h) {
                        row0[par][lane + 64 * h] = D[i][h];
                        row0[par][NBP + lane + 64 * h] = Q[i][h];
                        D[i][h] = Q[i][h] = 0.0;
                        asm volatile("" : "+v"(D[i][h]), "+v"(Q[i][h]));
                    }
                }
        }
        // column sums x^T (D, Q), x the first column below the first row
        double x[RW];
        {
            double pd[CH], pq[CH];
#pragma unroll
            for (int i = 0; i < RW; ++i) x[i] = first(D[i]);
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                pd[h] = pq[h] = 0.0;
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    pd[h] = fma(x[i], D[i][h], pd[h]);
                    pq[h] = fma(x[i], Q[i][h], pq[h]);
                }
                part[w][lane + 64 * h] = pd[h];
                part[w][NBP + lane + 64 * h] = pq[h];
            }
        }
        if (!ok) fail[par] = 1;
        wait_memory();                          // inbox words set back in the last sweep
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(fail[par]) != 0) return;
        {
            const int col = w * 16 * CH + lane % (16 * CH), sub = lane / (16 * CH);
            double s = 0.0;
#pragma unroll
            for (int h = 0; h < PARTS; ++h) s += part[sub * PARTS + h][col];
            if constexpr (CH == 1) s = sum_rows(s);
            if constexpr (CH == 2) s = sum_halves(s);
            if constexpr (GROUPED) {
                // the members' sums and, from the one that has it, row 0
                const int64_t slot = par * (int64_t)box_sums(CH, G);
                const int holder = i0 / (8 * RW);
                const double r0 = row0[par][col];
                for (int o = 1; o < G; ++o) {
                    const int to = m + o < G ? m + o : m + o - G;
                    double* other = box_x + (int64_t)(to - m) * size + slot;
                    send(other + m * 2 * NBP + col, s);
                    if (m == holder) send(other + G * 2 * NBP + col, r0);
                }
                bool from[5];
                double y[5];
#pragma unroll
                for (int h = 0; h < 4; ++h) from[h] = h < G && h != m;
                from[4] = m != holder;
                // four members at most, row 0 behind them
                bool ok2 = true;
                {
                    const bool f4[4] = {from[0], from[1], from[2], from[3]};
                    double y4[4], y1[1];
                    const bool f1[1] = {from[4]};
                    ok2 = await(a, box_x + slot + col, 2 * NBP, f4, y4);
                    ok2 = await(a, box_x + slot + G * 2 * NBP + col, 0, f1, y1) && ok2;
#pragma unroll
                    for (int h = 0; h < 4; ++h) y[h] = h == m ? s : y4[h];
                    y[4] = y1[0];
                }
#pragma unroll
                for (int h = 0; h < 4; ++h)
                    if (from[h]) set_back(box_x + slot + h * 2 * NBP + col);
                if (from[4]) set_back(box_x + slot + G * 2 * NBP + col);
                s = ((y[0] + y[1]) + (y[2] + y[3]));
                if (from[4]) row0[par][col] = y[4];
                if (!ok2) fail[par] = 1;
            }
            if (sub == 0) total[col] = s;
        }
        lds_barrier();
        if (GROUPED && __builtin_amdgcn_readfirstlane(fail[par]) != 0) return;

        // left reflector; the new first row
        const Refl fl = reflector(row0[par][i0], total[i0]);
        double td[CH], tq[CH], g[CH], last[CH];
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const double rd = row0[par][lane + 64 * h], rq = row0[par][NBP + lane + 64 * h];
            td[h] = fl.tau * fma(fl.scale, total[lane + 64 * h], rd);
            tq[h] = fl.tau * fma(fl.scale, total[NBP + lane + 64 * h], rq);
            last[h] = rd - td[h];
            g[h] = rq - tq[h];
            td[h] *= -fl.scale;
            tq[h] *= -fl.scale;
        }
        if (w == 0 && k < Kn) {
            double* to = box + (int64_t)G * size + par * box_row(CH) + lane;
#pragma unroll
            for (int h = 0; h < CH; ++h)
                if (use[h]) send(to + 64 * h, g[h]);
        }
        const Refl fg = clear(g);
        if (w == 1) {
            if (b > 0) {
                if (!GROUPED || m == i0 / (8 * RW)) {
                    double* to = box_l - (int64_t)G * size + par * box_last(CH);
#pragma unroll
                    for (int h = 0; h < CH; ++h)
                        if (use[h]) send(to + lane + 64 * h, lane + 64 * h == i0 ? fg.beta : last[h]);
                    if (lane == 0) send(to + NBP, fl.beta);
                }
            } else {
                if (k + 1 < K) {
                    double* to = box + (par ^ 1) * box_row(CH) + lane;
#pragma unroll
                    for (int h = 0; h < CH; ++h)
                        if (use[h]) send(to + 64 * h, lane + 64 * h == i0 ? fg.beta : last[h]);
                }
                if (m == 0 && lane == 0) a.d[k + 1] = fl.beta;
            }
        }
        // words read in this sweep are set back
        if (w == NW - 1 && (b > 0 || k > 0)) {
#pragma unroll
            for (int h = 0; h < CH; ++h)
                if (use[h]) set_back(box + par * box_row(CH) + lane + 64 * h);
        }
        if (takes) {
#pragma unroll
            for (int h = 0; h < CH; ++h)
                if (use[h]) set_back(box_l + (par ^ 1) * box_last(CH) + lane + 64 * h);
            if (lane == 0) set_back(box_l + (par ^ 1) * box_last(CH) + NBP);
        }
        // the other rows: from the left, then Q from the right
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                D[i][h] = fma(x[i], td[h], D[i][h]);
                Q[i][h] = fma(x[i], tq[h], Q[i][h]);
            }
        from_right(Q, g, fg.tau);
        // Q's first column becomes D's last
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const bool moves = lane + 64 * h == i0;
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                D[i][h] = moves ? Q[i][h] : D[i][h];
                Q[i][h] = moves ? 0.0 : Q[i][h];
            }
        }
        ip = i0;
        i0 = i0 + 1 < nb ? i0 + 1 : 0;
    }
}

// Control words and inboxes before hold_kernel.
__global__ void hold_init_kernel(int32_t* ctrl, double* box, int64_t words, int keep_error) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < G_WORDS && !(keep_error && g == G_ERROR)) ctrl[g] = 0;
    for (int64_t i = g; i < words; i += (int64_t)gridDim.x * blockDim.x) box[i] = __builtin_bit_cast(double, MARK);
}

// Copy the upper band of B into W (zero elsewhere), clear the control words
// (the error word too unless keep_error: then a status already there, such as
// the band reduction's in the one-shot pipeline, stops the chase at its
// first wait and stays visible) and the progress counters.  Entry (i, j) of
// the band is B[i rs + j cs]: rs = 1, cs = ldb for an upper band stored as
// is, rs = ldb, cs = 1 for the transpose of a lower band.
__global__ void pack_kernel(const double* B, int64_t rs, int64_t cs, int64_t n, int nb, double* W, int64_t ldw,
                            int32_t* ctrl, int32_t* prog, int32_t* bar, int nsweeps, int group, int keep_error,
                            const int32_t* met) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (met && aload(met) == MET_GO) return;
    if (g < G_WORDS && g != G_MET && !(keep_error && g == G_ERROR)) ctrl[g] = 0;
    for (int64_t s = g; s < (int64_t)nsweeps * group; s += stride) prog[s] = 0;
    for (int64_t s = g; s < nsweeps; s += stride) bar[s] = 0;
    const int64_t total = ldw * n;
    for (int64_t x = g; x < total; x += stride) {
        const int64_t j = x / ldw;
        const int64_t i = j + (x - j * ldw) - (2 * nb - 1);
        W[x] = (i >= 0 && i <= j && j - i <= nb) ? B[i * rs + j * cs] : 0.0;
    }
}

__global__ void extract_kernel(const double* W, int64_t ldw, int64_t n, int nb, double* d, double* e,
                               const int32_t* met) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n || (met && aload(met) == MET_GO)) return;
    d[i] = W[(2 * nb - 1) + i * ldw];
    if (i + 1 < n) e[i] = W[(2 * nb - 2) + (i + 1) * ldw];
}

// Largest of v over the workgroup, in every thread; red holds a value a wave.
__device__ __forceinline__ double block_max(double v, double* red) {
#pragma unroll
    for (int o = 1; o < 64; o *= 2) v = fmax(v, __shfl_xor(v, o, 64));
    __syncthreads();
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int w = 1; w < BT / 64; ++w) v = fmax(v, red[w]);
    return v;
}

// One pivot of B^T B - x^2 I as the quotient of successive M: with
// t = N / M the pivot is d^2 + t and the next t is e^2 t / pivot - x^2, so
//     M' = d^2 M + N,   N' = e^2 N - x^2 M'
// with no division; the pivot's sign is the change of M's.
__device__ __forceinline__ void sturm_step(double2 de, double x2, double& M, double& N, uint32_t& signs) {
    const double Mn = fma(de.x, M, N);
    N = fma(-x2, Mn, de.y * N);
    M = Mn;
    signs = __builtin_amdgcn_alignbit(signs, (uint32_t)(__builtin_bit_cast(uint64_t, Mn) >> 32), 31);
}

// M and N by the power of two that brings the larger to [1, 2).
__device__ __forceinline__ void sturm_scale(double& M, double& N) {
    const uint32_t hm = (uint32_t)(__builtin_bit_cast(uint64_t, M) >> 32) & 0x7FFFFFFFu;
    const uint32_t hn = (uint32_t)(__builtin_bit_cast(uint64_t, N) >> 32) & 0x7FFFFFFFu;
    const uint32_t h = (hm > hn ? hm : hn) & 0x7FF00000u;
    const double f = __builtin_bit_cast(double, (uint64_t)((2046u << 20) - h) << 32);
    M *= f;
    N *= f;
}

// MS lanes per singular value (multisection): each round, lane l counts
// below x_l = lo + (l+1)(hi-lo)/(MS+1), and the interval shrinks to the
// one between the largest x with at most s values below it and the
// smallest x with more, a factor MS+1 a round (13 rounds to full precision
// at MS = 16, against 53 for bisection), with MS times the lanes.
//
// The entries are scaled by a power of two to at most one and squared once
// per staging, in LDS, where every lane reads the same pair; squares below
// 2^-124 are raised to it (entries by 2^-62 of the largest at most, a
// thousandth of the bisection's own 2^-52), so the map of (M, N) a step makes
// (determinant d^2 e^2) takes neither both to zero nor, in the four steps
// between scalings, to underflow.  Every rounding is a relative change of one
// d^2, e^2 or x^2, as in the recurrence with divisions.
//
// What bounds it: a round is a chain of n steps of two dependent FMAs, and
// the lanes of all values fill the chip at one wave a SIMD; a step issues
// about 28 cycles (three FP64 operations, the sign, a quarter of a scaling;
// measured 39 at n = 16384, with the staging).  Against two divisions a pair
// of pivots on twice the lanes: n = 2000 5.6 -> 0.43 ms, 8192 29.5 -> 2.4 ms,
// 16384 75.9 -> 6.1 ms, 33000 255 -> 28 ms.
constexpr int STAGE = 4096;             // pairs staged at a time (64 KiB, two workgroups a CU)

template <int MS>
__global__ __launch_bounds__(BT) void bisect_kernel(const double* d, const double* e, int64_t n, double* sigma) {
    static_assert(64 % MS == 0, "a value's lanes lie in one wave");
    __shared__ double2 pair[STAGE];
    __shared__ double red[BT / 64];
    const int64_t gt = (int64_t)blockIdx.x * BT + threadIdx.x;
    const int64_t j = gt / MS;
    const int lane = (int)(gt % MS);
    // largest entry and half the Gershgorin bound of the Golub-Kahan matrix
    double amax = 0.0, half = 0.0, bad = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += BT) {
        const double di = fabs(d[i]);
        const double ei = i + 1 < n ? fabs(e[i]) : 0.0, ep = i > 0 ? fabs(e[i - 1]) : 0.0;
        if (di != di || ei != ei) bad = 1.0;
        half = fmax(half, 0.5 * di + 0.5 * fmax(ei, ep));
        amax = fmax(amax, fmax(di, ei));
    }
    amax = block_max(amax, red);
    half = block_max(half, red);
    bad = block_max(bad, red);
    if (bad != 0.0 || amax == 0.0 || amax > DBL_MAX) {      // NaN, zero or infinity throughout
        if (lane == 0 && j < n) sigma[j] = bad != 0.0 ? __builtin_nan("") : amax;
        return;
    }
    int ex;
    (void)frexp(amax, &ex);             // entries times 2^-ex are at most one
    const double bound = ldexp(half, 1 - ex);
    const double abstol = DBL_EPSILON * bound;
    double lo = 0.0, hi = bound * (1.0 + 4.0 * DBL_EPSILON);
    const int64_t s = n - 1 - j;        // sigma[j] is the s-th smallest (decreasing order)
    bool active = j < n;
    for (int it = 0; it < 128; ++it) {
        active = active && hi - lo > fmax(abstol, 2.0 * DBL_EPSILON * hi);
        if (!__syncthreads_or(active)) break;
        const double x = lo + (hi - lo) * (double)(lane + 1) / (double)(MS + 1);
        const double x2 = x * x;
        const bool any = __builtin_amdgcn_ballot_w64(active) != 0;
        double M = 1.0, N = -x2;
        uint32_t signs = 0;             // the latest signs of M, the newest lowest
        int cnt = 0;
        for (int64_t c = 0; c < n; c += STAGE) {
            const int len = (int)(n - c < STAGE ? n - c : STAGE);
            if (it == 0 || n > STAGE) {
                __syncthreads();
                for (int i = threadIdx.x; i < len; i += BT) {
                    const double di = ldexp(d[c + i], -ex), ei = c + i + 1 < n ? ldexp(e[c + i], -ex) : 0.0;
                    pair[i] = {fmax(di * di, 0x1p-124), fmax(ei * ei, 0x1p-124)};
                }
                __syncthreads();
            }
            if (!any) continue;
            int i = 0;
            for (; i + 16 <= len; i += 16) {
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    sturm_step(pair[i + u], x2, M, N, signs);
                    if (u % 4 == 3) sturm_scale(M, N);
                }
                cnt += __builtin_popcount((signs ^ signs >> 1) & 0xFFFFu);
            }
            for (; i < len; ++i) {
                sturm_step(pair[i], x2, M, N, signs);
                sturm_scale(M, N);
                cnt += (signs ^ signs >> 1) & 1u;
            }
        }
        const bool inside = x > lo && x < hi;
        const bool below = inside && cnt <= s;                  // x <= sigma_j
        double nlo = below ? x : lo;
        double nhi = inside && !below ? x : hi;
#pragma unroll
        for (int o = 1; o < MS; o *= 2) {
            nlo = fmax(nlo, __shfl_xor(nlo, o, 64));
            nhi = fmin(nhi, __shfl_xor(nhi, o, 64));
        }
        if (nlo >= nhi || (nlo == lo && nhi == hi)) active = false;     // counts out of order, or no progress
        if (active) {
            lo = nlo;
            hi = nhi;
        }
    }
    if (lane == 0 && j < n) sigma[j] = ldexp(0.5 * (lo + hi), ex);
}

// workspace: control words (256 B), the band array (3 nb n doubles), the
// members' progress counters and the exchange counters (int32 per sweep and
// member, and per sweep), the exchange areas
inline int64_t round256(int64_t b) { return (b + 255) / 256 * 256; }

inline int nsweeps_of(int64_t n, int nb) { return nb <= 1 || n <= 2 ? 0 : (int)(n - 2); }

inline int64_t ws_prog_off(int64_t n, int nb) { return round256(256 + (int64_t)3 * nb * n * 8); }
inline int64_t ws_bar_off(int64_t n, int nb) {
    return ws_prog_off(n, nb) + round256((int64_t)nsweeps_of(n, nb) * group_of(nb) * 4);
}
inline int64_t ws_xch_off(int64_t n, int nb) {
    return ws_bar_off(n, nb) + round256((int64_t)nsweeps_of(n, nb) * 4);
}

inline int64_t ws_sweep_bytes(int64_t n, int nb) {
    const int g = group_of(nb);
    const int64_t xch = g > 1 && nsweeps_of(n, nb) > 0 ? 8 * nareas_of(g) * area_doubles(nb, g) : 0;
    return round256(ws_xch_off(n, nb) + xch);
}

// Workgroups of a block and all inboxes of hold_kernel; none (0) where the
// blocks do not fit on the chip at once, or nothing is chased.  Workgroups a
// compute unit: what the registers of the instance allow (72, 88, 200, 224 of
// 512 a lane and SIMD, two waves a workgroup and SIMD).
inline int hold_ch(int nb) { return width_of(nb) / 64; }
inline int hold_group(int nb) { return nb <= 128 ? 1 : (nb + 63) / 64; }
inline int hold_per_cu(int nb) { return nb <= 32 ? 3 : nb <= 64 ? 2 : 1; }
inline int64_t hold_workgroups(int64_t n, int nb) {
    const int64_t wg = (n - 1 + nb - 1) / nb * hold_group(nb);
    return nsweeps_of(n, nb) > 0 && wg <= MAX_WG * hold_per_cu(nb) ? wg : 0;
}
inline int64_t hold_words(int64_t n, int nb) {
    return hold_workgroups(n, nb) * box_doubles(hold_ch(nb), hold_group(nb));
}

inline size_t ws_bytes(int64_t n, int nb) {
    return (size_t)(ws_sweep_bytes(n, nb) + 8 * hold_words(n, nb));
}

int device_attr(hipDeviceAttribute_t attr, int fallback) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, attr, dev) != hipSuccess) return fallback;
    return v;
}

}  // namespace bbg

extern "C" {

int bb_bnd2bd_workspace(int64_t n, int nb, size_t* ws_bytes) {
    if (n < 0) return -1;
    if (nb < 1 || nb > bbg::MAX_NB) return -2;
    if (!ws_bytes) return -3;
    *ws_bytes = bbg::ws_bytes(n, nb);
    return BB_OK;
}

}  // extern "C"

namespace bbg {

// The chase after argument checks: band entry (i, j) at B[i rs + j cs].
int bnd2bd_launch(const double* B, int64_t rs, int64_t cs, int64_t n, int nb, double* d, double* e, void* ws,
                  double watchdog_s, bool keep_error, void* stream);

}  // namespace bbg

extern "C" {

int bb_bnd2bd_group(const double* B, int64_t ldb, int64_t n, int nb, double* d, double* e, void* ws,
                    size_t ws_bytes, double watchdog_s, int group, void* stream) {
    if (group < 0 || group > bbg::GROUP_MAX) return -10;
    if (n < 0) return -3;
    if (!B && n > 0) return -1;
    if (ldb < (n > 1 ? n : 1)) return -2;
    if (nb < 1 || nb > bbg::MAX_NB) return -4;
    if (!d && n > 0) return -5;
    if (!e && n > 1) return -6;
    if (!ws && n > 0) return -7;
    if (ws_bytes < bbg::ws_bytes(n, nb)) return BB_EWORKSPACE;
    if (n == 0) return BB_OK;
    return bbg::bnd2bd_launch(B, 1, ldb, n, nb, d, e, ws, watchdog_s, false, stream);
}

}  // extern "C"

int bbg::bnd2bd_launch(const double* B, int64_t rs, int64_t cs, int64_t n, int nb, double* d, double* e,
                       void* ws, double watchdog_s, bool keep_error, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    const int nsw = bbg::nsweeps_of(n, nb);
    bbg::ChaseArgs a;
    a.W = (double*)((char*)ws + 256);
    a.ldw = 3 * (int64_t)nb;
    a.n = n;
    a.nb = nb;
    a.nsweeps = nsw;
    a.ctrl = (int32_t*)ws;
    a.prog = (int32_t*)((char*)ws + bbg::ws_prog_off(n, nb));
    a.bar = (int32_t*)((char*)ws + bbg::ws_bar_off(n, nb));
    a.xch = (double*)((char*)ws + bbg::ws_xch_off(n, nb));
    a.group = bbg::group_of(nb);
    a.nareas = bbg::nareas_of(a.group);
    const double khz = (double)bbg::device_attr(hipDeviceAttributeWallClockRate, 100000);
    a.watchdog_ticks = (int64_t)((watchdog_s > 0 ? watchdog_s : 30.0) * khz * 1000.0);
    const int cus = bbg::device_attr(hipDeviceAttributeMultiprocessorCount, 256);
    const int64_t wgs = bbg::hold_workgroups(n, nb);
    a.met = nullptr;
    if (wgs > 0 && wgs <= (int64_t)cus * bbg::hold_per_cu(nb)) {
        bbg::HoldArgs h;
        h.B = B;
        h.rs = rs;
        h.cs = cs;
        h.n = n;
        h.nb = nb;
        h.group = bbg::hold_group(nb);
        h.ctrl = a.ctrl;
        h.box = (double*)((char*)ws + bbg::ws_sweep_bytes(n, nb));
        h.d = d;
        h.e = e;
        h.watchdog_ticks = a.watchdog_ticks;
        h.meet_ticks = (int64_t)(bbg::MEET_SECONDS * khz * 1000.0);
        const int64_t words = bbg::hold_words(n, nb);
        hipLaunchKernelGGL(bbg::hold_init_kernel, dim3((unsigned)std::min<int64_t>((words + 255) / 256, cus)),
                           dim3(256), 0, s, a.ctrl, h.box, words, keep_error ? 1 : 0);
        if (hipGetLastError() != hipSuccess) return BB_EHIP;
        const dim3 grid((unsigned)wgs), block(bbg::NT);
        if (nb <= 32)
            hipLaunchKernelGGL((bbg::hold_kernel<1, 4>), grid, block, 0, s, h);
        else if (nb <= 64)
            hipLaunchKernelGGL((bbg::hold_kernel<1, 8>), grid, block, 0, s, h);
        else if (nb <= 128)
            hipLaunchKernelGGL((bbg::hold_kernel<2, 16>), grid, block, 0, s, h);
        else
            hipLaunchKernelGGL((bbg::hold_kernel<4, 8>), grid, block, 0, s, h);
        if (hipGetLastError() != hipSuccess) return BB_EHIP;
        a.met = &a.ctrl[bbg::G_MET];
        keep_error = true;
    }
    // the chase by sweeps; after a launch above that held the band, these end at once
    const int64_t total = a.ldw * n;
    int blocks = (int)std::min<int64_t>((total + 255) / 256, 8 * (int64_t)cus);
    hipLaunchKernelGGL(bbg::pack_kernel, dim3(blocks < 1 ? 1 : blocks), dim3(256), 0, s, B, rs, cs, n, nb, a.W,
                       a.ldw, a.ctrl, a.prog, a.bar, nsw, a.group, keep_error ? 1 : 0, a.met);
    if (hipGetLastError() != hipSuccess) return BB_EHIP;
    if (nsw > 0) {
        // whole groups, at least one, one workgroup a CU (MAX_WG at most: the
        // exchange areas are counted for that)
        const int wg = std::min(cus, bbg::MAX_WG);
        if (wg < a.group) return BB_ENOTSUP;
        const dim3 grid((unsigned)std::min<int64_t>((int64_t)nsw * a.group, wg / a.group * a.group));
        switch (bbg::width_of(nb)) {
            case 64: hipLaunchKernelGGL(bbg::chase_kernel<64>, grid, dim3(bbg::NT), 0, s, a); break;
            case 128: hipLaunchKernelGGL(bbg::chase_kernel<128>, grid, dim3(bbg::NT), 0, s, a); break;
            default: hipLaunchKernelGGL(bbg::chase_kernel<256>, grid, dim3(bbg::NT), 0, s, a); break;
        }
        if (hipGetLastError() != hipSuccess) return BB_EHIP;
    }
    hipLaunchKernelGGL(bbg::extract_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a.W, a.ldw, n,
                       nb, d, e, a.met);
    return hipGetLastError() == hipSuccess ? BB_OK : BB_EHIP;
}

extern "C" {

int bb_bnd2bd(const double* B, int64_t ldb, int64_t n, int nb, double* d, double* e, void* ws,
              size_t ws_bytes, double watchdog_s, void* stream) {
    return bb_bnd2bd_group(B, ldb, n, nb, d, e, ws, ws_bytes, watchdog_s, 0, stream);
}

int bb_bd2val(const double* d, const double* e, int64_t n, double* sigma, void* stream) {
    if (n < 0) return -3;
    if (!d && n > 0) return -1;
    if (!e && n > 1) return -2;
    if (!sigma && n > 0) return -4;
    if (n == 0) return BB_OK;
    // as many lanes a value as leave one wave a SIMD (rounds go with
    // 1 / log2(ms + 1), a second wave on a SIMD doubles their time: n = 9000
    // takes 3.4 ms at 4, where half the SIMDs idle, 16385 8.6 ms at 2)
    int ms = 1;
    while (ms < 64 && n * 2 * ms <= bbg::MS_LANES) ms *= 2;
    const dim3 grid((unsigned)((n * ms + bbg::BT - 1) / bbg::BT)), block(bbg::BT);
    hipStream_t s = (hipStream_t)stream;
    switch (ms) {
        case 1: hipLaunchKernelGGL(bbg::bisect_kernel<1>, grid, block, 0, s, d, e, n, sigma); break;
        case 2: hipLaunchKernelGGL(bbg::bisect_kernel<2>, grid, block, 0, s, d, e, n, sigma); break;
        case 4: hipLaunchKernelGGL(bbg::bisect_kernel<4>, grid, block, 0, s, d, e, n, sigma); break;
        case 8: hipLaunchKernelGGL(bbg::bisect_kernel<8>, grid, block, 0, s, d, e, n, sigma); break;
        case 16: hipLaunchKernelGGL(bbg::bisect_kernel<16>, grid, block, 0, s, d, e, n, sigma); break;
        case 32: hipLaunchKernelGGL(bbg::bisect_kernel<32>, grid, block, 0, s, d, e, n, sigma); break;
        default: hipLaunchKernelGGL(bbg::bisect_kernel<64>, grid, block, 0, s, d, e, n, sigma); break;
    }
    return hipGetLastError() == hipSuccess ? BB_OK : BB_EHIP;
}

// bb_ge2val's workspace: the band reduction's, and after it (stream order)
// the chase's with the bidiagonal (d, e) behind it.
static int ge2val_sizes(int64_t m, int64_t n, int nb, int tree, int variant, int prec, const bb_opts* opts,
                        size_t* vt_bytes, size_t* ws_bytes, size_t* de_off) {
    size_t vt = 0, wsb = 0;
    const int rc = bb_query(m, n, nb, tree, variant, prec, opts, &vt, &wsb);
    if (rc != BB_OK) return rc;
    const int64_t k = m < n ? m : n;
    const size_t chase = bbg::ws_bytes(k, nb);
    const size_t off = (chase + 255) / 256 * 256;
    const size_t need = off + (size_t)(2 * (k > 0 ? k : 1)) * sizeof(double);
    if (vt_bytes) *vt_bytes = vt;
    if (ws_bytes) *ws_bytes = wsb > need ? wsb : need;
    if (de_off) *de_off = off;
    return BB_OK;
}

int bb_ge2val_workspace(int64_t m, int64_t n, int nb, int tree, int variant, int prec, const bb_opts* opts,
                        size_t* vt_bytes, size_t* ws_bytes) {
    if (!vt_bytes || !ws_bytes) return -8;
    return ge2val_sizes(m, n, nb, tree, variant, prec, opts, vt_bytes, ws_bytes, nullptr);
}

int bb_ge2val(void* A, int64_t m, int64_t n, int64_t lda, int nb, int tree, int variant, int prec, double* sigma,
              void* vt, size_t vt_bytes, void* ws, size_t ws_bytes, const bb_opts* opts, void* stream) {
    size_t need_vt = 0, need_ws = 0, de_off = 0;
    int rc = ge2val_sizes(m, n, nb, tree, variant, prec, opts, &need_vt, &need_ws, &de_off);
    if (rc != BB_OK) return rc;
    const int64_t k = m < n ? m : n;
    if (!sigma && k > 0) return -9;
    if (vt_bytes < need_vt || ws_bytes < need_ws) return BB_EWORKSPACE;
    rc = bidiag_band(A, m, n, lda, nb, tree, variant, prec, vt, vt_bytes, ws, ws_bytes, opts, stream);
    if (rc != BB_OK || k == 0) return rc;
    double* d = (double*)((char*)ws + de_off);
    double* e = d + k;
    // m >= n: upper band in the leading n x n part; m < n: lower band in the
    // leading m x m part, chased as its transpose
    const double* B = (const double*)A;
    rc = m >= n ? bbg::bnd2bd_launch(B, 1, lda, k, nb, d, e, ws, opts ? opts->watchdog_s : 0.0, true, stream)
                : bbg::bnd2bd_launch(B, lda, 1, k, nb, d, e, ws, opts ? opts->watchdog_s : 0.0, true, stream);
    if (rc != BB_OK) return rc;
    return bb_bd2val(d, e, k, sigma, stream);
}

}  // extern "C"
