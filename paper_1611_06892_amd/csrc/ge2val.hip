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
// Blocks: block b of sweep k is the nb rows from c = k + 1 + b nb on, with the
// columns c .. c + 2 nb - 1.  One block of one sweep (block_step) is the unit
// of work, and there are two ways to bring the blocks to it:
//   * where all blocks' workgroups find room on the chip at once, they hold
//     the blocks in registers and the sweeps pass through them (hold_blocks);
//   * else, for larger matrices or beside work that holds compute units, each
//     sweep is run by workgroups of its own over the band in memory
//     (run_sweeps), any number of them.
// Both run the same block_step on the same values in the same lanes, so the
// result does not depend on the way, bit by bit.  Multiply-adds are written
// out and contraction is off, so that the compiler cannot round the two
// copies of the step differently.
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

#pragma clang fp contract(off)

namespace bbg {

constexpr int NT = 512;                 // threads of the chase kernels (8 waves)
constexpr int NW = NT / 64;
constexpr int BT = 256;                 // threads of a bisection workgroup
constexpr int MS_LANES = 1 << 16;       // lanes of the bisection: one wave a SIMD
constexpr int MAX_NB = 256;
constexpr int GROUP_MAX = 16;           // of bb_bnd2bd_group's argument
constexpr int MAX_WG = 256;             // compute units
enum : int { G_ERROR = 1, G_MET = 2, G_RUNNING = 3, G_HEAD = 32, G_WORDS = 64 };

// What a wait needs: the control words and the watchdog.
struct Waits {
    int32_t* ctrl;
    int64_t watchdog_ticks;
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
// zero tail gives the identity, tau = 0.  Its sums are taken as zeros, so that
// infinities and NaN elsewhere stay where they are (0.6 % of a chase at nb = 128,
// 1.2 % at 256).  1 / nrm and scale take one step of third
// order from the hardware approximations.
struct Refl {
    double beta, tau, scale;
};
__device__ __forceinline__ Refl reflector(double al, double ss) {
    if (ss == 0.0) return {al, 0.0, 0.0};
    const double t = fma(al, al, ss), ts = copysign(t, al), r0 = __builtin_amdgcn_rsq(t);
    const double s0 = ts * r0, y0 = __builtin_amdgcn_rcp(fma(ts, r0, al));
    const double e0 = fma(-fabs(s0), r0, 1.0);
    const double r = fma(r0 * e0, fma(e0, 0.375, 0.5), r0);
    const double s1 = ts * r;
    const double e1 = fma(-fma(ts, r, al), y0, 1.0);
    return {-fma(fma(-s1, s1, t), copysign(0.5 * r, al), s1), fma(fabs(al), r, 1.0), fma(y0, fma(e1, e1, e1), y0)};
}

// Called by a whole wave: polls *p (each lane's own) until all have reached
// target; false when an error was reported or the watchdog fired.
__device__ __forceinline__ bool poll(const Waits& a, const int32_t* p, int target) {
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

// ---- one block of one sweep -------------------------------------------------
//
// Block b holds the nb rows below row c - 1, c = k + 1 + b nb, and in them the
// columns c .. c + nb - 1 (D) and c + nb .. c + 2 nb - 1 (Q).  In sweep k it
//   * takes the row above that the right reflector clears (its columns are
//     D's; from block b - 1, or row k), forms the reflector and applies it to D;
//   * forms the left reflector of D's first column and applies it to D and Q;
//   * gives the new first row of Q to block b + 1, as the row to be cleared
//     there, and applies its reflector to its own other rows of Q;
//   * moves its window one row and one column on: its first row, finished for
//     this block, becomes block b - 1's new last row (of block 0, the row the
//     next sweep clears), its last row was the first one of block b + 1.
// Rows and columns are held in rings of nb: row or column c + i of sweep k,
// of D and of Q, is in slot (k + i) mod nb, so a row keeps its slot through all
// sweeps and the window moves without moving anything but one column of Q, which
// becomes D's in the same lanes.  Rows and columns past the matrix are +0 and
// stay so; a zero column or row gives the identity.
//
// Lane l holds the columns of slots l + 64 h, wave w and register i row slot
// 8 i + w (+ 8 RW m for member m of a group of ceil(nb / 64) workgroups, nb >
// 128).  Row sums go over the lanes of a wave; column sums over a wave's
// registers, then the waves (LDS) and, in a group, the members.
//
// Members exchange values through boxes whose words hold MARK, a NaN no
// arithmetic gives (and senders replace), until a value comes; the receiver
// polls the words it needs and sets them back.  Two boxes by the parity of the
// step are enough: what a receiver reads in one step is set back before it
// sends anything in the next, and no value of the one after that can be sent to
// it before.
constexpr uint64_t MARK = 0x7FF4B1D1A60CA11Eull;

__device__ __forceinline__ bool marked(double v) { return __builtin_bit_cast(uint64_t, v) == MARK; }
__device__ __forceinline__ void send(double* p, double v) {
    st(p, v != v ? __builtin_bit_cast(double, 0x7FF8000000000000ull) : v);
}
__device__ __forceinline__ void set_back(double* p) { st(p, __builtin_bit_cast(double, MARK)); }

// Called by a whole wave: v[h] = p[h * stride] where use, once none of them
// is MARK; false when an error was reported or the watchdog fired.
template <int N>
__device__ __forceinline__ bool await(const Waits& a, const double* p, int stride, const bool (&use)[N],
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
// none: zeros instead.
template <int RW>
__device__ __forceinline__ void wave_sums(double (&p)[RW], bool none) {
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
    q[0] = none ? 0.0 : q[0];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int half = i / (RW / 2), r = i % (RW / 2), row = r / (RW / 4), s = r % (RW / 4);
        const int lane_of = 32 * half + 16 * row + (RW == 16 ? 8 * (s / 2) + 4 * (s % 2) : RW == 8 ? 8 * s : 0);
        p[i] = lane_value(q[0], lane_of);
    }
}

constexpr int box_sums(int ch, int group) { return ch <= 2 ? 0 : (group + 1) * 128 * ch; }

// Workgroups that run a block: how many, which one this is, its boxes for the
// others' column sums and row 0 (two parities), doubles between two members'.
struct Group {
    int G, m;
    double* box;
    int64_t stride;
};

template <int CH>
struct StepLds {
    double part[NW][128 * CH];          // column sums of each wave
    double total[128 * CH];             // of the block
    double row0[2][128 * CH];           // the first row, by parity of the step
    int fail[2];
};

// par: the step's parity; i0: slot of the first row and column; v: the row to
// clear; ok: whether the caller's waits were.  send_row(g) is given the row the
// next block clears, send_last(fr, fl, fg, last) the rest of the finished first
// row: last with fg's beta in slot i0, fl's beta on the diagonal.  The first
// row's registers end as zeros.  Ends the workgroup where a wait failed (an exit
// of the kernel, not a result: D and Q would be copied where the paths meet).
template <int CH, int RW, class Row, class Last>
__device__ __forceinline__ void block_step(const Waits& a, StepLds<CH>& s, const Group& gr, int par, int i0, bool ok,
                                           double (&D)[RW][CH], double (&Q)[RW][CH], double (&v)[CH], Row&& send_row,
                                           Last&& send_last) {
    constexpr int NBP = 64 * CH;
    constexpr int PARTS = NW * CH / 4;          // waves' sums a lane adds: 2, 4, 8
    constexpr bool GROUPED = CH == 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = GROUPED ? gr.G : 1, m = GROUPED ? gr.m : 0;
    const int l0 = i0 % 64, h0 = i0 / 64;
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
    auto from_right = [&](double (&M)[RW][CH], const double (&x)[CH], const Refl& f) {
        double p[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            p[i] = M[i][0] * x[0];
#pragma unroll
            for (int h = 1; h < CH; ++h) p[i] = fma(M[i][h], x[h], p[i]);
        }
        wave_sums<RW>(p, f.tau == 0.0);
        double tx[CH];
#pragma unroll
        for (int h = 0; h < CH; ++h) tx[h] = -f.tau * x[h];
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int h = 0; h < CH; ++h) M[i][h] = fma(p[i], tx[h], M[i][h]);
    };
    const Refl fr = clear(v);
    from_right(D, v, fr);

    // the first row leaves the registers
    const bool gives = w == i0 % 8 && (!GROUPED || m == i0 / (8 * RW));
    if (gives) {
        // (a bit a register: comparisons of one value become a switch, at whose
        // end every register that its cases change would be copied)
        const uint32_t reg = 1u << i0 / 8 % RW;
#pragma unroll
        for (int i = 0; i < RW; ++i)
            if (__builtin_expect(reg >> i & 1, 0)) {
#pragma unroll
                for (int h = 0; h < CH; ++h) {
                    s.row0[par][lane + 64 * h] = D[i][h];
                    s.row0[par][NBP + lane + 64 * h] = Q[i][h];
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
            s.part[w][lane + 64 * h] = pd[h];
            s.part[w][NBP + lane + 64 * h] = pq[h];
        }
    }
    if (!ok) s.fail[par] = 1;
    wait_memory();                          // words set back in the last step
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(s.fail[par]) != 0) __builtin_amdgcn_endpgm();
    {
        const int col = w * 16 * CH + lane % (16 * CH), sub = lane / (16 * CH);
        double each[PARTS], sum = 0.0;
#pragma unroll
        for (int h = 0; h < PARTS; ++h) each[h] = s.part[sub * PARTS + h][col];
        __builtin_amdgcn_sched_barrier(0);      // (all of them are read before the first is added)
#pragma unroll
        for (int h = 0; h < PARTS; ++h) sum += each[h];
        if constexpr (CH == 1) sum = sum_rows(sum);
        if constexpr (CH == 2) sum = sum_halves(sum);
        if constexpr (GROUPED) {
            // the members' sums and, from the one that has it, row 0
            double* own = gr.box + par * (int64_t)box_sums(CH, G);
            const int holder = i0 / (8 * RW);
            const double r0 = s.row0[par][col];
            for (int o = 1; o < G; ++o) {
                const int to = m + o < G ? m + o : m + o - G;
                double* other = own + (to - m) * gr.stride;
                send(other + m * 2 * NBP + col, sum);
                if (m == holder) send(other + G * 2 * NBP + col, r0);
            }
            // four members at most, row 0 behind them
            bool from[4];
            const bool from0[1] = {m != holder};
#pragma unroll
            for (int h = 0; h < 4; ++h) from[h] = h < G && h != m;
            double y[4], y0[1];
            bool ok2 = await(a, own + col, 2 * NBP, from, y);
            ok2 = await(a, own + G * 2 * NBP + col, 0, from0, y0) && ok2;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                if (from[h]) set_back(own + h * 2 * NBP + col);
                y[h] = h == m ? sum : y[h];
            }
            if (from0[0]) {
                set_back(own + G * 2 * NBP + col);
                s.row0[par][col] = y0[0];
            }
            sum = (y[0] + y[1]) + (y[2] + y[3]);
            if (!ok2) s.fail[par] = 1;
        }
        if (sub == 0) s.total[col] = sum;
    }
    lds_barrier();
    if (GROUPED && __builtin_amdgcn_readfirstlane(s.fail[par]) != 0) __builtin_amdgcn_endpgm();

    // left reflector; the new first row (its terms are read while the reflector
    // is formed)
    double td[CH], tq[CH], g[CH], last[CH];
#pragma unroll
    for (int h = 0; h < CH; ++h) {
        last[h] = s.row0[par][lane + 64 * h];
        g[h] = s.row0[par][NBP + lane + 64 * h];
        td[h] = s.total[lane + 64 * h];
        tq[h] = s.total[NBP + lane + 64 * h];
    }
    const Refl fl = reflector(s.row0[par][i0], s.total[i0]);
#pragma unroll
    for (int h = 0; h < CH; ++h) {
        td[h] = fma(fl.scale, td[h], last[h]);
        tq[h] = fma(fl.scale, tq[h], g[h]);
        td[h] = fl.tau == 0.0 ? 0.0 : td[h];
        tq[h] = fl.tau == 0.0 ? 0.0 : tq[h];
        last[h] = fma(-fl.tau, td[h], last[h]);
        g[h] = fma(-fl.tau, tq[h], g[h]);
        td[h] *= -fl.tau * fl.scale;
        tq[h] *= -fl.tau * fl.scale;
    }
    send_row(g);
    const Refl fg = clear(g);
    send_last(fr, fl, fg, last);
    // the other rows: from the left, then Q from the right
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            D[i][h] = fma(x[i], td[h], D[i][h]);
            Q[i][h] = fma(x[i], tq[h], Q[i][h]);
        }
    from_right(Q, g, fg);
}

// ---- the chase with the band held in registers -----------------------------
//
// Every block has its workgroups, which keep it through all sweeps: nothing of
// the band moves, and what blocks give each other are messages of one row.  A
// message is its values, in inboxes of MARK words as above, by the parity of
// the sweep; indexed by slot, it needs no rotation.
//
// What bounds it: the chain of 2 n steps, a message (about 1.3 us from the
// store to the polling load that sees it) and the step's own chain (reflector,
// row sums, column sums over the waves, reflector) each; the rest of a step's
// work falls into the time the block waits anyway, as a block works in every
// other step only.  A step takes 1.8 us (nb = 32), 2.1 (64), 2.9 (128) and 4.6
// (256, with the exchange between four members).
//
// All workgroups have to run at once, so they meet first; if they have not
// met within MEET_SECONDS (other work holds compute units), those that run do
// the chase by sweeps, which needs no more than one group, and those that start
// later join them.
constexpr double MEET_SECONDS = 2e-3;

struct HoldArgs {
    Waits wait;
    const double* W;      // the band array
    int64_t n;
    int nb;
    int group;            // workgroups per block
    double* box;          // inboxes, per workgroup
    double* d;
    double* e;
    int64_t meet_ticks;
};

// An inbox: two rows to clear, two last rows (and a diagonal entry behind
// each), for groups the exchange's boxes.
constexpr int box_row(int ch) { return 64 * ch; }
constexpr int box_last(int ch) { return 64 * ch + 8; }
constexpr int box_doubles(int ch, int group) { return 2 * (box_row(ch) + box_last(ch) + box_sums(ch, group)); }

enum : int { MET_GO = 1, MET_GIVE_UP = 2 };     // the word G_MET

// One thread of each workgroup: whether all of them are running (MET_GO).
__device__ __forceinline__ int meet(const HoldArgs& a) {
    const uint64_t t0 = wall_clock64();
    int none = 0;
    if (__hip_atomic_fetch_add(&a.wait.ctrl[G_RUNNING], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
        (int)gridDim.x - 1)
        __hip_atomic_compare_exchange_strong(&a.wait.ctrl[G_MET], &none, (int)MET_GO, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    for (;;) {
        const int met = aload(&a.wait.ctrl[G_MET]);
        if (met != 0) return met;
        if ((int64_t)(wall_clock64() - t0) > a.meet_ticks) {
            none = 0;
            __hip_atomic_compare_exchange_strong(&a.wait.ctrl[G_MET], &none, (int)MET_GIVE_UP, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_s_sleep(4);
    }
}

template <int CH, int RW>
__device__ __forceinline__ void hold_blocks(const HoldArgs& a, StepLds<CH>& lds) {
    constexpr int NBP = 64 * CH;
    constexpr bool GROUPED = CH == 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = a.nb, G = GROUPED ? a.group : 1;
    const int b = (int)blockIdx.x / G, m = (int)blockIdx.x % G;
    const int size = box_doubles(CH, G);
    double* box = a.box + (int64_t)blockIdx.x * size;
    double* box_l = box + 2 * box_row(CH);
    const Group gr{G, m, box_l + 2 * box_last(CH), size};
    const int64_t K = a.n - 1 - (int64_t)b * nb, Kn = K - nb;   // sweeps of this block, of the next
    // (from the band array, not from B: d and e, written from here on, may lie there)
    const int64_t rowp = 3 * (int64_t)nb - 1;           // from entry (i, j) to (i + 1, j)
    const double* w0 = a.W + nb - 1;                    // entry (0, 0)
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
            D[i][h] = in && col < a.n ? w0[row * rowp + col] : 0.0;
            Q[i][h] = in && col + nb < a.n ? w0[row * rowp + col + nb] : 0.0;
        }
    }
    if (blockIdx.x == 0 && tid == 0) a.d[0] = w0[0];

    int i0 = 0, ip = 0;                         // slots of the first row and column: of this sweep, of the last
    for (int64_t k = 0; k < K; ++k) {
        const int par = (int)(k & 1);
        bool ok = true;
        // the last row, which was the first one of the next block
        const bool takes = k > 0 && k <= Kn && w == ip % 8 && (!GROUPED || m == ip / (8 * RW));
        if (takes) {
            double x[CH], diag[1];
            const bool one[1] = {true};
            ok = await(a.wait, box_l + (par ^ 1) * box_last(CH) + lane, 64, use, x);
            ok = ok && await(a.wait, box_l + (par ^ 1) * box_last(CH) + NBP, 0, one, diag);
            const uint32_t reg = 1u << ip / 8 % RW;
#pragma unroll
            for (int i = 0; i < RW; ++i)
                if (__builtin_expect(reg >> i & 1, 0)) {
#pragma unroll
                    for (int h = 0; h < CH; ++h) {
                        D[i][h] = lane + 64 * h == ip ? diag[0] : 0.0;
                        Q[i][h] = x[h];
                        asm volatile("" : "+v"(D[i][h]), "+v"(Q[i][h]));
                    }
                }
        }
        // the row to clear
        double v[CH];
        if (b > 0 || k > 0) {
            ok = await(a.wait, box + par * box_row(CH) + lane, 64, use, v) && ok;
        } else {
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                const int64_t col = 1 + lane + 64 * h;
                v[h] = use[h] && col < a.n ? w0[col] : 0.0;
            }
        }
        block_step<CH, RW>(
            a.wait, lds, gr, par, i0, ok, D, Q, v,
            [&](const double (&g)[CH]) {
                if (w == 0 && k < Kn) {
                    double* to = box + (int64_t)G * size + par * box_row(CH) + lane;
#pragma unroll
                    for (int h = 0; h < CH; ++h)
                        if (use[h]) send(to + 64 * h, g[h]);
                }
            },
            [&](const Refl& fr, const Refl& fl, const Refl& fg, const double (&last)[CH]) {
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
                        if (m == 0 && lane == 0) {
                            a.e[k] = fr.beta;
                            a.d[k + 1] = fl.beta;
                        }
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
            });
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

// ---- the chase by sweeps ----------------------------------------------------
//
// The band is copied into an array with room for the fill of the chase (nb - 1
// diagonals below the main one, 2 nb - 1 above), by rows:
//     W[(j - i + nb - 1) + i * 3 nb]  holds entry (i, j).
// One persistent launch: each workgroup takes the next sweep, or the next
// member's place in a group that runs one (tickets from an atomic counter, so
// a sweep is only ever waited for by a later one that running workgroups hold:
// no deadlock for any grid), and runs its blocks in order: it loads a member's
// rows of the block, does the step, stores them, and keeps the row the next
// block clears.  A row keeps its slot and so its member, and block b of sweep k
// takes the rows that block b of sweep k - 1 left and, as its last one, the first
// row of block b + 1, so member m waits for member m of the sweep ahead alone
// (for row k also for the one that has it).  A block publishes its first row
// before its others: less than two steps separate consecutive sweeps.
//
// The band array is written and read with agent-scope stores and loads (past
// the XCD's L2, at the coherence point), so a counter is published once every
// wave has waited for its own memory operations, with no L2 write-back, and the
// loads that follow a counter's load see every store performed before it was
// written, with no L2 invalidation; a wall-clock watchdog bounds every wait.
//
// What bounds it: the chain of about 2 n steps, in each the round trips to the
// coherence point (the poll of the sweep ahead, a member's rows in, up to 256
// KB, and out, for groups the exchange) and the step itself.  A block's stores
// complete while the next one's wait is polled and its rows are loaded.
// Measured, with slices of rows in LDS on up to 16 workgroups a sweep (whose sums
// were others than the held chase's) and so: 20000 at nb = 16 300 and 172 ms, 50000
// at nb = 64 760 and 649 ms, 40000 at nb = 128 1326 and 1138 ms, 20000 at nb =
// 256 983 and 650 ms.  Where the band can be held: 2000 at nb = 64 16 ms (held
// 7.7), 16384 at nb = 128 450 (96), 8192 at nb = 256 255 ms (75).
struct SweepArgs {
    Waits wait;
    double* W;
    int64_t n;
    int nb;
    int nsweeps;
    int group;            // workgroups per sweep
    int32_t* prog;        // t + 1: blocks < t and the first row of block t stored, per sweep and member
                          // (T + 1: all T blocks)
    double* xch;          // exchange areas (group > 1): two parities a member
    int nareas;
    double* d;
    double* e;
};

template <int CH, int RW>
__device__ __forceinline__ void run_sweeps(const SweepArgs& a, StepLds<CH>& lds, int& sk, int& flag) {
    constexpr bool GROUPED = CH == 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = a.nb, G = GROUPED ? a.group : 1;
    const int64_t rowp = 3 * (int64_t)nb - 1;           // from entry (i, j) to (i + 1, j)

    for (;;) {
        // ticket = sweep * G + member: a group's members are consecutive
        // tickets, all taken by running workgroups before any of them can
        // be needed by a later sweep
        if (tid == 0) sk = __hip_atomic_fetch_add(&a.wait.ctrl[G_HEAD], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const int ticket = __builtin_amdgcn_readfirstlane(sk);
        __syncthreads();
        const int64_t k = ticket / G;
        const int m = ticket - (int)k * G;
        if (k >= a.nsweeps) return;
        const int T = (int)nsteps(a.n, nb, k);
        const int Tp = k > 0 ? (int)nsteps(a.n, nb, k - 1) : 0;
        int32_t* prog = a.prog + k * G;
        const int64_t sums = 2 * (int64_t)box_sums(CH, G);
        const Group gr{G, m, GROUPED ? a.xch + (k % a.nareas * G + m) * sums : nullptr, sums};
        const int i0 = (int)(k % nb);                       // slot of the first row and column
        const int ahead_holder = GROUPED && k > 0 ? (int)((k - 1) % nb) / (8 * RW) : 0;     // has row k
        bool use[CH];
        int off[CH];                                        // column of a slot, from the block's first
        double v[CH];
#pragma unroll
        for (int h = 0; h < CH; ++h) {
            const int q = lane + 64 * h;
            use[h] = q < nb;
            off[h] = q < i0 ? q - i0 + nb : q - i0;
        }

        for (int t = 0; t < T; ++t) {
            const int64_t c = k + 1 + (int64_t)t * nb;
            double* w0 = a.W + c * rowp + c + nb - 1;       // entry (c, c)
            // block t of the sweep ahead and the first row of its block t + 1;
            // at the start also its row k and the area's last user
            if (k > 0 && w == 0) {
                const int32_t* ahead = a.prog + (k - 1) * G + (lane == 1 && t == 0 ? ahead_holder : m);
                int target = t + 1 < Tp ? t + 2 : Tp + 1;
                if (GROUPED && t == 0 && k >= a.nareas && lane >= 2 && lane < 2 + G) {
                    ahead = a.prog + (k - a.nareas) * G + lane - 2;
                    target = (int)nsteps(a.n, nb, k - a.nareas) + 1;
                }
                const bool ok = poll(a.wait, ahead, target);
                if (lane == 0) flag = ok;
            }
            lds_barrier();
            if (k > 0 && __builtin_amdgcn_readfirstlane(flag) == 0) return;

            // what does not exist is loaded from entry (c, c) or the row's
            // first, so that no load is behind a branch, and taken as zero
            const int64_t left = a.n - c;                   // rows and columns from c on
            double D[RW][CH], Q[RW][CH];
            int row[RW];                                    // from c; nb: does not exist
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                const int r = 8 * (RW * m + i) + w, o = r < i0 ? r - i0 + nb : r - i0;
                row[i] = r < nb && o < left ? o : nb;
                const double* p = w0 + (row[i] < nb ? row[i] * rowp : 0);
#pragma unroll
                for (int h = 0; h < CH; ++h) {
                    D[i][h] = ld(p + (use[h] && off[h] < left ? off[h] : 0));
                    Q[i][h] = ld(p + (use[h] && off[h] + nb < left ? off[h] + nb : 0));
                }
            }
            if (t == 0) {
#pragma unroll
                for (int h = 0; h < CH; ++h) {
                    const bool in = use[h] && off[h] < left;
                    v[h] = ld(w0 - rowp + (in ? off[h] : 0));       // row k
                    v[h] = in ? v[h] : 0.0;
                }
                if (k == 0 && m == 0 && tid == 0) a.d[0] = ld(a.W + nb - 1);
            }
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int h = 0; h < CH; ++h) {
                    D[i][h] = row[i] < nb && use[h] && off[h] < left ? D[i][h] : 0.0;
                    Q[i][h] = row[i] < nb && use[h] && off[h] + nb < left ? Q[i][h] : 0.0;
                }

            double next[CH];
            block_step<CH, RW>(
                a.wait, lds, gr, t & 1, i0, true, D, Q, v,
                [&](const double (&g)[CH]) {
#pragma unroll
                    for (int h = 0; h < CH; ++h) next[h] = g[h];
                },
                [&](const Refl& fr, const Refl& fl, const Refl& fg, const double (&last)[CH]) {
                    if (w == 1 && (!GROUPED || m == i0 / (8 * RW))) {       // the finished first row
#pragma unroll
                        for (int h = 0; h < CH; ++h) {
                            if (use[h] && off[h] < left) st(w0 + off[h], off[h] == 0 ? fl.beta : last[h]);
                            if (use[h] && off[h] + nb < left) st(w0 + off[h] + nb, off[h] == 0 ? fg.beta : 0.0);
                        }
                    }
                    if (w == 1 && lane == 0 && t == 0 && m == 0) {
                        a.e[k] = fr.beta;
                        a.d[k + 1] = fl.beta;
                    }
                });
            // The previous block's stores had completed in every wave at the
            // step's first barrier, and the first row, which this block's
            // rows below no longer touch, has in the wave that stored it.
            if (w == 1) {
                wait_memory();
                if (lane == 0) __hip_atomic_store(&prog[m], t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int h = 0; h < CH; ++h) {
                v[h] = next[h];
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    if (row[i] == 0 || row[i] == nb) continue;      // uniform
                    double* p = w0 + row[i] * rowp + off[h];
                    if (use[h] && off[h] < left) st(p, off[h] == 0 ? 0.0 : D[i][h]);
                    if (use[h] && off[h] + nb < left) st(p + nb, Q[i][h]);
                }
            }
        }
        // the whole sweep
        wait_memory();
        __syncthreads();
        if (tid == 0) __hip_atomic_store(&prog[m], T + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// tries: the blocks are held if the workgroups (as many as they need) meet; one
// kernel for both ways, as a launch that finds nothing left to do waits for
// room beside other work like any other.
template <int CH, int RW>
__global__ __launch_bounds__(NT) void chase_kernel(HoldArgs h, SweepArgs a, int tries) {
    __shared__ StepLds<CH> lds;
    __shared__ int met, flag;
    if (threadIdx.x == 0) {
        lds.fail[0] = lds.fail[1] = 0;
        met = tries ? meet(h) : (int)MET_GIVE_UP;
        if (aload(&a.wait.ctrl[G_ERROR]) != 0) met = 0;     // an error reported before stops the chase
    }
    __syncthreads();
    const int way = __builtin_amdgcn_readfirstlane(met);
    __syncthreads();
    if (way == MET_GO) {
        hold_blocks<CH, RW>(h, lds);
        __builtin_amdgcn_endpgm();          // (what the sweeps need is not kept through this)
    }
    if (way == MET_GIVE_UP) run_sweeps<CH, RW>(a, lds, met, flag);
}

// Everything the chase finds in the workspace, for either way: the control
// words cleared (not the error word where keep_error: a status already there,
// such as the band reduction's in the one-shot pipeline, stops the chase at its
// start and stays visible) and the progress counters, exchange areas and
// inboxes marked, the upper band of B copied into W (zero elsewhere).  Entry
// (i, j) of the band is B[i rs + j cs]: rs = 1, cs = ldb for an upper band stored
// as is, rs = ldb, cs = 1 for the transpose of a lower band.
// One launch for both ways: beside work that fills the chip every launch waits
// for room of its own (a matrix product's last workgroups, say).
struct PrepareArgs {
    const double* B;
    int64_t rs, cs, n;
    int nb;
    int32_t* ctrl;
    int keep_error;
    double* W;
    int32_t* prog;
    int64_t nprog;
    double *xch, *box;
    int64_t nxch, nbox;
};

__global__ void prepare_kernel(PrepareArgs a) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const double mark = __builtin_bit_cast(double, MARK);
    if (g < G_WORDS && !(a.keep_error && g == G_ERROR)) a.ctrl[g] = 0;
    for (int64_t x = g; x < a.nprog; x += stride) a.prog[x] = 0;
    for (int64_t x = g; x < a.nxch; x += stride) a.xch[x] = mark;
    for (int64_t x = g; x < a.nbox; x += stride) a.box[x] = mark;
    const int64_t ldw = 3 * (int64_t)a.nb, total = ldw * a.n;
    for (int64_t x = g; x < total; x += stride) {
        const int64_t i = x / ldw;
        const int64_t j = i + (x - i * ldw) - (a.nb - 1);
        a.W[x] = j >= i && j - i <= a.nb && j < a.n ? a.B[i * a.rs + j * a.cs] : 0.0;
    }
}

// A band that is bidiagonal as it is (nb = 1 or n <= 2), from the band array.
__global__ void diagonals_kernel(const double* W, int64_t n, int nb, double* d, double* e) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double* w = W + nb - 1 + i * 3 * nb;
    if (i < n) d[i] = w[0];
    if (i + 1 < n) e[i] = w[1];
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

// Instance for a bandwidth: slots of 64 CH columns, workgroups a block or a
// sweep (of 8 RW row slots each), workgroups a compute unit that the workspace
// has room for: what the registers of chase_kernel's instance allow (69, 86, 227,
// 247 of 512 a lane and SIMD, two waves a workgroup and SIMD).
inline int ch_of(int nb) { return nb <= 64 ? 1 : nb <= 128 ? 2 : 4; }
inline int group_of(int nb) { return nb <= 128 ? 1 : (nb + 63) / 64; }
inline int per_cu(int nb) { return nb <= 32 ? 3 : nb <= 64 ? 2 : 1; }

inline int64_t round256(int64_t b) { return (b + 255) / 256 * 256; }

inline int nsweeps_of(int64_t n, int nb) { return nb <= 1 || n <= 2 ? 0 : (int)(n - 1); }

// Exchange areas of the chase by sweeps (groups only): sweep k uses area k %
// nareas, once every member of the sweep that had it before has ended (and with
// it set its words back).  So many that this is never waited for: no more than
// MAX_WG / group + 1 sweeps have running workgroups.
inline int nareas_of(int64_t n, int nb) {
    return group_of(nb) > 1 ? std::min(nsweeps_of(n, nb), MAX_WG / group_of(nb) + 2) : 0;
}

// Workspace: control words (256 B), the band array (3 nb n doubles), the
// members' progress counters (int32 per sweep and member), the exchange areas,
// the held blocks' inboxes.
inline int64_t prog_words(int64_t n, int nb) { return (int64_t)nsweeps_of(n, nb) * group_of(nb); }
inline int64_t xch_words(int64_t n, int nb) {
    return (int64_t)nareas_of(n, nb) * group_of(nb) * 2 * box_sums(ch_of(nb), group_of(nb));
}
// Workgroups of all blocks; none (0) where they do not fit on the chip at
// once, or nothing is chased.
inline int64_t hold_workgroups(int64_t n, int nb) {
    const int64_t wg = (n - 1 + nb - 1) / nb * group_of(nb);
    return nsweeps_of(n, nb) > 0 && wg <= MAX_WG * per_cu(nb) ? wg : 0;
}
inline int64_t hold_words(int64_t n, int nb) {
    return hold_workgroups(n, nb) * box_doubles(ch_of(nb), group_of(nb));
}
inline int64_t ws_prog_off(int64_t n, int nb) { return round256(256 + (int64_t)3 * nb * n * 8); }
inline int64_t ws_xch_off(int64_t n, int nb) { return ws_prog_off(n, nb) + round256(prog_words(n, nb) * 4); }
inline int64_t ws_hold_off(int64_t n, int nb) { return ws_xch_off(n, nb) + round256(xch_words(n, nb) * 8); }
inline size_t ws_bytes(int64_t n, int nb) { return (size_t)(ws_hold_off(n, nb) + 8 * hold_words(n, nb)); }

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

// f(chase_kernel) of the instance for nb.
template <class F>
void with_instance(int nb, F&& f) {
    if (nb <= 32) f(chase_kernel<1, 4>);
    else if (nb <= 64) f(chase_kernel<1, 8>);
    else if (nb <= 128) f(chase_kernel<2, 16>);
    else f(chase_kernel<4, 8>);
}

// The chase after argument checks: band entry (i, j) at B[i rs + j cs].
// by_sweeps: not held, whatever the size.
int bnd2bd_launch(const double* B, int64_t rs, int64_t cs, int64_t n, int nb, double* d, double* e, void* ws,
                  double watchdog_s, bool by_sweeps, bool keep_error, void* stream);

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
    return bbg::bnd2bd_launch(B, 1, ldb, n, nb, d, e, ws, watchdog_s, group > 0, false, stream);
}

}  // extern "C"

int bbg::bnd2bd_launch(const double* B, int64_t rs, int64_t cs, int64_t n, int nb, double* d, double* e,
                       void* ws, double watchdog_s, bool by_sweeps, bool keep_error, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    int32_t* ctrl = (int32_t*)ws;
    const int nsw = bbg::nsweeps_of(n, nb);
    const double khz = (double)bbg::device_attr(hipDeviceAttributeWallClockRate, 100000);
    const bbg::Waits wait{ctrl, (int64_t)((watchdog_s > 0 ? watchdog_s : 30.0) * khz * 1000.0)};
    const int cus = bbg::device_attr(hipDeviceAttributeMultiprocessorCount, 256);
    const int group = bbg::group_of(nb);
    if (nsw > 0 && cus < group) return BB_ENOTSUP;
    // A chase's workgroups take their compute units' LDS, each an equal part of
    // it, so that no other kernel's that use LDS run there: a matrix product's waves
    // on the same SIMDs, whose FP64 pipe they share, make a step of 2 us take 45.
    // Beside FP64 products on another stream, with 11 KB a workgroup and so: 300 at
    // nb = 64 28 and 12 ms, 1000 at nb = 64 62 and 14 ms.  Alone it costs nothing.
    const int64_t blocks = std::max<int64_t>(1, (n - 1 + nb - 1) / nb) * group;
    const int per = (int)std::min<int64_t>(bbg::per_cu(nb), (blocks + cus - 1) / cus);
    const int64_t wgs = bbg::hold_workgroups(n, nb);
    int room = 0;                               // workgroups of this build a compute unit runs
    size_t lds = 0;
    bbg::with_instance(nb, [&](auto kernel) {
        const int all = bbg::device_attr(hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, 65536);
        hipFuncAttributes fa;
        if (hipFuncGetAttributes(&fa, (const void*)kernel) == hipSuccess) {
            const int most = all - (int)fa.sharedSizeBytes;     // (the same for every call)
            if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most) == hipSuccess)
                lds = (size_t)std::max(0, most - (all - all / per)) / 1280 * 1280;
        }
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&room, kernel, bbg::NT, lds) != hipSuccess) room = 0;
        (void)hipGetLastError();                // (without an answer the sweeps run, in the LDS they need)
    });
    const bool hold = !by_sweeps && wgs > 0 && wgs <= (int64_t)cus * room;
    double* box = (double*)((char*)ws + bbg::ws_hold_off(n, nb));
    double* W = (double*)((char*)ws + 256);
    const bbg::HoldArgs h{wait, W, n, nb, group, box, d, e, (int64_t)(bbg::MEET_SECONDS * khz * 1000.0)};
    const bbg::SweepArgs a{wait, W, n, nb, nsw, group,
                           (int32_t*)((char*)ws + bbg::ws_prog_off(n, nb)),
                           (double*)((char*)ws + bbg::ws_xch_off(n, nb)), std::max(1, bbg::nareas_of(n, nb)), d, e};
    const bbg::PrepareArgs p{B, rs, cs, n, nb, ctrl, keep_error ? 1 : 0, W, a.prog, bbg::prog_words(n, nb),
                             a.xch, box, bbg::xch_words(n, nb), hold ? bbg::hold_words(n, nb) : 0};
    const int64_t total = (int64_t)3 * nb * n;
    hipLaunchKernelGGL(bbg::prepare_kernel, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 8 * (int64_t)cus)),
                       dim3(256), 0, s, p);
    if (hipGetLastError() != hipSuccess) return BB_EHIP;
    if (nsw == 0) {
        hipLaunchKernelGGL(bbg::diagonals_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, W, n, nb, d, e);
        return hipGetLastError() == hipSuccess ? BB_OK : BB_EHIP;
    }
    // A workgroup (group) a block: to hold it, and for the sweeps, of which no
    // more than blocks are in progress (two are never at one block).  Without
    // room for all, whole groups, one workgroup a CU and MAX_WG at most (the
    // exchange areas are counted for that), without groups as many as run.
    const int64_t grid = hold ? wgs
                              : std::min<int64_t>(blocks, group > 1 ? std::min(cus, bbg::MAX_WG) / group * group
                                                                    : (int64_t)cus * per);
    bbg::with_instance(nb, [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(bbg::NT), lds, s, h, a, hold ? 1 : 0);
    });
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
    rc = m >= n ? bbg::bnd2bd_launch(B, 1, lda, k, nb, d, e, ws, opts ? opts->watchdog_s : 0.0, false, true, stream)
                : bbg::bnd2bd_launch(B, lda, 1, k, nb, d, e, ws, opts ? opts->watchdog_s : 0.0, false, true, stream);
    if (rc != BB_OK) return rc;
    return bb_bd2val(d, e, k, sigma, stream);
}

}  // extern "C"
