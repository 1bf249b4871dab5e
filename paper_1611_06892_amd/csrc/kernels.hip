// gfx950 kernels of the tiled band bidiagonalization.
//
// Every task of the graph is one tile kernel of Table 1 (Section 3.2):
//   panel  : GEQRT (factor a square tile into a triangle), TSQRT (zero a square
//            tile below a triangle), TTQRT (zero a triangle below a triangle);
//   update : UNMQR, TSMQR, TTMQR (apply those reflectors to a trailing tile or
//            tile pair).
// LQ steps use the same kernels on transposed tiles (Section 3.4, Algorithm 4):
// each task carries a transpose flag and all arithmetic is written in a
// "logical" frame where logical element (r, c) of a tile is physical element
// (r, c) for QR steps and (c, r) for LQ steps.
//
// Reflector convention (the LAPACK/PLASMA kernels the paper builds on): for
// x = (alpha, x_tail), beta = -sign(alpha) ||x||, tau = (beta - alpha)/beta,
// v = (1, x_tail/(alpha - beta)); tau = 0 when x_tail == 0.  The k reflectors
// of a panel are kept in compact WY form Q = H_1 ... H_k = I - V T V^T with T
// upper triangular, and an update applies Q^T: C <- C - V T^T V^T C.
//
// One workgroup of 512 threads (8 wave64, two per SIMD) executes one work
// unit.  Panels are blocked by 16 columns, each factored by one wave in its
// registers and applied by the others with MFMA; updates apply the 16-column
// blocks of a panel's reflectors with FP64 MFMA (v_mfma_f64_16x16x4) to
// register-resident 16-column slices of the trailing tile(s), one slice per
// wave.  Two waves per SIMD let one wave's MFMA chain run while the other
// waits on a dependency.
#include <mutex>
#include <type_traits>
#include <utility>

#include "../../include/bidiag.h"
#include "kernels.hpp"

namespace bbk {

namespace {

constexpr int NT = 512;          // threads per workgroup
typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

enum : int { K_GEQRT = 0, K_TSQRT = 1, K_TTQRT = 2, K_UNMQR = 3, K_TSMQR = 4, K_TTMQR = 5, K_HQ = 3 };

template <int NB>
struct Shape {
    static constexpr int MT = NB / 16;                 // 16 x 16 tiles per tile side
    static constexpr int LDV = NB + 2;                 // LDS column stride of an update's block V_b: 16-byte
                                                       // aligned, and rows and columns spread over the banks
    // doubles: a panel's block U_b with its T_b, and all of a panel (two of
    // those, a diagonal block of column stride 17 per column tile of a round,
    // the Gram columns); an update's two staged blocks V_b, T_b take less
    static constexpr int UBUF = MT * 336 + 256;
    static constexpr int LDS = 2 * UBUF + (MT < 8 ? MT : 8) * 272 + 274;
    static_assert(LDS >= 2 * (16 * LDV + 256), "update buffers");
};

// Keeps the scheduler from hoisting loads of later 16-row steps of a fully
// unrolled product above this point (bounds register pressure).
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// Workgroup barrier that orders LDS only.  The tile kernels exchange data
// between waves through LDS alone; their global stores (outputs) are not read
// back by the same workgroup, so barriers need not wait for them.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Global store of a task output.  CO (coherent outputs) selects agent-scope
// stores, which are made coherent across the L2s of all XCDs as they
// complete; the persistent scheduler uses them so that finishing a task needs
// only a wait for its stores instead of an L2 write-back.
// Matrix tiles and records are global memory.  Accessing them through
// global-address-space pointers (not generic ones) keeps them off the LDS
// counter, so LDS waits in the products do not also wait for global loads.
typedef __attribute__((address_space(1))) double gdouble;
__device__ __forceinline__ gdouble* gptr(double* p) { return (gdouble*)p; }

template <bool CO>
__device__ __forceinline__ void gstore(double* p, double v) {
    gdouble* q = gptr(p);
    if (CO) __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *q = v;
}

// v, opaque to the compiler: what is formed from it (addresses, lane masks)
// stays where it is used.  Hoisted out of the scheduler's loop or a panel's
// it would be held through code that leaves no registers for it at nb = 256.
__device__ __forceinline__ int here(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// A tile seen in the logical frame: logical element (r, c) is base[r rs + c cs].
// vr/vc: logical rows/columns that exist in the matrix (the rest of the nb x nb
// tile is zero padding, never accessed).
struct TileView {
    double* base;
    int64_t rs, cs;
    int vr, vc;
};

// One lane's part of the 16 columns from c0: column c0 + lane % 16, rows
// 16 i + 4 (lane / 16) .. + 3 of row tile i, read and written four at a time.
// Tiles whose columns are contiguous (QR steps) take buffer accesses: one
// byte offset per lane, the row in the instruction, 16 bytes at a time (the
// accesses need 4-byte alignment only, so any leading dimension does for nb <= 128), by
// element in the row tile in which a ragged tile ends; what does not exist has
// an offset past the buffer's end, where loads give zero and stores do
// nothing.  Everything else (LQ steps) is addressed by element; in a ragged
// tile a load of a missing element reads the tile's first one instead and
// yields zero, so that no load is behind a branch.
// ENDS: ragged tiles go through the buffer too.  In panels, whose chain they
// lengthen (1 % at nb = 64), and at nb = 256, where the branches cost 400
// spills, they go by element.
template <int NB, bool ENDS = NB <= 128>
struct TileLane {
    static constexpr int PAST = (int)0xC0000000u;
    __amdgpu_buffer_rsrc_t rsrc;
    int voff, vr;
    bool vec, whole;
    gdouble *p, *first;
    int64_t rs;
    int rlim;                       // rows r0 + r < rlim exist (r0 a multiple of 16, r < 4)
    __device__ __forceinline__ TileLane(const TileView& t, int c0) {
        const int lane = here(threadIdx.x) & 63, c = c0 + (lane & 15), r = 4 * (lane >> 4);
        whole = t.vr == NB && t.vc == NB;
        // contiguous columns within a buffer's 32-bit offsets (nb = 256: aligned
        // too; without that condition, or with it a value of its own, the
        // compiler spills 445 registers, not 401, and 16384^2 takes 360 ms, not 352)
        vec = (ENDS || whole) && t.rs == 1 &&
              (NB <= 128 || (((uint64_t)t.base & 15) == 0 && (t.cs & 1) == 0)) && t.cs * NB < (1 << 27);
        vr = t.vr;
        rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)t.base, (short)0, 0x7fffffff, 0x00020000);
        voff = !ENDS || c < t.vc ? 8 * (r + c * (int)t.cs) : PAST;
        first = gptr(t.base);
        p = first + r * t.rs + c * t.cs;
        rs = t.rs;
        rlim = c < t.vc ? t.vr - r : 0;
    }
    // Keeps addresses formed from this lane's offsets from being hoisted
    // above this point.
    __device__ __forceinline__ void renew() { asm volatile("" : "+v"(p), "+v"(voff)); }
    // The lane's offset where it has row `row` + 4 (lane / 16) of the tile.
    __device__ __forceinline__ int element(int row) const {
        return row + 4 * ((threadIdx.x & 63) >> 4) < vr ? voff : PAST;
    }
    template <int MT>
    __device__ __forceinline__ void load(int r0, d4 (&x)[MT]) const {
        if (vec) {
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int row = r0 + 16 * i;
                if (!ENDS || row + 16 <= vr) {
                    const u4 lo = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, 8 * row, 0);
                    const u4 hi = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff + 16, 8 * row, 0);
                    const d2 l = __builtin_bit_cast(d2, lo), h = __builtin_bit_cast(d2, hi);
                    x[i] = d4{l[0], l[1], h[0], h[1]};
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        x[i][r] = __builtin_bit_cast(
                            double, __builtin_amdgcn_raw_buffer_load_b64(rsrc, element(row + r), 8 * (row + r), 0));
                }
            }
        } else if (whole) {
            gdouble* q = p + r0 * rs;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x[i][r] = *q;
                    q += r < 3 ? rs : 13 * rs;
                }
            }
        } else {
            gdouble* q = p + r0 * rs;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x[i][r] = *(r0 + 16 * i + r < rlim ? q : first);
                    q += r < 3 ? rs : 13 * rs;
                }
            }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) x[i][r] = r0 + 16 * i + r < rlim ? x[i][r] : 0.0;
        }
    }
    __device__ __forceinline__ d4 load(int r0) const {
        d4 x[1];
        load<1>(r0, x);
        return x[0];
    }
    // LINES: the stores of a row tile take 64 bytes of each column; without,
    // 16 of each 32 (panels, which wait for nothing but their own chain, and
    // nb = 256, where the exchange costs registers: 16384^2 352 and 356 ms).
    // Together with 16-byte accesses at any leading dimension and in ragged
    // tiles, nb = 128 updates of uneven matrices (4096 of 64 to 1024 rows in
    // a batch): TSMQR 62.7 -> 49.3, UNMQR 36.6 -> 32.8 us.
    template <bool CO, bool LINES = NB <= 128>
    __device__ __forceinline__ void store(int r0, d4 x) const {
        if (ENDS && vec && r0 + 16 > vr) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double v = x[r];          // (a bit cast of the vector's element takes element 0)
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rsrc, element(r0 + r), 8 * (r0 + r),
                                                      CO ? 16 : 0);
            }
        } else if (vec && !LINES) {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, d2{x[0], x[1]}), rsrc, voff, 8 * r0,
                                                   CO ? 16 : 0);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, d2{x[2], x[3]}), rsrc, voff + 16, 8 * r0,
                                                   CO ? 16 : 0);
        } else if (vec) {
            // Each store takes 64 contiguous bytes of every column: lane g of
            // a column has rows 2 g, 2 g + 1 of the tile's first eight for the
            // one, of its last eight for the other.
            u4 lo = __builtin_bit_cast(u4, d2{x[0], x[1]}), hi = __builtin_bit_cast(u4, d2{x[2], x[3]});
            u4 a, b;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const auto p = __builtin_amdgcn_permlane16_swap(lo[k], hi[k], false, false);
                const auto q = __builtin_amdgcn_permlane32_swap(p[0], p[1], false, false);
                a[k] = q[0];
                b[k] = q[1];
            }
            // cache policy 16 (sc1): performed at the agent's coherence point,
            // as gstore's agent-scope stores
            const int v = voff - 16 * ((threadIdx.x & 63) >> 4);
            __builtin_amdgcn_raw_buffer_store_b128(a, rsrc, v, 8 * r0, CO ? 16 : 0);
            __builtin_amdgcn_raw_buffer_store_b128(b, rsrc, v + 64, 8 * r0, CO ? 16 : 0);
        } else if (whole) {
            gdouble* q = p + r0 * rs;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gstore<CO>((double*)q, x[r]);
                q += rs;
            }
        } else {
            gdouble* q = p + r0 * rs;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (r0 + r < rlim) gstore<CO>((double*)q, x[r]);
                q += rs;
            }
        }
    }
};

// Descriptor of the task's matrix.  A single-matrix launch carries it in the
// kernel arguments.  A batched launch reads it from the workspace, where an
// earlier kernel of the stream wrote it: the loads are agent-scope atomics,
// so no cache level can serve a value left there by an earlier launch that
// used the same workspace.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ MatDesc mat_desc(const KArgs& a, int mat) {
    if (a.mats == nullptr) return a.single;
    const uint64_t* w = reinterpret_cast<const uint64_t*>(a.mats + mat);
    uint64_t f[5];
#pragma unroll
    for (int k = 0; k < 5; ++k)
        f[k] = uniform64(__hip_atomic_load(w + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    MatDesc d;
    d.A = reinterpret_cast<double*>(f[0]);
    d.lda = (int64_t)f[1];
    d.m = (int64_t)f[2];
    d.n = (int64_t)f[3];
    d.rec = reinterpret_cast<double*>(f[4]);
    return d;
}

// The V/T record of a task (slot within its matrix's records).
template <int NB>
__device__ __forceinline__ double* record(const MatDesc& d, const DevTask& tk) {
    return d.rec + (int64_t)tk.slot * (int64_t)(NB * NB + 16 * NB);
}

__device__ __forceinline__ TileView view(const MatDesc& d, const DevTask& tk, int pr, int pc, int nb) {
    const int trans = tk.trans & 1;
    TileView t;
    t.base = d.A + (int64_t)pr * nb + (int64_t)pc * nb * d.lda;
    t.rs = trans ? d.lda : 1;
    t.cs = trans ? 1 : d.lda;
    int prow = (int)min((int64_t)nb, d.m - (int64_t)pr * nb);
    int pcol = (int)min((int64_t)nb, d.n - (int64_t)pc * nb);
    t.vr = trans ? pcol : prow;
    t.vc = trans ? prow : pcol;
    return t;
}

// Register layout of a 16-column slice of a tile, shared by every MFMA of this
// file: element r (0..3) of lane l of row tile i holds logical
// (16 i + 4 (l/16) + r, c0 + l%16), four consecutive rows a lane.
// v_mfma_f64_16x16x4 returns its row m = 4 r + l/16 in element r of lane l and
// takes the k index k = l/16 of its step from lane l, so with row m of the
// first operand taken as row perm16(m) = 4 (m % 4) + m / 4, results come in this layout,
// and element r is the second operand of the k-step that covers rows
// 4 (l/16) + r: a slice held this way feeds the next product without any
// data movement.
__device__ __forceinline__ int perm16(int m) { return 4 * (m & 3) + (m >> 2); }

template <int MT, class Lane>
__device__ __forceinline__ void load_slice(const Lane& t, d4 (&x)[MT]) {
    t.template load<MT>(0, x);
}

template <bool CO, int MT>
__device__ __forceinline__ void store_slice(const TileLane<16 * MT>& t, const d4 (&x)[MT]) {
#pragma unroll
    for (int i = 0; i < MT; ++i) t.template store<CO>(16 * i, x[i]);
}

// Reads of one V/T record through a buffer descriptor: every load of a
// product shares one per-lane byte offset and adds a wave-uniform constant,
// so unrolled products need no per-load address registers.  Reads past the
// record's end return zero.
struct Rec {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ Rec(const double* base, int nb) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0,
                                                 (int)(8 * (nb * nb + 16 * nb)), 0x00020000);
    }
    __device__ __forceinline__ double ld(int voff, int soff) const {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsrc, voff, soff, 0));
    }
};

// The unit a workgroup of the persistent scheduler finished last, whose
// output stores may still be in flight.  The next unit retires it once its own
// first loads are issued, so that the store drain and the load latency
// overlap: every wave waits for all of its memory operations, then thread 0
// counts the unit as done.
struct Prev {
    int task;                      // -1: nothing to retire
    int ticket;
    uint64_t wait, run, end;       // trace times of the finished unit
};

__device__ __forceinline__ int aload(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Thread 0, after the unit's outputs are complete: count down the
// successors' dependency counters, then count the unit as done.
__device__ __forceinline__ void complete_unit(const KArgs& a, int task) {
    const int s0 = a.succ_off[task], s1 = a.succ_off[task + 1];
    for (int e = s0; e < s1; ++e)
        __hip_atomic_fetch_add(&a.deps[a.succ_idx[e]], -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&a.ctrl[CTRL_DONE], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by all 64 lanes of wave 0 (the results are the same in every lane).
// take_ticket: the next priority position, or -1 when all are taken.
// unit_ready: whether that unit's task has no unfinished predecessor now.
// wait_unit: wait until it has none; returns the ticket, or -1 to stop.
__device__ __forceinline__ int take_ticket(const KArgs& a, int lane) {
    int u = 0;
    if (lane == 0)
        u = __hip_atomic_fetch_add(&a.ctrl[CTRL_HEAD], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    u = __builtin_amdgcn_readfirstlane(u);
    return u >= a.nunits ? -1 : u;
}

__device__ __forceinline__ bool unit_ready(const KArgs& a, int u, int lane) {
    const int task = __builtin_amdgcn_readfirstlane(a.units[u].x);
    int d = 0;
    if (lane == 0) d = aload(&a.deps[task]);
    return __builtin_amdgcn_readfirstlane(d) <= 0;
}

__device__ __forceinline__ int wait_unit(const KArgs& a, int u, int lane) {
    const int task = __builtin_amdgcn_readfirstlane(a.units[u].x);
    const uint64_t t0 = wall_clock64();
    for (;;) {
        int d = 0, err = 0;
        if (lane == 0) {
            d = aload(&a.deps[task]);
            if (d > 0) err = aload(&a.ctrl[CTRL_ERROR]);
        }
        d = __builtin_amdgcn_readfirstlane(d);
        if (d <= 0) return u;
        if (__builtin_amdgcn_readfirstlane(err) != 0) return -1;
        if ((int64_t)(wall_clock64() - t0) > a.watchdog_ticks) {
            if (lane == 0) __hip_atomic_store(&a.ctrl[CTRL_ERROR], 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return -1;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// Scheduler words in LDS (persistent kernel): the next ticket, whether its
// unit was ready when taken, and the wall-clock time it was taken at.
enum : int { SCH_TICKET = 0, SCH_READY = 1, SCH_TIME = 2, SCH_WORDS = 4 };

// Wave 0 takes the next ticket and checks its unit once.  An update kernel
// does this before its final stores: a wait for the returned values then
// does not also wait for those stores (one in-order counter covers loads and
// stores), and the next unit's loads can be issued while they drain.
__device__ __forceinline__ void take_next(const KArgs& a, int* sch) {
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const uint64_t tw = wall_clock64();
        const int u = take_ticket(a, lane);
        const bool ready = u >= 0 && unit_ready(a, u, lane);
        if (lane == 0) {
            sch[SCH_TICKET] = u;
            sch[SCH_READY] = ready;
            *(uint64_t*)(sch + SCH_TIME) = tw;
        }
    }
}

__device__ __forceinline__ void retire(const KArgs& a, Prev& p) {
    if (p.task < 0) return;        // uniform
    __builtin_amdgcn_s_waitcnt(0);
    lds_barrier();
    if (threadIdx.x == 0) {
        if (a.trace != nullptr) {
            int64_t* tr = a.trace + 4 * (int64_t)p.ticket;
            tr[0] = (int64_t)p.wait;
            tr[1] = (int64_t)p.run;
            tr[2] = (int64_t)p.end;
            tr[3] = blockIdx.x;
        }
        complete_unit(a, p.task);
    }
    p.task = -1;
}

// ---------------------------------------------------------------------------
// Application of the first NBLK 16-column blocks of a panel record to a
// 16-column slice per wave (the body of UNMQR/TSMQR/TTMQR, Table 1).  Wave
// w's slice c2 (logical columns c0 .. c0 + 15 of C2, all NB rows, in the
// MFMA result layout) is already in registers; block b+1 of the record is
// fetched from memory while block b is applied, then staged in LDS for all
// eight waves:
//   W = C1(block-row b) + V_b^T C2     (UNMQR: no C1)
//   W = T_b^T W
//   C1(block-row b) -= W,   C2 -= V_b W
// which is Q^T [C1; C2] for Q = Q_0 Q_1 ... (Section 3.2).  Zero 16 x 16
// blocks of V are skipped: V is unit lower triangular after GEQRT and upper
// triangular after TTQRT.  HQ applies Q itself (used to form Q C and P C
// from the records): the blocks in reverse order, each with T_b instead of
// T_b^T.  The previous unit of the workgroup is retired once the first
// record block's loads are issued.
// ---------------------------------------------------------------------------
template <int NB, int NBLK, int KIND, bool CO, bool HQ>
__device__ __forceinline__ void apply_blocks(const Rec& rec, const TileLane<NB>& T1, bool active, d4* c2,
                                             double* lds, const KArgs& a, Prev& prev) {
    constexpr int MT = NB / 16;
    constexpr int LDV = Shape<NB>::LDV;
    constexpr int BUF = 16 * LDV + 256;       // V_b (NB x 16, stride LDV) then T_b^T (16 x 16)
    constexpr int PRE = 16 * NB / NT + 1;     // staged doubles per thread and block
    constexpr bool HASC1 = KIND != K_UNMQR;
    const int tid = here(threadIdx.x), lane = tid & 63, j = lane & 15, g = lane >> 4, pj = perm16(j);

    // Block b of the record: V(:, 16b..16b+15) is contiguous (column-major),
    // T_b^T follows the nb x nb matrix.  Thread t stages elements t + NT k of
    // V_b and element t of T_b^T (t < 256).
    auto fetch = [&](int b, double (&pre)[PRE]) {
#pragma unroll
        for (int k = 0; k < PRE - 1; ++k) pre[k] = rec.ld(8 * (tid + NT * k), 8 * (16 * b * NB));
        pre[PRE - 1] = tid < 256 ? rec.ld(8 * tid, 8 * (NB * NB + 256 * b)) : 0.0;
    };
    auto stage = [&](int buffer, const double (&pre)[PRE]) {
        double* buf = lds + buffer * BUF;
#pragma unroll
        for (int k = 0; k < PRE - 1; ++k) {
            const int e = tid + NT * k;
            buf[(e % NB) + (e / NB) * LDV] = pre[k];
        }
        if (tid < 256) buf[16 * LDV + tid] = pre[PRE - 1];
    };
    auto blk = [](int step) { return HQ ? NBLK - 1 - step : step; };

    double pre[PRE];
    fetch(blk(0), pre);
    retire(a, prev);
    stage(0, pre);
    d4 C1n = {0.0, 0.0, 0.0, 0.0};
    if (HASC1 && active) C1n = T1.load(16 * blk(0));
    lds_barrier();
#pragma unroll
    for (int st = 0; st < NBLK; ++st) {
        const int b = blk(st);
        const double* Vs = lds + (st & 1) * BUF;
        const double* Ts = Vs + 16 * LDV;
        if (st + 1 < NBLK) fetch(blk(st + 1), pre);
        const d4 C1b = C1n;
        if (HASC1 && active && st + 1 < NBLK) C1n = T1.load(16 * blk(st + 1));
        if (active) {
            // Two accumulators halve the dependent-MFMA chain of W.
            d4 Wp[2] = {C1b, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (KIND == K_UNMQR && i < b) continue;
                if (KIND == K_TTMQR && i > b) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    Wp[r & 1] = mfma(Vs[(16 * i + 4 * g + r) + pj * LDV], c2[i][r], Wp[r & 1]);
                // at nb = 256 the slice takes half the registers: keep the
                // operand loads of later row tiles from being hoisted
                if (MT > 8 && (i & 1)) SCHED_FENCE();
            }
            const d4 W = Wp[0] + Wp[1];
            d4 W2 = {0.0, 0.0, 0.0, 0.0};
            // Ts holds T_b^T column-major: T_b(k, i) at i + 16 k.
#pragma unroll
            for (int r = 0; r < 4; ++r)
                W2 = mfma(-(HQ ? Ts[(4 * g + r) + 16 * pj] : Ts[pj + 16 * (4 * g + r)]), W[r], W2);
            // W2 holds -T_b^T W: negating the 4 T operands spares negating
            // the V operands of the update below.
            if (HASC1) T1.template store<CO>(16 * b, C1b + W2);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (KIND == K_UNMQR && i < b) continue;
                if (KIND == K_TTMQR && i > b) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) c2[i] = mfma(Vs[(16 * i + pj) + (4 * g + r) * LDV], W2[r], c2[i]);
                if (MT > 8 && (i & 1)) SCHED_FENCE();
            }
        }
        if (st + 1 < NBLK) stage((st + 1) & 1, pre);
        lds_barrier();
    }
}

// ---------------------------------------------------------------------------
// Panel kernels: GEQRT, TSQRT, TTQRT (Table 1), blocked by 16 columns.
//
// GEQRT factors the tile X = T1 (R overwrites its upper triangle, zeros below).
// TSQRT / TTQRT factor [R1; X2] with R1 = T1 upper triangular and X2 = T2
// square (TS) or upper triangular (TT): R1 is updated in place and X2 zeroed.
// The reflector of column c is u_c = e_c + (tail below the diagonal) for
// GEQRT and u_c = [e_c ; v2_c] for TS/TT; V stores the tails (with the unit
// diagonal made explicit for GEQRT), which are full for TS and upper
// triangular for TT.
//
// Column tile w (nb x 16) stays in the registers of wave w, in the MFMA
// result layout, from its first load to its factorization.  Block b (the
// paper's inner blocking ib = 16):
//  1. leaf: wave b factors its own column tile alone (leaf_columns) and writes
//     U_b and T_b to LDS; one workgroup barrier.
//  2. the waves right of it apply Q_b^T to their tiles with three 16-wide MFMA
//     products (W = R1 + U_b^T X, W = T_b^T W, X -= U_b W), wave b + 1 first
//     (it holds the next leaf), while wave b writes the block's outputs.
// Record (FP64): V (nb x nb, column-major), then the nb/16 blocks T_b^T
// (16 x 16 column-major) -- the same blocked compact-WY form the update
// kernels apply.
// ---------------------------------------------------------------------------

// Broadcasts within rows of 16 lanes: DPP row_newbcast, the 64-bit DPP control,
// as the first operand of an FMA (dst += src0[lane C of the row] * src1).  The
// compiler does not fold its broadcast moves into FMAs, and unfolded they
// double the leaf's instructions, so these are written out.  A DPP operand
// must not have been written by the two preceding instructions, which the
// compiler does not check for inline assembly: every block starts with two
// wait states, and inside a block an operand is written at least three
// instructions before it is broadcast.
#define BB_BC " row_newbcast:%c[c] row_mask:0xf bank_mask:0xf\n\t"
#define BB_BN " row_newbcast:%c[n] row_mask:0xf bank_mask:0xf\n\t"

// Lane C's value in the whole row.  WAIT: wait states before the read, two
// after a vector instruction; six after the 4 x 4 x 4 matrix product (which
// the compiler keeps only for its own instructions).
template <int C, int WAIT = 2>
__device__ __forceinline__ double bcast16(double v) {
    double r;
    asm("s_nop %[w]\n\tv_mov_b64_dpp %[r], %[v]" BB_BC : [r] "=v"(r) : [v] "v"(v), [c] "n"(C), [w] "n"(WAIT - 1));
    return r;
}

// v += coef * (lane C's v) for eight values, then acc += (lane C + 1's v) * v
// (two sums: an FMA's result is ready for the next but one).
template <int C>
__device__ __forceinline__ void update_dot8(double* v, double coef, double (&acc)[2]) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %[v0], %[v0], %[f]" BB_BC "v_fmac_f64_dpp %[v1], %[v1], %[f]" BB_BC
        "v_fmac_f64_dpp %[v2], %[v2], %[f]" BB_BC "v_fmac_f64_dpp %[v3], %[v3], %[f]" BB_BC
        "v_fmac_f64_dpp %[v4], %[v4], %[f]" BB_BC "v_fmac_f64_dpp %[v5], %[v5], %[f]" BB_BC
        "v_fmac_f64_dpp %[v6], %[v6], %[f]" BB_BC "v_fmac_f64_dpp %[v7], %[v7], %[f]" BB_BC
        "v_fmac_f64_dpp %[a0], %[v0], %[v0]" BB_BN "v_fmac_f64_dpp %[a1], %[v1], %[v1]" BB_BN
        "v_fmac_f64_dpp %[a0], %[v2], %[v2]" BB_BN "v_fmac_f64_dpp %[a1], %[v3], %[v3]" BB_BN
        "v_fmac_f64_dpp %[a0], %[v4], %[v4]" BB_BN "v_fmac_f64_dpp %[a1], %[v5], %[v5]" BB_BN
        "v_fmac_f64_dpp %[a0], %[v6], %[v6]" BB_BN "v_fmac_f64_dpp %[a1], %[v7], %[v7]" BB_BN
        : [v0] "+v"(v[0]), [v1] "+v"(v[1]), [v2] "+v"(v[2]), [v3] "+v"(v[3]), [v4] "+v"(v[4]), [v5] "+v"(v[5]),
          [v6] "+v"(v[6]), [v7] "+v"(v[7]), [a0] "+v"(acc[0]), [a1] "+v"(acc[1])
        : [f] "v"(coef), [c] "n"(C), [n] "n"(C + 1));
}

// v += coef * (lane C's v) for four values (two wait states at the end: a
// matrix product reads them next).
template <int C>
__device__ __forceinline__ void update4(double (&v)[4], double coef) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %[v0], %[v0], %[f]" BB_BC "v_fmac_f64_dpp %[v1], %[v1], %[f]" BB_BC
        "v_fmac_f64_dpp %[v2], %[v2], %[f]" BB_BC "v_fmac_f64_dpp %[v3], %[v3], %[f]" BB_BC
        "s_nop 1"
        : [v0] "+v"(v[0]), [v1] "+v"(v[1]), [v2] "+v"(v[2]), [v3] "+v"(v[3])
        : [f] "v"(coef), [c] "n"(C));
}

// acc += (lane C's v) * v for four values.
template <int C>
__device__ __forceinline__ void dot4(const double* v, double (&acc)[2]) {
    asm volatile(
        "s_nop 1\n\t"
        "v_fmac_f64_dpp %[a0], %[v0], %[v0]" BB_BC "v_fmac_f64_dpp %[a1], %[v1], %[v1]" BB_BC
        "v_fmac_f64_dpp %[a0], %[v2], %[v2]" BB_BC "v_fmac_f64_dpp %[a1], %[v3], %[v3]" BB_BC
        : [a0] "+v"(acc[0]), [a1] "+v"(acc[1])
        : [v0] "v"(v[0]), [v1] "v"(v[1]), [v2] "v"(v[2]), [v3] "v"(v[3]), [c] "n"(C));
}

// s += sum of (lane L .. L + 3's v) * u[0 .. 3], in two sums.
template <int L>
__device__ __forceinline__ void row_dot4(double v, const double* u, double (&s)[2]) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %[s0], %[v], %[u0] row_newbcast:%c[l0] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %[s1], %[v], %[u1] row_newbcast:%c[l1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %[s0], %[v], %[u2] row_newbcast:%c[l2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %[s1], %[v], %[u3] row_newbcast:%c[l3] row_mask:0xf bank_mask:0xf"
        : [s0] "+v"(s[0]), [s1] "+v"(s[1])
        : [v] "v"(v), [u0] "v"(u[0]), [u1] "v"(u[1]), [u2] "v"(u[2]), [u3] "v"(u[3]), [l0] "n"(L), [l1] "n"(L + 1),
          [l2] "n"(L + 2), [l3] "n"(L + 3));
}

// f(0), f(1), .. f(N - 1) with the index as a compile-time constant (the lane
// of a DPP broadcast is part of the instruction).
template <class F, int... I>
__device__ __forceinline__ void for_constants_of(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void for_constants(F f) {
    for_constants_of(f, std::make_integer_sequence<int, N>{});
}

// Sum over the four rows of 16 lanes (f = 1), or row k's value (f = 1 in row k's
// lanes, else 0), in every lane: four 4 x 4 x 4 matrix products whose k index
// is the row, one instruction where lane exchanges take a dozen.
__device__ __forceinline__ double across_rows(double f, double v) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(f, v, 0.0, 0, 0, 0);
}

// LDS words through which the leaf of a block hands its T_b column by column
// to the wave that forms it: G(l, c) at 16 c + l, tau_c, and the number of
// columns handed over since the panel began.
struct GramLds {
    double* G;                      // 256
    double* tau;                    // 16
    int* done;
};

// Factors one column tile in the registers of one wave.  Lane (g, j) =
// (lane / 16, lane % 16) holds column j: in x rows 16 i + 4 g + r (element r
// of row tile i) below the block's diagonal 16 x 16 block, in xd that block's
// rows 4 g + r (GEQRT) and in LDS at D[row + 17 j] the block itself (TS/TT:
// the rows of R1, zero below its diagonal, so that reflectors have no entries
// there).  Only row tiles clo CH .. chi CH - 1 of x can be nonzero.
//
// One pass over the rows per column: the dot products of column c with every
// column j give the reflector's norm (j = c), the products w_j that update
// the columns right of it (j > c) and its Gram column with the finished
// reflectors (j < c), which T_b needs and another wave works on meanwhile.
// Reflector tails stay unscaled; lane j keeps column j's factor
// 1 / (alpha - beta) in sc.  The update with column c and the dot products
// of column c + 1 share a loop.  Row c of the diagonal block is taken out of
// xd before column c's dot products and finished in D.
//
// What bounds it: the issue of one wave, about 2 (rows / 4) + 50 FP64
// instructions a column at five cycles each, with a chain of about 16
// dependent ones (eight cycles each) between two columns.  A column needs no
// signal from another wave and no barrier.
//
// On return D holds R on and above the diagonal (and GEQRT's unscaled tails
// below).
template <int MT>
__device__ __forceinline__ void leaf_columns(double (&x)[4 * MT], double (&xd)[4], double* D, double& sc, bool pair,
                                             int clo, int chi, const GramLds& gram, int done0) {
    constexpr int CH = MT < 4 ? MT : 4, NC = MT / CH;   // row tiles per chunk, chunks
    const int lane = threadIdx.x & 63;
    // Row R of the diagonal block, taken out of xd.
    auto take_row = [&](auto rc) {
        constexpr int R = decltype(rc)::value;
        const bool in = (here(lane) >> 4) == R / 4;
        const double v = across_rows(in ? 1.0 : 0.0, xd[R % 4]);
        xd[R % 4] = in ? 0.0 : xd[R % 4];
        return v;
    };
    double acc[2] = {0.0, 0.0};
    double a = D[17 * (lane & 15)];
    if (!pair) {
        a = take_row(std::integral_constant<int, 0>{});
        dot4<0>(xd, acc);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k)
        if (k >= clo && k < chi) {
#pragma unroll
            for (int e = 4 * CH * k; e < 4 * CH * (k + 1); e += 4) dot4<0>(x + e, acc);
        }
    sc = 0.0;
    for_constants<16>([&](auto cc) {
        constexpr int C = decltype(cc)::value;
        const int j = here(lane) & 15;
        const double dot = across_rows(1.0, acc[0] + acc[1]);
        // With nrm = sqrt(al^2 + ss) and r = 1 / nrm: beta = -sign(al) nrm,
        // tau = (beta - al) / beta = 1 + |al| r, scale = 1 / (al - beta).
        // r and the reciprocal each take one step of third order from the
        // hardware approximations (r (1 + e/2 + 3 e^2/8), y (1 + e + e^2)),
        // the second's from an approximation formed beside the first's step;
        // s0 and s1 (~ nrm) carry al's sign.
        const double al = bcast16<C, 6>(a), ss = bcast16<C, 6>(dot);
        const double tn = fma(al, al, ss), ts = copysign(tn, al), r0 = __builtin_amdgcn_rsq(tn);
        const double s0 = ts * r0;
        const double y0 = __builtin_amdgcn_rcp(al + s0);
        const double e0 = fma(-fabs(s0), r0, 1.0);
        const double r = fma(r0 * e0, fma(e0, 0.375, 0.5), r0);
        const double s1 = ts * r;
        const double e1 = fma(-(al + s1), y0, 1.0);
        double tau = fma(fabs(al), r, 1.0), scale = fma(y0, fma(e1, e1, e1), y0);
        double bt = -fma(fma(-s1, s1, tn), copysign(0.5 * r, al), s1);
        if (__builtin_amdgcn_ballot_w64(ss == 0.0) != 0) {      // zero tail: H_c = I
            asm volatile("");                                   // (a branch, not selects)
            tau = 0.0;
            scale = 0.0;
            bt = al;
        }
        const double h = fma(scale, dot, a);            // u_c . column j
        const double tj = j > C ? tau : 0.0;            // columns right of c
        const double coef = h * (-tj * scale);
        double an = 0.0;
        if constexpr (C < 15) {
            acc[0] = acc[1] = 0.0;
            an = D[C + 1 + 17 * j];
            if (!pair) {
                update4<C>(xd, coef);
                an = take_row(std::integral_constant<int, C + 1>{});
                dot4<C + 1>(xd, acc);
            }
#pragma unroll
            for (int k = 0; k < NC; ++k)
                if (k >= clo && k < chi) {
#pragma unroll
                    for (int e = 4 * CH * k; e < 4 * CH * (k + 1); e += 8) update_dot8<C>(x + e, coef, acc);
                }
        }
        // hand over G(:, c) and tau_c; LDS writes of a wave complete in order
        gram.G[16 * C + j] = sc * h;
        gram.tau[C] = tau;
        asm volatile("" ::: "memory");
        __hip_atomic_store(gram.done, done0 + C + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        asm volatile("" ::: "memory");
        D[C + 17 * j] = j == C ? bt : fma(-tj, h, a);
        sc = j == C ? scale : sc;
        a = an;
        asm volatile("" : "+v"(sc));                    // (formed here, not where it is used)
    });
}

// Forms T_b beside the leaf of block b, one column behind it, by the forward
// recurrence T(c,c) = tau_c, T(0:c-1,c) = -tau_c T(0:c-1,0:c-1) G(0:c-1,c):
// lane j (of each row of 16) holds row j of T.  Writes T(i, l) to Tb[l + 16 i].
// The leaf waits for nothing, so neither wait here can last.
__device__ __forceinline__ void form_t(const GramLds& gram, int done0, double* Tb) {
    const int lane = threadIdx.x & 63, j = lane & 15;
    double t[16];
#pragma unroll
    for (int l = 0; l < 16; ++l) t[l] = 0.0;
    for_constants<16>([&](auto cc) {
        constexpr int C = decltype(cc)::value;
        while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(
                   gram.done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < done0 + C + 1)
            __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
        const double gc = gram.G[16 * C + j], tau = gram.tau[C];
        double s[2] = {0.0, 0.0};
        // (entries of t not formed yet are zero)
        for_constants<(C + 3) / 4>([&](auto lc) {
            constexpr int L = 4 * decltype(lc)::value;
            row_dot4<L>(gc, t + L, s);
        });
        t[C] = j < C ? -tau * (s[0] + s[1]) : (j == C ? tau : 0.0);
    });
    if (lane < 16) {
#pragma unroll
        for (int l = 0; l < 16; ++l) Tb[l + 16 * j] = t[l];
    }
}

// Matrix results must not be read by a vector instruction within 19 issue
// slots of the MFMA that writes them; the compiler keeps that distance for
// its own instructions but does not look into the leaf's assembly, which x
// reaches here.
template <int N>
__device__ __forceinline__ void settle(double (&x)[N]) {
#pragma unroll
    for (int e = 0; e < N; e += 8)
        asm volatile("" : "+v"(x[e]), "+v"(x[e + 1]), "+v"(x[e + 2]), "+v"(x[e + 3]), "+v"(x[e + 4]),
                          "+v"(x[e + 5]), "+v"(x[e + 6]), "+v"(x[e + 7]));
    asm volatile("s_nop 15\n\ts_nop 7");
}

// A block U_b in LDS: element (16 i + 4 g + r, c) at 336 i + 84 g + 4 c + r.  A
// lane's four values of a row tile lie together (16-byte accesses for the
// leaf's output and for U^T X), and the rows of a column, which the record
// and U W read, spread over the banks.  T_b (T(i, l) at l + 16 i) follows.
constexpr int U_TILE = 336, U_G = 84;
__device__ __forceinline__ int u_at(int row, int col) {
    return U_TILE * (row >> 4) + U_G * ((row >> 2) & 3) + 4 * col + (row & 3);
}

// Panel of any kind (pair: TS or TT, tt: TT) and tile size.  For nb <= 128
// every column tile has its wave.  A 256-wide tile takes two rounds of eight
// column tiles (a 256 x 16 tile is half of a wave's registers): in the second,
// the first round's blocks are staged from the record just written, as an
// update does, and applied first.
//
// A wave's work is one sequence: it applies the blocks left of its column
// tile, factors the tile, and then only takes its share of the outputs.
// Barrier b of a round follows leaf b, so a block's LDS buffer is rewritten
// (two blocks later) only after every wave has finished with it.
//
// What bounds it: the chain of leaves (leaf_columns) and of the next column
// tile's applications between them.  Leaves shared by four waves, one column
// after the other through LDS and a barrier (or a counter), took 2000 cycles
// a column at nb = 128; one wave alone takes 600 to 800, and the other waves
// are free for the applications and the outputs.  Unit times in a lightly
// loaded run, before and after: nb = 32 TTQRT 17 -> 12 us, nb = 64 TSQRT
// 39 -> 27 us, nb = 128 GEQRT 86 -> 74 and TTQRT 90 -> 65 us, nb = 256 (its
// trailing tiles used to wait in scratch memory between blocks) GEQRT
// 390 -> 347 us.
template <int NB, bool CO>
__device__ __forceinline__ void panel(const KArgs& a, const DevTask& tk, double* lds, Prev& prev) {
    using S = Shape<NB>;
    constexpr int MT = S::MT, BUF = S::UBUF, NW = NT / 64;
    constexpr int HT = MT < NW ? MT : NW, NH = MT / HT; // column tiles per round, rounds
    constexpr int CH = MT < 4 ? MT : 4;
    const bool pair = tk.kind != K_GEQRT, tt = tk.kind == K_TTQRT;
    const int tid = here(threadIdx.x), lane = tid & 63, j = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool own = HT == NW || w < HT;

    const MatDesc md = mat_desc(a, tk.mat);
    const TileView T1 = view(md, tk, tk.r1, tk.c1, NB);
    const TileView TX = pair ? view(md, tk, tk.r2, tk.c2, NB) : T1;
    double* gV = record<NB>(md, tk);
    double* gTt = gV + NB * NB;
    double* Ds = lds + 2 * BUF + 272 * (w % HT);        // the wave's diagonal block, column stride 17
    double* gl = lds + 2 * BUF + 272 * HT;
    const GramLds gram{gl, gl + 256, (int*)(gl + 272)};
    if (tid == 0) *gram.done = 0;                       // (barriers follow before the first leaf)
    lds_barrier();

#pragma unroll 1
    for (int h = 0; h < NH; ++h) {
        const int ct = HT * h + w;                      // this wave's column tile
        TileLane<NB, false> l1(T1, 16 * ct), lx(TX, 16 * ct);
        d4 x[MT], R1n = {0.0, 0.0, 0.0, 0.0};
        if (own) load_slice<MT>(lx, x);
        // R1's rows are changed by the block of the same index only: the
        // diagonal block is read here, the others one block ahead.
        if (pair && own) {
            const d4 r = l1.load(16 * ct);
            if (ct > 0) R1n = l1.load(0);
#pragma unroll
            for (int k = 0; k < 4; ++k) Ds[(4 * g + k) + 17 * j] = 4 * g + k <= j ? r[k] : 0.0;
        }
        // Zeros below R (GEQRT) or in all of X2 (TS; TT: its triangle).
        auto clear = [&]() {
            const int r0 = pair ? 0 : 16 * (ct + 1), r1 = min(tt ? 16 * (ct + 1) : NB, TX.vr);
            if (TX.rs == 1) {
                // columns are contiguous: whole lines along them (the slice
                // layout would write 16 bytes of each line at a time)
                const int c1 = min(16, TX.vc - 16 * ct), ln = here(lane);
#pragma unroll 1
                for (int c = 0; c < c1; ++c)
#pragma unroll 1
                    for (int row = r0 + ln; row < r1; row += 64)
                        gstore<CO>(TX.base + row + (16 * ct + c) * TX.cs, 0.0);
            } else {
                const d4 zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
                for (int i = r0; i < r1; i += 16) lx.template store<CO, false>(i, zero);
            }
        };

        // Q_cb^T on this wave's tile, the block at U: W = R1 + U^T X,
        // W = T^T W, X -= U W, on the rows U can change.  Row tiles go in
        // pairs with a sum each, so that consecutive MFMAs are independent.
        auto apply = [&](int cb, const double* U, auto ahead) {
            constexpr bool AHEAD = decltype(ahead)::value;
            const double* Tb = U + MT * U_TILE;
            const int ln = here(lane), j = ln & 15, g = ln >> 4, pj = perm16(j);
            l1.renew();
            lx.renew();
            const d4 R1b = R1n;
            if (pair && cb + 1 < ct) R1n = l1.load(16 * (cb + 1));
            const int plo = pair ? 0 : cb / 2, phi = tt ? cb / 2 + 1 : MT / 2;
            const double* uw = U + U_G * g + 4 * pj;
            d4 Wk[2] = {R1b, {0.0, 0.0, 0.0, 0.0}};
            // AHEAD: operands of the next pair are read while this one's run
            d2 u[2][2][2];
            auto read_w = [&](int p) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        u[p & 1][k][q] = *(const d2*)(uw + U_TILE * (2 * p + k) + 2 * q);
            };
            if (AHEAD) read_w(0);
#pragma unroll
            for (int p = 0; p < MT / 2; ++p) {
                if (AHEAD && p + 1 < MT / 2) read_w(p + 1);
                if (p >= plo && p < phi) {
                    if (!AHEAD) read_w(p);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int k = 0; k < 2; ++k) Wk[k] = mfma(u[p & 1][k][r / 2][r % 2], x[2 * p + k][r], Wk[k]);
                }
                SCHED_FENCE();
            }
            const double* ux = U + U_G * (j & 3) + 16 * g + (j >> 2);
            auto read_x = [&](int p) {
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int r = 0; r < 4; ++r) u[p & 1][k][r / 2][r % 2] = ux[U_TILE * (2 * p + k) + 4 * r];
            };
            double tb[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) tb[r] = -Tb[pj + 16 * (4 * g + r)];
            if (AHEAD) read_x(0);
            const d4 W = Wk[0] + Wk[1];
            d4 W2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int r = 0; r < 4; ++r) W2 = mfma(tb[r], W[r], W2);
            if (pair) l1.template store<CO, false>(16 * cb, R1b + W2);
#pragma unroll
            for (int p = 0; p < MT / 2; ++p) {
                if (AHEAD && p + 1 < MT / 2) read_x(p + 1);
                if (p >= plo && p < phi) {
                    if (!AHEAD) read_x(p);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int k = 0; k < 2; ++k)
                            x[2 * p + k] = mfma(u[p & 1][k][r / 2][r % 2], W2[r], x[2 * p + k]);
                }
                SCHED_FENCE();
            }
            if (!pair) {                                // row tile cb is final: rows of R
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    if (i == cb) {
                        lx.template store<CO, false>(16 * i, x[i]);
                        x[i] = d4{0.0, 0.0, 0.0, 0.0};
                    }
            }
        };
        // A wave's share of block b's record, the idle waves' in turn.
        auto write_record = [&](int b) {
            const double* U = lds + (b & 1) * BUF;
            const int cb = HT * h + b, n = b + 1 + (NW - HT), k0 = w <= b ? w : w - HT + b + 1;
            const int ln = here(lane);
#pragma unroll 1
            for (int k = k0; k < NB / 4; k += n) {
                const int e = ln + 64 * k;
                gstore<CO>(gV + (int64_t)cb * 16 * NB + e, U[u_at(e % NB, e / NB)]);
            }
            if (w == b) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    gstore<CO>(gTt + 256 * cb + 64 * k + ln, U[MT * U_TILE + 64 * k + ln]);
            }
        };
        // Before barrier b: the wave two after the leaf's (on another SIMD)
        // forms T_b.
        auto meet = [&](int b) {
            if (w == ((b + 2) & (NW - 1))) form_t(gram, 16 * (HT * h + b), lds + (b & 1) * BUF + MT * U_TILE);
            lds_barrier();
        };

        if (h == 0) {
            retire(a, prev);
        } else {
            // the record's first half: every wave's stores done, then stale
            // lines dropped as at the start of a unit
            __builtin_amdgcn_s_waitcnt(0);
            lds_barrier();
            asm volatile("buffer_inv sc1" ::: "memory");
            const Rec rec(gV, NB);
            constexpr int PRE = 16 * NB / NT;
            double pre[PRE], pt = 0.0;
            const int tid = here(threadIdx.x);
            auto fetch = [&](int cb) {
#pragma unroll
                for (int k = 0; k < PRE; ++k) pre[k] = rec.ld(8 * (tid + NT * k), 8 * 16 * NB * cb);
                if (tid < 256) pt = rec.ld(8 * tid, 8 * (NB * NB + 256 * cb));
            };
            fetch(0);
#pragma unroll 1
            for (int cb = 0; cb < HT; ++cb) {
                double* U = lds + (cb & 1) * BUF;
#pragma unroll
                for (int k = 0; k < PRE; ++k) {
                    const int e = tid + NT * k;
                    U[u_at(e % NB, e / NB)] = pre[k];
                }
                if (tid < 256) U[MT * U_TILE + tid] = pt;
                if (cb + 1 < HT) fetch(cb + 1);
                lds_barrier();
                // (two waves a SIMD hide each other's operand reads, and the
                // fetched block takes the registers)
                apply(cb, U, std::false_type{});
            }
            lds_barrier();
        }
        // the tile is in registers: its zeros are stored while the first leaf
        // runs (by wave 0 after its own)
        if (own && w > 0) {
            __builtin_amdgcn_s_waitcnt(0);
            asm volatile("" ::: "memory");
            clear();
        }

#pragma unroll 1
        for (int b = 0; b < HT && b < w; ++b) {
            if (b + 1 == w) __builtin_amdgcn_s_setprio(3);      // the next leaf
            meet(b);
            if (own) apply(HT * h + b, lds + (b & 1) * BUF, std::true_type{});
            else write_record(b);
        }
        if (!own) continue;

        double xs[4 * MT], xd[4] = {0.0, 0.0, 0.0, 0.0}, sc;
        if (!pair) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
                if (i == ct) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) xd[r] = x[i][r];
                    x[i] = d4{0.0, 0.0, 0.0, 0.0};
                }
        }
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) xs[4 * i + r] = x[i][r];
        asm volatile("" : "+v"(xd[0]), "+v"(xd[1]), "+v"(xd[2]), "+v"(xd[3]));
        settle(xs);
        leaf_columns<MT>(xs, xd, Ds, sc, pair, pair ? 0 : (ct + 1) / CH, tt ? ct / CH + 1 : MT / CH, gram, 16 * ct);

        double* U = lds + (w & 1) * BUF;
        const int ln = here(lane), j = ln & 15, g = ln >> 4;
        d4 dt;                                          // the diagonal block in the tile layout
#pragma unroll
        for (int r = 0; r < 4; ++r) dt[r] = Ds[(4 * g + r) + 17 * j];
        double* uw = U + U_G * g + 4 * j;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            *(d2*)(uw + U_TILE * i) = d2{xs[4 * i] * sc, xs[4 * i + 1] * sc};
            *(d2*)(uw + U_TILE * i + 2) = d2{xs[4 * i + 2] * sc, xs[4 * i + 3] * sc};
        }
        if (!pair) {                                    // explicit unit lower triangle
            double v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 4 * g + r;
                v[r] = row > j ? dt[r] * sc : (row == j ? 1.0 : 0.0);
            }
            *(d2*)(uw + U_TILE * ct) = d2{v[0], v[1]};
            *(d2*)(uw + U_TILE * ct + 2) = d2{v[2], v[3]};
        }
        lds_barrier();
        __builtin_amdgcn_s_setprio(0);
        l1.renew();
        lx.renew();
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * g + r > j) dt[r] = 0.0;
        l1.template store<CO, false>(16 * ct, dt);                   // R (GEQRT) or R1's diagonal block
        write_record(w);
        if (w == 0) clear();
#pragma unroll 1
        for (int b = w + 1; b < HT; ++b) {
            meet(b);
            write_record(b);
        }
    }
    lds_barrier();
}

// ---------------------------------------------------------------------------
// Update kernels: UNMQR, TSMQR, TTMQR (Table 1) on a strip of the trailing
// tile (or tile pair): the whole tile for nb <= 128, a 128-column half for
// nb = 256, or (PART_NARROW, applications only) 64 columns.  Wave w owns the 16 logical columns c0 = part * NS + 16 w ..
// c0 + 15 of C2 (and C1); waves past the tile's width only stage and
// synchronize.  All nb/16 blocks of the record are applied (apply_blocks).
// ---------------------------------------------------------------------------
template <int NB, int KIND, bool CO, bool HQ>
__device__ __forceinline__ void update(const KArgs& a, const DevTask& tk, int part, double* lds, Prev& prev,
                                       int* sch) {
    constexpr int MT = NB / 16;
    constexpr bool HASC1 = KIND != K_UNMQR;
    // strip width: one 16-column slice per wave at most
    const int ns = NB < 128 ? NB : part & PART_NARROW ? 64 : 128;
    if (NB >= 128) part &= PART_NARROW - 1;
    const int tid = here(threadIdx.x), w = tid >> 6;
    const int c0 = part * ns + 16 * w;
    const MatDesc md = mat_desc(a, tk.mat);
    const TileView T2 = view(md, tk, tk.r2, tk.c2, NB);
    const TileView T1 = HASC1 ? view(md, tk, tk.r1, tk.c1, NB) : T2;
    // Waves without columns still take part in staging and barriers.
    const bool active = 16 * w < ns && c0 < T2.vc;
    const Rec rec(record<NB>(md, tk), NB);

    TileLane<NB> l1(T1, c0), l2(T2, c0);
    d4 c2[MT];
    if (active) load_slice<MT>(l2, c2);
    apply_blocks<NB, MT, KIND, CO, HQ>(rec, l1, active, &c2[0], lds, a, prev);
    if (sch != nullptr) take_next(a, sch);
    l2.renew();
    if (active) store_slice<CO, MT>(l2, c2);
}

// ---------------------------------------------------------------------------
// Updates on FP32 MFMA (v_mfma_f32_16x16x4f32), for the precision variants:
// the V/T block operands and the C operands are rounded to FP32 (RNE), each
// product accumulates in FP32, and its result is added into the FP64 tiles.
// SPLIT: every operand x is also carried as x_lo = fp32(x - x_hi) and a
// product A B is taken as A_hi B_hi + A_hi B_lo + A_lo B_hi, accumulated in
// FP32 over 16-row chunks and in FP64 across chunks.  Panels, V and T stay
// FP64 in either case.
//
// The FP32 instruction returns element r of lane l at row 4(l/16) + r (the
// FP64 one at row 4r + l/16), which is the slices' layout as it is: no row is
// permuted, and the k-step r of a 16-row block takes the rows
// {4g + r : g = 0..3}, of which lane l holds its own element r.
// ---------------------------------------------------------------------------
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma32(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float lo32(double x, float hi) { return (float)(x - (double)hi); }

template <int NB, int KIND, bool CO, bool SPLIT>
__device__ __forceinline__ void update32(const KArgs& a, const DevTask& tk, int part, double* lds, Prev& prev,
                                         int* sch) {
    constexpr int MT = NB / 16;
    constexpr int NS = NB < 128 ? NB : 128;  // strip width: one 16-column slice per wave
    constexpr int LDV = NB + 1;
    constexpr int PL = 16 * LDV + 256;        // floats per plane: V_b (NB x 16) then T_b^T
    constexpr int BUF = (SPLIT ? 2 : 1) * PL; // hi plane [, lo plane]
    constexpr int PRE = 16 * NB / NT + 1;
    constexpr bool HASC1 = KIND != K_UNMQR;
    const int tid = here(threadIdx.x), lane = tid & 63, w = tid >> 6, j = lane & 15, g = lane >> 4;
    const int c0 = part * NS + 16 * w;
    const MatDesc md = mat_desc(a, tk.mat);
    const TileView T2 = view(md, tk, tk.r2, tk.c2, NB);
    const TileView T1 = HASC1 ? view(md, tk, tk.r1, tk.c1, NB) : T2;
    const bool active = 16 * w < NS && c0 < T2.vc;
    const Rec rec(record<NB>(md, tk), NB);
    float* fl = reinterpret_cast<float*>(lds);

    auto fetch = [&](int b, double (&pre)[PRE]) {
#pragma unroll
        for (int k = 0; k < PRE - 1; ++k) pre[k] = rec.ld(8 * (tid + NT * k), 8 * (16 * b * NB));
        pre[PRE - 1] = tid < 256 ? rec.ld(8 * tid, 8 * (NB * NB + 256 * b)) : 0.0;
    };
    auto stage = [&](int b, const double (&pre)[PRE]) {
        float* hi = fl + (b & 1) * BUF;
        float* lo = hi + PL;
#pragma unroll
        for (int k = 0; k < PRE - 1; ++k) {
            const int e = tid + NT * k;
            const int at = (e % NB) + (e / NB) * LDV;
            const float h = (float)pre[k];
            hi[at] = h;
            if (SPLIT) lo[at] = lo32(pre[k], h);
        }
        if (tid < 256) {
            const float h = (float)pre[PRE - 1];
            hi[16 * LDV + tid] = h;
            if (SPLIT) lo[16 * LDV + tid] = lo32(pre[PRE - 1], h);
        }
    };
    // Product of a (16 x 4) A-fragment pair with a B-fragment given in FP64.
    auto prod = [&](float ah, float al, double bv, f4 acc) {
        const float bh = (float)bv;
        acc = mfma32(ah, bh, acc);
        if (SPLIT) {
            acc = mfma32(ah, lo32(bv, bh), acc);
            acc = mfma32(al, bh, acc);
        }
        return acc;
    };

    d4 c2[MT];
    TileLane<NB> l1(T1, c0), l2(T2, c0);
    if (active) load_slice<MT>(l2, c2);
    double pre[PRE];
    fetch(0, pre);
    retire(a, prev);
    stage(0, pre);
    d4 C1n = {0.0, 0.0, 0.0, 0.0};
    if (HASC1 && active) C1n = l1.load(0);
    lds_barrier();
#pragma unroll
    for (int b = 0; b < MT; ++b) {
        const float* Vh = fl + (b & 1) * BUF;
        const float* Vl = Vh + PL;
        const float* Th = Vh + 16 * LDV;
        const float* Tl = Vl + 16 * LDV;
        if (b + 1 < MT) fetch(b + 1, pre);
        const d4 C1b = C1n;
        if (HASC1 && active && b + 1 < MT) C1n = l1.load(16 * (b + 1));
        if (active) {
            // W = C1_b + V_b^T C2, FP64 across 16-row chunks.
            d4 W = C1b;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (KIND == K_UNMQR && i < b) continue;
                if (KIND == K_TTMQR && i > b) continue;
                f4 ch = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int at = (16 * i + 4 * g + r) + j * LDV;
                    ch = prod(Vh[at], SPLIT ? Vl[at] : 0.f, c2[i][r], ch);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) W[r] += (double)ch[r];
            }
            // W2 = T_b^T W
            f4 w2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int at = j + 16 * (4 * g + r);
                w2 = prod(Th[at], SPLIT ? Tl[at] : 0.f, W[r], w2);
            }
            d4 W2;
#pragma unroll
            for (int r = 0; r < 4; ++r) W2[r] = (double)w2[r];
            if (HASC1) l1.template store<CO>(16 * b, C1b - W2);
            // C2 -= V_b W2
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                if (KIND == K_UNMQR && i < b) continue;
                if (KIND == K_TTMQR && i > b) continue;
                f4 ch = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int at = (16 * i + j) + (4 * g + r) * LDV;
                    ch = prod(-Vh[at], SPLIT ? -Vl[at] : 0.f, W2[r], ch);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) c2[i][r] += (double)ch[r];
            }
        }
        if (b + 1 < MT) stage(b + 1, pre);
        lds_barrier();
    }
    if (sch != nullptr) take_next(a, sch);
    l2.renew();
    if (active) store_slice<CO, MT>(l2, c2);
}

// PREC: 0 = FP64 updates, 2 = FP32-MFMA updates, 3 = split-FP32 updates
// (reductions: panels and updates); PREC_APPLY = the applications of Q and
// P from finished records (FP64 updates of both directions, no panels).
// Reductions and applications are separate kernels, so that neither carries
// the register demand of the other's code.
template <int NB, bool CO, int PREC>
__device__ __forceinline__ void run_unit(const KArgs& a, int task, int part, double* lds, Prev& prev, int* sch) {
    const DevTask tk = a.tasks[task];      // task is wave-uniform: scalar loads
    if constexpr (PREC == PREC_APPLY) {
        switch (tk.kind) {
        case K_UNMQR: update<NB, K_UNMQR, CO, false>(a, tk, part, lds, prev, sch); break;
        case K_TSMQR: update<NB, K_TSMQR, CO, false>(a, tk, part, lds, prev, sch); break;
        case K_TTMQR: update<NB, K_TTMQR, CO, false>(a, tk, part, lds, prev, sch); break;
        case K_UNMQR + K_HQ: update<NB, K_UNMQR, CO, true>(a, tk, part, lds, prev, sch); break;
        case K_TSMQR + K_HQ: update<NB, K_TSMQR, CO, true>(a, tk, part, lds, prev, sch); break;
        default: update<NB, K_TTMQR, CO, true>(a, tk, part, lds, prev, sch); break;
        }
    } else {
        switch (tk.kind) {
        case K_GEQRT:
        case K_TSQRT:
        case K_TTQRT: panel<NB, CO>(a, tk, lds, prev); break;
        case K_UNMQR:
            if (PREC == 0) update<NB, K_UNMQR, CO, false>(a, tk, part, lds, prev, sch);
            else update32<NB, K_UNMQR, CO, PREC == 3>(a, tk, part, lds, prev, sch);
            break;
        case K_TSMQR:
            if (PREC == 0) update<NB, K_TSMQR, CO, false>(a, tk, part, lds, prev, sch);
            else update32<NB, K_TSMQR, CO, PREC == 3>(a, tk, part, lds, prev, sch);
            break;
        default:
            if (PREC == 0) update<NB, K_TTMQR, CO, false>(a, tk, part, lds, prev, sch);
            else update32<NB, K_TTMQR, CO, PREC == 3>(a, tk, part, lds, prev, sch);
            break;
        }
    }
    retire(a, prev);               // a kind that ran nothing
}

// A unit of a launch that mixes tile sizes: the task's own size, from its
// descriptor.
template <bool CO, int PREC>
__device__ __forceinline__ void run_unit_mixed(const KArgs& a, int task, int part, double* lds, Prev& prev,
                                               int* sch) {
    const int code = __builtin_amdgcn_readfirstlane(a.tasks[task].trans) >> 1;
    switch (code) {
    case 0: run_unit<32, CO, PREC>(a, task, part, lds, prev, sch); break;
    case 1: run_unit<64, CO, PREC>(a, task, part, lds, prev, sch); break;
    default: run_unit<128, CO, PREC>(a, task, part, lds, prev, sch); break;
    }
}

template <int NB, bool CO, int PREC>
__device__ __forceinline__ void run_any(const KArgs& a, int task, int part, double* lds, Prev& prev, int* sch) {
    if constexpr (NB == NB_MIXED) run_unit_mixed<CO, PREC>(a, task, part, lds, prev, sch);
    else run_unit<NB, CO, PREC>(a, task, part, lds, prev, sch);
}

// LDS of a kernel (doubles): the mixed kernels hold the largest size they run.
template <int NB>
constexpr int kernel_lds() { return NB == NB_MIXED ? Shape<128>::LDS : Shape<NB>::LDS; }

}  // namespace

// One launch per topological level: block b runs unit unit_base + b.
template <int NB, int PREC>
__global__ __launch_bounds__(NT) void level_kernel(KArgs a, int32_t unit_base) {
    __shared__ alignas(16) double lds[kernel_lds<NB>()];
    const int2 u = a.units[unit_base + blockIdx.x];
    Prev none{-1, 0, 0, 0, 0};
    run_any<NB, false, PREC>(a, u.x, u.y, lds, none, nullptr);
}

// Persistent scheduler.  The work units are listed in one priority order:
// the start order of a list-scheduling simulation of the task graph on the
// GPU's workgroups (most urgent ready unit first), which is topological (a
// unit's predecessors all come earlier).  Each workgroup takes the next
// position of that order (one atomic add on the ticket counter) and waits
// until the unit's task has no unfinished predecessor unit.  Tickets go only
// to running workgroups and every predecessor holds an earlier ticket, so the
// earliest unfinished ticket can always proceed: no deadlock for any grid
// size.  A finished unit is counted done only after the workgroup's next unit
// has issued its first loads (its output stores drain meanwhile), and never
// later than the workgroup's next wait on a dependency, so that argument still
// holds.  A wall-clock watchdog bounds every wait (error 3 after
// watchdog_ticks), and an error reported by any workgroup stops all of them.

template <int NB, int PREC>
__global__ __launch_bounds__(NT) void persistent_kernel(KArgs a) {
    __shared__ alignas(16) double lds[kernel_lds<NB>() + SCH_WORDS / 2];
    int* sch = (int*)(lds + kernel_lds<NB>());
    const int tid = threadIdx.x;
    Prev prev{-1, 0, 0, 0, 0};
    if (tid == 0) sch[SCH_TICKET] = -2;     // -2: no ticket taken yet
    for (;;) {
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(sch[SCH_TICKET]) == -2) take_next(a, sch);
        lds_barrier();
        // Uniform in the workgroup; readfirstlane lets the compiler see that,
        // which keeps the loop's exits uniform.
        int u = __builtin_amdgcn_readfirstlane(sch[SCH_TICKET]);
        const bool ready = __builtin_amdgcn_readfirstlane(sch[SCH_READY]) != 0;
        const uint64_t t_wait = *(const uint64_t*)(sch + SCH_TIME);
        lds_barrier();
        if (tid == 0) sch[SCH_TICKET] = -2;
        // Never wait while holding an unfinished unit: its successors may be
        // the units waited for.
        if (!ready) retire(a, prev);
        if (u < 0) break;
        if (!ready) {
            if (tid < 64) {
                const int r = wait_unit(a, u, tid);
                if (tid == 0) sch[SCH_READY] = r;
            }
            lds_barrier();
            u = __builtin_amdgcn_readfirstlane(sch[SCH_READY]);
            if (u < 0) break;
        }
        const int2 un0 = a.units[u];
        const int2 un = make_int2(__builtin_amdgcn_readfirstlane(un0.x),
                                  __builtin_amdgcn_readfirstlane(un0.y));
        // Acquire: drop stale lines of the inputs from this CU's caches and
        // this XCD's L2 (the predecessors' completion was observed above).
        // Release: a unit writes its outputs with agent-scope stores, and
        // waiting for them to complete publishes them to every XCD.  The
        // invalidation is issued without the full memory wait a fence would
        // add, which would also wait for the previous unit's stores.
        asm volatile("buffer_inv sc1" ::: "memory");
        const uint64_t t_run = a.trace != nullptr && tid == 0 ? wall_clock64() : 0;
        run_any<NB, true, PREC>(a, un.x, un.y, lds, prev, sch);
        prev.task = un.x;
        prev.ticket = u;
        prev.wait = t_wait;
        prev.run = t_run;
        prev.end = a.trace != nullptr && tid == 0 ? wall_clock64() : 0;
    }
}

#ifdef BB_KERNELS_COMMON
__global__ void init_kernel(int32_t* deps, const int32_t* ndeps, int32_t ntasks, int32_t* ctrl) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < CTRL_WORDS) ctrl[i] = 0;
    for (int t = i; t < ntasks; t += gridDim.x * blockDim.x) deps[t] = ndeps[t];
}

hipError_t launch_init(const KArgs& a, const int32_t* ndeps_init, int32_t ntasks, hipStream_t s) {
    int blocks = (ntasks + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(init_kernel, dim3(blocks), dim3(256), 0, s, a.deps, ndeps_init, ntasks, a.ctrl);
    return hipGetLastError();
}

__global__ void batch_desc_kernel(MatDesc* mats, int32_t nmats, const int64_t* gidx, const int64_t* dims,
                                  const int64_t* recoff, double* const* A, const int64_t* lda, double* vt) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nmats; i += gridDim.x * blockDim.x) {
        const int64_t g = gidx[i];
        mats[i] = MatDesc{A[g], lda[g], dims[2 * i], dims[2 * i + 1], vt + recoff[i]};
    }
}

hipError_t launch_batch_desc(MatDesc* mats, int32_t nmats, const int64_t* gidx, const int64_t* dims,
                             const int64_t* recoff, double* const* A, const int64_t* lda, double* vt,
                             hipStream_t s) {
    if (nmats <= 0) return hipSuccess;
    int blocks = (nmats + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(batch_desc_kernel, dim3(blocks), dim3(256), 0, s, mats, nmats, gidx, dims, recoff, A,
                       lda, vt);
    return hipGetLastError();
}

bool nb_supported(int nb) { return nb == 32 || nb == 64 || nb == 128 || nb == 256; }

// Workspace of bb_execute_noalloc: a file-scope device array, one copy per
// device for the life of the process.  Host code never passes the array's
// name to a kernel or a copy (on the host it is only a stand-in for the
// symbol): the device address of each device's copy is looked up once, with
// that device current, and used everywhere instead.
static __device__ __align__(256) unsigned char scratch[BB_NOALLOC_WS_MAX];

hipError_t noalloc_scratch(void** ptr, size_t* bytes) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *bytes = BB_NOALLOC_WS_MAX;
    return hipSuccess;
}

#endif  // BB_KERNELS_COMMON

// This file is compiled once per (tile size, arithmetic) pair (BB_KERNELS_NB,
// BB_KERNELS_PREC: that pair's kernels, the translation units built in
// parallel) and once for the size-independent part (BB_KERNELS_COMMON), which
// sees the launchers' declarations only and so compiles no kernel twice.
#if defined(BB_KERNELS_NB) && defined(BB_KERNELS_PREC)
template <int NB, int PREC>
hipError_t launch_level_np(const KArgs& a, int32_t unit_base, int32_t count, hipStream_t s) {
    hipLaunchKernelGGL((level_kernel<NB, PREC>), dim3(count), dim3(NT), 0, s, a, unit_base);
    return hipGetLastError();
}

template <int NB, int PREC>
hipError_t launch_persistent_np(const KArgs& a, int32_t workgroups, hipStream_t s) {
    hipLaunchKernelGGL((persistent_kernel<NB, PREC>), dim3(workgroups), dim3(NT), 0, s, a);
    return hipGetLastError();
}

template hipError_t launch_level_np<BB_KERNELS_NB, BB_KERNELS_PREC>(const KArgs&, int32_t, int32_t, hipStream_t);
template hipError_t launch_persistent_np<BB_KERNELS_NB, BB_KERNELS_PREC>(const KArgs&, int32_t, hipStream_t);
#endif

#ifdef BB_KERNELS_COMMON
#define BB_NP_CASES(F, ...)                                                        \
    switch (nb * 4 + prec) {                                                       \
    case NB_MIXED * 4 + 0: return F<NB_MIXED, 0>(__VA_ARGS__);                     \
    case NB_MIXED * 4 + 2: return F<NB_MIXED, 2>(__VA_ARGS__);                     \
    case NB_MIXED * 4 + 3: return F<NB_MIXED, 3>(__VA_ARGS__);                     \
    case 32 * 4 + 0: return F<32, 0>(__VA_ARGS__);                                 \
    case 32 * 4 + 2: return F<32, 2>(__VA_ARGS__);                                 \
    case 32 * 4 + 3: return F<32, 3>(__VA_ARGS__);                                 \
    case 64 * 4 + 0: return F<64, 0>(__VA_ARGS__);                                 \
    case 64 * 4 + 2: return F<64, 2>(__VA_ARGS__);                                 \
    case 64 * 4 + 3: return F<64, 3>(__VA_ARGS__);                                 \
    case 128 * 4 + 0: return F<128, 0>(__VA_ARGS__);                               \
    case 128 * 4 + 2: return F<128, 2>(__VA_ARGS__);                               \
    case 128 * 4 + 3: return F<128, 3>(__VA_ARGS__);                               \
    case 256 * 4 + 0: return F<256, 0>(__VA_ARGS__);                               \
    case 256 * 4 + 2: return F<256, 2>(__VA_ARGS__);                               \
    case 256 * 4 + 3: return F<256, 3>(__VA_ARGS__);                               \
    case 32 * 4 + PREC_APPLY: return F<32, PREC_APPLY>(__VA_ARGS__);               \
    case 64 * 4 + PREC_APPLY: return F<64, PREC_APPLY>(__VA_ARGS__);               \
    case 128 * 4 + PREC_APPLY: return F<128, PREC_APPLY>(__VA_ARGS__);             \
    case 256 * 4 + PREC_APPLY: return F<256, PREC_APPLY>(__VA_ARGS__);             \
    default: return hipErrorInvalidValue;                                          \
    }

hipError_t launch_level(int nb, int prec, const KArgs& a, int32_t unit_base, int32_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    BB_NP_CASES(launch_level_np, a, unit_base, count, s)
}

hipError_t launch_persistent(int nb, int prec, const KArgs& a, int32_t workgroups, hipStream_t s) {
    BB_NP_CASES(launch_persistent_np, a, workgroups, s)
}
#endif  // BB_KERNELS_COMMON

}  // namespace bbk
