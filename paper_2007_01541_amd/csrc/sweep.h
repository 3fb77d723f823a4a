// Triangular sweeps for few right-hand sides as one persistent launch.
//
// What bounds a sweep with few right-hand sides is neither memory nor
// arithmetic but the chain of dependent steps from the leaves to the root and
// back: level by level, super-block by super-block.  As separate launches
// every link of that chain costs a launch and the cold start of its kernel
// (descriptor loads, operand loads, drain), 8-12 us for work of well under
// 1 us.  Here the whole sweep is one launch of a few workgroups per compute
// unit that take tasks from a queue; a task polls for the values it needs.
// Its matrix operand does not depend on them, so it is loaded into registers
// before the wait, and a link costs about 0.6 us from a store to the poll that
// sees it and a 64-deep product.  Measured (one right-hand side, FP64): a
// solve at N = 4,096 445 -> 78 us (60 launches before), a theta step at N =
// 65,536 (solve and product) 2.40 -> 0.76 ms.
//
// Order and progress: the queue lists every task after all tasks it waits
// for, and tasks are claimed in queue order.  A workgroup runs its tasks in the
// order it claimed them and holds at most one that it has not started (the
// short kinds claim their successor first, see run), later in the queue than
// the one it runs.  The first unfinished task therefore is always being run,
// not held, and waits for nothing, so the launch finishes however few
// workgroups are resident.  Every wait is bounded all the same: a workgroup
// that polls too often raises an abort word, which ends all waits and turns
// what is published from then on into NaN, and the factor's give-up word, from
// which the host reports it.
//
// Exchanged values are written and read with relaxed device-scope atomics,
// which are coherent across the eight dies' caches, and a value is its own
// flag: everything that tasks exchange (the results and right-hand sides of
// pivot blocks, the update rows, the split partial sums) is filled with a bit
// pattern (all ones, a NaN that no task publishes) before the launch, and a
// reader polls the elements it needs until none is empty.  No task relies on
// the order in which two different stores become visible, and none waits for
// its own stores.
//
// Arithmetic: forward, a row subtracts one sum per 256-pivot super-block;
// backward, a column subtracts one sum per 256 rows; each is formed from the
// waves' partial sums, the forward solves' diagonal term last.  All orders are
// fixed, so results are deterministic; they depend on the number of right-hand
// sides through the kernel's width (1, 4 or 8 columns) alone.
#pragma once
#include "common.h"

namespace wcs {
namespace dev {

// Kinds of task.  A narrow front (at most 64 pivots) is one task for its
// pivots and the first 256 update rows, and one per further 256 update rows
// (a wave takes 64 rows and the whole contraction).  Any other front: the
// tasks along its chain (FWD_PIV, BWD_COL) take 32 pivots each, so that the
// next operand and the super-block inverse fit the registers together and a
// compute unit fetches half as much per link; its update rows are one task
// per 64 rows forward (FWD_TILE) and per 64 columns and 256 rows backward
// (BWD_PART).  A wave takes 64 of every 256 pivots or rows contracted over.
enum SweepKind { SW_FWD_TILE = 0, SW_FWD_PIV = 1, SW_FWD_FRONT = 2, SW_FWD_ROWS = 3, SW_BWD_PART = 4, SW_BWD_COL = 5, SW_BWD_FRONT = 6 };
// a task with its front's descriptors (one scalar load gives all it needs).
// idx: 32-pivot block (FWD_PIV, BWD_COL) or 64-column block (BWD_PART); r0:
// first row; [i0, i1): items or partial slots
struct SweepTask {
    int64_t foff, xoff, rptr, woff;    // elements of the front buffer and of its super-block inverses; row offsets
    int32_t m, p, first, kind;
    int32_t idx, r0, i0, i1;
};
// update rows of one child that land in a forward task's rows: first row of W, position in rel, count
struct SweepItem {
    int32_t src, rel, cnt, pad;
};

constexpr int SW_ROWS = 256;        // update rows per task
constexpr int SW_POLLS = 1 << 21;   // polls, of about a microsecond, before a wait gives up

template <typename T> struct SweepArgs {
    const SweepTask *tasks;
    const SweepItem *items;
    const int32_t *rel, *rows;
    const T *fronts, *xinv;         // forward factor
    const T *fronts_u, *xinv_u;     // backward factor (the same unless LU)
    T *W, *Y, *part;                // update rows, input and output rows, partial sums of the update rows
    T *ex;                          // exchange arrays of n x k each: z, w (forward), v, x (backward)
    int64_t nk;
    int32_t *ctl;                   // [0] queue position, [1] abort
    int32_t *gave_up;               // set to 1 when a wait gives up; cleared by the host
    int32_t polls;                  // ... after this many polls
    int32_t t0, t1, k;              // tasks [t0, t1)
    int32_t part_l, from_z;         // Y takes the forward result; the backward sweep starts from it (else from Y)
};
// every 32-bit word of what is exchanged, and of ctl, before a launch
constexpr int32_t SW_UNSET = -1;

// the fill before a launch: three ranges of n0, n1, n2 words (all 16-byte aligned)
__global__ __launch_bounds__(256) void k_sweep_fill(int32_t *p0, int64_t n0, int32_t *p1, int64_t n1, int32_t *p2,
                                                    int64_t n2)
{
    const int64_t stride = (int64_t)gridDim.x * 256, t0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
    auto fill = [&](int32_t *p, int64_t n) {
        const int4 v = make_int4(SW_UNSET, SW_UNSET, SW_UNSET, SW_UNSET);
        for (int64_t i = t0; i < n / 4; i += stride) reinterpret_cast<int4 *>(p)[i] = v;
        if (t0 < n % 4) p[n / 4 * 4 + t0] = SW_UNSET;
    };
    fill(p0, n0);
    fill(p1, n1);
    fill(p2, n2);
}

template <typename T> __device__ __forceinline__ T ld_dev(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T> __device__ __forceinline__ void st_dev(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T, int KT> struct Sweep {
    static constexpr int NEL = 64 * KT;                        // elements of a 64-row tile
    static constexpr int NE = (NEL + THREADS - 1) / THREADS;   // ... per thread
    static constexpr int MAXR = 64 + SW_ROWS;
    typedef typename Vec4<T>::type V4;

    struct Lds {
        T z[256 * KT];               // contraction operand
        T part[256 * KT];            // partial sums of the four waves
        T w[MAXR * KT];              // rows of the task
        int32_t task;                // the next task
        int32_t abort;
    };

    typedef typename std::conditional<sizeof(T) == 8, unsigned long long, unsigned int>::type Bits;
    static constexpr Bits EMPTY = ~(Bits)0;

    const SweepArgs<T> &a;
    Lds &sh;
    const int tid, wave, lane, k;
    T *const xz, *const xw, *const xx;               // exchange arrays

    __device__ __forceinline__ Sweep(const SweepArgs<T> &a_, Lds &s)
        : a(a_), sh(s), tid(threadIdx.x), wave(__builtin_amdgcn_readfirstlane(threadIdx.x / 64)),
          lane(threadIdx.x % 64), k(a_.k), xz(a_.ex), xw(a_.ex + a_.nk), xx(a_.ex + 3 * a_.nk)
    {
    }

    // Workgroup barrier after the LDS accesses issued so far.  The explicit wait
    // is needed: hipcc 7.2 drops the one that __syncthreads() implies where the
    // pending LDS write reaches the barrier over a loop's back edge (seen in the
    // generated code; with two workgroups on a compute unit waves then read the
    // previous task number).
    __device__ __forceinline__ static void sync()
    {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
    }
    __device__ __forceinline__ T *xv_() const { return a.ex + 2 * a.nk; }
    // one more poll without success: true if the wave gives up
    __device__ __forceinline__ bool stuck(int spin)
    {
        __builtin_amdgcn_s_sleep(1);
        if (spin < a.polls && ((spin & 1023) != 0 || ld_dev(a.ctl + 1) == SW_UNSET)) return false;
        st_dev(a.ctl + 1, 1);
        st_dev(a.gave_up, 1);
        sh.abort = 1;
        return true;
    }
    // what is published: never the pattern of an empty element, NaN after an abort
    __device__ __forceinline__ T out(T v) const
    {
        Bits b;
        __builtin_memcpy(&b, &v, sizeof(T));
        return (sh.abort || b == EMPTY) ? (T)__builtin_nan("") : v;
    }
    // N elements at p(q) for need(q), polled until none of the wave's is empty; 0 where not needed
    template <int N, typename NeedFn, typename PtrFn>
    __device__ __forceinline__ void poll(T (&v)[N], NeedFn need, PtrFn p)
    {
        for (int spin = 1;; spin++) {
            bool all = true;
#pragma unroll
            for (int q = 0; q < N; q++) {
                v[q] = need(q) ? ld_dev(p(q)) : (T)0;
                Bits b;
                __builtin_memcpy(&b, &v[q], sizeof(T));
                all = all && b != EMPTY;
            }
            if (__all(all) || stuck(spin)) break;
        }
    }
    // the same for rows [n0, n) alone
    __device__ __forceinline__ void stage_after(int n0, int n, const T *src)
    {
        T v[KT];
        poll(
            v, [&](int q) { int r = (tid + THREADS * q) / KT; return r >= n0 && r < n && (tid + THREADS * q) % KT < k; },
            [&](int q) { int e = tid + THREADS * q; return src + (int64_t)(e / KT) * k + e % KT; });
#pragma unroll
        for (int q = 0; q < KT; q++) sh.z[tid + THREADS * q] = v[q];
    }
    // sh.z[r KT + c] = rows [0, n) of src (row-major, k columns), polled; zero beyond and past column k
    __device__ __forceinline__ void stage(int n, const T *src)
    {
        T v[KT];
        poll(
            v, [&](int q) { int e = tid + THREADS * q; return e / KT < n && e % KT < k; },
            [&](int q) { int e = tid + THREADS * q; return src + (int64_t)(e / KT) * k + e % KT; });
#pragma unroll
        for (int q = 0; q < KT; q++) sh.z[tid + THREADS * q] = v[q];
    }
    // acc = sum_j v[j] z[z0 + STEP j].  The rows of z are read G at a time (the
    // empty asm keeps the compiler from reading all of them ahead or moving the
    // products behind the next operand's loads, both of which spill); NA sums
    // in turn, because one chain of products is latency-bound (64 dependent
    // FP64 products and their reads took 1.25 us of a 7 us link).
    template <int STEP, int N> __device__ __forceinline__ void dot(const T (&v)[N], int z0, T (&acc)[KT])
    {
        constexpr int G = KT >= 8 ? 4 : KT >= 4 ? 8 : 16, NA = KT >= 8 ? 1 : KT >= 4 ? 2 : 4;
        static_assert(N % G == 0 && G % NA == 0, "groups");
        T s[NA][KT];
#pragma unroll
        for (int i = 0; i < NA; i++)
#pragma unroll
            for (int c = 0; c < KT; c++) s[i][c] = 0;
        const T *z = sh.z + z0 * KT;
#pragma unroll
        for (int g = 0; g < N; g += G) {
#pragma unroll
            for (int j = g; j < g + G; j++)
#pragma unroll
                for (int c = 0; c < KT; c++) s[j % NA][c] += v[j] * z[STEP * j * KT + c];
#pragma unroll
            for (int i = 0; i < NA; i++)
#pragma unroll
                for (int c = 0; c < KT; c++) asm volatile("" : "+v"(s[i][c])::"memory");
        }
#pragma unroll
        for (int c = 0; c < KT; c++) {
            if constexpr (NA == 4) acc[c] = (s[0][c] + s[1][c]) + (s[2][c] + s[3][c]);
            else if constexpr (NA == 2) acc[c] = s[0][c] + s[1][c];
            else acc[c] = s[0][c];
        }
    }
    // 64 rows: the four waves' sums per (lane, column), added in wave order: element e of this thread in s[]
    __device__ __forceinline__ void reduce(const T (&acc)[KT], T (&s)[NE])
    {
#pragma unroll
        for (int c = 0; c < KT; c++) sh.part[(wave * 64 + lane) * KT + c] = acc[c];
        sync();
#pragma unroll
        for (int q = 0; q < NE; q++) {
            int e = tid + THREADS * q;
            s[q] = e < NEL ? (sh.part[e] + sh.part[NEL + e]) + (sh.part[2 * NEL + e] + sh.part[3 * NEL + e]) : (T)0;
        }
    }
    // 32 rows: the eight half-waves' sums (a lane's row is lane % 32), in order: element tid in the return value
    __device__ __forceinline__ T reduce32(const T (&acc)[KT])
    {
        constexpr int H = 32 * KT;
#pragma unroll
        for (int c = 0; c < KT; c++) sh.part[(wave * 64 + lane) * KT + c] = acc[c];
        sync();
        T s = 0;
        if (tid < H)
            s = ((sh.part[tid] + sh.part[H + tid]) + (sh.part[2 * H + tid] + sh.part[3 * H + tid])) +
                ((sh.part[4 * H + tid] + sh.part[5 * H + tid]) + (sh.part[6 * H + tid] + sh.part[7 * H + tid]));
        return s;
    }
    // Transposed products (backward).  Lane l holds rows l % 16 + 16 t (t < NT)
    // and columns 4 j + l / 16 (j < NJ) of the wave's rows of L, v[t NJ + j]: each
    // load instruction covers whole cache lines (a column per lane took four
    // times as many line accesses, 3-6 us for a super-block's inverse).
    template <int NT, int NJ>
    __device__ __forceinline__ void load_t(const T *base, int64_t ld, int nc, int r0, int lo, int hi, T (&v)[NT * NJ])
    {
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            const T *col = base + (int64_t)min(4 * j + lane / 16, nc - 1) * ld;
#pragma unroll
            for (int t = 0; t < NT; t++) v[t * NJ + j] = col[min(max(r0 + 16 * t + lane % 16, lo), hi - 1)];
        }
    }
    template <int CTRL> __device__ __forceinline__ static T dpp(T v)
    {
        if constexpr (sizeof(T) == 4) {
            return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
        } else {
            const long long b = __double_as_longlong(v);
            const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
            const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
            return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
        }
    }
    // one halving of the sums over the 16 lanes of a row: N values to N / 2, the
    // lanes with `up` keeping the second half; CTRL pairs a lane with one on the other side
    template <int CTRL, int N> __device__ __forceinline__ static void halve(T *p, bool up)
    {
#pragma unroll
        for (int i = 0; i < N / 2; i++) {
            const T give = up ? p[i] : p[i + N / 2], keep = up ? p[i + N / 2] : p[i];
            p[i] = keep + dpp<CTRL>(give);
        }
    }
    // acc[c] = sum over the wave's rows of v(row, col) z[z0 + row] for this lane's
    // column tcol(): NJ = 16, one column per lane; NJ = 8, one per pair of lanes
    template <int NT, int NJ> __device__ __forceinline__ void dot_t(const T (&v)[NT * NJ], int z0, T (&acc)[KT])
    {
        const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
#pragma unroll
        for (int c = 0; c < KT; c++) {
            T x[NT], p[NJ];
#pragma unroll
            for (int t = 0; t < NT; t++) x[t] = sh.z[(z0 + 16 * t + lane % 16) * KT + c];
#pragma unroll
            for (int j = 0; j < NJ; j++) {
                p[j] = v[j] * x[0];
#pragma unroll
                for (int t = 1; t < NT; t++) p[j] += v[t * NJ + j] * x[t];
            }
            // lane ^ 8, lane ^ 7, lane ^ 3, lane ^ 1
            halve<0x128, NJ>(p, b3);            // row_ror:8
            halve<0x141, NJ / 2>(p, b2);        // row_half_mirror
            halve<0x1B, NJ / 4>(p, b1);         // quad_perm [3,2,1,0]
            if constexpr (NJ == 16) halve<0xB1, 2>(p, b0);   // quad_perm [1,0,3,2]
            else p[0] += dpp<0xB1>(p[0]);
            acc[c] = p[0];
            asm volatile("" : "+v"(acc[c])::"memory");
        }
    }
    template <int NJ> __device__ __forceinline__ int tcol() const
    {
        const int j = NJ == 16 ? (lane & 8) + (lane & 4) + (lane & 2) + (lane & 1)
                               : (lane & 8) / 2 + (lane & 4) / 2 + (lane & 2) / 2;
        return 4 * j + lane / 16;
    }
    // the four waves' sums of the columns (NJ = 16: 64 columns, as reduce; NJ = 8: 32, element tid)
    __device__ __forceinline__ void reduce_t(const T (&acc)[KT], T (&s)[NE])
    {
        const int col = tcol<16>();
#pragma unroll
        for (int c = 0; c < KT; c++) sh.part[(wave * 64 + col) * KT + c] = acc[c];
        sync();
#pragma unroll
        for (int q = 0; q < NE; q++) {
            int e = tid + THREADS * q;
            s[q] = e < NEL ? (sh.part[e] + sh.part[NEL + e]) + (sh.part[2 * NEL + e] + sh.part[3 * NEL + e]) : (T)0;
        }
    }
    __device__ __forceinline__ T reduce_t32(const T (&acc)[KT])
    {
        constexpr int H = 32 * KT;
        const int col = tcol<8>();
        if ((lane & 1) == 0)
#pragma unroll
            for (int c = 0; c < KT; c++) sh.part[(wave * 32 + col) * KT + c] = acc[c];
        sync();
        T s = 0;
        if (tid < H) s = (sh.part[tid] + sh.part[H + tid]) + (sh.part[2 * H + tid] + sh.part[3 * H + tid]);
        return s;
    }
    // own elements (row r, column c) of the 64-row tile
    template <typename Fn> __device__ __forceinline__ void own(int nr, Fn fn)
    {
#pragma unroll
        for (int q = 0; q < NE; q++) {
            int e = tid + THREADS * q, r = e / KT, c = e % KT;
            if (e < NEL && r < nr && c < k) fn(q, r, c);
        }
    }
    // sh.w[(row - r0) KT + c] += update rows of the task's children, in their order
    __device__ __forceinline__ void add_items(const SweepTask &D)
    {
        for (int i = D.i0; i < D.i1; i++) {
            const SweepItem it = a.items[i];
            const T *src = a.W + (int64_t)it.src * k;
            for (int e0 = tid; e0 < it.cnt * KT + tid; e0 += 2 * THREADS) {
                auto need = [&](int q) { int e = e0 + THREADS * q; return e < it.cnt * KT && e % KT < k; };
                int d[2];
                T v[2];
#pragma unroll
                for (int q = 0; q < 2; q++) d[q] = need(q) ? a.rel[it.rel + (e0 + THREADS * q) / KT] - D.r0 : 0;
                poll(v, need, [&](int q) {
                    int e = e0 + THREADS * q;
                    return src + (int64_t)(e / KT) * k + e % KT;
                });
#pragma unroll
                for (int q = 0; q < 2; q++)
                    if (need(q)) sh.w[d[q] * KT + (e0 + THREADS * q) % KT] += v[q];
            }
            sync();
        }
    }

    __device__ __forceinline__ void put_z(int64_t o, T v)
    {
        st_dev(xz + o, out(v));
        if (a.part_l) st_dev(a.Y + o, out(v));
    }
    __device__ __forceinline__ void put_x(int64_t o, T v)
    {
        st_dev(xx + o, out(v));
        st_dev(a.Y + o, out(v));
    }

    // 64 update rows: minus one product per super-block of pivots
    __device__ void fwd_tile(const SweepTask &D)
    {
        const int ld = front_ld(D.m), r0 = D.r0, nr = min(64, D.m - r0), nS = (D.p + 255) / 256;
        // operands past the end of the rows or columns repeat the last one: their
        // results are not stored, or meet a zero of sh.z
        const T *L = a.fronts + D.foff + r0;
        const int lr = min(lane, nr - 1);
        T lv[64];
        auto load = [&](int S) {
            const int c0 = S * 256 + wave * 64;
#pragma unroll
            for (int j = 0; j < 64; j++) lv[j] = (L + (int64_t)min(c0 + j, D.p - 1) * ld)[lr];
        };
        load(0);
        for (int e = tid; e < NEL; e += THREADS) sh.w[e] = 0;
        sync();
        add_items(D);
        T v[NE], s[NE], acc[KT];
#pragma unroll
        for (int q = 0; q < NE; q++) v[q] = tid + THREADS * q < NEL ? sh.w[tid + THREADS * q] : (T)0;
        for (int S = 0; S < nS; S++) {
            const int s0 = S * 256;
            stage(min(256, D.p - s0), xz + (int64_t)(D.first + s0) * k);
            sync();
            dot<1>(lv, wave * 64, acc);
            if (S + 1 < nS) load(S + 1);
            reduce(acc, s);
#pragma unroll
            for (int q = 0; q < NE; q++) v[q] -= s[q];
            sync();
        }
        own(nr, [&](int q, int r, int c) { st_dev(a.W + (D.woff + r0 + r) * k + c, out(v[q])); });
    }

    // The forward solves' rows of X = L_SS^-1 end with their largest element, the
    // diagonal one.  Summed with the others, in whatever order, it is rounded
    // at every later addition; so the lanes take a zero instead (from above the
    // diagonal, where the inverse of a 64-block is zero) and the thread that
    // owns the row adds X_rr w_r last.  (Relative error of FP32 L^-1 b at N =
    // 16,384, 1, 4 and 7 right-hand sides: 8.16, 7.85 and 7.48e-8 without,
    // 6.84, 6.89 and 6.90e-8 so; the level-by-level kernels 7.04, 7.07 and
    // 7.87e-8.  Full solves take 0-1% longer at 1-4, 0-2% less at 8.)  Offset
    // in X of that zero for row r:
    __device__ __forceinline__ static int above(int r) { return r % 64 ? -1 : 256; }

    // 32 pivots: w minus one product per earlier super-block, then z = X w over
    // their own super-block.  Lane l takes row l % 32 and the columns of parity
    // l / 32; element (tid / KT, tid % KT) is this thread's.
    __device__ void fwd_piv(const SweepTask &D)
    {
        const int ld = front_ld(D.m), r0 = D.r0, nr = min(32, D.p - r0), nS = D.idx / 8, ib = D.idx % 8, s0 = nS * 256;
        const int half = lane / 32, er = tid / KT, ec = tid % KT;
        const bool mine = er < nr && ec < k;
        const T *L = a.fronts + D.foff + r0 + min(lane % 32, nr - 1);
        // the super-block's rows of X, up to its own columns (zero above its diagonal blocks)
        const int xr = ib * 32 + lane % 32, xc = min(wave, ib / 2) * 64 + half;
        const T *XS = a.xinv + D.xoff + (int64_t)nS * 256 * 256;
        const int ed = ib * 32 + min(er, 31);
        const T xd = XS[(int64_t)ed * 256 + ed];
        T lv[32], xv[32], acc[KT];
        auto load = [&](int S) {
            const T *c = L + (int64_t)(S * 256 + wave * 64 + half) * ld;
#pragma unroll
            for (int j = 0; j < 32; j++) lv[j] = c[(int64_t)(2 * j) * ld];
        };
        if (nS > 0) load(0);
        if (tid < 32 * KT) sh.w[tid] = mine ? ld_dev(a.Y + (int64_t)(D.first + r0 + er) * k + ec) : (T)0;
        sync();
        add_items(D);
        T v = tid < 32 * KT ? sh.w[tid] : (T)0;
#pragma unroll
        for (int j = 0; j < 32; j++) {
            const int c = xc + 2 * j;
            xv[j] = XS[c * 256 + xr + (c == xr ? above(xr) : 0)];
        }
        for (int S = 0; S < nS; S++) {
            stage(256, xz + (int64_t)(D.first + S * 256) * k);
            sync();
            dot<2>(lv, wave * 64 + half, acc);
            if (S + 1 < nS) load(S + 1);
            v -= reduce32(acc);
            sync();
        }
        if (mine && r0 + nr < min(D.p, s0 + 256)) st_dev(xw + (int64_t)(D.first + r0 + er) * k + ec, out(v));
        stage(ib * 32, xw + (int64_t)(D.first + s0) * k);
        sync();
        if (tid < 32 * KT) sh.z[ib * 32 * KT + tid] = mine ? v : (T)0;
        sync();
        dot<2>(xv, wave * 64 + half, acc);
        v = reduce32(acc) + xd * v;
        if (mine) put_z((int64_t)(D.first + r0 + er) * k + ec, v);
    }

    // a narrow front: its pivots and the first SW_ROWS update rows
    __device__ void fwd_front(const SweepTask &D)
    {
        const int ld = front_ld(D.m), r = D.p + wave * 64 + lane;
        T xv[16], lv[64], xd[NE];
        const T *X = a.xinv + D.xoff, *L = a.fronts + D.foff;
        const int lr = min(r, D.m - 1);
        int ln = lane;
        asm volatile("" : "+v"(ln));     // or the offsets are computed once for all tasks, and spilled
#pragma unroll
        for (int j = 0; j < 16; j++) {
            const int c = wave * 16 + j;
            xv[j] = X[c * 256 + ln + (c == ln ? above(ln) : 0)];
        }
#pragma unroll
        for (int j = 0; j < 64; j++) lv[j] = (L + (int64_t)min(j, D.p - 1) * ld)[lr];
#pragma unroll
        for (int q = 0; q < NE; q++) {
            const int e = min((tid + THREADS * q) / KT, 63);
            xd[q] = X[e * 256 + e];
        }
        for (int e = tid; e < MAXR * KT; e += THREADS) {
            int rr = e / KT, c = e % KT;
            sh.w[e] = (rr < D.p && c < k) ? ld_dev(a.Y + (int64_t)(D.first + rr) * k + c) : (T)0;
        }
        sync();
        add_items(D);
        T acc[KT], s[NE];
        for (int e = tid; e < NEL; e += THREADS) sh.z[e] = e / KT < D.p ? sh.w[e] : (T)0;
        sync();
        dot<1>(xv, wave * 16, acc);
        reduce(acc, s);
#pragma unroll
        for (int q = 0; q < NE; q++) {
            const int e = tid + THREADS * q;
            if (e < NEL) s[q] += xd[q] * sh.w[e];
        }
        own(D.p, [&](int q, int rr, int c) { put_z((int64_t)(D.first + rr) * k + c, s[q]); });
#pragma unroll
        for (int q = 0; q < NE; q++) {
            int e = tid + THREADS * q;
            if (e < NEL) sh.z[e] = e / KT < D.p ? s[q] : (T)0;
        }
        sync();
        dot<1>(lv, 0, acc);
        if (r < D.m)
#pragma unroll
            for (int c = 0; c < KT; c++)
                if (c < k) st_dev(a.W + (D.woff + r) * k + c, out(sh.w[r * KT + c] - acc[c]));
    }

    // ... and SW_ROWS further update rows from r0
    __device__ void fwd_rows(const SweepTask &D)
    {
        const int ld = front_ld(D.m), rr = wave * 64 + lane, r = D.r0 + rr;
        T lv[64], acc[KT];
        const T *L = a.fronts + D.foff;
        const int lr = min(r, D.m - 1);
#pragma unroll
        for (int j = 0; j < 64; j++) lv[j] = (L + (int64_t)min(j, D.p - 1) * ld)[lr];
        for (int e = tid; e < SW_ROWS * KT; e += THREADS) sh.w[e] = 0;
        sync();
        add_items(D);
        stage(D.p, xz + (int64_t)D.first * k);
        sync();
        dot<1>(lv, 0, acc);
        if (r < D.m)
#pragma unroll
            for (int c = 0; c < KT; c++)
                if (c < k) st_dev(a.W + (D.woff + r) * k + c, out(sh.w[rr * KT + c] - acc[c]));
    }

    // part[slot] = -L(update rows [r0, r0 + 256), 64 columns)^T x
    __device__ void bwd_part(const SweepTask &D)
    {
        const int ld = front_ld(D.m), ab = D.idx * 64, na = min(64, D.p - ab);
        T lv[64], acc[KT], s[NE], x[KT];
        load_t<4, 16>(a.fronts_u + D.foff + (int64_t)ab * ld, ld, na, D.r0 + wave * 64, D.p, D.m, lv);
        const int r = D.r0 + tid;
        const bool ok = r >= D.p && r < D.m;
        const int row = ok ? a.rows[D.rptr + r] : 0;
        poll(x, [&](int c) { return ok && c < k; }, [&](int c) { return xx + (int64_t)row * k + c; });
#pragma unroll
        for (int c = 0; c < KT; c++) sh.z[tid * KT + c] = x[c];
        sync();
        dot_t<4, 16>(lv, wave * 64, acc);
        reduce_t(acc, s);
        T *o = a.part + (int64_t)D.i0 * 64 * k;
        own(na, [&](int q, int cc, int c) { st_dev(o + cc * k + c, out(-s[q])); });
    }

    // the rows the backward sweep starts from
    __device__ __forceinline__ void start(T (&v)[NE], int nr, int64_t o)
    {
        const T *src = a.from_z ? xz : a.Y;
        auto need = [&](int q) { int e = tid + THREADS * q; return e < NEL && e / KT < nr && e % KT < k; };
        auto ptr = [&](int q) { int e = tid + THREADS * q; return src + o + (int64_t)(e / KT) * k + e % KT; };
        if (a.from_z) poll(v, need, ptr);
        else
#pragma unroll
            for (int q = 0; q < NE; q++) v[q] = need(q) ? ld_dev(ptr(q)) : (T)0;
    }

    // v += the task's partial sums, in their order
    __device__ __forceinline__ void add_parts(const SweepTask &D, int na, T (&v)[NE])
    {
        constexpr int B = 4;
        for (int i = D.i0; i < D.i1; i += B)
#pragma unroll
            for (int q = 0; q < NE; q++) {
                const int e = tid + THREADS * q;
                const bool mine = e < NEL && e / KT < na && e % KT < k;
                const T *o = a.part + (int64_t)i * 64 * k + (int64_t)(e / KT) * k + e % KT;
                T u[B];
                poll(u, [&](int b) { return mine && i + b < D.i1; }, [&](int b) { return o + (int64_t)b * 64 * k; });
#pragma unroll
                for (int b = 0; b < B; b++) v[q] += u[b];
            }
    }

    // x of 32 pivots: v = y + partial sums, minus one product per later
    // super-block, then X^T v over their own; element (tid / KT, tid % KT) is this thread's
    __device__ void bwd_col(const SweepTask &D)
    {
        const int ld = front_ld(D.m), nS = (D.p + 255) / 256;
        const int ab = D.idx * 32, na = min(32, D.p - ab), own_s = D.idx / 8, jb = D.idx % 8, s0 = own_s * 256;
        const int er = tid / KT, ec = tid % KT, nrow = min(256, D.p - s0), base = jb / 2 * 64;
        const bool mine = er < na && ec < k;
        const T *L = a.fronts_u + D.foff + (int64_t)ab * ld;
        T lv[32], xv[32], acc[KT], u[4];
        if (nS - 1 > own_s) load_t<4, 8>(L, ld, na, (nS - 1) * 256 + wave * 64, 0, D.p, lv);
        // the super-block's columns of X from their diagonal block on: wave w takes the w-th block
        load_t<4, 8>(a.xinv_u + D.xoff + (int64_t)s0 * 256 + (int64_t)(jb * 32) * 256, 256, na, base + wave * 64, 0,
                     nrow, xv);
        const int64_t o = (int64_t)(D.first + ab + er) * k + ec;
        T v[1];
        if (a.from_z) poll(v, [&](int) { return mine; }, [&](int) { return xz + o; });
        else v[0] = mine ? ld_dev(a.Y + o) : (T)0;
        const T *ps = a.part + (int64_t)D.i0 * 64 * k + (int64_t)(D.idx % 2 * 32 + er) * k + ec;
        for (int i = D.i0; i < D.i1; i += 4, ps += 4 * 64 * k) {
            poll(u, [&](int b) { return mine && i + b < D.i1; }, [&](int b) { return ps + (int64_t)b * 64 * k; });
            v[0] += (u[0] + u[1]) + (u[2] + u[3]);
        }
        for (int S = nS - 1; S > own_s; S--) {
            stage(min(256, D.p - S * 256), xx + (int64_t)(D.first + S * 256) * k);
            sync();
            dot_t<4, 8>(lv, wave * 64, acc);
            if (S - 1 > own_s) load_t<4, 8>(L, ld, na, S * 256 - 256 + wave * 64, 0, D.p, lv);
            v[0] -= reduce_t32(acc);
            sync();
        }
        if (mine && jb > 0) st_dev(xv_() + o, out(v[0]));
        // v of the rows after these 32 up to the super-block's end; zero before and beyond
        const int lo = jb * 32 - base;
        stage_after(lo + na, nrow - base, xv_() + (int64_t)(D.first + s0 + base) * k);
        sync();
        if (mine) sh.z[lo * KT + tid] = v[0];
        sync();
        dot_t<4, 8>(xv, wave * 64, acc);
        v[0] = reduce_t32(acc);
        if (mine) put_x(o, v[0]);
    }

    // a narrow front: its pivots and the first SW_ROWS update rows
    __device__ void bwd_front(const SweepTask &D)
    {
        const int ld = front_ld(D.m), r4 = D.p & ~3;
        T xv[16], lv[64], acc[KT], s[NE], v[NE], x[KT];
        load_t<4, 16>(a.fronts_u + D.foff, ld, D.p, r4 + wave * 64, min(D.p, D.m - 1), D.m, lv);
        load_t<1, 16>(a.xinv_u + D.xoff, 256, D.p, wave * 16, 0, 256, xv);
        const int r = r4 + tid;
        const bool ok = r >= D.p && r < D.m;
        const int row = ok ? a.rows[D.rptr + r] : 0;
        start(v, D.p, (int64_t)D.first * k);
        poll(x, [&](int c) { return ok && c < k; }, [&](int c) { return xx + (int64_t)row * k + c; });
#pragma unroll
        for (int c = 0; c < KT; c++) sh.z[tid * KT + c] = x[c];
        sync();
        dot_t<4, 16>(lv, wave * 64, acc);
        reduce_t(acc, s);
#pragma unroll
        for (int q = 0; q < NE; q++) v[q] -= s[q];
        add_parts(D, D.p, v);
        sync();
#pragma unroll
        for (int q = 0; q < NE; q++) {
            int e = tid + THREADS * q;
            if (e < NEL) sh.z[e] = e / KT < D.p ? v[q] : (T)0;
        }
        sync();
        dot_t<1, 16>(xv, wave * 16, acc);
        reduce_t(acc, s);
        own(D.p, [&](int q, int rr, int c) { put_x((int64_t)(D.first + rr) * k + c, s[q]); });
    }

    // the short kinds claim their successor at once (it then waits for no more
    // than this task's time); the kinds that run along a front's chain do not
    __device__ void run()
    {
        if (tid == 0) {
            sh.abort = 0;
            sh.task = claim();
        }
        for (;;) {
            sync();
            const int i = __builtin_amdgcn_readfirstlane(sh.task);
            sync();
            if (i >= a.t1) break;
            const SweepTask D = a.tasks[i];
            const bool chain = D.kind == SW_FWD_TILE || D.kind == SW_FWD_PIV || D.kind == SW_BWD_COL;
            int next = 0;
            if (tid == 0 && !chain) next = claim();
            switch (D.kind) {
            case SW_FWD_TILE: fwd_tile(D); break;
            case SW_FWD_PIV: fwd_piv(D); break;
            case SW_FWD_FRONT: fwd_front(D); break;
            case SW_FWD_ROWS: fwd_rows(D); break;
            case SW_BWD_PART: bwd_part(D); break;
            case SW_BWD_COL: bwd_col(D); break;
            default: bwd_front(D); break;
            }
            if (tid == 0) sh.task = chain ? claim() : next;
        }
    }
    __device__ __forceinline__ int claim() const { return a.t0 + 1 + atomicAdd(a.ctl, 1); }   // ctl[0] starts at SW_UNSET
};

// workgroups per compute unit that the registers of the prefetched operand allow
template <typename T, int KT> constexpr int sweep_per_cu() { return sizeof(T) == 4 && KT <= 4 ? 3 : 2; }

template <typename T, int KT>
__global__ __launch_bounds__(THREADS, (sweep_per_cu<T, KT>())) void k_sweep(SweepArgs<T> a)
{
    __shared__ typename Sweep<T, KT>::Lds sh;
    Sweep<T, KT>(a, sh).run();
}

}  // namespace dev
}  // namespace wcs
