// fk_walk.hip -- the walk kernels: every lane steps one Brownian walk at a
// time by Euler-Maruyama, accumulates the trapezoid sum of the density along
// it, detects the exit from the box and stores the exit point and the sum
// (arXiv:1709.07469, section 2.3, steps 1-4).  The Dirichlet data is read at
// the stored exit points by the reduction pass, where every lane evaluates it
// at once instead of one lane at a time inside the stepping loop.
//
// One kernel template covers FP64 and mixed precision, single problems and
// batches of problems, and the adjoint replay (which walks the same paths and
// scatters trapezoid weights instead of storing exit records).
//
// Scheduling (gfx950, wave64):
//   - persistent blocks, sized from the occupancy calculator;
//   - a wavefront's first run of consecutive walks is given by its place in
//     the launch; further runs it claims from a global counter (one atomic per
//     claim; the run shrinks as the queue drains so the last walks spread over
//     all wavefronts);
//   - lanes whose walk has ended are refilled at macro-step boundaries, where
//     every active lane is at the start of a Philox block triple: FP64 walks
//     take 2 steps (6 normals = 3 blocks), mixed walks take 4 steps
//     (12 normals = 3 blocks) per macro-step; a wavefront whose walks end
//     often waits for several idle lanes and starts their walks together;
//   - a macro-step in which no walk of the wavefront ends runs its steps as
//     straight-line code;
//   - drain rounds: once the queue is empty, all 64 lanes of a wavefront
//     generate Philox blocks and normals for its remaining live walks into
//     LDS (any lane can compute any walk's block, the generator being
//     counter based) -- up to 128 (FP64) or 256 (mixed) steps per round for a
//     lone walk.  With few live walks the whole round is shared by the lanes
//     (coop_round below): only the chains of positions run step after step,
//     one lane per walk and axis, while densities and exit tests are taken
//     for all steps at once.  The longest walks decide when a launch ends;
//   - a launch of fewer walks than lanes gives every resident wavefront the
//     same few walks (Queue::cap) instead of filling wavefronts one by one,
//     and works in drain rounds from its start;
//   - a walk's record is written to its own slot (task index), so the result
//     does not depend on which lane or wavefront ran it, nor on the mode.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fk_stats.hpp"

namespace fk {

namespace {

constexpr int kMaxWaves = 4;        // 256 threads per block at most

// The task queue can be split into contiguous stripes with a claim counter
// each (the queue slot of a workspace holds kMaxStripes counters).  Block b
// starts on stripe b mod stripes -- consecutive blocks are placed on the 8
// XCDs in turn, so with 8 stripes each XCD walks its own contiguous range of
// tasks and, in a batch of problems with separate sources, its wavefronts
// hold walks of one problem at a time (the problem-uniform fast path applies,
// and an XCD's L2 serves one problem's grid) -- and a wavefront whose stripe
// runs out takes the next.  The launch settings choose the count: 8 for
// batches of separate sources, 1 for other launches (their lanes share a
// source anyway, and stripes that end on long walks lengthen the drain).
constexpr uint32_t kMaxStripes = 32;

// Blocks b < n of a launch with b mod m = r.
__host__ __device__ inline uint32_t blocks_of(uint32_t n, uint32_t m, uint32_t r)
{
    return (n + m - 1u - r) / m;
}

// per_block: tasks of the first runs of a block's wavefronts
__global__ void zero_queue_kernel(unsigned long long* q, uint32_t grid, uint32_t stripes, uint32_t per_block,
                                  uint32_t* status, uint32_t flags)
{
    const uint32_t s = threadIdx.x;
    if (s < kMaxStripes) q[s] = s < stripes ? (unsigned long long)blocks_of(grid, stripes, s) * per_block : 0ull;
    if (status && threadIdx.x == 0) *status = flags;
}

__device__ __forceinline__ uint64_t first_lane_u64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// The value lane l (the same for the whole wavefront) holds.
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ double lane_value(double v, int l)
{
    return __longlong_as_double((long long)lane_u64((uint64_t)__double_as_longlong(v), l));
}
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-uniform claim state over the striped task queue.  Claims of one counter
// are served one after the other, some 35 ns each, so a launch's wavefronts
// take their first run of tasks by their place in it (start_pool), and the
// counters, set past those runs, give out the rest.  A capped launch (cap < 64)
// has no more tasks than first runs, and claims none: with a claim each at the
// start and a failing one at the end, 2000 wavefronts of one short walk spent
// 4/5 of the launch on them.
struct Queue {
    unsigned long long* counter;   // one claim counter per stripe
    uint64_t n_tasks;
    uint32_t grab;
    uint32_t total_waves;
    uint32_t stripes;              // 1 .. kMaxStripes
    uint32_t refill_cost;          // 128 R of the refill rule below
    uint32_t cap;                  // most live walks of a wavefront (1 .. 64)
};

struct Pool {
    uint64_t next, end, left;
    bool exhausted;
    uint32_t stripe, tried;
    uint64_t rounds;    // refill calls (one per macro-step or drain round)
    int64_t started;    // walks started after the first fill
};

// RUNS: with a first run, of as many tasks as the wavefront may hold.
template <bool RUNS>
__device__ __forceinline__ Pool start_pool(const Queue& Q)
{
    const uint32_t stripe = blockIdx.x % Q.stripes;
    Pool pool{0ull, 0ull, Q.n_tasks, false, stripe, 0u, 0ull, -64};
    if constexpr (RUNS) {
        // the wavefront's place among those of its stripe
        const uint32_t waves = blockDim.x / 64;
        uint64_t place = (uint64_t)(blockIdx.x / Q.stripes) * waves + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
        uint64_t lo = Q.n_tasks * stripe / Q.stripes, hi = Q.n_tasks * (stripe + 1) / Q.stripes;
        if (Q.cap < 64u) {              // the tasks in equal runs, the stripes' wavefronts in order
            for (uint32_t s = 0; s < stripe; ++s) place += (uint64_t)blocks_of(gridDim.x, Q.stripes, s) * waves;
            lo = 0ull;
            hi = Q.n_tasks;
            pool.exhausted = true;
        }
        lo += place * Q.cap;
        pool.next = lo < hi ? lo : hi;
        pool.end = lo + Q.cap < hi ? lo + Q.cap : hi;
        const uint64_t runs = (uint64_t)Q.total_waves * Q.cap;
        pool.left = runs < Q.n_tasks ? Q.n_tasks - runs : 0ull;
    }
    return pool;
}

// Starting walks costs the wavefront about half a macro-step however many
// lanes take one (the set-up code runs once for all of them), while a lane
// left idle loses its share of every macro-step.  With walks ending at a rate
// of lambda per macro-step, waiting for k idle lanes costs (k - 1)/(128 lambda)
// + R/k macro-steps per walk (R = 1/2 the set-up), least for the smallest k
// with k (k + 1) >= 128 R lambda.  lambda is the wavefront's own count of
// walks started over its macro-steps so far: long walks (rare ends) refill
// every lane at once, short ones wait for several.  The launch settings give
// 128 R (default 64: R = 1/2; R = 1/4 measured the same).

// Refills idle lanes from the wavefront's claimed run, claiming a new run
// from its stripe when it is empty (and moving to the next stripe when that
// one is used up).  Returns the task of this lane if it was idle and got
// one, else ~0.  Called by the whole wavefront once per macro-step.
__device__ __forceinline__ uint64_t refill(Pool& pool, const Queue& Q, bool active)
{
    pool.rounds += 1;
    const uint64_t idle = __ballot(!active);
    const uint32_t live = 64u - (uint32_t)__popcll(idle);
    if (live >= Q.cap) return ~0ull;
    const uint32_t n_idle = Q.cap - live;
    // an all-idle wavefront always passes: started <= 64 rounds
    if (!pool.exhausted && pool.started > 0 &&
        (uint64_t)n_idle * (n_idle + 1) * pool.rounds < (uint64_t)Q.refill_cost * (uint64_t)pool.started)
        return ~0ull;
    const uint32_t stripes = Q.stripes;
    // each pass claims a run or uses up one stripe: stripes passes at most
    for (uint32_t pass = 0; pass < stripes && pool.next == pool.end && !pool.exhausted; ++pass) {
        const uint64_t lo = Q.n_tasks * pool.stripe / stripes;
        const uint64_t hi = Q.n_tasks * (pool.stripe + 1) / stripes;
        uint64_t want = pool.left / (4ull * Q.total_waves);
        if (want < n_idle) want = n_idle;
        if (want > (uint64_t)Q.grab) want = (uint64_t)Q.grab;
        unsigned long long old = 0ull;
        if (__lane_id() == 0) old = atomicAdd(Q.counter + pool.stripe, (unsigned long long)want);
        old = first_lane_u64(__shfl(old, 0));
        if (old < hi - lo) {
            pool.next = lo + old;
            pool.end = lo + old + want < hi ? lo + old + want : hi;
            pool.left = (hi - pool.end) * stripes;   // the whole queue's, estimated
        } else if (stripes == 1 || ++pool.tried == stripes) {
            pool.exhausted = true;
        } else {
            pool.stripe = (pool.stripe + 1) % stripes;
        }
    }
    const uint64_t avail = pool.end - pool.next;
    const uint32_t rank = (uint32_t)__popcll(idle & __lanemask_lt());
    uint64_t mine = ~0ull;
    const uint64_t taken = (n_idle < avail) ? n_idle : avail;
    if (!active && rank < taken) mine = pool.next + rank;
    pool.next += taken;
    pool.started += (int64_t)taken;
    return mine;
}

struct TaskInfo {
    double x0[3];
    uint64_t s;      // station
    uint32_t w;      // 0: the walk from x0 (+h e_z for g_z), 1: from x0 - h e_z
    uint32_t sctr;   // station word of the Philox counter
    uint32_t pctr;   // path word
};

// Local task t of a problem: (station s, local path i, walk w) with
// t = (s * N + i) * npair + w.
__device__ __forceinline__ TaskInfo decode(const WalkCommon& C, uint64_t t)
{
    TaskInfo ti;
    const uint64_t q = (C.npair == 2) ? (t >> 1) : t;
    const uint32_t w = (C.npair == 2) ? (uint32_t)(t & 1ull) : 0u;
    const uint64_t s = q / (uint64_t)C.N;
    const uint64_t i = q - s * (uint64_t)C.N;
    const double* st = C.stations + 3 * s;
    ti.x0[0] = st[0];
    ti.x0[1] = st[1];
    ti.x0[2] = st[2];
    if (C.npair == 2) ti.x0[2] = (w == 0) ? st[2] + C.h : st[2] - C.h;
    ti.sctr = (C.npair == 2 && C.pairing == FK_PAIR_INDEPENDENT) ? (uint32_t)(2 * s + w) : (uint32_t)s;
    ti.pctr = (uint32_t)((uint64_t)C.path_offset + i);
    ti.s = s;
    ti.w = w;
    return ti;
}

__device__ __forceinline__ bool strictly_inside(const WalkCommon& C, const double x[3])
{
    if (C.domain == FK_DOMAIN_BALL) return dist2(x[0], x[1], x[2], C.ctr[0], C.ctr[1], C.ctr[2]) < C.r2;
    return (x[0] > C.lo[0]) & (x[0] < C.hi[0]) & (x[1] > C.lo[1]) & (x[1] < C.hi[1]) & (x[2] > C.lo[2]) &
           (x[2] < C.hi[2]);
}

// Adjoint replay: a walk whose sample (or pair) the forward solve excluded
// is skipped.
__device__ __forceinline__ bool forward_capped(const WalkCommon& C, uint64_t t)
{
    if (C.npair == 2) {
        const uint64_t j = t & ~1ull;
        return ((C.fwd_steps[j] | C.fwd_steps[j + 1]) & kCapFlag) != 0;
    }
    return (C.fwd_steps[t] & kCapFlag) != 0;
}

// The adjoint's signed trapezoid weights are gathered in a block-shared LDS
// table before they reach the global int64 counts.  A walk crosses a voxel
// face on most steps of a fine grid, and every global atomic on device memory
// is performed at the memory side (hundreds of cycles, limited in flight), so
// the walks of a block -- which start from the same stations and crowd the
// same voxels -- first add into the table.  Each slot is one 32-bit word,
// (index + 1) << 11 | 11-bit signed count, updated by compare-and-swap only,
// so it is atomic across the block's wavefronts; a different index evicts the
// slot's entry to the global counts, a count that would leave +-1024 goes
// there as well, and so does every weight whose index + 1 needs more than 21
// bits or whose size is 1024 or more.  The table is flushed when the block's
// walks are done.  Integer sums in any order: the counts are exact and the
// same as without the table.
constexpr int kAdjTableBits = 13;
constexpr int kAdjSlots = 1 << kAdjTableBits;    // 32 KiB of LDS per block
constexpr int kAdjCountBits = 11;
constexpr uint32_t kAdjKeyLimit = 1u << (32 - kAdjCountBits);
constexpr int64_t kAdjBound = 1ll << (kAdjCountBits - 1);

__device__ __forceinline__ void global_add(int64_t* counts, int64_t idx, int64_t w)
{
    atomicAdd(reinterpret_cast<unsigned long long*>(counts + idx), (unsigned long long)w);
}

// The key (index + 1, 0 = empty) and the signed count of a table word.
__device__ __forceinline__ uint32_t adj_key(uint32_t e) { return e >> kAdjCountBits; }
__device__ __forceinline__ int64_t adj_count(uint32_t e)
{
    return (int64_t)((int32_t)(e << (32 - kAdjCountBits)) >> (32 - kAdjCountBits));
}

__device__ __forceinline__ void adj_emit(uint32_t* tab, int64_t* counts, int64_t idx, int64_t w)
{
    if ((uint64_t)idx + 1 >= kAdjKeyLimit || w >= kAdjBound || w <= -kAdjBound) {
        global_add(counts, idx, w);
        return;
    }
    const uint32_t k1 = (uint32_t)idx + 1u;
    const uint32_t slot = ((uint32_t)idx * 2654435761u) >> (32 - kAdjTableBits);
    uint32_t cur = __hip_atomic_load(&tab[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    for (;;) {
        const uint32_t ck = adj_key(cur);
        const int64_t cc = adj_count(cur);
        int64_t keep = w, out_idx = -1, out_c = 0;   // out: what leaves the table if this swap wins
        if (ck == k1) {
            keep = cc + w;
            if (keep >= kAdjBound || keep <= -kAdjBound) {
                out_idx = idx;
                out_c = keep;
                keep = 0;
            }
        } else if (ck != 0) {
            out_idx = (int64_t)ck - 1;
            out_c = cc;
        }
        const uint32_t want = (k1 << kAdjCountBits) | ((uint32_t)keep & ((1u << kAdjCountBits) - 1u));
        const uint32_t prev = atomicCAS(&tab[slot], cur, want);
        if (prev == cur) {
            if (out_c != 0) global_add(counts, out_idx, out_c);
            return;
        }
        cur = prev;
    }
}

// Dense station tables: when a grid has at most kDenseVoxels voxels, each
// block of the adjoint works on one station at a time and adds its walks'
// weights into a plain int32 count per voxel in LDS (128 KiB: an LDS atomic
// add, no key, no eviction), flushed to the global counts when the block
// moves on to another station.  A weight of 2^19 or more goes straight to
// the global counts; a count that reaches +-2^30 is taken out of the table by
// an atomic exchange and moved there too (concurrent adds of the block's
// 1024 threads, each below 2^19, cannot carry it past 2^31 meanwhile).
constexpr int kDenseVoxels = (int)kAdjDenseVoxels;
constexpr int64_t kDenseDirect = 1ll << 19;
constexpr int64_t kDenseLimit = 1ll << 30;
static_assert(kAdjDenseBlock * kDenseDirect + kDenseLimit < (1ll << 31), "a dense count must stay within int32");

__device__ __forceinline__ void dense_emit(int* tab, int64_t* counts, int64_t row, int64_t v, int64_t w)
{
    if (w >= kDenseDirect || w <= -kDenseDirect) {
        global_add(counts, row + v, w);
        return;
    }
    const int old = atomicAdd(&tab[v], (int)w);
    const int64_t now = (int64_t)old + w;
    if (now >= kDenseLimit || now <= -kDenseLimit) global_add(counts, row + v, (int64_t)atomicExch(&tab[v], 0));
}

// Run-length coalesced scatter of one walk's signed trapezoid weights, into
// the block's hashed table or (DENSE) its dense station table.
template <bool DENSE>
struct Scatter {
    int64_t* counts;            // the problem's counts
    void* tab;                  // the block's table
    int64_t row;                // station offset into counts
    int64_t v;                  // pending voxel (-1: none)
    int64_t c;                  // pending weight
    int64_t sign;
    __device__ __forceinline__ void flush()
    {
        if (v >= 0 && c != 0) {
            if constexpr (DENSE)
                dense_emit(static_cast<int*>(tab), counts, row, v, c);
            else
                adj_emit(static_cast<uint32_t*>(tab), counts, row + v, c);
        }
        c = 0;
    }
    __device__ __forceinline__ void add(int64_t voxel, int64_t weight)
    {
        if (voxel != v) {
            flush();
            v = voxel;
        }
        c += sign * weight;
    }
};

// The launch's one generator key, in scalar registers and, by the empty asm's
// dependence on the round's number, a new value in every round: the ten
// rounds' keys are then scalar additions of every macro-step (the scalar unit
// is idle) instead of twenty values kept over the whole loop, which overflow
// the scalar registers and come back through VALU lane reads, 16 to 20 a
// macro-step.  Mixed batches hold the twenty without spilling and are 1.5 %
// faster so (the 32-model batch).
__device__ __forceinline__ void scalar_key(uint32_t& key0, uint32_t& key1, uint64_t round)
{
    asm("" : "+s"(key0), "+s"(key1) : "s"((uint32_t)round));
}

// ---------------------------------------------------------------------------
// Precision traits.
// ---------------------------------------------------------------------------
template <bool F64>
struct Prec;

// x, from here on held in a vector register (an empty asm with a vector
// operand: no instruction is emitted)
template <class T>
__device__ __forceinline__ T in_vgpr(T x)
{
    asm("" : "+v"(x));
    return x;
}

template <>
struct Prec<true> {
    using T = double;
    using Src = SourceF64;
    static constexpr int kNormals = 2;   // per Philox block
    static constexpr int kMacro = 2;     // steps per 3 blocks
    __device__ static void normals(const Block& b, T* z, const BmTables* t) { normals_f64(b, *t, z[0], z[1]); }
    __device__ static T fmat(T a, T b, T c) { return fma(a, b, c); }
    template <bool LEVELS>
    __device__ static GridProbe grid_fetch(const Src& s, T x, T y, T z) { return grid_fetch_f64<LEVELS>(s, x, y, z); }
    template <bool LEVELS>
    __device__ static T grid_keep(const Src& s, const GridProbe& p) { return grid_keep_f64<LEVELS>(s, p); }
    __device__ static int64_t voxel(const Src& s, T x, T y, T z) { return voxel_f64(s, x, y, z); }
    __device__ static T lo(const WalkCommon& C, int c) { return C.lo[c]; }
    __device__ static T hi(const WalkCommon& C, int c) { return C.hi[c]; }
    __device__ static T ctr(const WalkCommon& C, int c) { return C.ctr[c]; }
    __device__ static T r2(const WalkCommon& C) { return C.r2; }
    __device__ static T radius(const WalkCommon& C) { return C.R; }
    __device__ static T dt(const WalkCommon& C) { return C.dt; }
    __device__ static T delta(const WalkCommon& C) { return C.delta; }
    __device__ static T deep2(const WalkCommon& C) { return C.deep2; }
    __device__ static T uniform(const Block& b, int j)
    {
        const uint32_t hi = j ? b.w3 : b.w1, lo = j ? b.w2 : b.w0;
        return uniform53(hi, lo);
    }
    __device__ static T sdt(const WalkCommon& C) { return C.sdt; }
};

template <>
struct Prec<false> {
    using T = float;
    using Src = SourceF32;
    static constexpr int kNormals = 4;
    static constexpr int kMacro = 4;
    __device__ static void normals(const Block& b, T* z, const BmTables*)
    {
        normals_f32(b.w0, b.w1, z[0], z[1]);
        normals_f32(b.w2, b.w3, z[2], z[3]);
    }
    __device__ static T fmat(T a, T b, T c) { return fmaf(a, b, c); }
    template <bool LEVELS>
    __device__ static GridProbe grid_fetch(const Src& s, T x, T y, T z) { return grid_fetch_f32<LEVELS>(s, x, y, z); }
    template <bool LEVELS>
    __device__ static T grid_keep(const Src& s, const GridProbe& p) { return grid_keep_f32<LEVELS>(s, p); }
    __device__ static int64_t voxel(const Src& s, T x, T y, T z) { return voxel_f32(s, x, y, z); }
    __device__ static T lo(const WalkCommon& C, int c) { return C.lo_f[c]; }
    __device__ static T hi(const WalkCommon& C, int c) { return C.hi_f[c]; }
    __device__ static T ctr(const WalkCommon& C, int c) { return C.ctr_f[c]; }
    __device__ static T r2(const WalkCommon& C) { return C.r2_f; }
    __device__ static T radius(const WalkCommon& C) { return C.R_f; }
    __device__ static T dt(const WalkCommon& C) { return C.dt_f; }
    __device__ static T delta(const WalkCommon& C) { return C.delta_f; }
    __device__ static T deep2(const WalkCommon& C) { return C.deep2_f; }
    __device__ static T uniform(const Block& b, int j)
    {
        const uint32_t w = j == 0 ? b.w0 : j == 1 ? b.w1 : j == 2 ? b.w2 : b.w3;
        return uniform24(w);
    }
    __device__ static T sdt(const WalkCommon& C) { return C.sdt_f; }
};

template <bool F64>
struct SourceOf;
template <>
struct SourceOf<true> {
    __device__ static const SourceF64& get(const BatchDesc& D) { return D.s64; }
};
template <>
struct SourceOf<false> {
    __device__ static const SourceF32& get(const BatchDesc& D) { return D.s32; }
};

// The batch's shared source, in the kernel arguments.
template <bool F64>
__device__ __forceinline__ const typename std::conditional<F64, SourceF64, SourceF32>::type& shared_source(
    const BatchArgs& A)
{
    if constexpr (F64)
        return A.src64;
    else
        return A.src32;
}

// The lanes' common source when every live lane of the wavefront points at
// the same one (a wavefront claims consecutive walks, so it almost always
// works on one problem), re-addressed through the constant address space so
// that its fields load with scalar instructions into scalar registers; null
// when the lanes' problems differ.  Called with only the live lanes active.
template <class Src>
__device__ __forceinline__ const Src* wave_uniform(const Src* p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    const uint64_t f = ((uint64_t)hi << 32) | lo;
    if (!__all(a == f)) return nullptr;
    return (const Src*)(const __attribute__((address_space(4))) Src*)f;
}

// Stepping parameters of the problem a lane is walking.  In single-problem
// launches they are the same for every lane; in a batch each lane loads its
// problem's at the start of a walk.
template <bool F64>
struct LaneProblem {
    using T = typename Prec<F64>::T;
    const WalkCommon* C;
    const typename Prec<F64>::Src* src;
    T sdt;
    // box domain: the bounds; ball domain: (lo0, lo1, lo2) = centre,
    // hi0 = squared radius, hi1 = radius, hi2 = (R - delta)^2 (the two never
    // coexist, so they share registers)
    T lo0, lo1, lo2, hi0, hi1, hi2;
    T dt, delta;               // Brownian-bridge test
    bool ball, bridge;
    uint32_t key0, key1, pid;
    uint32_t max_steps;        // at most 2^31 - 1

    // keys = false leaves key0 and key1 as they are (a batch whose problems
    // share the generator key holds it in scalar registers, set once).
    __device__ __forceinline__ void load(const WalkCommon& c, const typename Prec<F64>::Src& s, bool keys = true)
    {
        C = &c;
        src = &s;
        sdt = Prec<F64>::sdt(c);
        lo0 = Prec<F64>::lo(c, 0);
        lo1 = Prec<F64>::lo(c, 1);
        lo2 = Prec<F64>::lo(c, 2);
        hi0 = Prec<F64>::hi(c, 0);
        hi1 = Prec<F64>::hi(c, 1);
        hi2 = Prec<F64>::hi(c, 2);
        ball = c.domain == FK_DOMAIN_BALL;
        bridge = c.exit_rule == FK_EXIT_BRIDGE;
        dt = Prec<F64>::dt(c);
        delta = Prec<F64>::delta(c);
        if (ball) {
            lo0 = Prec<F64>::ctr(c, 0);
            lo1 = Prec<F64>::ctr(c, 1);
            lo2 = Prec<F64>::ctr(c, 2);
            hi0 = Prec<F64>::r2(c);
            hi1 = Prec<F64>::radius(c);
            hi2 = Prec<F64>::deep2(c);
        }
        if (keys) {
            key0 = c.key0;
            key1 = c.key1;
        }
        pid = c.problem_id;
        max_steps = (uint32_t)c.max_steps;
    }

    // Takes lane l's problem (the same in every lane afterwards).
    __device__ __forceinline__ void from_lane(const LaneProblem& o, int l, bool keys)
    {
        C = (const WalkCommon*)lane_u64((uint64_t)o.C, l);
        src = (const typename Prec<F64>::Src*)lane_u64((uint64_t)o.src, l);
        sdt = lane_value(o.sdt, l);
        lo0 = lane_value(o.lo0, l);
        lo1 = lane_value(o.lo1, l);
        lo2 = lane_value(o.lo2, l);
        hi0 = lane_value(o.hi0, l);
        hi1 = lane_value(o.hi1, l);
        hi2 = lane_value(o.hi2, l);
        dt = lane_value(o.dt, l);
        delta = lane_value(o.delta, l);
        ball = __builtin_amdgcn_readlane((int)o.ball, l) != 0;
        bridge = __builtin_amdgcn_readlane((int)o.bridge, l) != 0;
        if (keys) {
            key0 = (uint32_t)__builtin_amdgcn_readlane((int)o.key0, l);
            key1 = (uint32_t)__builtin_amdgcn_readlane((int)o.key1, l);
        }
        pid = (uint32_t)__builtin_amdgcn_readlane((int)o.pid, l);
        max_steps = (uint32_t)__builtin_amdgcn_readlane((int)o.max_steps, l);
    }
};

// The stepping loop a kernel instance is built for.  Bits 0-1: 0 = the box
// domain's loop with the step-end exit test only; 1 = with the ball domain's
// exit test; 2 = also with the Brownian-bridge test.  Bit 2: the density
// source has a voxel grid, whose values each macro-step loads ahead; bit 3
// (with bit 2): the grids are given by levels (an index grid and its
// densities); bit 4 (with bit 2, box exit test only): every problem has a grid
// that covers its box (Walker::covered).  A launch uses the least general loop
// its problems need.
constexpr int kLoopGrid = 4;
constexpr int kLoopLevels = 8;
constexpr int kLoopCover = 16;
constexpr int loop_exit(int loop) { return loop & 3; }
constexpr bool loop_grid(int loop) { return (loop & kLoopGrid) != 0; }
constexpr bool loop_levels(int loop) { return (loop & kLoopLevels) != 0; }
constexpr bool loop_cover(int loop) { return (loop & kLoopCover) != 0; }

// One lane's walk.
template <bool F64, bool KAHAN, bool ADJ, int LOOP, bool DENSE = false>
struct Walker {
    using T = typename Prec<F64>::T;
    uint64_t rec;    // the walk's record slot (its task minus the launch's first task)
    ExitRecord* exits;
    uint32_t* steps_out;
    T x0, x1, x2;
    double S;        // sum of densities (add_density), FP64 accumulation
    float Sf, Sc;    // or Kahan sum and compensation
    uint32_t n, k, sctr, pctr;
    bool active;
    bool deep;       // the current point lies delta inside every face (bridge test)
    Scatter<DENSE> sc;

    // delta inside every face (ball: |x - c|^2 <= (R - delta)^2)
    __device__ __forceinline__ static bool deep_inside(const LaneProblem<F64>& P, T y0, T y1, T y2, T d2)
    {
        if (P.ball) return d2 <= P.hi2;
        return y0 - P.lo0 >= P.delta && P.hi0 - y0 >= P.delta && y1 - P.lo1 >= P.delta && P.hi1 - y1 >= P.delta &&
               y2 - P.lo2 >= P.delta && P.hi2 - y2 >= P.delta;
    }

    // Brownian-bridge test of step m of the walk with counter words pctr and
    // sctr, from (x0, x1, x2) to y (both inside): returns the face the walk stopped at (0..5; 6 = the sphere) or -1.
    __device__ __forceinline__ static int bridge_stop(const LaneProblem<F64>& P, uint32_t pctr, uint32_t sctr,
                                                      uint32_t m, T x0, T x1, T x2, T y0, T y1, T y2)
    {
        constexpr int q = Prec<F64>::kNormals;
        const Block b = philox10(0x80000000u + m / q, pctr, sctr, P.pid, P.key0, P.key1);
        const T U = Prec<F64>::uniform(b, (int)(m % q));
        if (P.ball) {
            const T a = P.hi1 - sqrt(dist2(x0, x1, x2, P.lo0, P.lo1, P.lo2));
            const T c = P.hi1 - sqrt(dist2(y0, y1, y2, P.lo0, P.lo1, P.lo2));
            const T p = exp(T(-2) * a * c / P.dt);
            return U <= p ? 6 : -1;
        }
        const T lo[3] = {P.lo0, P.lo1, P.lo2}, hi[3] = {P.hi0, P.hi1, P.hi2};
        const T x[3] = {x0, x1, x2}, y[3] = {y0, y1, y2};
        T keep = T(1), pbest = T(-1);
        int fbest = 0;
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int j = f >> 1;
            const T a = (f & 1) ? hi[j] - x[j] : x[j] - lo[j];
            const T c = (f & 1) ? hi[j] - y[j] : y[j] - lo[j];
            const T p = exp(T(-2) * a * c / P.dt);
            keep *= T(1) - p;
            if (p > pbest) {
                pbest = p;
                fbest = f;
            }
        }
        return U <= T(1) - keep ? fbest : -1;
    }

    // Turns the normals of the next MACRO steps into the points those steps
    // reach (as if none ended the walk).  Points past the walk's end are never
    // used.
    __device__ __forceinline__ void advance(const LaneProblem<F64>& P, T* z) const
    {
        T p0 = x0, p1 = x1, p2 = x2;
#pragma unroll
        for (int s = 0; s < Prec<F64>::kMacro; ++s) {
            p0 = Prec<F64>::fmat(P.sdt, z[3 * s], p0);
            p1 = Prec<F64>::fmat(P.sdt, z[3 * s + 1], p1);
            p2 = Prec<F64>::fmat(P.sdt, z[3 * s + 2], p2);
            z[3 * s] = p0;
            z[3 * s + 1] = p1;
            z[3 * s + 2] = p2;
        }
    }

    // The source's densities at N points: the grid's, all loads issued before
    // the first is used, then the analytic bodies' added in their order.
    template <int N>
    __device__ __forceinline__ static void densities(const typename Prec<F64>::Src& src, const T* y, T* r)
    {
#pragma unroll
        for (int i = 0; i < N; ++i) r[i] = T(0);
        // A launch takes the grid loop when any of its problems has a grid,
        // but a batch may mix sources with and without one: the lane's own
        // source is checked, once for all the points' loads.
        if (loop_grid(LOOP) && src.has_grid) {
            GridProbe pr[N];
#pragma unroll
            for (int i = 0; i < N; ++i)
                pr[i] = Prec<F64>::template grid_fetch<loop_levels(LOOP)>(src, y[3 * i], y[3 * i + 1], y[3 * i + 2]);
#pragma unroll
            for (int i = 0; i < N; ++i) r[i] = Prec<F64>::template grid_keep<loop_levels(LOOP)>(src, pr[i]);
        }
        bodies<N>(src, y, r);
    }

    // The least and greatest of one coordinate of a macro-step's points (y[0],
    // y[3], ...), in single instructions: positions are never NaN, and the
    // library's minimum would quiet its operands first.
    __device__ __forceinline__ static void extremes(const double* y, double& low, double& high)
    {
        static_assert(!F64 || Prec<F64>::kMacro == 2, "");
        asm("v_min_f64 %0, %1, %2" : "=v"(low) : "v"(y[0]), "v"(y[3]));
        asm("v_max_f64 %0, %1, %2" : "=v"(high) : "v"(y[0]), "v"(y[3]));
    }
    __device__ __forceinline__ static void extremes(const float* y, float& low, float& high)
    {
        static_assert(F64 || Prec<F64>::kMacro == 4, "");
        asm("v_min3_f32 %0, %1, %2, %3" : "=v"(low) : "v"(y[0]), "v"(y[3]), "v"(y[6]));
        asm("v_min_f32 %0, %1, %2" : "=v"(low) : "v"(low), "v"(y[9]));
        asm("v_max3_f32 %0, %1, %2, %3" : "=v"(high) : "v"(y[0]), "v"(y[3]), "v"(y[6]));
        asm("v_max_f32 %0, %1, %2" : "=v"(high) : "v"(high), "v"(y[9]));
    }

    // Covering loops, the wavefront's walks on one source: the densities of a
    // macro-step's points, and whether it is a plain one -- every point of
    // every live lane strictly inside its box and in its grid (between the
    // source's inner bounds), no walk at its last steps.  A plain macro-step
    // needs no clamp, in-grid test, select or exit test (18 compares of the
    // points' extremes instead of 48 compares, clamps and selects in a mixed
    // walk).  Otherwise densities outside the grid are put to zero here, and
    // steps tests the exits.
    // Measured on the 32-model batch, mixed: 137.0 -> 132.3 ms; 11 models FP64:
    // 39.7 -> 37.0 ms; 97-voxel g_z by levels, FP64: 7.28 -> 7.13 ms.  The
    // 128^3 grid, whose walks are short and whose loads miss, gains 0.4 %.
    __device__ __forceinline__ bool covered(const LaneProblem<F64>& P, const typename Prec<F64>::Src& src, const T* y,
                                            T* rn) const
    {
        constexpr int MACRO = Prec<F64>::kMacro;
        const uint32_t voxels = src.nxy * (uint32_t)src.n[2];
        // the bodies' counts with the source's other scalars, in one wait
        int n_prisms = src.n_prisms, n_spheres = src.n_spheres;
        asm volatile("" : "+s"(n_prisms), "+s"(n_spheres));
        const void* base = loop_levels(LOOP) ? (const void*)src.idx : (const void*)src.rho;
        const auto grid = grid_buffer(base, loop_levels(LOOP) ? voxels : 4u * voxels);
        int i[MACRO][3];
        uint32_t v[MACRO];
        T worst = T(0);
#pragma unroll
        for (int s = 0; s < MACRO; ++s) {
            covered_index(src, y + 3 * s, i[s], worst);
            const uint32_t flat = covered_flat(src, i[s]);
            v[s] = loop_levels(LOOP) ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(grid, flat, 0, 0)
                                     : __builtin_amdgcn_raw_buffer_load_b32(grid, 4u * flat, 0, 0);
        }
        bool in = n + MACRO < P.max_steps;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            T low, high;
            extremes(y + c, low, high);
            in = in & (low > src.in_lo[c]) & (high < src.in_hi[c]);
        }
        if constexpr (F64) {
            // a point too near a voxel face for the short lookup, anywhere in
            // the box: the general one
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(worst > src.near) != 0ull, 0)) {
                densities<MACRO>(src, y, rn);
                return false;
            }
        }
        if (loop_levels(LOOP)) {
            const auto levels = grid_buffer(src.levels, 1024u);
#pragma unroll
            for (int s = 0; s < MACRO; ++s) v[s] = __builtin_amdgcn_raw_buffer_load_b32(levels, 4u * v[s], 0, 0);
        }
        const bool plain = __builtin_amdgcn_ballot_w64(!in) == 0ull;
#pragma unroll
        for (int s = 0; s < MACRO; ++s) rn[s] = (T)__uint_as_float(v[s]);
        if (!plain)
#pragma unroll
            for (int s = 0; s < MACRO; ++s)
                rn[s] = (in_axis(i[s][0], src.n[0]) & in_axis(i[s][1], src.n[1]) & in_axis(i[s][2], src.n[2])) ? rn[s]
                                                                                                             : T(0);
        if (n_prisms + n_spheres > 0) bodies<MACRO>(src, y, rn);
        return plain;
    }

    // One macro-step through the points y: densities, sums and exit tests.
    // Returns whether the walk ended, and where and how (steps).  ONE: the
    // wavefront's walks share the source, and the covering lookup is taken.
    template <bool ONE>
    __device__ __forceinline__ bool take(const LaneProblem<F64>& P, const typename Prec<F64>::Src& src, const T* y,
                                         int& at, int& how)
    {
        constexpr int MACRO = Prec<F64>::kMacro;
        T rn[MACRO];
        if constexpr (!ADJ && loop_cover(LOOP) && ONE) {
            if (covered(P, src, y, rn)) {
#pragma unroll
                for (int s = 0; s < MACRO; ++s) add_density(rn[s]);
                n += MACRO;
                x0 = y[3 * MACRO - 3];
                x1 = y[3 * MACRO - 2];
                x2 = y[3 * MACRO - 1];
                return false;
            }
        } else if constexpr (!ADJ) {
            densities<MACRO>(src, y, rn);
        }
        return steps(P, src, y, rn, at, how);
    }

    // Adds a point's density r to the walk's sum of densities, in which the
    // walk's first and last point count half: half the trapezoid sum
    // sum_n (rho_n + rho_{n+1}), in one addition a step (two, and the density
    // of the step before in registers, when every step added its two ends).
    // Kahan g_z of the SI prism 93.5 -> 88.8 ms, the paper's bridge g_z, mixed,
    // 2.61 -> 2.43 ms (with the round keys of scalar_key).
    __device__ __forceinline__ void add_density(T r)
    {
        if (KAHAN && !F64) {
            const float t0 = (float)r - Sc;
            const float t = Sf + t0;
            Sc = (t - Sf) - t0;
            Sf = t;
        } else {
            S = S + (double)r;
        }
    }

    __device__ __forceinline__ void start_sum(T r)
    {
        S = KAHAN && !F64 ? 0.0 : 0.5 * (double)r;
        Sf = KAHAN && !F64 ? 0.5f * (float)r : 0.0f;
        Sc = 0.0f;
    }

    // Whether y has left the domain (on the boundary counts as left); d2 is
    // the squared distance from the ball's centre (ball domains only).
    __device__ __forceinline__ static bool leaves(const LaneProblem<F64>& P, T y0, T y1, T y2, T& d2)
    {
        if (loop_exit(LOOP) >= 1 && P.ball) {
            d2 = dist2(y0, y1, y2, P.lo0, P.lo1, P.lo2);
            return d2 >= P.hi0;
        }
        d2 = T(0);
        return (y0 <= P.lo0) | (y0 >= P.hi0) | (y1 <= P.lo1) | (y1 >= P.hi1) | (y2 <= P.lo2) | (y2 >= P.hi2);
    }

    // The macro-step's Euler-Maruyama steps through the points y (advance),
    // each with its density and exit test, up to the first that ends the
    // walk.  Returns true when the walk ended, at step at, with how = 0: it
    // left the domain; how = 1: it reached max_steps; how = 2 + f: the bridge
    // test stopped it at face f.  The walk's point x moves to the macro-step's
    // last point only when the walk goes on, so a walk that ended keeps it at
    // the macro-step's start (finish recovers the last step's two ends from x
    // and y).  rn holds the density at each point (densities; the
    // adjoint has none).
    __device__ __forceinline__ bool steps(const LaneProblem<F64>& P, const typename Prec<F64>::Src& src, const T* y,
                                          const T* rn, int& at, int& how)
    {
        constexpr int MACRO = Prec<F64>::kMacro;
        bool done = false;
        if constexpr (!ADJ && loop_exit(LOOP) < 2) {
            // Exit tests of all the points first.  When no walk of the
            // wavefront ends in this macro-step -- nearly always for walks of
            // hundreds of steps -- the steps run as straight-line code,
            // without the per-step masking of walks that ended.
            bool out[MACRO];
            bool end = n + MACRO >= P.max_steps;
#pragma unroll
            for (int s = 0; s < MACRO; ++s) {
                T d2;
                out[s] = leaves(P, y[3 * s], y[3 * s + 1], y[3 * s + 2], d2);
                end = end | out[s];
            }
            if (__ballot(end) == 0ull) {
#pragma unroll
                for (int s = 0; s < MACRO; ++s) add_density(rn[s]);
                n += MACRO;
            } else {
#pragma unroll
                for (int s = 0; s < MACRO; ++s) {
                    if (done) break;
                    n += 1;
                    T r = rn[s];
                    if (out[s]) {
                        how = 0;
                        at = s;
                        done = true;
                        r = T(0.5) * r;
                    } else if (n == P.max_steps) {
                        how = 1;
                        at = s;
                        done = true;
                    }
                    add_density(r);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < MACRO; ++s) {
                if (done) break;
                const T y0 = y[3 * s], y1 = y[3 * s + 1], y2 = y[3 * s + 2];
                n += 1;
                T d2;
                const bool out = leaves(P, y0, y1, y2, d2);
                int stop = -1;
                if (loop_exit(LOOP) == 2 && P.bridge && !out) {
                    const bool deep_y = deep_inside(P, y0, y1, y2, d2);
                    if (!(deep && deep_y)) {
                        const T p0 = s ? y[3 * s - 3] : x0, p1 = s ? y[3 * s - 2] : x1, p2 = s ? y[3 * s - 1] : x2;
                        stop = bridge_stop(P, pctr, sctr, n - 1, p0, p1, p2, y0, y1, y2);
                    }
                    deep = deep_y;
                }
                if (ADJ) sc.add(Prec<F64>::voxel(src, y0, y1, y2), (out || stop >= 0) ? 1 : 2);
                if (out || stop >= 0) {
                    how = out ? 0 : 2 + stop;
                    at = s;
                    done = true;
                } else if (n == P.max_steps) {
                    how = 1;
                    at = s;
                    done = true;
                }
                if (!ADJ) add_density(done ? T(0.5) * rn[s] : rn[s]);
            }
        }
        if (!done) {
            x0 = y[3 * MACRO - 3];
            x1 = y[3 * MACRO - 2];
            x2 = y[3 * MACRO - 1];
        }
        return done;
    }

    // Ends the walk: y holds the macro-step's points (advance) and the walk
    // ended at step at of them: the end point is y[at], the last point inside
    // the one before it (x for the first step).
    __device__ __forceinline__ void finish(const LaneProblem<F64>& P, const T* y, int at, int how)
    {
        constexpr int MACRO = Prec<F64>::kMacro;
        T a0 = x0, a1 = x1, a2 = x2, e0 = y[0], e1 = y[1], e2 = y[2];
#pragma unroll
        for (int s = 1; s < MACRO; ++s) {
            if (at == s) {
                a0 = y[3 * s - 3];
                a1 = y[3 * s - 2];
                a2 = y[3 * s - 1];
                e0 = y[3 * s];
                e1 = y[3 * s + 1];
                e2 = y[3 * s + 2];
            }
        }
        finish_at(P, a0, a1, a2, e0, e1, e2, how);
    }

    // Stores the exit record (or flushes the scatter) of a walk whose last
    // step went from a to e, and frees the lane.
    __device__ __forceinline__ void finish_at(const LaneProblem<F64>& P, T a0, T a1, T a2, T e0, T e1, T e2, int how)
    {
        const bool capped = how == 1;
        if (ADJ) {
            sc.flush();
        } else {
            const WalkCommon& C = *P.C;
            double e[3] = {0.0, 0.0, 0.0};
            if (loop_exit(LOOP) == 2 && how >= 2) {
                // bridge stop: the step's end projected onto the face
                e[0] = (double)e0;
                e[1] = (double)e1;
                e[2] = (double)e2;
                const int f = how - 2;
                if (f == 6) {
                    const double r = sqrt(dist2(e[0], e[1], e[2], C.ctr[0], C.ctr[1], C.ctr[2]));
#pragma unroll
                    for (int j = 0; j < 3; ++j) e[j] = C.ctr[j] + C.R * ((e[j] - C.ctr[j]) / r);
                } else {
                    e[f >> 1] = (f & 1) ? C.hi[f >> 1] : C.lo[f >> 1];
                }
            } else if (!capped) {
                e[0] = (double)e0;
                e[1] = (double)e1;
                e[2] = (double)e2;
                if (C.exit_rule != FK_EXIT_OVERSHOOT) {
                    const double a[3] = {(double)a0, (double)a1, (double)a2};
                    const double b[3] = {(double)e0, (double)e1, (double)e2};
                    if (C.domain == FK_DOMAIN_BALL)
                        intersect_ball(C.ctr, C.r2, a, b, e);
                    else
                        intersect_exit(C.lo, C.hi, a, b, e);
                }
            }
            const double sum = 2.0 * ((!F64 && KAHAN) ? ((double)Sf - (double)Sc) : S);
            exits[rec] = ExitRecord{e[0], e[1], e[2], sum};
            steps_out[rec] = n | (capped ? kCapFlag : 0u);
        }
        active = false;
    }
};

// ---------------------------------------------------------------------------
// Shared drain rounds.  A lone walk stepping in its own lane issues every
// instruction of a step -- some 60 of them, 5 cycles each with one wavefront
// per SIMD -- for one step's worth of work.  Of a step only the move
// x + sqrt(dt) z and the sum of densities depend on the step before; densities
// and exit tests do not.  So in a round with at most coop_live live walks of
// one problem
//   1. the chain of moves runs in one lane per walk and axis, which replaces
//      its row of normals in LDS by the positions they lead to (rows, so that
//      16 bytes go with one LDS instruction: a move is one fused multiply-add
//      and 0.5 (FP32) or 1 (FP64) LDS instructions);
//   2. all 64 lanes take densities and exit tests of the round's points, up
//      to MACRO points each, all grid loads in flight together;
//   3. the walks' densities are added in step order, up to the first point
//      that ends a walk: only those that are not zero, one at a time from the
//      lane that has it, or all of them from LDS where most are not.
// The arithmetic of every step and its order are those of a macro-step, so a
// walk's record does not depend on the rounds it ran in.
// Measured, with the even shares of Queue::cap, against lanes stepping alone:
// a lone walk 213 -> 33 ns a step in FP64 (37 on a grid), 175 to 214 -> 20 to
// 21 ns mixed;
// 8 stations x 250 walks in FP64 1329 -> 141 us (a call returning host
// arrays, with the first runs of start_pool); Table 1's cells Delta t = 0.01,
// N = 5120: 6.67 -> 3.11 ms, and 0.001, N = 25600 (with the FP64 normals):
// 129 -> 84.0 ms.
constexpr int kCoopLive = 21;     // the chains fill a wavefront
// Without the bridge test (whose tests of every point sharing spreads best)
// rounds of 17 to 21 walks are sooner done unshared: 48 small grid models 674
// -> 657 us, the cell of 5120 walks 3114 -> 3059 us with at most 16 shared,
// and the bridge g_z 1915 -> 2019 (32 shared: 3118 -> 3407 and 1944 -> 2005).
constexpr int coop_live(int loop) { return loop_exit(loop) == 2 ? kCoopLive : 16; }

// A wavefront's LDS in a shared round.  Row (axis c, walk w) starts at
// (c m + w) pitch, pitch = the round's steps and 16 bytes (so that rows start
// in different banks); kRow holds the m rows of an axis for every m.
template <bool F64>
struct CoopRound {
    using T = typename Prec<F64>::T;
    static constexpr int kV = 16 / (int)sizeof(T);        // elements per 16 bytes
    // an axis's rows, m (macros MACRO + kV) for macros = 64 / m and m <= kCoopLive
    // (85 MACRO at most), and room beside them for the slots of a round that is
    // not shared
    static constexpr int kRow = 96 * Prec<F64>::kMacro;
    static_assert(kRow >= 64 * Prec<F64>::kMacro + kCoopLive * kV, "the rows of every shared round");
    alignas(16) T pos[3 * kRow];
    static constexpr int kPad = 128 / (int)sizeof(T);     // read past a row's end (for_row)
    alignas(16) T dens[kRow + kPad];
    int end[kCoopLive];           // 16 x the first step that ends walk w + how (Walker::steps)
    uint8_t near[64 * Prec<F64>::kMacro];   // bridge test: points to test
};

template <class T>
struct alignas(16) Quad {
    T v[16 / sizeof(T)];
};

// fma(s, z, p) in z's register: the compiler's choice, the form that adds to
// p's, needs a copy for each position stored.
__device__ __forceinline__ double fma_into(double z, double s, double p)
{
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(s), "v"(z), "v"(p));
    return r;
}

__device__ __forceinline__ float fma_into(float z, float s, float p)
{
    float r;
    asm("v_fma_f32 %0, %1, %2, %3" : "=v"(r) : "v"(s), "v"(z), "v"(p));
    return r;
}

// Reads the row's quads two batches of 64 bytes ahead of f(quad index, quad),
// which is called on its n quads in order: a lone chain of additions then waits
// for itself, not for the LDS.  Up to 128 bytes past the row are read, and not
// used (CoopRound::kPad).
template <bool F64, class T = typename Prec<F64>::T, class F>
__device__ __forceinline__ void for_row(const Quad<T>* row, int n, F&& f)
{
    constexpr int J = 4;
    Quad<T> a[J], b[J];
#pragma unroll
    for (int k = 0; k < J; ++k) a[k] = row[k];
#pragma unroll
    for (int k = 0; k < J; ++k) b[k] = row[J + k];
    int j = 0;
#pragma unroll 1
    for (; j + 2 * J <= n; j += 2 * J) {
#pragma unroll
        for (int k = 0; k < J; ++k) f(j + k, a[k]);
#pragma unroll
        for (int k = 0; k < J; ++k) a[k] = row[j + 2 * J + k];
#pragma unroll
        for (int k = 0; k < J; ++k) f(j + J + k, b[k]);
        __builtin_amdgcn_sched_barrier(0);        // moved up, the reads would need registers of their own, and copies
#pragma unroll
        for (int k = 0; k < J; ++k) b[k] = row[j + 3 * J + k];
    }
#pragma unroll
    for (int k = 0; k < 2 * J; ++k)
        if (j + k < n) f(j + k, k < J ? a[k < J ? k : 0] : b[k < J ? 0 : k - J]);
}

// Replaces a row of normals by the positions they lead to from p.  A lone walk
// spends 2/5 of its round here, bound by the latency of the dependent
// operation: with one batch ahead, positions copied into store order and
// guarded reads a step of a lone walk took 37 ns in FP64 and 30 in mixed
// precision; it takes 33 and 20 to 21 now.
template <bool F64, class T = typename Prec<F64>::T>
__device__ __forceinline__ void chain_row(Quad<T>* row, int n, T sdt, T p)
{
    for_row<F64>(row, n, [&](int j, Quad<T> q) {
#pragma unroll
        for (int e = 0; e < CoopRound<F64>::kV; ++e) p = q.v[e] = fma_into(q.v[e], sdt, p);
        row[j] = q;
    });
}

// One shared round: m live walks (walk w is held by lane lanes[w]; rank is w
// in the lanes that hold one), `macros` macro-steps each, whose normals are
// in R.pos.  P is the live walks' problem.
template <bool F64, bool KAHAN, int LOOP>
__device__ __forceinline__ void coop_round(Walker<F64, KAHAN, false, LOOP>& W, const LaneProblem<F64>& P,
                                           const typename Prec<F64>::Src& src, CoopRound<F64>& R, const uint8_t* lanes,
                                           int m, int macros, int rank)
{
    using T = typename Prec<F64>::T;
    constexpr int MACRO = Prec<F64>::kMacro;
    constexpr int V = CoopRound<F64>::kV;
    const int lane = (int)__lane_id();
    const int L = macros * MACRO;                 // steps per walk, a multiple of V
    const int pitch = L + V;
    const int over_m = 65536 / m + 1;             // q / m = q * over_m >> 16 for q < 128
    const int over_L = 65536 / L + 1;             // t / L = t * over_L >> 16 for t < 256

    // 1. positions: chain q = c m + w moves axis c of walk w
#pragma unroll 1
    for (int q0 = 0; q0 < 3 * m; q0 += 64) {
        const int q = q0 + lane;
        const int c = (q * over_m) >> 16, w = q - c * m;
        const int from = lanes[w];
        const T s0 = __shfl(W.x0, from), s1 = __shfl(W.x1, from), s2 = __shfl(W.x2, from);
        if (c < 3) {
            chain_row<F64>(reinterpret_cast<Quad<T>*>(R.pos + q * pitch), L / V, P.sdt, c == 0 ? s0 : c == 1 ? s1 : s2);
        }
    }
    if (lane < m) R.end[lane] = 16 * L;
    wave_sync_lds();

    // 2. densities and exit tests: point t = w L + s in lane t mod 64
    auto at = [&](int c, int w, int s) { return (c * m + w) * pitch + s; };
    auto before = [&](int w, int s, T& a0, T& a1, T& a2) {   // the point before step s > 0
        a0 = R.pos[at(0, w, s - 1)];
        a1 = R.pos[at(1, w, s - 1)];
        a2 = R.pos[at(2, w, s - 1)];
    };
    T y[3 * MACRO], rn[MACRO];
    int ws[MACRO], ss[MACRO];
#pragma unroll
    for (int i = 0; i < MACRO; ++i) {
        const int t = lane + 64 * i < L * m ? lane + 64 * i : 0;    // no point: any other
        ws[i] = (t * over_L) >> 16;
        ss[i] = t - ws[i] * L;
#pragma unroll
        for (int c = 0; c < 3; ++c) y[3 * i + c] = R.pos[at(c, ws[i], ss[i])];
    }
    Walker<F64, KAHAN, false, LOOP>::template densities<MACRO>(src, y, rn);
    bool some = false;
    uint64_t mass[MACRO];                         // lanes whose point i has a density
    int n_mass = 0, n_near = 0;
    // a walk's end as 16 step + how: the earliest step, and there a stop at a
    // face before a cap
    auto ends = [&](int w, int s, int how) {
        atomicMin(&R.end[w], 16 * s + (how == 1 ? 15 : how));
        some = true;
    };
#pragma unroll
    for (int i = 0; i < MACRO; ++i) {
        const bool valid = lane + 64 * i < L * m;
        const int w = ws[i], s = ss[i];
        const uint32_t nw = (uint32_t)__shfl((int)W.n, lanes[w]);
        const T y0 = y[3 * i], y1 = y[3 * i + 1], y2 = y[3 * i + 2];
        if (valid) R.dens[w * pitch + s] = rn[i];
        mass[i] = __builtin_amdgcn_ballot_w64(valid & !(rn[i] == T(0)));
        n_mass += __popcll(mass[i]);
        T d2;
        const bool out = Walker<F64, KAHAN, false, LOOP>::leaves(P, y0, y1, y2, d2);
        if (valid & (out | (nw + (uint32_t)s + 1u >= P.max_steps))) ends(w, s, out ? 0 : 1);
        if constexpr (loop_exit(LOOP) == 2) {
            const int from = lanes[w];
            T a0 = __shfl(W.x0, from), a1 = __shfl(W.x1, from), a2 = __shfl(W.x2, from);
            const bool test = P.bridge && valid && !out;
            if (test && s > 0) before(w, s, a0, a1, a2);
            const T da = P.ball ? dist2(a0, a1, a2, P.lo0, P.lo1, P.lo2) : T(0);
            const bool near = test && !(W.deep_inside(P, a0, a1, a2, da) && W.deep_inside(P, y0, y1, y2, d2));
            const uint64_t nears = __builtin_amdgcn_ballot_w64(near);
            if (near) R.near[n_near + __popcll(nears & __lanemask_lt())] = (uint8_t)(lane + 64 * i);
            n_near += __popcll(nears);
        }
    }
    if constexpr (loop_exit(LOOP) == 2) {
        // the steps that may cross a face on the way, 64 at a time (tested where
        // they are, each of the MACRO passes over the points that holds one
        // would pay for a test of its own: 1930 against 1900 us for 31 stations
        // of 2 x 2048 walks)
        wave_sync_lds();
        for (int p0 = 0; p0 < n_near; p0 += 64) {
            const bool mine = p0 + lane < n_near;
            const int t = R.near[mine ? p0 + lane : 0];
            const int w = (t * over_L) >> 16, s = t - w * L, from = lanes[w];
            const uint32_t pw = (uint32_t)__shfl((int)W.pctr, from), sw = (uint32_t)__shfl((int)W.sctr, from);
            const uint32_t nw = (uint32_t)__shfl((int)W.n, from);
            T a0 = __shfl(W.x0, from), a1 = __shfl(W.x1, from), a2 = __shfl(W.x2, from);
            if (mine) {
                if (s > 0) before(w, s, a0, a1, a2);
                const int stop = W.bridge_stop(P, pw, sw, nw + (uint32_t)s, a0, a1, a2, R.pos[at(0, w, s)],
                                               R.pos[at(1, w, s)], R.pos[at(2, w, s)]);
                if (stop >= 0) ends(w, s, 2 + stop);
            }
        }
    }
    const bool any_end = __builtin_amdgcn_ballot_w64(some) != 0ull;
    wave_sync_lds();

    // 3. the walks' sums and ends
    const int end = any_end && W.active ? R.end[rank] : 16 * L;
    const int f = end >> 4, how = (end & 15) == 15 ? 1 : end & 15;
    const int taken = f < L ? f + 1 : L;
    // Adding a zero leaves an uncompensated sum as it is.  One density costs
    // some 8 instructions from its lane, a step of every walk 3 from LDS.
    if (!KAHAN && 8 * n_mass <= 3 * L) {
#pragma unroll
        for (int i = 0; i < MACRO; ++i)
            for (uint64_t left = mass[i]; left != 0ull; left &= left - 1ull) {
                const int b = __ffsll((unsigned long long)left) - 1;
                const T r = lane_value(rn[i], b);
                const int w = __builtin_amdgcn_readlane(ws[i], b), s = __builtin_amdgcn_readlane(ss[i], b);
                if (W.active & (rank == w) & (s <= f)) W.add_density(s == f ? T(0.5) * r : r);
            }
    } else if (W.active) {
        const T* row = R.dens + rank * pitch;
        const int whole = f < L ? f : L;          // densities of full weight
        for_row<F64>(reinterpret_cast<const Quad<T>*>(row), whole / V, [&](int, const Quad<T>& d) {
#pragma unroll
            for (int e = 0; e < V; ++e) W.add_density(d.v[e]);
        });
        for (int s = whole & ~(V - 1); s < whole; ++s) W.add_density(row[s]);
        if (f < L) W.add_density(T(0.5) * row[f]);
    }
    if (W.active) {
        W.n += (uint32_t)taken;
        W.k += (uint32_t)(3 * macros);
        const int l = taken - 1;                  // the last point reached
        const T e0 = R.pos[at(0, rank, l)], e1 = R.pos[at(1, rank, l)], e2 = R.pos[at(2, rank, l)];
        if (f < L) {
            T a0 = W.x0, a1 = W.x1, a2 = W.x2;
            if (f > 0) {
                a0 = R.pos[at(0, rank, f - 1)];
                a1 = R.pos[at(1, rank, f - 1)];
                a2 = R.pos[at(2, rank, f - 1)];
            }
            W.finish_at(P, a0, a1, a2, e0, e1, e2, how);
        } else {
            W.x0 = e0;
            W.x1 = e1;
            W.x2 = e2;
            W.deep = false;                       // tested again where it matters
        }
    }
}

// ---------------------------------------------------------------------------
// The kernel body.
// ---------------------------------------------------------------------------
// DENSE (adjoint only): blocks of kAdjDenseBlock threads with a dense
// per-station table,
// working through the stations one at a time (each station's tasks have
// their own claim counter; a block starts on station blockIdx mod S and,
// when its station's tasks are all claimed and its walks done, flushes the
// table and moves on to the next station with unclaimed tasks).
// UKEY (batches): every problem has the same generator key, passed in the
// launch arguments, so the Philox key schedule is scalar work.
template <bool F64, bool KAHAN, bool ADJ, bool BATCH, int LOOP, bool SHARED, bool DENSE, bool UKEY, class Args>
__device__ __forceinline__ void walk_body(const Args& A)
{
    using T = typename Prec<F64>::T;
    constexpr int NPB = Prec<F64>::kNormals;
    constexpr int MACRO = Prec<F64>::kMacro;
    // Drain rounds need a buffer per wavefront; the dense instance runs
    // without them (its LDS holds the table), so its last walks of a station
    // step in ordinary macro-steps.
    constexpr bool DRAIN = !DENSE;
    constexpr int TAIL_WAVES = DRAIN ? kMaxWaves : 1;
    static_assert(!DENSE || (ADJ && !BATCH), "dense tables are the adjoint's");

    __shared__ uint8_t tail_lane[TAIL_WAVES][64];
    // a drain round's normals: block slots of NPB, or a shared round's rows
    // (the adjoint's blocks have LDS for half as many slots beside its table)
    constexpr int kSlots = ADJ ? 192 : 384;
    struct Slots {
        Quad<T> z[kSlots];
    };
    static_assert(NPB == 16 / (int)sizeof(T), "a slot is 16 bytes");
    using Tail = typename std::conditional<ADJ, Slots, CoopRound<F64>>::type;
    static_assert(sizeof(Tail) >= sizeof(Slots), "the slots of a round that is not shared lie in its LDS");
    __shared__ Tail tail[TAIL_WAVES];
    const BmTables* bmt = nullptr;
    if constexpr (F64) {
        BmTables* t = bm_tables();
        fill_bm_tables(*t);
        bmt = t;
    }

    Queue Q;
    LaneProblem<F64> P;
    if constexpr (BATCH) {
        Q = Queue{A.queue, (uint64_t)A.n_tasks, (uint32_t)A.grab, A.total_waves, A.stripes, A.refill_cost, A.cap};
        P.C = nullptr;
        P.src = nullptr;
        P.sdt = T(0);
        P.lo0 = P.lo1 = P.lo2 = P.hi0 = P.hi1 = P.hi2 = T(0);
        P.ball = false;
        P.key0 = P.key1 = P.pid = 0;
        if constexpr (UKEY) {
            P.key0 = A.key0;
            P.key1 = A.key1;
        }
        P.max_steps = 0u;
    } else {
        Q = Queue{A.c.queue, (uint64_t)A.c.n_tasks, (uint32_t)A.c.grab, A.c.total_waves, A.c.stripes,
                  A.c.refill_cost, A.c.cap};
        P.load(A.c, A.src);
        // held in vector registers, as a batch holds them: kept in scalar
        // registers beside the source's bodies they overflow the scalar file,
        // and every step then reloads them from spill lanes
        P.sdt = in_vgpr(P.sdt);
        P.lo0 = in_vgpr(P.lo0);
        P.lo1 = in_vgpr(P.lo1);
        P.lo2 = in_vgpr(P.lo2);
        P.hi0 = in_vgpr(P.hi0);
        P.hi1 = in_vgpr(P.hi1);
        P.hi2 = in_vgpr(P.hi2);
    }
    // the density source of the lane's walk: the launch's (kernel arguments),
    // the batch's shared one (kernel arguments), or the lane's problem's
    auto source = [&]() -> const typename Prec<F64>::Src& {
        if constexpr (!BATCH) return A.src;
        else if constexpr (SHARED) return shared_source<F64>(A);
        else return *P.src;
    };
    // runs f on the source of the live lanes' walks (called with only those
    // lanes active), and on whether they share it as a compile-time constant:
    // in a batch of separate sources, through wave_uniform when they do
    auto with_source = [&](auto&& f) {
        if constexpr (BATCH && !SHARED) {
            if (const auto* u = wave_uniform(P.src))
                f(*u, std::true_type{});
            else
                f(*P.src, std::false_type{});
        } else if constexpr (!BATCH) {
            // the source in the kernel arguments (the launch's one argument,
            // at the start of the argument segment), re-addressed through an
            // opaque scalar pointer each macro-step: its bodies are reloaded
            // with scalar loads instead of being held live (and spilled)
            // across the loop
            uint64_t a = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(Args, src);
            asm volatile("" : "+s"(a));
            f(*(const typename Prec<F64>::Src*)(const __attribute__((address_space(4))) typename Prec<F64>::Src*)a,
              std::true_type{});
        } else {
            f(source(), std::true_type{});
        }
    };
    Pool pool = start_pool<!DENSE>(Q);
    Walker<F64, KAHAN, ADJ, LOOP, DENSE> W;
    W.active = false;
    W.rec = 0;
    if constexpr (BATCH) {
        W.exits = A.exits;
        W.steps_out = A.steps;
    } else {
        W.exits = A.c.exits;
        W.steps_out = A.c.steps;
    }
    W.x0 = W.x1 = W.x2 = T(0);
    W.S = 0.0;
    W.Sf = W.Sc = 0.0f;
    W.n = W.k = W.sctr = W.pctr = 0;
    W.deep = false;
    W.sc = Scatter<DENSE>{nullptr, nullptr, 0, -1, 0, 1};
    void* adj_tab = nullptr;
    int* dirty = nullptr;       // dense: set when the block starts a walk of its station
    if constexpr (ADJ && !DENSE) {
        static_assert(!BATCH, "the adjoint runs single-problem launches");
        __shared__ uint32_t tab[kAdjSlots];
        for (int i = threadIdx.x; i < kAdjSlots; i += blockDim.x) tab[i] = 0u;
        __syncthreads();
        adj_tab = tab;
    }
    if constexpr (DENSE) {
        __shared__ int dtab[kDenseVoxels];
        __shared__ int dflag;
        for (int i = threadIdx.x; i < kDenseVoxels; i += blockDim.x) dtab[i] = 0;
        if (threadIdx.x == 0) dflag = 0;
        __syncthreads();
        adj_tab = dtab;
        dirty = &dflag;
    }
    const int wave = threadIdx.x >> 6;
    const int lane = (int)__lane_id();
    uint64_t task_base = 0;   // task of queue index 0
    if constexpr (!BATCH) task_base = (uint64_t)A.c.task0;

    // Fills the wavefront's free lanes with walks from the queue.
    auto start_walks = [&]() {
        const uint64_t got = refill(pool, Q, W.active);
        if (got != ~0ull) {
            const WalkCommon* Cp;
            uint64_t t;
            if constexpr (BATCH) {
                const int64_t T = A.task0 + (int64_t)got;
                const int m = find_problem(A.task_off, A.n_problems, T);
                const BatchDesc& D = A.desc[m];
                t = (uint64_t)(T - A.task_off[m]);
                if constexpr (SHARED)
                    P.load(D.c, shared_source<F64>(A), !UKEY);
                else
                    P.load(D.c, SourceOf<F64>::get(D), !UKEY);
                Cp = &D.c;
            } else {
                t = task_base + got;
                Cp = &A.c;
            }
            const WalkCommon& C = *Cp;
            const TaskInfo ti = decode(C, t);
            W.rec = got;
            const bool inside = strictly_inside(C, ti.x0);
            if (ADJ && (!inside || forward_capped(C, t))) {
                // excluded in the forward solve: contributes nothing
            } else if (!ADJ && !inside) {
                // a start point on or outside the boundary yields no sample
                const double q = __builtin_nan("");
                W.exits[got] = ExitRecord{q, q, q, q};
                W.steps_out[got] = kCapFlag;
            } else {
                W.x0 = (T)ti.x0[0];
                W.x1 = (T)ti.x0[1];
                W.x2 = (T)ti.x0[2];
                W.sctr = ti.sctr;
                W.pctr = ti.pctr;
                W.n = 0;
                W.k = 0;
                W.S = 0.0;
                W.Sf = W.Sc = 0.0f;
                if (ADJ) {
                    if (DENSE) __hip_atomic_store(dirty, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    W.sc.counts = C.counts;
                    W.sc.tab = adj_tab;
                    W.sc.row = (int64_t)ti.s * C.nvox;
                    W.sc.v = -1;
                    W.sc.c = 0;
                    W.sc.sign = ti.w ? -1 : 1;
                    W.sc.add(Prec<F64>::voxel(source(), W.x0, W.x1, W.x2), 1);
                } else {
                    const T start[3] = {W.x0, W.x1, W.x2};
                    T r;
                    Walker<F64, KAHAN, ADJ, LOOP, DENSE>::template densities<1>(source(), start, &r);
                    W.start_sum(r);
                }
                W.deep = false;
                if (loop_exit(LOOP) == 2 && P.bridge) {
                    const T d2 = P.ball ? dist2(W.x0, W.x1, W.x2, P.lo0, P.lo1, P.lo2) : T(0);
                    W.deep = W.deep_inside(P, W.x0, W.x1, W.x2, d2);
                }
                W.active = true;
            }
        }
    };

    // The wavefront's walks until its queue is used up and they are done: in
    // macro-steps while there are walks to refill its lanes with, then in
    // drain rounds.  (Two loops, so that what the drain rounds keep in
    // registers is not live through the macro-steps.)
    auto run_waves = [&]() {
        if (DRAIN && Q.cap < 64u) start_walks();     // a capped launch: its one run
        while (!DRAIN || Q.cap == 64u) {
            start_walks();
            if (__ballot(W.active) == 0ull) {
                if (pool.exhausted) break;
                continue;
            }
            if (DRAIN && pool.exhausted) break;
            if (!W.active) continue;

            // ---- macro-step: 3 blocks of this lane's own walk ----
            T z[3 * NPB];
            uint32_t key0 = P.key0, key1 = P.key1;
            if constexpr (!BATCH || (F64 && UKEY)) scalar_key(key0, key1, pool.rounds);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const Block bl = philox10(W.k + b, W.pctr, W.sctr, P.pid, key0, key1);
                Prec<F64>::normals(bl, z + NPB * b, bmt);
            }
            W.k += 3;
            W.advance(P, z);
            bool done = false;
            int how = 0, at = 0;
            with_source([&](const typename Prec<F64>::Src& src, auto one) {
                done = W.template take<decltype(one)::value>(P, src, z, at, how);
            });
            if (done) W.finish(P, z, at, how);
        }
        while (DRAIN) {
            const uint64_t live = __ballot(W.active);
            if (live == 0ull) break;
            const int m = __popcll(live);
            // ---- drain round: the queue is empty, or the launch gives no
            // wavefront more walks than these, so every lane generates Philox
            // blocks for the live walks of its wavefront (block slot
            // g = r * m + w holds block r of live walk w), for as many
            // macro-steps of each as the slots hold: of the lanes' passes at
            // most a fifth is then unused, however many walks are live.
            const int rank = __popcll(live & __lanemask_lt());
            if (W.active) tail_lane[wave][rank] = (uint8_t)lane;
            wave_sync_lds();
            // shared: few enough live walks, all of one problem
            const int first = __ffsll((unsigned long long)live) - 1;
            bool shared = !ADJ && m <= coop_live(LOOP);
            if constexpr (!ADJ && BATCH) {
                const uint64_t pc = lane_u64((uint64_t)P.C, first);
                shared = shared && __builtin_amdgcn_ballot_w64(W.active && (uint64_t)P.C != pc) == 0ull;
            }
            // macro-steps per live walk this round
            const int macros = shared ? 64 / m : kSlots / (3 * m);
            const int B = 3 * macros;                  // blocks per live walk
            const int passes = (B * m + 63) / 64;
            T* const slots = reinterpret_cast<T*>(&tail[wave]);
            const int over = 65536 / m + 1;            // g / m = g * over >> 16 for g < 384
            const int pitch = macros * MACRO + CoopRound<F64>::kV;
#pragma unroll 1
            for (int i = 0; i < passes; ++i) {
                const int g = lane + 64 * i;
                const int r = (g * over) >> 16;
                const int w = g - r * m;
                const int src = tail_lane[wave][w];
                const uint32_t ks = (uint32_t)__shfl((int)W.k, src);
                const uint32_t ps = (uint32_t)__shfl((int)W.pctr, src);
                const uint32_t ss = (uint32_t)__shfl((int)W.sctr, src);
                uint32_t key0 = P.key0, key1 = P.key1, pid = P.pid;
                if constexpr (!BATCH || (F64 && UKEY)) scalar_key(key0, key1, pool.rounds);
                if constexpr (BATCH) {
                    if constexpr (!UKEY) {
                        key0 = (uint32_t)__shfl((int)P.key0, src);
                        key1 = (uint32_t)__shfl((int)P.key1, src);
                    }
                    pid = (uint32_t)__shfl((int)P.pid, src);
                }
                if (r < B) {
                    const Block bl = philox10(ks + (uint32_t)r, ps, ss, pid, key0, key1);
                    T z[NPB];
                    Prec<F64>::normals(bl, z, bmt);
                    if (shared) {
                        // normal e = NPB r + j of walk w: step e / 3, axis e mod 3
                        int s = (NPB * r * 21846) >> 16, c = NPB * r - 3 * s;
#pragma unroll
                        for (int j = 0; j < NPB; ++j) {
                            slots[(c * m + w) * pitch + s] = z[j];
                            s += c == 2;
                            c = c == 2 ? 0 : c + 1;
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < NPB; ++j) slots[g * NPB + j] = z[j];
                    }
                }
            }
            wave_sync_lds();
            if constexpr (!ADJ) {
                if (shared) {
                    LaneProblem<F64> PE = P;
                    const typename Prec<F64>::Src* sp;
                    if constexpr (BATCH) PE.from_lane(P, first, !UKEY);
                    if constexpr (BATCH && !SHARED)
                        sp = (const typename Prec<F64>::Src*)(const __attribute__((address_space(4)))
                                                              typename Prec<F64>::Src*)(uint64_t)PE.src;
                    else
                        sp = &source();
                    coop_round(W, PE, *sp, tail[wave], tail_lane[wave], m, macros, rank);
                    wave_sync_lds();
                    continue;
                }
            }
            if (W.active) {
                const int n_steps = MACRO * macros;
                bool done = false;
                int how = 0;
                for (int s0 = 0; s0 < n_steps && !done; s0 += MACRO) {
                    T zz[3 * MACRO];
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        const Quad<T> q = reinterpret_cast<const Quad<T>*>(slots)[(3 * (s0 / MACRO) + b) * m + rank];
#pragma unroll
                        for (int j = 0; j < NPB; ++j) zz[NPB * b + j] = q.v[j];
                    }
                    int at = 0;
                    W.advance(P, zz);
                    with_source([&](const typename Prec<F64>::Src& src, auto) {
                        done = W.template take<false>(P, src, zz, at, how);
                    });
                    if (done) W.finish(P, zz, at, how);
                }
                W.k += (uint32_t)B;
            }
            wave_sync_lds();
        }
    };

    if constexpr (DENSE) {
        __shared__ int next_station;
        const int64_t S = A.c.n_stations;
        const uint64_t per = (uint64_t)A.c.N * (uint64_t)A.c.npair;   // tasks of one station
        const int64_t nvox = A.c.nvox;
        int* tab = static_cast<int*>(adj_tab);
        const uint32_t waves_per_station = A.c.total_waves / (uint32_t)S > 0 ? A.c.total_waves / (uint32_t)S : 1u;
        if (threadIdx.x == 0) next_station = (int)(blockIdx.x % (uint32_t)S);
        __syncthreads();
        for (;;) {
            const int s = next_station;
            if (s < 0) break;
            Q = Queue{A.c.queue + s, per, (uint32_t)A.c.grab, waves_per_station, 1u, A.c.refill_cost, 64u};
            pool = start_pool<false>(Q);
            task_base = (uint64_t)s * per;
            run_waves();
            __syncthreads();    // the block's walks of station s are done
            if (*dirty) {
                for (int64_t v = threadIdx.x; v < nvox; v += blockDim.x) {
                    const int c = tab[v];
                    if (c != 0) {
                        global_add(A.c.counts, (int64_t)s * nvox + v, c);
                        tab[v] = 0;
                    }
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                *dirty = 0;
                int nxt = -1;
                for (int64_t k = 1; k <= S; ++k) {
                    const int c = (int)((s + k) % S);
                    if (__hip_atomic_load(A.c.queue + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < per) {
                        nxt = c;
                        break;
                    }
                }
                next_station = nxt;
            }
            __syncthreads();
        }
    } else {
        run_waves();
    }
    if constexpr (ADJ && !DENSE) {
        // every wavefront has left the loop: the table's entries go out
        __syncthreads();
        const uint32_t* tab = static_cast<const uint32_t*>(adj_tab);
        for (int i = threadIdx.x; i < kAdjSlots; i += blockDim.x) {
            const uint32_t e = tab[i];
            const int64_t c = adj_count(e);
            if (adj_key(e) != 0 && c != 0) global_add(A.c.counts, (int64_t)adj_key(e) - 1, c);
        }
    }
}

// Minimum resident 256-thread blocks per CU the compiler must allow (this
// bounds the VGPRs per lane: 4 blocks = 4 wavefronts per SIMD = 128 VGPRs).
// FP64 walks are held to 4 wavefronts per SIMD: measured faster than 3
// wavefronts without the limit, when the box loop spilled a little.  Now the box,
// ball and grid loops take 115 to 117 VGPRs and spill none; with the bridge test
// they spill 14 to 16 (52 to 60 bytes a lane).
#ifndef FK_F64_BLOCKS_PER_CU
#define FK_F64_BLOCKS_PER_CU 4
#endif
// Mixed-precision walks are held to 6 (80 VGPRs; 3 to 6 spilled, 14 to 18 with
// the bridge test).
#ifndef FK_F32_BLOCKS_PER_CU
#define FK_F32_BLOCKS_PER_CU 6
#endif
// Batches (box loop): 4 blocks for FP64 (128 VGPRs; 2 spilled with a key per
// lane) and 5 for mixed precision (96 VGPRs, a 12-byte spill) measured 7-10 %
// faster than the unconstrained 3 and 4.  The ball and bridge loops are left free:
// 94 to 150 VGPRs and 113 to 199, 2 to 5 blocks.
#ifndef FK_BATCH_F64_BLOCKS_PER_CU
#define FK_BATCH_F64_BLOCKS_PER_CU 4
#endif
#ifndef FK_BATCH_F32_BLOCKS_PER_CU
#define FK_BATCH_F32_BLOCKS_PER_CU 5
#endif

// Grid loops keep several grid loads in flight, which takes registers: mixed
// single-problem walks measured best at 5 blocks (96 VGPRs: 88 to 91 taken, and
// 5 to 13 spilled with the bridge test), mixed batches of
// separate sources at 4 (128 VGPRs; per-lane source fields), while a batch
// sharing one source stays at 5.
#ifndef FK_F32_GRID_BLOCKS_PER_CU
#define FK_F32_GRID_BLOCKS_PER_CU 5
#endif
#ifndef FK_BATCH_F32_GRID_BLOCKS_PER_CU
#define FK_BATCH_F32_GRID_BLOCKS_PER_CU 4
#endif
// FP64 batches of separate grids: 3 blocks (up to 170 VGPRs, 148 to 149 taken)
// hold the walk without the 28-register spill that 4 blocks cost when it was
// tried (whose stores reached memory at about 130 GB/s), and measured 3 % faster.
#ifndef FK_BATCH_F64_GRID_BLOCKS_PER_CU
#define FK_BATCH_F64_GRID_BLOCKS_PER_CU 3
#endif

// The adjoint's blocks are held to 3 per CU by their LDS (the 32 KiB table
// and the drain buffers), so their registers are bounded for 3.
constexpr int kAdjBlocksPerCu = 3;

template <bool F64, bool KAHAN, bool ADJ, int LOOP>
__global__ void __launch_bounds__(256, ADJ                ? kAdjBlocksPerCu
                                       : F64             ? FK_F64_BLOCKS_PER_CU
                                       : loop_grid(LOOP) ? FK_F32_GRID_BLOCKS_PER_CU
                                                         : FK_F32_BLOCKS_PER_CU)
    walk_kernel(const typename std::conditional<F64, WalkArgsF64, WalkArgsF32>::type A)
{
    walk_body<F64, KAHAN, ADJ, false, LOOP, false, false, false>(A);
}

// The adjoint with dense station tables: one block of kAdjDenseBlock threads
// per CU (the 128 KiB table takes most of the CU's 160 KiB of LDS).  FP64 spills
// 4 VGPRs of its 128 (20 bytes a lane; 28 with the bridge test), mixed none.
template <bool F64, bool KAHAN, int LOOP>
__global__ void __launch_bounds__(kAdjDenseBlock, 1)
    adjoint_dense_kernel(const typename std::conditional<F64, WalkArgsF64, WalkArgsF32>::type A)
{
    walk_body<F64, KAHAN, true, false, LOOP, false, true, false>(A);
}

template <bool F64, bool KAHAN, int LOOP, bool SHARED, bool UKEY>
__global__ void __launch_bounds__(256, loop_exit(LOOP)   ? 1
                                       : (F64 && loop_grid(LOOP) && !SHARED) ? FK_BATCH_F64_GRID_BLOCKS_PER_CU
                                       : F64             ? FK_BATCH_F64_BLOCKS_PER_CU
                                       : (loop_grid(LOOP) && !SHARED) ? FK_BATCH_F32_GRID_BLOCKS_PER_CU
                                                                      : FK_BATCH_F32_BLOCKS_PER_CU)
    batch_walk_kernel(const BatchArgs A)
{
    walk_body<F64, KAHAN, false, true, LOOP, SHARED, false, UKEY>(A);
}

}  // namespace

hipError_t launch_zero_queue(unsigned long long* queue, const LaunchCfg& cfg, hipStream_t stream, uint32_t* status,
                             uint32_t flags)
{
    hipLaunchKernelGGL(zero_queue_kernel, dim3(1), dim3(64), 0, stream, queue, (uint32_t)cfg.grid, cfg.stripes,
                       cfg.cap == 64u ? (uint32_t)cfg.block : 0u, status, flags);
    return hipGetLastError();
}

namespace {

// Calls f with the loop variant as a compile-time constant.
template <class F>
void with_loop(int loop, F&& f)
{
    switch (loop) {
    case 28: f(std::integral_constant<int, 28>{}); break;
    case 20: f(std::integral_constant<int, 20>{}); break;
    case 14: f(std::integral_constant<int, 14>{}); break;
    case 13: f(std::integral_constant<int, 13>{}); break;
    case 12: f(std::integral_constant<int, 12>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 1: f(std::integral_constant<int, 1>{}); break;
    default: f(std::integral_constant<int, 0>{});
    }
}

// The adjoint samples no density (it counts voxel visits), so its loop never
// carries the grid bit.
template <bool F64, bool KAHAN, bool ADJ, class A>
void launch_walk(const A& a, int loop, const LaunchCfg& cfg, hipStream_t stream, bool dense)
{
    with_loop(ADJ ? loop_exit(loop) : loop, [&](auto L) {
        constexpr int LOOP = ADJ ? loop_exit(decltype(L)::value) : decltype(L)::value;
        if constexpr (ADJ) {
            if (dense) {
                hipLaunchKernelGGL((adjoint_dense_kernel<F64, KAHAN, LOOP>), dim3(cfg.grid), dim3(cfg.block), 0, stream,
                                   a);
                return;
            }
        }
        hipLaunchKernelGGL((walk_kernel<F64, KAHAN, ADJ, LOOP>), dim3(cfg.grid), dim3(cfg.block), 0, stream, a);
    });
}

template <int VARIANT, bool ADJ>
const void* walk_fn(int precision, bool dense)
{
    constexpr int LOOP = ADJ ? loop_exit(VARIANT) : VARIANT;
    if constexpr (ADJ) {
        if (dense)
            return precision == FK_F64 ? (const void*)adjoint_dense_kernel<true, false, LOOP>
                 : precision == FK_MIXED_KAHAN ? (const void*)adjoint_dense_kernel<false, true, LOOP>
                                               : (const void*)adjoint_dense_kernel<false, false, LOOP>;
    }
    return precision == FK_F64 ? (const void*)walk_kernel<true, false, ADJ, LOOP>
         : precision == FK_MIXED_KAHAN ? (const void*)walk_kernel<false, true, ADJ, LOOP>
                                       : (const void*)walk_kernel<false, false, ADJ, LOOP>;
}

// FP64 batches take the uniform key only with one shared source (+2 % on
// the SI-prism FP64 batch).  Batches of separate sources keep the per-lane
// key: their walks already fill the scalar registers, and with the key
// schedule there too they spill more and measured 1.6 % slower (the
// 32-model FP64 grid batch).
template <bool SHARED, bool UKEY>
constexpr bool kF64Ukey = SHARED && UKEY;

template <int LOOP, bool SHARED, bool UKEY>
const void* batch_fn(int precision)
{
    return precision == FK_F64 ? (const void*)batch_walk_kernel<true, false, LOOP, SHARED, kF64Ukey<SHARED, UKEY>>
         : precision == FK_MIXED_KAHAN ? (const void*)batch_walk_kernel<false, true, LOOP, SHARED, UKEY>
                                       : (const void*)batch_walk_kernel<false, false, LOOP, SHARED, UKEY>;
}

template <int LOOP, bool SHARED, bool UKEY>
void launch_batch(const BatchArgs& a, const LaunchCfg& cfg, hipStream_t stream)
{
    if (a.precision == FK_F64)
        hipLaunchKernelGGL((batch_walk_kernel<true, false, LOOP, SHARED, kF64Ukey<SHARED, UKEY>>), dim3(cfg.grid),
                           dim3(cfg.block), 0, stream, a);
    else if (a.precision == FK_MIXED_KAHAN)
        hipLaunchKernelGGL((batch_walk_kernel<false, true, LOOP, SHARED, UKEY>), dim3(cfg.grid), dim3(cfg.block), 0,
                           stream, a);
    else
        hipLaunchKernelGGL((batch_walk_kernel<false, false, LOOP, SHARED, UKEY>), dim3(cfg.grid), dim3(cfg.block), 0,
                           stream, a);
}

// Calls f with (shared source, uniform key) as compile-time constants.
template <class F>
void with_batch_mode(bool shared, bool ukey, F&& f)
{
    if (shared) {
        if (ukey) f(std::true_type{}, std::true_type{});
        else f(std::true_type{}, std::false_type{});
    } else {
        if (ukey) f(std::false_type{}, std::true_type{});
        else f(std::false_type{}, std::false_type{});
    }
}

}  // namespace

hipError_t launch_walk_f64(const WalkArgsF64& a, const LaunchCfg& cfg, hipStream_t stream, int loop, bool adjoint,
                           bool dense)
{
    if (adjoint)
        launch_walk<true, false, true>(a, loop, cfg, stream, dense);
    else
        launch_walk<true, false, false>(a, loop, cfg, stream, false);
    return hipGetLastError();
}

hipError_t launch_walk_f32(const WalkArgsF32& a, bool kahan, const LaunchCfg& cfg, hipStream_t stream, int loop,
                           bool adjoint, bool dense)
{
    if (adjoint) {
        if (kahan)
            launch_walk<false, true, true>(a, loop, cfg, stream, dense);
        else
            launch_walk<false, false, true>(a, loop, cfg, stream, dense);
    } else {
        if (kahan)
            launch_walk<false, true, false>(a, loop, cfg, stream, false);
        else
            launch_walk<false, false, false>(a, loop, cfg, stream, false);
    }
    return hipGetLastError();
}

hipError_t walk_occupancy(int precision, int block, int* blocks_per_cu, int loop, bool adjoint, bool dense)
{
    const void* fn = nullptr;
    if (adjoint)
        with_loop(loop_exit(loop), [&](auto L) { fn = walk_fn<decltype(L)::value, true>(precision, dense); });
    else
        with_loop(loop, [&](auto L) { fn = walk_fn<decltype(L)::value, false>(precision, false); });
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, block, 0);
}

hipError_t launch_batch_walk(const BatchArgs& a, const LaunchCfg& cfg, hipStream_t stream, int loop, bool shared)
{
    with_loop(loop, [&](auto L) {
        with_batch_mode(shared, a.uniform_key != 0, [&](auto S, auto U) {
            launch_batch<decltype(L)::value, decltype(S)::value, decltype(U)::value>(a, cfg, stream);
        });
    });
    return hipGetLastError();
}

hipError_t batch_occupancy(int precision, int block, int* blocks_per_cu, int loop, bool shared, bool ukey)
{
    const void* fn = nullptr;
    with_loop(loop, [&](auto L) {
        with_batch_mode(shared, ukey, [&](auto S, auto U) {
            fn = batch_fn<decltype(L)::value, decltype(S)::value, decltype(U)::value>(precision);
        });
    });
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, block, 0);
}

// ---------------------------------------------------------------------------
// Diagnostic: the random stream as the walk kernels compute it.
// ---------------------------------------------------------------------------
namespace {

__global__ void stream_blocks_kernel(const uint32_t* ctr, int64_t n, uint32_t key0, uint32_t key1, uint32_t* words,
                                     double* z64, float* z32)
{
    BmTables* bmt = bm_tables();
    fill_bm_tables(*bmt);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Block b = philox10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], key0, key1);
    if (words) {
        words[4 * i] = b.w0;
        words[4 * i + 1] = b.w1;
        words[4 * i + 2] = b.w2;
        words[4 * i + 3] = b.w3;
    }
    if (z64) normals_f64(b, *bmt, z64[2 * i], z64[2 * i + 1]);
    if (z32) {
        normals_f32(b.w0, b.w1, z32[4 * i], z32[4 * i + 1]);
        normals_f32(b.w2, b.w3, z32[4 * i + 2], z32[4 * i + 3]);
    }
}

}  // namespace

hipError_t launch_stream_blocks(const uint32_t* ctr, int64_t n, uint32_t key0, uint32_t key1, uint32_t* words,
                                double* z64, float* z32, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(stream_blocks_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, ctr, n, key0,
                       key1, words, z64, z32);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Adjoint helpers.
// ---------------------------------------------------------------------------
namespace {

__global__ void fill_zero_kernel(int64_t* p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// grad_rho[v] = sum_s coef_s counts[s][v], s in order, with
// coef_s = grad_out[s] * scale / n_s (n_s = untruncated samples of station s).
__global__ void combine_kernel(const int64_t* counts, int64_t n_stations, int64_t nvox, const double* grad_out,
                               const fk_stat* fwd, double scale, double* grad_rho)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (int64_t)gridDim.x * blockDim.x) {
        double acc = 0.0;
        for (int64_t s = 0; s < n_stations; ++s) {
            const int64_t ns = fwd[s].n;
            if (ns <= 0) continue;
            const double coef = grad_out[s] * scale / (double)ns;
            acc += coef * (double)counts[s * nvox + v];
        }
        grad_rho[v] = acc;
    }
}

}  // namespace

hipError_t launch_fill_zero(int64_t* p, int64_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const int64_t blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p, n);
    return hipGetLastError();
}

hipError_t launch_adjoint_combine(const int64_t* counts, int64_t n_stations, int64_t nvox, const double* grad_out,
                                  const fk_stat* fwd, double scale, double* grad_rho, hipStream_t stream)
{
    const int64_t blocks = (nvox + 255) / 256 < 8192 ? (nvox + 255) / 256 : 8192;
    hipLaunchKernelGGL(combine_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, counts, n_stations, nvox,
                       grad_out, fwd, scale, grad_rho);
    return hipGetLastError();
}

}  // namespace fk
