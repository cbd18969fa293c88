// The chain program of the register-resident Gaussian kernels: one chain per wavefront, kC pairs of components per lane.
//
// The recursion over the trajectory's tree needs no return stack here.  Leaf m (1-based) of a doubling of 2^j leaves
// completes the subtrees of levels 1 .. ctz(m), and unless it is the last leaf the subtree it leaves behind is the left
// half of the one of level ctz(m) + 1: the pair (j, m) says where the program stands, and a leaf or a span that must not
// be continued ends the whole doubling.  The lanes of a wave agree on it; what is decided by vector arithmetic becomes a scalar
// by a vote (agreed), so every branch is a scalar one and the program's state stays in scalar registers.
//
// A step of one chain is a serial chain of instructions, and with few chains its latency is all that counts (d = 100
// banded, 1024 chains, one wave per SIMD: a step takes 0.9 us).  What is done about it here:
//   * the lowest level of the tree stays in registers (an odd leaf is kept until its neighbour has been merged with it),
//   * the first leaves of the next levels and the pool's first buffers are in LDS as far as it reaches (n_first, n_pool),
//   * the other end of the trajectory and the proposal are in registers (kHeld),
//   * the uniforms of the merges of four leaves come from one generator pass,
//   * the sums of a leaf and of the two-leaf span it closes are taken together (wave_sum_rows), sums stay in vector registers,
//     and memory is addressed in its own space: 10.8 -> 9.26 ms (d = 2, 4 chains: 673 -> 581 us; d = 1000 binary32, 16384 chains,
//     where instructions bound it: 53.8 -> 48.0 ms).
// d = 100 banded, 1024 chains, 100 iterations: 15.3 ms (tree storage in global memory, a return stack) -> 9.26 ms.
#pragma once
#include "nuts_dev.h"
#include "nuts_fastmath.h"
#include "nuts_rng.h"

namespace nuts {

constexpr int kRowMaxDepth = 20;

// Workspace vectors of one slot (128 kC elements each), D = max_tree_depth:
//   2*b + c                 proposal pool, b <= D, c in {theta, grad}
//   2*(D+1) + 2*s + c       first-leaf slots, s <= D, c in {theta, r}
//   4*(D+1) + x             x < 5: the other end (theta, r, grad) and the proposal (theta, grad), unless kHeld
enum : int { kRowOtherTh = 0, kRowOtherR = 1, kRowOtherG = 2, kRowTop = 3, kRowTopG = 4, kRowRest = 5 };
__host__ __device__ inline int row_num_vectors(int max_depth) { return 4 * (max_depth + 1) + kRowRest; }

template <typename T>
struct RowVec;
template <>
struct RowVec<float> {
    typedef float2 type;
};
template <>
struct RowVec<double> {
    typedef double2 type;
};

// How much of the tree's storage a slot has in LDS.
struct RowLds {
    int n_first;  // first-leaf slots 2 .. n_first + 1
    int n_pool;   // pool buffers 0 .. n_pool - 1
};
inline size_t row_entry_bytes(int kc, size_t elem) { return (size_t)2 * 128 * kc * elem; }  // one slot or buffer
// Of `bytes` of LDS per slot: the first leaves are read back by every merge, so they come first.
// (without gradients pool buffers are written and hardly ever read: they stay in memory)
inline RowLds row_lds_split(size_t bytes, int kc, size_t elem, int max_depth, bool grad)
{
    const int n = (int)(bytes / row_entry_bytes(kc, elem)), most = max_depth > 1 ? max_depth - 1 : 0;
    RowLds r;
    r.n_first = n < most ? n : most;
    r.n_pool = !grad ? 0 : n - r.n_first < max_depth + 1 ? n - r.n_first : max_depth + 1;
    return r;
}

// Chains that take turns.  A slot that keeps a chain to its end leaves the chip half idle while the last chains finish.  So the last chains of
// a call are handed over between two iterations, when little more than the position belongs to a chain: a slot that has
// taken so many steps (kTurnSteps) with one of them puts it at the end of a queue and takes the one that has waited longest, unless none
// waits.  Every chain that is neither waiting nor finished has a slot, so a slot that finds the queue empty has nothing to wait
// for: it goes on with its chain, or ends.
// A turn costs some 10 us, and 70 where 2048 slots turn at once, as they do while all chains take about as many steps: hence so many steps
// between two of them, fewer where the chains' lengths differ less and a call has fewer of them (dense kernels).  Time without turns over time with, after 256, 512 (dense:
// 400) and 1024 (512) steps: diagonal, d = 130 binary64, 3000 chains, 1.25 1.24 1.24; d = 1000 binary32, 16384 chains, 1.05 1.06 1.07; equal scales, d = 100
// binary32, 16384 chains, 0.76 0.88 0.98, d = 200 binary64, 4096 chains, 0.81 0.94 1.00; banded, d = 100, 4096 chains, 1.12 1.11 1.12, d = 120 with four
// steps a leaf, 0.4 ms, 0.78 0.97 0.98; full, d = 60 binary64, 1500 chains, 1.27 1.18 1.10.  (A time between turns, in place of steps, fills
// itself with turns where many slots turn at once: 0.15 ms 0.43 to 1.1.)  Which calls take turns, and kTurnStepsEven: turn_steps in nuts_api.hip.
// More chains than kTurnChains per slot would not shorten the end.
constexpr int kTurnChains = 8;
constexpr unsigned kTurnSteps = 1024, kTurnStepsDense = 400, kTurnStepsEven = 256;
// What a slot needs for that is read from memory where a turn ends: in scalar registers throughout it would cost every step
// (d = 2, 4 chains 1.02 times as long).
struct RowTurns {
    unsigned mask;      // the ring has mask + 1 words: 0, or 1 + a chain's number from `first`; at least as many as there are chains in turns
    unsigned row_bytes;
    unsigned steps;     // that a slot takes with a chain while others wait
    char* rows;         // of each chain in turns: position (and gradient), log-density, iteration
    long first;         // chains from here on take turns
};
// words of the queue: head, tail and count, each in a line of its own, the plan above, the ring
enum : int { kTurnHead = 0, kTurnTail = 32, kTurnCount = 64, kTurnPlan = 96, kTurnRing = 128 };
__host__ __device__ inline size_t row_turn_bytes(int kc, size_t elem, bool grad) { return ((size_t)(grad ? 2 : 1) * 128 * kc * elem + 16 + 127) & ~(size_t)127; }

// Chains whose vectors take up more of a lane than this keep their slot: their kernels have no register left for more code.  (The element-wise one
// with the code for turns spills to accumulation registers and to scratch memory at once, and the compiler then lost a register of a
// reload: faults_in_assembly in build.py.  The code for turns had no part in the wrong values that this gave.)
constexpr int kTurnLaneBytes = 128;
template <typename T, int kC>
constexpr bool row_takes_turns() { return 2 * kC * (int)sizeof(T) <= kTurnLaneBytes; }

// What a slot takes up: nothing is left, a chain that begins (the caller owes start_chain its gradient), or one that goes on.
enum : int { kTakeNone = 0, kTakeFresh = 1, kTakeAgain = 2 };

// kGrad: the gradient belongs to the state (otherwise the kernel recomputes it from the position and g is not touched).
// kAhead: an iteration's random numbers that do not depend on where the trajectory goes may be drawn before it begins.
// kTurns: the call's last chains may take turns (take() in place of fetch()).
template <typename T, int kC, bool kHeld, bool kGrad, bool kAhead = false, bool kTurns = false>
struct RowChain {
    static constexpr int kVpl = 2 * kC, kPitch = 128 * kC;
    typedef T VecN __attribute__((ext_vector_type(2)));
    // (pointers of their address spaces: where one of two addresses of different spaces is taken the compiler would
    // otherwise make a generic pointer of both and flat instructions, which wait for both memories)
    typedef __attribute__((address_space(1))) T* GlobalPtr;
    typedef __attribute__((address_space(3))) T* LdsPtr;
    static __device__ __forceinline__ __attribute__((address_space(1))) VecN* vec_at(GlobalPtr p) { return (__attribute__((address_space(1))) VecN*)p; }
    static __device__ __forceinline__ __attribute__((address_space(3))) VecN* vec_at(LdsPtr p) { return (__attribute__((address_space(3))) VecN*)p; }

    const DevSample& sa;
    const int lane, d, D;
    const GlobalPtr ws;  // this slot's vectors in global memory
    const LdsPtr lds;    // this slot's vectors in LDS: n_first pairs, then n_pool pairs
    const RowLds rl;

    T th[kVpl], r[kVpl], g[kGrad ? kVpl : 1];     // the end of the trajectory that the current doubling extends
    T pth[kVpl], pr[kVpl], pg[kGrad ? kVpl : 1];  // the last odd leaf, until the leaf after it has been merged with it
    T rest[kHeld ? kRowRest : 1][kHeld ? kVpl : 1];
    static constexpr uint32_t kNoSeveral = 1u << 31;  // (no iteration follows it)
    static constexpr int kInEdge = -1, kInPrev = -2;  // cur_idx / frame_idx: the proposal is th, or pth

    int j = 0, m = 0, v = 0, nleap = 0, iter = 0;  // v: direction of the end in th (0: both ends are the same point)
    long chain = 0;
    uint32_t gchain = 0, free_mask = 0;
    // Weights of trajectory points are numbers, not logarithms: a leaf weighs exp(H0 - H) / unit (slice sampler: 1 or 0),
    // a subtree the sum of its leaves, so a merge is an add and a selection one product and a comparison.  log_unit_w is
    // the logarithm of the unit: 0 until a leaf's energy falls more than 600 below what the unit can represent; then
    // that leaf becomes the unit and what the iteration holds is rescaled.
    double H0 = 0, w_tree = 0, cur_w = 0, log_unit_w = 0, edge_logp = 0, prev_logp = 0, top_logp = 0, log_slice = 0;
    // Random numbers that do not depend on where the trajectory goes, one generator pass for many: lane j < 32 votes the
    // direction of doubling j into dirbits and lane 32 + j holds the TOP uniform of doubling j (once per iteration);
    // lane 16 q + l holds the SUBTREE uniform of level u_sub_base + l for the leaf that ends q leaf pairs after leapfrog count
    // u_sub_leaf: only every second leaf can complete a merge.
    double u_top = 0, u_sub = 0;
    uint32_t dirbits = 0;
    int u_sub_leaf = 0, u_sub_base = 0;
    int cur_s = 0, cur_idx = kInEdge;
    double frame_w = 0, pool_logp = 0;  // lane k: level k / pool buffer k
    int frame_idx = 0;
    unsigned long long n_leaf = 0, n_extra = 0;
    T r_next[kAhead ? kVpl : 1];  // drawn for iteration `ahead`: the momentum, |r|^2, and what dirbits, u_top and log_slice will be
    double kin_next = 0, u_top_next = 0, log_slice_next = 0;
    uint32_t dirbits_next = 0;
    int ahead = -1;
    T several[2] = {};             // momenta of the iterations from several_from on (draw_momentum)
    uint32_t several_from = kNoSeveral;
    unsigned* const turns;   // NULL: no turns
    unsigned turn_from = 0;  // n_leaf when the slot took its chain

    __device__ RowChain(const DevSample& sa_, int d_, int lane_, T* ws_, T* lds_, RowLds rl_, unsigned* turns_ = nullptr)
        : sa(sa_), lane(lane_), d(d_), D(sa_.max_depth), ws((GlobalPtr)ws_), lds((LdsPtr)lds_), rl(rl_), turns(turns_) {}

    __device__ int elem(int q, int e) const { return (q * kWave + lane) * 2 + e; }  // component of register 2q + e
    __device__ DrawKey key() const { return DrawKey{sa.key0, sa.key1}; }

    template <typename P>
    __device__ __forceinline__ void load(P src, T (&dst)[kVpl]) const
    {
#pragma unroll
        for (int q = 0; q < kC; ++q) {
            const VecN x = *vec_at(src + elem(q, 0));
            dst[2 * q] = x[0];
            dst[2 * q + 1] = x[1];
        }
    }
    template <typename P>
    __device__ __forceinline__ void store(P dst, const T (&src)[kVpl]) const
    {
#pragma unroll
        for (int q = 0; q < kC; ++q) *vec_at(dst + elem(q, 0)) = VecN{src[2 * q], src[2 * q + 1]};
    }
    __device__ __forceinline__ void copy(T (&dst)[kVpl], const T (&src)[kVpl]) const
    {
#pragma unroll
        for (int i = 0; i < kVpl; ++i) dst[i] = src[i];
    }
    // two vectors of a pool buffer or first-leaf slot (LDS and global memory are different instructions: no generic pointer)
    __device__ __forceinline__ void pair_load(int in_lds, int lds_entry, int vec, T (&a)[kVpl], T (&b)[kVpl]) const
    {
        if (in_lds) {
            load(lds + (size_t)(2 * lds_entry) * kPitch, a);
            load(lds + (size_t)(2 * lds_entry + 1) * kPitch, b);
        } else {
            load(ws + (size_t)vec * kPitch, a);
            load(ws + (size_t)(vec + 1) * kPitch, b);
        }
    }
    __device__ __forceinline__ void pair_store(int in_lds, int lds_entry, int vec, const T (&a)[kVpl], const T (&b)[kVpl]) const
    {
        if (in_lds) {
            store(lds + (size_t)(2 * lds_entry) * kPitch, a);
            store(lds + (size_t)(2 * lds_entry + 1) * kPitch, b);
        } else {
            store(ws + (size_t)vec * kPitch, a);
            store(ws + (size_t)(vec + 1) * kPitch, b);
        }
    }
    __device__ __forceinline__ void first_load(int s, T (&a)[kVpl], T (&b)[kVpl]) const
    {
        pair_load(s - 2 < rl.n_first, s - 2, 2 * (D + 1) + 2 * s, a, b);
    }
    __device__ __forceinline__ void first_store(int s, const T (&a)[kVpl], const T (&b)[kVpl]) const
    {
        pair_store(s - 2 < rl.n_first, s - 2, 2 * (D + 1) + 2 * s, a, b);
    }
    template <int kG>
    __device__ __forceinline__ void pool_load(int b, T (&t)[kVpl], T (&gr)[kG]) const
    {
        if constexpr (kGrad)
            pair_load(b < rl.n_pool, rl.n_first + b, 2 * b, t, gr);
        else
            load(ws + (size_t)(2 * b) * kPitch, t);
    }
    template <int kG>
    __device__ __forceinline__ void pool_store(int b, const T (&t)[kVpl], const T (&gr)[kG]) const
    {
        if constexpr (kGrad)
            pair_store(b < rl.n_pool, rl.n_first + b, 2 * b, t, gr);
        else
            store(ws + (size_t)(2 * b) * kPitch, t);
    }
    __device__ __forceinline__ void rest_load(int x, T (&a)[kVpl]) const
    {
        if constexpr (kHeld)
            copy(a, rest[x]);
        else
            load(ws + (size_t)(4 * (D + 1) + x) * kPitch, a);
    }
    __device__ __forceinline__ void rest_store(int x, const T (&a)[kVpl])
    {
        if constexpr (kHeld)
            copy(rest[x], a);
        else
            store(ws + (size_t)(4 * (D + 1) + x) * kPitch, a);
    }

    // Standard normals for every component, zero beyond d (components 2k, 2k + 1 share draw k: they are in one lane).
    __device__ __forceinline__ void draw_normals(uint32_t tag, uint32_t iteration, T (&out)[kVpl]) const
    {
#pragma unroll 1
        for (int q = 0; q < kC; ++q) {  // rolled: once per iteration, must not cost registers
            double z0 = 0.0, z1 = 0.0;
            const int i = elem(q, 0);
            if (i < d) {
                normal_pair(draw(key(), (uint32_t)(i >> 1), tag, 0, iteration, gchain), z0, z1);
                if (i + 1 >= d) z1 = 0.0;
            }
            // (the pairs move up by one each time: an index that depends on q would put the array in scratch memory)
#pragma unroll
            for (int i = 0; i + 2 < kVpl; ++i) out[i] = out[i + 2];
            out[kVpl - 2] = (T)z0;
            out[kVpl - 1] = (T)z1;
        }
    }

    // Momenta.  Of up to 64 components one pass of the generator, and the logarithm, root, sine and cosine after it, serves 64 / n
    // iterations, n the power of two from the number of pairs on: lane n k + p makes pair p of the k-th one.  d = 2, 4 chains, 100 iterations
    // 584 -> 530 us.  (Kernels that hold a gradient have no scalar registers for it: d = 100 banded 1.02 times as long.)
    __device__ __forceinline__ void draw_momentum(uint32_t iteration, T (&out)[kVpl])
    {
        if constexpr (kC > 1 || kGrad) {
            draw_normals(kDrawMomentum, iteration, out);
        } else {
            const int pairs = (d + 1) >> 1, shift = pairs > 1 ? 32 - __builtin_clz(pairs - 1) : 0, per = kWave >> shift;
            if (iteration - several_from >= (unsigned)per) {
                const int p = lane & ((1 << shift) - 1);
                double z0, z1;
                normal_pair(draw(key(), (uint32_t)p, kDrawMomentum, 0, iteration + (uint32_t)(lane >> shift), gchain), z0, z1);
                several[0] = p < pairs ? (T)z0 : T(0);
                several[1] = 2 * p + 1 < d ? (T)z1 : T(0);
                several_from = iteration;
            }
            const int from = lane < pairs ? ((int)(iteration - several_from) << shift) + lane : 0;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const T x = __shfl(several[e], from, kWave);
                out[e] = lane < pairs ? x : T(0);
            }
        }
    }

    __device__ uint32_t all_bufs() const { return (1u << (D + 1)) - 1u; }
    // The current proposal gets a pool buffer, unless it has one.
    __device__ __forceinline__ void materialise_cur()
    {
        if (cur_idx >= 0) return;
        const int b = __ffs(free_mask) - 1;
        free_mask &= ~(1u << b);
        if (cur_idx == kInPrev) {
            pool_store(b, pth, pg);
            if (lane == b) pool_logp = prev_logp;
        } else {
            pool_store(b, th, g);
            if (lane == b) pool_logp = edge_logp;
        }
        cur_idx = b;
    }

    // This lane's shares of (theta+ - theta-) . r at both ends of the span between the extended end and (xt, xr), times the
    // direction: the difference is taken edge minus (xt), and the sums' sign turned afterwards (negation is exact).
    __device__ __forceinline__ void span_dots(const T (&xt)[kVpl], const T (&xr)[kVpl], double& da, double& db) const
    {
        da = db = 0.0;
#pragma unroll
        for (int i = 0; i < kVpl; ++i) {
            const T delta = th[i] - xt[i];
            da = fma((double)delta, (double)xr[i], da);
            db = fma((double)delta, (double)r[i], db);
        }
    }
    __device__ __forceinline__ bool no_uturn(const T (&xt)[kVpl], const T (&xr)[kVpl]) const
    {
        double da, db;
        span_dots(xt, xr, da, db);
        return __ballot((double)v * wave_sum_halves(da, db) >= 0.0) == ~0ull;
    }

    // Takes the next chain from the queue; false if there is none.  Its starting point is in th, and the caller owes
    // start_chain() that point's gradient.
    __device__ bool fetch()
    {
        unsigned long long c = 0;
        if (lane == 0) c = atomicAdd(&sa.counters[kCtrQueue], 1ull);
        const unsigned lo = (unsigned)uni((int)(unsigned)c), hi = (unsigned)uni((int)(unsigned)(c >> 32));
        c = ((unsigned long long)hi << 32) | lo;
        if ((long)c >= sa.n_chains) return false;
        chain = (long)c;
        gchain = (uint32_t)(sa.first_chain + chain);
        iter = sa.iter_begin;
        ahead = -1;
        several_from = kNoSeveral;
        if (sa.init_states) {
            const T* src = (const T*)sa.init_states + (size_t)chain * d;
#pragma unroll
            for (int q = 0; q < kC; ++q)
#pragma unroll
                for (int e = 0; e < 2; ++e) th[2 * q + e] = elem(q, e) < d ? src[elem(q, e)] : T(0);
        } else {
            draw_normals(kDrawInit, 0, th);
        }
        return true;
    }
    // A chain's row goes past the caches, which the XCDs do not share: words at agent scope, and the queue's word after them.
    __device__ const RowTurns& turn_plan() const { return *reinterpret_cast<const RowTurns*>(turns + kTurnPlan); }
    __device__ unsigned long long* turn_row() const
    {
        const RowTurns& plan = turn_plan();
        return (unsigned long long*)(plan.rows + (size_t)(chain - plan.first) * plan.row_bytes);
    }
    static __device__ __forceinline__ void put(unsigned long long* p, unsigned long long x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    static __device__ __forceinline__ unsigned long long got(const unsigned long long* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ void turn_put(unsigned long long* row, const T (&x)[kVpl]) const
    {
#pragma unroll
        for (int q = 0; q < kC; ++q) {
            if constexpr (sizeof(T) == 4) {
                put(row + q * kWave + lane, ((unsigned long long)__float_as_uint(x[2 * q + 1]) << 32) | __float_as_uint(x[2 * q]));
            } else {
                put(row + elem(q, 0), (unsigned long long)__double_as_longlong(x[2 * q]));
                put(row + elem(q, 1), (unsigned long long)__double_as_longlong(x[2 * q + 1]));
            }
        }
    }
    __device__ __forceinline__ void turn_got(const unsigned long long* row, T (&x)[kVpl]) const
    {
#pragma unroll
        for (int q = 0; q < kC; ++q) {
            if constexpr (sizeof(T) == 4) {
                const unsigned long long w = got(row + q * kWave + lane);
                x[2 * q] = __uint_as_float((unsigned)w);
                x[2 * q + 1] = __uint_as_float((unsigned)(w >> 32));
            } else {
                x[2 * q] = __longlong_as_double((long long)got(row + elem(q, 0)));
                x[2 * q + 1] = __longlong_as_double((long long)got(row + elem(q, 1)));
            }
        }
    }
    static constexpr int kTurnWords = kPitch * (int)sizeof(T) / 8;  // of a vector

    // Whether a chain waits for a slot (it may be gone when it is asked for).
    __device__ bool others_wait() const
    {
        return agreed((long)got(&sa.counters[kCtrQueue]) < sa.n_chains) || uni(turns_waiting()) > 0;
    }
    __device__ __forceinline__ int turns_waiting() const { return (int)__hip_atomic_load(turns + kTurnCount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ void hand_over()
    {
        unsigned long long* row = turn_row();
        T x[kVpl];
        rest_load(kRowTop, x);
        turn_put(row, x);
        if constexpr (kGrad) {
            rest_load(kRowTopG, x);
            turn_put(row + kTurnWords, x);
        }
        if (lane == 0) {
            put(row + (kGrad ? 2 : 1) * kTurnWords, (unsigned long long)__double_as_longlong(top_logp));
            put(row + (kGrad ? 2 : 1) * kTurnWords + 1, (unsigned long long)iter);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) {
            const unsigned t = __hip_atomic_fetch_add(turns + kTurnTail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned* p = turns + kTurnRing + (t & turn_plan().mask);
            unsigned expected = 0u;  // (occupied only by a chain that another slot is about to take)
            while (!__hip_atomic_compare_exchange_strong(p, &expected, 1u + (unsigned)(chain - turn_plan().first), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT))
                expected = 0u;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __hip_atomic_fetch_add(turns + kTurnCount, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // The chain that has waited longest, if any waits.  Whoever hands a chain over, or takes back its claim on the count, looks at the
    // count after that: so no chain is left behind.
    __device__ bool take_again()
    {
        unsigned taken = 0;
        // (a look before the claim, unless this slot has just handed a chain over: claims made in vain by 2048 slots that end at the same time took 100 us, the
        // look of 1024 slots that turn at the same time 20 us)
        if (lane == 0 && (iter < sa.iter_end || turns_waiting() > 0)) {
            for (;;) {
                if ((int)__hip_atomic_fetch_add(turns + kTurnCount, ~0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0) {
                    const unsigned h = __hip_atomic_fetch_add(turns + kTurnHead, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    unsigned* p = turns + kTurnRing + (h & turn_plan().mask);
                    do  // (counted chains are in the ring, or an earlier place in it is being filled this moment)
                        taken = __hip_atomic_exchange(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    while (taken == 0u);
                    break;
                }
                const int left = (int)__hip_atomic_fetch_add(turns + kTurnCount, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
                if (left <= 0 && turns_waiting() <= 0) break;
            }
        }
        taken = (unsigned)uni((int)taken);
        if (taken == 0u) return false;
        asm volatile("" ::: "memory");
        chain = turn_plan().first + (long)taken - 1;
        gchain = (uint32_t)(sa.first_chain + chain);
        ahead = -1;
        several_from = kNoSeveral;
        const unsigned long long* row = turn_row();
        T x[kVpl];
        turn_got(row, x);
        rest_store(kRowTop, x);
        if constexpr (kGrad) {
            turn_got(row + kTurnWords, x);
            rest_store(kRowTopG, x);
        }
        top_logp = __longlong_as_double((long long)got(row + (kGrad ? 2 : 1) * kTurnWords));
        iter = uni((int)got(row + (kGrad ? 2 : 1) * kTurnWords + 1));
        return true;
    }
    __device__ int take()
    {
        if constexpr (!kTurns) {
            return fetch() ? kTakeFresh : kTakeNone;
        } else {
            turn_from = (unsigned)n_leaf;
            return fetch() ? kTakeFresh : turns && take_again() ? kTakeAgain : kTakeNone;
        }
    }

    __device__ void start_chain(double lp)  // lp: this lane's share of theta . grad
    {
        rest_store(kRowTop, th);
        if constexpr (kGrad) rest_store(kRowTopG, g);
        top_logp = 0.5 * wave_sum(lp);
        n_extra += 1;
    }

    __device__ __forceinline__ void draw_iteration(int it, T (&momentum)[kVpl], double& kin, double& tops, double& slice, uint32_t& dirs)
    {
        draw_momentum((uint32_t)it, momentum);
        kin = 0.0;
#pragma unroll
        for (int i = 0; i < kVpl; ++i) kin = fma((double)momentum[i], (double)momentum[i], kin);
        kin = wave_sum(kin);
        if (sa.sampler == kSamplerSlice) {
            const Words4 w = draw(key(), 0, kDrawSlice, 0, (uint32_t)it, gchain);
            slice = log(uniform52(w.w0, w.w1));
        }
        const Words4 wj = draw(key(), (uint32_t)(lane & 31), (lane & 32) ? kDrawTop : kDrawDirection, 0, (uint32_t)it, gchain);
        dirs = (uint32_t)__ballot(wj.w0 >> 31);
        tops = uniform52(wj.w0, wj.w1);
    }
    __device__ void draw_ahead(int it)
    {
        draw_iteration(it, r_next, kin_next, u_top_next, log_slice_next, dirbits_next);
        ahead = it;
    }

    __device__ void iter_begin()
    {
        rest_load(kRowTop, th);
        if constexpr (kGrad) rest_load(kRowTopG, g);
        double kin;
        if constexpr (kAhead) {
            if (ahead != iter) draw_ahead(iter);
            copy(r, r_next);
            kin = kin_next;
            u_top = u_top_next;
            log_slice = log_slice_next;
            dirbits = dirbits_next;
        } else {
            draw_iteration(iter, r, kin, u_top, log_slice, dirbits);
        }
        rest_store(kRowOtherTh, th);  // both ends of the trajectory start at the current point
        rest_store(kRowOtherR, r);
        if constexpr (kGrad) rest_store(kRowOtherG, g);
        v = 0;
        H0 = -top_logp + 0.5 * kin;
        w_tree = 1.0;  // the starting point: weight exp(0), or the first candidate
        log_unit_w = 0.0;
        u_sub_leaf = kNoLeaf;
        j = 0;
        nleap = 0;
    }

    __device__ void double_begin()
    {
        const int dir = ((dirbits >> j) & 1u) ? 1 : -1;
        if (v == -dir) {  // the doubling turns round: the two ends change places
            T xt[kVpl], xr[kVpl];
            rest_load(kRowOtherTh, xt);
            rest_load(kRowOtherR, xr);
            rest_store(kRowOtherTh, th);
            rest_store(kRowOtherR, r);
            copy(th, xt);
            copy(r, xr);
            if constexpr (kGrad) {
                rest_load(kRowOtherG, xt);
                rest_store(kRowOtherG, g);
                copy(g, xt);
            }
        }
        v = dir;
        m = 0;
        free_mask = all_bufs();  // nothing of the last doubling stays in the pool
    }

    // Half-kick and drift up to the position whose gradient is wanted, and the kick after it.
    __device__ __forceinline__ void kick_drift()
    {
        const T half = (T)(0.5 * (v * sa.eps)), full = (T)(v * sa.eps);
#pragma unroll
        for (int i = 0; i < kVpl; ++i) {
            r[i] = r[i] + half * g[i];
            th[i] = th[i] + full * r[i];
        }
    }
    __device__ __forceinline__ void kick()
    {
        const T half = (T)(0.5 * (v * sa.eps));
#pragma unroll
        for (int i = 0; i < kVpl; ++i) r[i] = r[i] + half * g[i];
    }

    // One subtree's halves become one: weights added, proposal selected, U-turn test over its span (of two leaves: pair_ok).
    __device__ __forceinline__ void merge(int level, bool pair_ok)
    {
        T xt[kVpl], xr[kVpl];
        if (level > 1) {
            // the subtree's first leaf is asked for before anything else: the latency runs under the random draw
            // and the weight arithmetic below
            const int f = m - (1 << level) + 1;  // first leaf of this subtree, 1-based
            first_load((f == 1) ? j : min(__ffs(f - 1) - 1, j), xt, xr);
        }
        const double l_w = read_lane(frame_w, level);
        const int l_idx = __builtin_amdgcn_readlane(frame_idx, level);
        const int gap = 2 * sa.leaf_steps;
        int ahead = nleap - u_sub_leaf;
        if ((ahead != 0 && ahead != gap && ahead != 2 * gap && ahead != 3 * gap) || (level & 16) != u_sub_base) {
            u_sub_base = level & 16;
            const Words4 w = draw(key(), (uint32_t)(nleap + (lane >> 4) * gap), kDrawSubtree, (uint32_t)(u_sub_base + (lane & 15)),
                                  (uint32_t)iter, gchain);
            u_sub = uniform52(w.w0, w.w1);
            u_sub_leaf = nleap;
            ahead = 0;
        }
        const int q = ahead == 0 ? 0 : (ahead == gap ? 1 : (ahead == 2 * gap ? 2 : 3));
        const double u = read_lane(u_sub, uni((level & 15) + 16 * q));
        // right with probability w_R / (w_L + w_R) (never when both are zero)
        const double w_new = l_w + cur_w;
        if (agreed(u * w_new < cur_w)) {
            if (l_idx >= 0) free_mask |= (1u << l_idx);
        } else {
            if (cur_idx >= 0) free_mask |= (1u << cur_idx);
            cur_idx = l_idx;
        }
        cur_w = w_new;
        cur_s = level > 1 ? no_uturn(xt, xr) : pair_ok;
    }

    // What follows a leaf's last leapfrog step (lp: this lane's share of theta . grad): its weight, then every merge it
    // completes.  True if the doubling wants another leaf.
    __device__ __forceinline__ bool finish_leaf(double lp)
    {
        double kin = 0.0;
#pragma unroll
        for (int i = 0; i < kVpl; ++i) kin = fma((double)r[i], (double)r[i], kin);
        m += 1;
        // An even leaf, if it is valid, is merged with the one before it: that span's two sums go with the leaf's own.
        bool pair_ok = false;
        if (m & 1) {
            wave_sum2(lp, kin);
        } else {
            double da, db;
            span_dots(pth, pr, da, db);
            const double x = wave_sum_rows(lp, kin, da, db);
            pair_ok = ((__ballot((double)v * x >= 0.0) >> 16) & 0xffff0000ffffull) == 0xffff0000ffffull;
            spread_halves(spread_even_rows(x), lp, kin);
        }
        edge_logp = 0.5 * lp;
        nleap += sa.leaf_steps;
        n_leaf += sa.leaf_steps;
        double delta = (-edge_logp + 0.5 * kin) - H0;
        if (!(fabs(delta) < INFINITY)) delta = INFINITY;
        if (sa.sampler == kSamplerSlice) {
            cur_w = (log_slice <= -delta) ? 1.0 : 0.0;
            cur_s = agreed(log_slice < kDeltaMax - delta);
        } else {
            double e = log_unit_w - delta;  // logarithm of the leaf's weight in the current unit
            if (agreed(e > 600.0)) {  // the energy has fallen far: this leaf becomes the unit
                const double shrink = exp_bounded(-e);
                w_tree *= shrink;
                frame_w *= shrink;
                log_unit_w = delta;
                e = 0.0;
            }
            cur_w = exp_bounded(e);
            cur_s = agreed(delta <= kDeltaMax);
        }
        cur_idx = kInEdge;
        if (!cur_s) return false;
        const int n_done = __ffs(m) - 1;  // levels that this leaf completes
        if (n_done == 0) {
            if (j == 0) return false;
            // the left half of a two-leaf subtree stays in registers; larger subtrees that it opens share one copy
            copy(pth, th);
            copy(pr, r);
            if constexpr (kGrad) copy(pg, g);
            prev_logp = edge_logp;
            cur_idx = kInPrev;
            const int s = (m == 1) ? j : min(__ffs(m - 1) - 1, j);
            if (s >= 2) first_store(s, th, r);
        } else {
            for (int level = 1; level <= n_done; ++level) {
                merge(uni(level), pair_ok);
                if (!cur_s) return false;
            }
            if (n_done == j) return false;
            materialise_cur();
        }
        if (lane == n_done + 1) {
            frame_w = cur_w;
            frame_idx = cur_idx;
        }
        return true;
    }

    // The end of a doubling; true if another one follows.
    __device__ bool double_end()
    {
        bool go_on = false;
        if (cur_s) {
            const double u = read_lane(u_top, uni(32 + j));
            if (agreed(u * w_tree < cur_w)) {  // accept the new half with probability min(1, w_new / w_tree)
                if (cur_idx == kInEdge) {
                    rest_store(kRowTop, th);
                    if constexpr (kGrad) rest_store(kRowTopG, g);
                    top_logp = edge_logp;
                } else if (cur_idx == kInPrev) {
                    rest_store(kRowTop, pth);
                    if constexpr (kGrad) rest_store(kRowTopG, pg);
                    top_logp = prev_logp;
                } else {
                    T t[kVpl], gr[kGrad ? kVpl : 1];
                    pool_load(cur_idx, t, gr);
                    rest_store(kRowTop, t);
                    if constexpr (kGrad) rest_store(kRowTopG, gr);
                    top_logp = read_lane(pool_logp, uni(cur_idx));
                }
            }
            w_tree += cur_w;
            T xt[kVpl], xr[kVpl];
            rest_load(kRowOtherTh, xt);
            rest_load(kRowOtherR, xr);
            go_on = no_uturn(xt, xr);
        }
        // (an invalid new half ends the iteration: the tree's weight is not needed any more)
        j += 1;
        return go_on && j < D;
    }

    // Emits the iteration's outputs; true if another iteration of the same chain follows.
    __device__ bool iter_end()
    {
        const size_t row = (size_t)iter * (size_t)sa.n_chains + (size_t)chain;
        if (sa.out_states) {
            T x[kVpl];
            rest_load(kRowTop, x);
            T* dst = (T*)sa.out_states + row * d;
#pragma unroll
            for (int q = 0; q < kC; ++q)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    if (elem(q, e) < d) dst[elem(q, e)] = x[2 * q + e];
        }
        if (lane == 0) {
            if (sa.out_depths) sa.out_depths[row] = j;
            if (sa.out_nleap) sa.out_nleap[row] = nleap;
        }
        iter += 1;
        if (iter >= sa.iter_end) return false;
        if constexpr (kTurns) {
            if (turns && (unsigned)n_leaf - turn_from >= turn_plan().steps && chain >= turn_plan().first && others_wait()) {
                hand_over();
                return false;
            }
        }
        return true;
    }
};

}  // namespace nuts
