// Wide tile kernel: logistic regression in either dtype with up to 128 features, NC = 16 or 4 chains per
// workgroup in lock step, their gradients together on the matrix cores.
//
// The round is that of the tile kernel (nuts_tile.h): 8 wavefronts; every chain has its program counter, return
// stack and tree state in the registers of 32 lanes, of which each owns up to 4 components of every state vector;
// control sweep, batched gradient  Z = X~ Theta, G = X~' s(Z)  on 16-row tiles of the same packed operand stream,
// completion.  What differs:
//   * any d <= 128 (MT = ceil(d / 16) feature tiles), binary64 arithmetic in the contraction for both dtypes (binary32
//     targets: state, momentum and gradient rounded to binary32 after every update, as in the general wave kernel);
//   * where it takes the general wave kernel's place (more than 32 features, or binary32), s is the residual sigma(-Z) as
//     there, and the log-likelihood is sum log sigma(|z~|) - sum max(-z~, 0), a product per row of a tile and lane.  The tile
//     kernel's s = sign(Z) F'(|Z|) with half the column sums added is cheaper, but a difference of large sums: 5000 x 60 at
//     the posterior, against 113 bits, gradient off by 2.9e-12 (wave kernel 4.9e-13, residuals 1.5e-13) and log-density
//     by 3.7e-12 (1.2e-13, 7.5e-14), other shapes alike;
//   * NC = 4 runs the two GEMMs on v_mfma_f64_4x4x4_4b: its four blocks are the four groups of 4 rows (first GEMM) or
//     of 4 features (second GEMM) of the 16x16x4 instruction's operands in the same lanes, and an element of the result
//     is accumulated in the same order, as is the log-likelihood: a chain has the same bits whichever form stepped it
//     (with up to 32 features and binary64 the 16-chain form is the kernel of nuts_tile.h).
//   * NC = 4 with kSplit: the rows of a group of four chains go to two workgroups of four waves, each of which has a SIMD to
//     itself and one of the eight sums over rows that a wave of the undivided form has, so the bits are the same.  Both workgroups
//     run the chain program of all four chains (it is deterministic: nothing but the sums has to be exchanged, once a round, and
//     one of them writes the outputs).
// The numbers of chains, rows and iterations decide between the forms (wide_chains_per_block, wide_split_pays below).
//
// What bounds it: with 16 chains the matrix instructions (1000 rows x 120 features: 63.5 k of the gradient phase's 83 k ticks,
// its logistic functions another 10 k; with few features the latter: 3000 x 5 in binary32 38 k of 58 k); with 4 chains the
// operand stream, which every compute unit reads from L2 at about 50 bytes per tick (1000 x 60: 1 MB in 20 k ticks, where
// the instructions would take 11 k) and, with few features, the instructions of two waves that share a SIMD: a tile of 1000 x 25 takes
// a wave 1310 ticks, and its transposition through LDS in place of half the stream made that 1620.  Divided, a wave issues alone:
// 770 ticks a tile of 25 features, two tiles interleaved, and 1340 of 60 (2450); the exchange takes 2.5 k ticks a round (3.0 k with
// more than 32 features).  5000 x 60, 512 chains: a round 101 k -> 63 k ticks; 20 000 x 25, 64 chains, 9.6 -> 5.0 ms, 3000 x 80, 128 chains 4.0 -> 2.7.  Measured against the wave kernel, which read X twice per chain and gradient with the
// vector ALUs: binary64, 512 chains, 5000 x 60: 1.1e5 -> 5.5e6 gradient evaluations per second; binary32, 250 chains, 700 x 17,
// slice sampler, four steps a leaf: 3.6e6 -> 5.0e7.  What the residuals cost against the tile kernel's functions: 700 x 17 in
// binary32, 4096 chains, 10 iterations 2.0 -> 2.5 ms; 1000 x 60, 4096 chains, 4 iterations 2.39 -> 2.55; 1000 x 120 3.74 -> 3.85;
// with four chains per workgroup nothing to 6 % (3000 x 5: 19 %).  Scratch memory per lane: with sixteen chains 48 bytes (MT = 3)
// to 492 (MT = 8) in binary64, 32 to 412 in binary32 (none at MT = 1 and 3); with four at most 44.
#pragma once
#include <hip/hip_runtime.h>

#include "nuts_dev.h"
#include "nuts_fastmath.h"
#include "nuts_rng.h"
#include "nuts_tile_common.h"

namespace nuts {

constexpr int kWideLds = 160 * 1024;

// Shape-dependent constants of one instantiation.
template <typename T, int MT, int NC, bool kSplit = false>
struct WideShape {
    static constexpr int kWaves = kSplit ? kTileWaves / 2 : kTileWaves;  // of a workgroup
    static constexpr int kTilesAtOnce = kSplit ? 2 : 1;                   // of a wave
    static constexpr int kCpl = (16 * MT + 31) / 32;     // components per lane
    static constexpr int kVec = kTileLanes * kCpl;       // elements of a stored vector
    static constexpr int kPitch = 16 * MT + 1;           // doubles per chain in the LDS tiles (odd: see nuts_tile.h)
    // residuals (see above), or the functions of the tile kernel and its bits
    static constexpr bool kResidual = sizeof(T) == 4 || MT > 2;
    static_assert(kResidual || NC == 4, "16 chains of a binary64 target with up to 32 features are the tile kernel's");
    static constexpr int kTab = (kResidual ? 0 : kFtabDoubles) + kLogTabDoubles;
    static constexpr int kQ = kResidual && NC == 16 ? 4 : 1;  // rows of a tile that a lane keeps log-likelihoods of apart
    // partial gradients: one slot per wave, or, where eight would take the tree levels' place, one per pair of waves
    static constexpr int kSlots = (NC == 16 && MT > 2) ? 4 : kTileWaves;
    // With more than two feature tiles the waves' partial sums are added in pairs (w, w + 4) first, in both forms.
    static constexpr bool kPairs = MT > 2;
    static constexpr int kFixed = (NC * kPitch + kSlots * NC * kPitch + kTileWaves * NC + 16 * MT +
                                   kTab + (kSplit ? 2 * kWaves * kWave : 0)) * 8 + 256;
    static constexpr int kEntry = NC * 2 * kVec * (int)sizeof(T);  // one pool buffer or first-leaf slot of every chain
    static constexpr int kRoom = (kWideLds - kFixed) / kEntry;
    // The vectors that only the start and the end of a doubling or of an iteration touch (the other end of the trajectory,
    // the proposal, the momentum drawn ahead) are in registers when a lane owns one component; with more they would crowd
    // the gradient loop out of the register file, and are kept in LDS or, if they do not fit, in global memory.
    static constexpr bool kHeld = kCpl == 1;
    static constexpr bool kRestLds = !kHeld && kRoom >= 5;
    static constexpr int kEntries = kRoom - (kRestLds ? 3 : 0);
    static constexpr int kLdsPool = kEntries >= 9 ? 5 : (kEntries + 1) / 2;   // shallow tree levels that live in LDS
    static constexpr int kLdsFirst = kEntries >= 9 ? 4 : kEntries / 2;
    static constexpr bool kHoldTheta = MT <= (kSplit ? 4 : 2);          // positions as operands in registers across a round's tiles
    // operands of a whole tile are requested one tile ahead, or (many features: not enough registers, and half a tile
    // of that many instructions covers the latency) half a tile ahead
    static constexpr bool kFullAhead = MT <= (NC == 4 ? 4 : 2);
};

// Which of the two the kernel takes for a target (elem: bytes of its dtype).
inline bool wide_uses_residuals(int64_t d, size_t elem) { return elem == 4 || d > 32; }

struct WideArgs {
    TileArgs ta;
    int ks1;  // k-steps of the first GEMM, 4 MT - 4 < ks1 <= 4 MT (with a constant column possibly 4 MT - 4)
    // divided rows (kSplit): the groups of four chains, a word of each for its workgroups to meet at, and their exchange buffers
    int n_pairs;
    unsigned* meet;
    char* exchange;
    int apart;  // (for tests) 1: the second of two workgroups behaves as if it had come too late; 2 + h: half h sends nothing after its third round
};

// Exchange between the two workgroups of a group of chains: [half][parity of the round][wave][vector][lane]{low, tag, high, tag}, a
// vector per feature tile and one of log-likelihoods.
__host__ __device__ constexpr int wide_exchange_half(int mt) { return 2 * (kTileWaves / 2) * (mt + 1) * kWave * 16; }  // bytes
constexpr int kWideAgent = 16;                       // cache policy of a buffer instruction: agent scope (sc1)
constexpr long long kWideMeetLimit = 20000;          // 0.2 ms (100 MHz)
constexpr long long kWideLostLimit = 6000000000ll;   // 60 s
enum : unsigned { kMeetBoth = 3u, kMeetAlone = 4u, kMeetLost = 8u };  // bit h: half h has come

// A workgroup that waits for its partner must have it resident: each announces itself before anything is done, and one whose
// partner has not come within 0.2 ms (a device or a mask of compute units without room for both) takes the whole group's rows, part
// after part; the partner, when it starts, finds that and returns.  Two that have met are both running and stay so.  Should one wait
// for the other's sums beyond kWideLostLimit all the same, the first half begins again and takes all rows, and the second ends: no wait is
// without an end, and the call returns the same bits.
//
// The other half of the group: true if it has come, and both go on together; false if this one goes on alone (`late`: not at
// all, the other one has gone on alone).
__device__ inline bool wide_meet(unsigned* word, int half, bool& late)
{
    const unsigned mine = 1u << half, other = 2u >> half;
    unsigned seen = __hip_atomic_fetch_or(word, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    late = (seen & kMeetAlone) != 0;
    if (late) return false;
    const long long t0 = wall_clock64();
    for (;;) {
        if (seen & other) return true;
        if (wall_clock64() - t0 > kWideMeetLimit) {
            unsigned expected = mine;
            if (__hip_atomic_compare_exchange_strong(word, &expected, mine | kMeetAlone, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                return false;
            return true;  // (it has come in between)
        }
        __builtin_amdgcn_s_sleep(1);
        seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Vectors of a chain that are kept outside the registers when !kHeld (after the level-indexed ones in the workspace).
enum : int { kRestOtherTh = 0, kRestOtherR = 1, kRestOtherG = 2, kRestTop = 3, kRestTopG = 4, kRestNext = 5, kRestCount = 6 };
__host__ __device__ inline int wide_num_vectors(int max_depth) { return tile_num_vectors(max_depth) + kRestCount; }

// State of one chain: as TileChain (nuts_tile.h), with kCpl components per lane.
template <typename T, int kCpl, bool kHeld>
struct WideChain {
    int pc, level, j, v, m, nleap, iter, cur_s, cur_idx, frame_idx, sub;
    uint64_t ret;
    uint32_t gchain, free_mask;  // gchain: global id of the chain
    double H0, w_tree, cur_w, log_unit_w, edge_logp, top_logp;
    double frame_w, pool_logp, u_sub;  // lane-distributed, see TileChain
    T tha[kCpl], ra[kCpl], ga[kCpl];                 // the end of the trajectory that the current doubling extends
    T rest[kHeld ? kRestCount : 1][kHeld ? kCpl : 1];  // kHeld: the vectors kRest*
    double kin_n;
    int ahead_iter, u_sub_leaf;
    uint32_t dirbits, dirbits_n;
};

// Quad s of every row of 16 lanes, in all four quads of the row.
template <int s>
__device__ __forceinline__ double spread_quad(double x)
{
    constexpr int kPattern = (s << 7) | 0x13;  // source lane = (lane & 0x13) | 4 s
    const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(x), kPattern);
    const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(x), kPattern);
    return __hiloint2double(hi, lo);
}

// What the lane s quads further on in its row of 16 holds (cyclically).
template <int s>
__device__ __forceinline__ double quad_after(double x)
{
    return dpp_rotate<0x130 - 4 * s>(x);  // row_ror: 16 - 4 s
}

template <typename T, int MT, int NC, bool kSplit>
__global__ __launch_bounds__((WideShape<T, MT, NC, kSplit>::kWaves * kWave)) void nuts_wide_kernel(WideArgs wa, DevSample sa)
{
    typedef WideShape<T, MT, NC, kSplit> S;
    constexpr int kThreads = S::kWaves * kWave;
    constexpr int kCpl = S::kCpl, kVec = S::kVec, kLP = S::kLdsPool, kLF = S::kLdsFirst;
    const TileArgs& ta = wa.ta;
    __shared__ double sTheta[NC][S::kPitch];
    __shared__ double sG[S::kSlots][NC][S::kPitch];
    __shared__ double sLL[kTileWaves][NC];
    __shared__ double sHalfCol[S::kResidual ? 1 : 16 * MT];  // column sums of X~, halved
    __shared__ __align__(16) double sSpread[kSplit ? S::kWaves : 1][S::kTilesAtOnce][kSplit ? kWave : 1];
    __shared__ int sHalted, sMeet, sLost;
    __shared__ __align__(16) double sFtab[S::kTab];
    const double* const log_tab = sFtab + S::kTab - kLogTabDoubles;
    __shared__ T sPool[NC][kLP > 0 ? kLP : 1][2][kLP > 0 ? kVec : 1];
    __shared__ T sFirst[NC][kLF > 0 ? kLF : 1][2][kLF > 0 ? kVec : 1];
    __shared__ T sRest[NC][kRestCount][S::kRestLds ? kVec : 1];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = uni(tid >> 6);
    // 16 chains: two per wave; 4 chains: one in the lower half of each of the first four waves (one per SIMD)
    const bool owns = NC == 16 || (wave < 4 && lane < kTileLanes);
    const int grp = NC == 16 ? tid / kTileLanes : (wave & 3);
    const int k = tid & (kTileLanes - 1);
    const int d = ta.d, D = sa.max_depth;
    const DrawKey key{sa.key0, sa.key1};
    const bool slice = sa.sampler == kSamplerSlice;
    const uint32_t all_bufs = (1u << (D + 1)) - 1u;
    // component e of this lane: pairs (2i, 2i + 1) that share a Box-Muller draw as far as they go, then single ones
    auto comp = [&](int e) __attribute__((always_inline)) -> int {
        return e < kCpl / 2 * 2 ? 64 * (e / 2) + 2 * k + (e & 1) : 64 * (kCpl / 2) + k;
    };

    // divided rows: workgroups b and b + 8 of every sixteen (which start on one XCD, one soon after the other) are a pair
    const int pair = kSplit ? (int)(blockIdx.x / 16 * 8 + blockIdx.x % 8) : 0, half_id = kSplit ? (int)(blockIdx.x / 8 % 2) : 0;
    if (kSplit && pair >= wa.n_pairs) return;
    const int wg = kSplit ? 2 * pair + half_id : (int)blockIdx.x;
    T* const wsc = reinterpret_cast<T*>(sa.workspace + (size_t)wg * sa.slot_bytes) +
                   (size_t)grp * wide_num_vectors(D) * kVec + k;
    // level-indexed tree storage: shallow levels in LDS, the others in global memory (a lane reads what it wrote itself)
    auto pool_load = [&](int b, int c, T (&v)[kCpl]) __attribute__((always_inline)) {
        if (b < kLP) {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) v[e] = sPool[grp][b < kLP ? b : 0][c][e * kTileLanes + k];
        } else {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) v[e] = wsc[(size_t)(2 * b + c) * kVec + e * kTileLanes];
        }
    };
    auto pool_store = [&](int b, int c, const T (&v)[kCpl]) __attribute__((always_inline)) {
        if (b < kLP) {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) sPool[grp][b < kLP ? b : 0][c][e * kTileLanes + k] = v[e];
        } else {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) wsc[(size_t)(2 * b + c) * kVec + e * kTileLanes] = v[e];
        }
    };
    auto first_load = [&](int s, int c, T (&v)[kCpl]) __attribute__((always_inline)) {
        if (s <= kLF) {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) v[e] = sFirst[grp][s <= kLF ? s - 1 : 0][c][e * kTileLanes + k];
        } else {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) v[e] = wsc[(size_t)(2 * (D + 1) + 2 * s + c) * kVec + e * kTileLanes];
        }
    };
    auto first_store = [&](int s, int c, const T (&v)[kCpl]) __attribute__((always_inline)) {
        if (s <= kLF) {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) sFirst[grp][s <= kLF ? s - 1 : 0][c][e * kTileLanes + k] = v[e];
        } else {
#pragma unroll
            for (int e = 0; e < kCpl; ++e) wsc[(size_t)(2 * (D + 1) + 2 * s + c) * kVec + e * kTileLanes] = v[e];
        }
    };

    for (int i = tid; i < S::kTab; i += kThreads) sFtab[i] = ta.ftab[kFtabDoubles + kLogTabDoubles - S::kTab + i];
    for (int i = tid; i < NC * S::kPitch; i += kThreads) (&sTheta[0][0])[i] = 0.0;
    for (int i = tid; i < (S::kResidual ? 0 : 16 * MT); i += kThreads) sHalfCol[i] = 0.5 * ta.colsum[i];
    if (tid == 0) sHalted = 0, sLost = 0;
    constexpr int kHalfBytes = wide_exchange_half(MT);
    const __amdgpu_buffer_rsrc_t other_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        wa.exchange + (size_t)(2 * pair + (1 - half_id)) * kHalfBytes, 0, kSplit ? kHalfBytes : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t own_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        wa.exchange + (size_t)(2 * pair + half_id) * kHalfBytes, 0, kSplit ? kHalfBytes : 0, 0x00020000);
    typedef __attribute__((ext_vector_type(4))) unsigned v4u;
    bool alone = true;  // (this workgroup has all rows)
    if (kSplit) {
        // Tags of an earlier launch go before the other half may look: rounds count from 1 in every launch.
        for (int i = tid * 16; i < kHalfBytes; i += kThreads * 16) __builtin_amdgcn_raw_buffer_store_b128(v4u{0, 0, 0, 0}, own_rsrc, i, 0, kWideAgent);
        __threadfence();
        __syncthreads();
        if (tid == 0) {
            bool late = false;
            const bool apart = wa.apart == 1, both = !apart && wide_meet(wa.meet + pair, half_id, late);
            sMeet = (apart ? half_id == 1 : late) ? 2 : both ? 1 : 0;
        }
        __syncthreads();
        const int met = uni(sMeet);
        if (met == 2) return;
        alone = met == 0;
    } else {
        __syncthreads();
    }
    const bool lead = !kSplit || alone || half_id == 0;  // writes what the call returns
    unsigned round = 0;
    const unsigned last_sent = wa.apart == 2 + half_id ? 3u : ~0u;  // (rounds beyond it are sent with its number)

    // where component i goes in the first GEMM's contraction (see feat1 in tile_pack_operands)
    auto slot_of = [&](int i) __attribute__((always_inline)) -> int {
        return S::kResidual || ta.z0_col < 0 ? i : (i == ta.z0_col ? d - 1 : (i == d - 1 ? ta.z0_col : i));
    };
    const __amdgpu_buffer_rsrc_t ops_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(ta.ops), 0, (int)ta.ops_bytes, 0x00020000);

    WideChain<T, kCpl, S::kHeld> c{};
    c.pc = owns ? kPcFetch : kPcHalt;
    c.cur_idx = -1;
    auto rest_load = [&](int x, T (&v)[kCpl]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < kCpl; ++e)
            v[e] = S::kHeld ? c.rest[S::kHeld ? x : 0][S::kHeld ? e : 0]
                            : (S::kRestLds ? sRest[grp][x][S::kRestLds ? e * kTileLanes + k : 0]
                                           : wsc[(size_t)(tile_num_vectors(D) + x) * kVec + e * kTileLanes]);
    };
    auto rest_store = [&](int x, const T (&v)[kCpl]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < kCpl; ++e) {
            if (S::kHeld) c.rest[S::kHeld ? x : 0][S::kHeld ? e : 0] = v[e];
            else if (S::kRestLds) sRest[grp][x][S::kRestLds ? e * kTileLanes + k : 0] = v[e];
            else wsc[(size_t)(tile_num_vectors(D) + x) * kVec + e * kTileLanes] = v[e];
        }
    };
    unsigned long long n_leaf = 0, n_rounds = 0;
    unsigned n_extra = 0;
    bool taken = false;
    long long cyc_control = 0, cyc_grad = 0, cyc_post = 0;

    // standard normals for this lane's components, in the dtype of the state
    auto draw_normals = [&](uint32_t tag, uint32_t it, T (&out)[kCpl]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < kCpl; ++e) {
            const int i = comp(e);
            if (e < kCpl / 2 * 2 && (e & 1)) continue;  // made with its neighbour
            double z0 = 0.0, z1 = 0.0;
            if (i < d) {
                const Words4 w = draw(key, (uint32_t)(i >> 1), tag, 0, it, c.gchain);
                const double rho = sqrt(-2.0 * log_unit(uniform52(w.w0, w.w1), log_tab));
                const double phi = 6.283185307179586476925286766559 * uniform52(w.w2, w.w3);
                if (e < kCpl / 2 * 2) {
                    z0 = rho * circle_point(phi, false);
                    z1 = i + 1 < d ? rho * circle_point(phi, true) : 0.0;
                } else {
                    z0 = rho * circle_point(phi, i & 1);
                }
            }
            out[e] = (T)z0;
            if (e < kCpl / 2 * 2) out[e + 1 < kCpl ? e + 1 : e] = (T)z1;
        }
    };
    auto push_ret = [&](unsigned code) __attribute__((always_inline)) { c.ret = (c.ret << 2) | code; };
    auto do_return = [&]() __attribute__((always_inline)) {
        c.pc = ret_to_pc((unsigned)(c.ret & 3u));
        c.ret >>= 2;
        c.level += 1;
    };
    auto descend_to_leaf = [&]() __attribute__((always_inline)) {
        c.ret <<= 2 * c.level;  // one kRetAfterLeft (= 0) per level
        c.level = 0;
        c.pc = kPcLeaf;
    };
    auto materialise_cur = [&]() __attribute__((always_inline)) {
        if (c.cur_idx >= 0) return;
        const int b = __ffs(c.free_mask) - 1;
        c.free_mask &= ~(1u << b);
        pool_store(b, 0, c.tha);
        pool_store(b, 1, c.ga);
        if (k == b) c.pool_logp = c.edge_logp;
        c.cur_idx = b;
    };
    // (theta+ - theta-) . r at both ends of the span between the extended end and (t, r); going backwards the span is the
    // negative of their difference, exactly, so the signs of the sums are turned by the direction
    auto no_uturn = [&](const T (&t)[kCpl], const T (&r)[kCpl]) __attribute__((always_inline)) -> bool {
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int e = 0; e < kCpl; ++e) {
            const T span = c.v > 0 ? c.tha[e] - t[e] : t[e] - c.tha[e];
            a = fma((double)span, (double)r[e], a);
            b = fma((double)span, (double)c.ra[e], b);
        }
        return group_both_nonnegative(a, b, lane);
    };

    // ---- blocks of the chain program; each runs for the lanes whose chain waits at it (see nuts_tile.h) ----
    auto block_after_right = [&]() __attribute__((always_inline)) {
        if (c.cur_s) {
            const int f = c.m - (1 << c.level) + 1;  // first leaf of this subtree, 1-based
            const int s = (f == 1) ? c.j : min(__ffs(f - 1) - 1, c.j);
            T tf[kCpl], rf[kCpl];
            first_load(s, 0, tf);
            first_load(s, 1, rf);
            const double l_w = __shfl(c.frame_w, c.level, kTileLanes);
            const int l_idx = __shfl(c.frame_idx, c.level, kTileLanes);
            const double u = __shfl(c.u_sub, c.level + (c.u_sub_leaf != c.nleap ? 16 : 0), kTileLanes);
            const double w_new = l_w + c.cur_w;
            if (u * w_new < c.cur_w) {  // right with probability w_R / (w_L + w_R)
                c.free_mask |= (1u << l_idx);
            } else {
                if (c.cur_idx >= 0) c.free_mask |= (1u << c.cur_idx);
                c.cur_idx = l_idx;
            }
            c.cur_w = w_new;
            c.cur_s = no_uturn(tf, rf);
        }
        do_return();
    };
    auto block_after_left = [&]() __attribute__((always_inline)) {
        if (!c.cur_s) {  // the right half is never built
            do_return();
            return;
        }
        materialise_cur();
        if (k == c.level) {
            c.frame_w = c.cur_w;
            c.frame_idx = c.cur_idx;
        }
        c.level -= 1;
        push_ret(kRetAfterRight);
        descend_to_leaf();
    };
    auto block_double_end = [&]() __attribute__((always_inline)) {
        bool go_on = false;
        if (c.cur_s) {
            const double u = __shfl(c.pool_logp, 16 + c.j, kTileLanes);
            if (u * c.w_tree < c.cur_w) {  // accept the new half with probability min(1, w_new / w_tree)
                if (c.cur_idx < 0) {
                    rest_store(kRestTop, c.tha);
                    rest_store(kRestTopG, c.ga);
                    c.top_logp = c.edge_logp;
                } else {
                    T t[kCpl], g[kCpl];
                    pool_load(c.cur_idx, 0, t);
                    pool_load(c.cur_idx, 1, g);
                    rest_store(kRestTop, t);
                    rest_store(kRestTopG, g);
                    c.top_logp = __shfl(c.pool_logp, c.cur_idx, kTileLanes);
                }
            }
            c.w_tree += c.cur_w;
            T to[kCpl], ro[kCpl];
            rest_load(kRestOtherTh, to);
            rest_load(kRestOtherR, ro);
            go_on = no_uturn(to, ro);
        }
        c.j += 1;
        c.free_mask = all_bufs;  // nothing of the finished doubling stays in the pool
        c.pc = (go_on && c.j < D) ? kPcDoubleBegin : kPcIterEnd;
    };
    auto block_iter_end = [&]() __attribute__((always_inline)) {
        const size_t row = (size_t)c.iter * (size_t)sa.n_chains + (size_t)(c.gchain - (uint32_t)sa.first_chain);
        if (lead && sa.out_states) {
            T* dst = static_cast<T*>(sa.out_states) + row * d;
            T t[kCpl];
            rest_load(kRestTop, t);
#pragma unroll
            for (int e = 0; e < kCpl; ++e)
                if (comp(e) < d) dst[comp(e)] = t[e];
        }
        if (lead && k == 0) {
            if (sa.out_depths) sa.out_depths[row] = c.j;
            if (sa.out_nleap) sa.out_nleap[row] = c.nleap;
        }
        c.iter += 1;
        c.pc = (c.iter < sa.iter_end) ? kPcIterBegin : kPcFetch;
    };
    auto block_fetch = [&]() __attribute__((always_inline)) {
        unsigned long long q = 0;
        if (kSplit) {  // (both halves have to know: a chain for every lane group, and no queue)
            q = taken ? (unsigned long long)sa.n_chains : (unsigned long long)(NC * pair + grp);
            taken = true;
        } else {
            if (k == 0) q = atomicAdd(&sa.counters[kCtrQueue], 1ull);
            q = __shfl(q, 0, kTileLanes);
        }
        T t[kCpl];
#pragma unroll
        for (int e = 0; e < kCpl; ++e) t[e] = (T)0;
        if ((long)q >= sa.n_chains) {
            c.pc = kPcHalt;
            if (k == 0) atomicAdd(&sHalted, 1);
            return;
        }
        c.gchain = (uint32_t)(sa.first_chain + (long)q);
        c.iter = sa.iter_begin;
        c.ahead_iter = -1;
        c.u_sub_leaf = kNoLeaf;
        c.free_mask = all_bufs;
        if (sa.init_states) {
            const T* src = static_cast<const T*>(sa.init_states) + (size_t)q * d;
#pragma unroll
            for (int e = 0; e < kCpl; ++e)
                if (comp(e) < d) t[e] = src[comp(e)];
        } else {
            draw_normals(kDrawInit, 0, t);
        }
        rest_store(kRestTop, t);
        c.pc = kPcInitEval;
    };
    // every random number of an iteration that does not depend on where the trajectory goes
    auto draw_iteration = [&](int it) __attribute__((always_inline)) {
        T r[kCpl];
        draw_normals(kDrawMomentum, (uint32_t)it, r);
        rest_store(kRestNext, r);
        double kin = 0.0;
#pragma unroll
        for (int e = 0; e < kCpl; ++e) kin = fma((double)r[e], (double)r[e], kin);
        c.kin_n = group_sum(kin);
        const bool slice_lane = slice && k == kTileLanes - 1;
        const Words4 w = draw(key, slice_lane ? 0u : (uint32_t)(k & 15),
                              k < 16 ? kDrawDirection : (slice_lane ? kDrawSlice : kDrawTop), 0, (uint32_t)it, c.gchain);
        const unsigned long long votes = __ballot((k < 16) && (w.w0 >> 31));
        c.dirbits_n = (uint32_t)(votes >> (lane & 32)) & 0xffffu;
        if (k >= 16) c.frame_w = uniform52(w.w0, w.w1);
        if (slice_lane) c.frame_w = log(c.frame_w);
        c.ahead_iter = it;
    };
    auto block_iter_begin = [&]() __attribute__((always_inline)) {
        if (c.ahead_iter != c.iter) draw_iteration(c.iter);
        c.dirbits = c.dirbits_n;
        if (k >= 16) c.pool_logp = c.frame_w;
        rest_load(kRestTop, c.tha);
        rest_load(kRestTopG, c.ga);
        rest_load(kRestNext, c.ra);
        rest_store(kRestOtherTh, c.tha);
        rest_store(kRestOtherG, c.ga);
        rest_store(kRestOtherR, c.ra);
        c.H0 = -c.top_logp + 0.5 * c.kin_n;
        c.w_tree = 1.0;
        c.log_unit_w = 0.0;
        c.j = 0;
        c.nleap = 0;
        c.u_sub_leaf = kNoLeaf;
        c.pc = kPcDoubleBegin;
    };
    auto block_double_begin = [&]() __attribute__((always_inline)) {
        const int v = ((c.dirbits >> c.j) & 1u) ? 1 : -1;
        if (v != c.v) {  // the doubling turns round: the two ends change places
            T t[kCpl], r[kCpl], g[kCpl];
            rest_load(kRestOtherTh, t);
            rest_load(kRestOtherR, r);
            rest_load(kRestOtherG, g);
            rest_store(kRestOtherTh, c.tha);
            rest_store(kRestOtherR, c.ra);
            rest_store(kRestOtherG, c.ga);
#pragma unroll
            for (int e = 0; e < kCpl; ++e) {
                c.tha[e] = t[e];
                c.ra[e] = r[e];
                c.ga[e] = g[e];
            }
        }
        c.v = v;
        c.m = 0;
        c.level = c.j;
        push_ret(kRetDoubleEnd);
        descend_to_leaf();
    };

    const int pairs1 = (wa.ks1 + 1) / 2;                // operand pairs of the first GEMM that the stream holds
    const int tile_bytes = (pairs1 + 2 * MT) * 64 * 16;  // bytes of a tile in the stream
    auto load_at = [&](int byte_off) __attribute__((always_inline)) -> double2 {
        return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(ops_rsrc, lane * 16, byte_off, 0));
    };

    for (;;) {
        const long long t0 = clock64();
        // ---- 1. control ----
        if (c.pc == kPcAfterRight && c.cur_s && c.u_sub_leaf != c.nleap && c.u_sub_leaf + 2 * sa.leaf_steps != c.nleap) {
            const Words4 w = draw(key, (uint32_t)(c.nleap + (k >= 16 ? 2 * sa.leaf_steps : 0)), kDrawSubtree, (uint32_t)(k & 15),
                                  (uint32_t)c.iter, c.gchain);
            c.u_sub = uniform52(w.w0, w.w1);
            c.u_sub_leaf = c.nleap;
        }
        for (;;) {
            const int pa = __builtin_amdgcn_readlane(c.pc, 0), pb = __builtin_amdgcn_readlane(c.pc, kTileLanes);
            const bool any_right = pa == kPcAfterRight || pb == kPcAfterRight;
            const bool any_left = pa == kPcAfterLeft || pb == kPcAfterLeft;
            if (!any_right && !any_left) break;
            if (any_right && c.pc == kPcAfterRight) block_after_right();
            if (c.pc == kPcAfterLeft) block_after_left();
        }
        const bool wave_busy = __any(c.pc == kPcDoubleEnd);
        if (c.pc == kPcDoubleEnd) block_double_end();
        if (c.pc == kPcIterEnd) block_iter_end();
        if (c.pc == kPcFetch) block_fetch();
        if (c.pc == kPcIterBegin) block_iter_begin();
        if (c.pc == kPcDoubleBegin) block_double_begin();
        if (!wave_busy && c.pc == kPcLeaf && c.ahead_iter != c.iter + 1 && c.nleap >= 1 && c.iter + 1 < sa.iter_end)
            draw_iteration(c.iter + 1);

        // ---- 2. batched gradient ----
        const bool at_leaf = c.pc == kPcLeaf, at_init = c.pc == kPcInitEval;
        const T half = (T)(0.5 * (c.v * sa.eps)), full = (T)(c.v * sa.eps);
        if (owns) {
            if (at_init) rest_load(kRestTop, c.tha);  // (the ends of the trajectory are set when the iteration begins)
#pragma unroll
            for (int e = 0; e < kCpl; ++e) {
                if (at_leaf) {  // first half-kick and drift, in place
                    c.ra[e] = c.ra[e] + half * c.ga[e];
                    c.tha[e] = c.tha[e] + full * c.ra[e];
                }
                if (comp(e) < 16 * MT) sTheta[grp][slot_of(comp(e))] = (at_leaf || at_init) ? (double)c.tha[e] : 0.0;
            }
        }
        constexpr bool kTwo = S::kTilesAtOnce == 2;
        double2 a1[2 * MT], a2[S::kFullAhead ? 2 * MT : 1], b1_[kTwo ? 2 * MT : 1], b2_[kTwo && S::kFullAhead ? 2 * MT : 1];
        // divided rows: operands of tiles t and t + kTileWaves (what is asked for beyond the last tile is that tile's)
        auto offset_of = [&](int t) __attribute__((always_inline)) -> int { return min(t, ta.n_tiles - 1) * tile_bytes; };
        auto ask_first = [&](int t) __attribute__((always_inline)) {
            const int p = offset_of(t), q = offset_of(t + kTileWaves);
#pragma unroll
            for (int i = 0; i < 2 * MT; ++i)
                if (i < 2 * MT - 2 || i < pairs1) {
                    a1[i] = load_at(p + i * 1024);
                    if (kTwo) b1_[kTwo ? i : 0] = load_at(q + i * 1024);
                }
        };
        auto ask_second = [&](int t) __attribute__((always_inline)) {
            if (!S::kFullAhead) return;
            const int p = offset_of(t) + pairs1 * 1024, q = offset_of(t + kTileWaves) + pairs1 * 1024;
#pragma unroll
            for (int i = 0; i < 2 * MT; ++i) {
                a2[S::kFullAhead ? i : 0] = load_at(p + i * 1024);
                if (kTwo) b2_[kTwo && S::kFullAhead ? i : 0] = load_at(q + i * 1024);
            }
        };
        // (not all operands fit ahead: the second GEMM's take the registers that the first has just used up)
        auto ask_second_pair = [&](int t, int p) __attribute__((always_inline)) {
            a1[p] = load_at(offset_of(t) + (pairs1 + p) * 1024);
            if (kTwo) b1_[kTwo ? p : 0] = load_at(offset_of(t + kTileWaves) + (pairs1 + p) * 1024);
        };
        const int first_part = alone ? 0 : half_id, last_part = kSplit && alone ? 1 : first_part;
        if (kSplit) {
            ask_first(first_part * S::kWaves + wave);
            ask_second(first_part * S::kWaves + wave);
        } else {
            const int base = wave * tile_bytes;
#pragma unroll
            for (int i = 0; i < 2 * MT; ++i)
                if (i < 2 * MT - 2 || i < pairs1) a1[i] = load_at(base + i * 1024);
            if (S::kFullAhead) {
#pragma unroll
                for (int i = 0; i < 2 * MT; ++i) a2[i] = load_at(base + (pairs1 + i) * 1024);
            }
        }
        tile_lds_barrier();
        // (a vote: begun again behind a vector branch, the loop over rounds is taken to differ from lane to lane, and every load of operands becomes a
        // loop over its addresses, 1.35 to 1.57 times the time; with one word for sHalted and sLost, and scalar branches on it, up to 1.04 times)
        if (kSplit && __builtin_expect(__any(*const_cast<volatile int*>(&sLost) != 0), 0)) {  // (before anything else: the last round's sums were not all there)
            tile_lds_barrier();
            if (half_id == 1) break;
            if (tid == 0) {
                sHalted = sLost = 0;
                atomicOr(wa.meet + pair, (unsigned)kMeetLost);
            }
            tile_lds_barrier();
            alone = true;
            if (owns) c.pc = kPcFetch;  // (what a chain that is fetched does not set itself)
            c.ret = 0;
            c.sub = 0;
            taken = false;
            n_leaf = n_rounds = 0;
            n_extra = 0;
            continue;
        }
        if (*const_cast<volatile int*>(&sHalted) == NC) break;  // every chain of the workgroup has halted
        n_rounds += 1;
        round += 1;
        const long long t1 = clock64();
        bool lost = false;  // (divided rows) the other half's sums did not come
        // (divided rows, alone: the other half's four sums, too)
        for (int part = first_part; part <= last_part; ++part) {
            const int turn = kSplit ? part * S::kWaves + wave : wave;  // which of the eight sums
            if (kSplit && part != first_part) {
                ask_first(turn);
                ask_second(turn);
            }
            typedef __attribute__((ext_vector_type(4))) double acc16;
            acc16 G16[NC == 16 ? MT : 1];
            double G4[NC == 4 ? MT : 1];
#pragma unroll
            for (int u = 0; u < MT; ++u) {
                if (NC == 16) G16[NC == 16 ? u : 0] = acc16{0.0, 0.0, 0.0, 0.0};
                else G4[NC == 4 ? u : 0] = 0.0;
            }
            // sum of |z| (residual form: of |z| - z), and the product of sigma(|z|) as it stands and as logarithms
            double sum_abs[S::kQ], prod[S::kQ], log_prod[S::kQ];
#pragma unroll
            for (int q = 0; q < S::kQ; ++q) sum_abs[q] = 0.0, prod[q] = 1.0, log_prod[q] = 0.0;
            // B operand of the first GEMM: component 4 s + lane/16 of the position of chain lane % NC
            const double* const b_src = &sTheta[lane & (NC - 1)][lane >> 4];
            double b1[S::kHoldTheta ? 4 * MT : 1];
            if (S::kHoldTheta) {
#pragma unroll
                for (int s = 0; s < 4 * MT; ++s) b1[s] = b_src[4 * s];
            }
            const double z0 = !S::kResidual && ta.z0_col >= 0 ? ta.z0_val * sTheta[lane & (NC - 1)][d - 1] : 0.0;
            auto row_tile = [&](const int t, const bool ragged, const bool more) __attribute__((always_inline)) {
                const int here = t * tile_bytes, next = (t + kTileWaves) * tile_bytes;
                // (the positions are read from LDS again for every tile: kept across tiles they would fill 8 MT registers)
                if (!S::kHoldTheta) asm volatile("" ::: "memory");
                acc16 z;
                double z4;
                if (NC == 16) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) z[q] = 0.0;
                } else {
                    z4 = (!ragged || 4 * ((lane >> 2) & 3) + (lane >> 4) < ta.rem_rows) ? z0 : 0.0;
                }
#pragma unroll
                for (int s = 0; s < 4 * MT; ++s) {
                    if (s < 4 * MT - 4 || s < wa.ks1) {
                        const double a = (s & 1) ? a1[s >> 1].y : a1[s >> 1].x;
                        const double b = S::kHoldTheta ? b1[S::kHoldTheta ? s : 0] : b_src[4 * s];
                        if (NC == 16) z = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, z, 0, 0, 0);
                        else z4 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, z4, 0, 0, 0);
                    }
                    // the second GEMM's operand takes the register pair that has just been used up
                    if (!S::kFullAhead && (s & 1)) a1[s >> 1] = load_at(here + (pairs1 + (s >> 1)) * 1024);
                }
                if (S::kFullAhead && more) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < 2 * MT; ++i)
                        if (i < 2 * MT - 2 || i < pairs1) a1[i] = load_at(next + i * 1024);
                }
                // residual of one row, and its share of the log-likelihood (an infinite or NaN logit makes the sum a NaN; rows
                // beyond the last one count nothing)
                auto row = [&](const double zr, const int first, double& sum, double& product) __attribute__((always_inline)) -> double {
                    double resid, sig;
                    logistic_residual(zr, resid, sig);
                    sum += fabs(zr) - zr;
                    product *= (!ragged || first + (lane >> 4) < ta.rem_rows) ? sig : 1.0;
                    return resid;
                };
                double sg[4];
                if (NC == 16) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        sg[q] = row(z[q], 4 * q, sum_abs[q < S::kQ ? q : 0], prod[q < S::kQ ? q : 0]);
                        if (q == 1) __builtin_amdgcn_sched_barrier(0);  // (two at a time: fewer registers)
                    }
                } else {
                    const double x = S::kResidual ? row(z4, 4 * ((lane >> 2) & 3), sum_abs[0], prod[0])
                                                  : __builtin_copysign(logistic_slope(z4, sFtab), z4);
                    // rows 4s + k of the tile sit in quad s: every block of the second GEMM wants them
                    sg[0] = spread_quad<0>(x);
                    sg[1] = spread_quad<1>(x);
                    sg[2] = spread_quad<2>(x);
                    sg[3] = spread_quad<3>(x);
                    if (!S::kResidual) {
                        // Sums and products in the order of the tile kernel, where one lane holds the tile's rows k, 4 + k, 8 + k
                        // and 12 + k: here quad 0 of every row of 16 lanes gets them so (what the other quads add up is not used).
                        // They run while the swizzles above are under way.  (1000 x 25, 512 chains, 20 iterations: 2.21 ms with
                        // a sum per lane, 2.39 so.)
                        const double a = fabs(z4), f = fabs(x) + 0.5, f2 = f * quad_after<1>(f);
                        sum_abs[0] = (((sum_abs[0] + a) + quad_after<1>(a)) + quad_after<2>(a)) + quad_after<3>(a);
                        prod[0] *= f2 * quad_after<2>(f2);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int u = 0; u < MT; ++u)
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const int p = u * 2 + (s >> 1);
                        const double2 pr = S::kFullAhead ? a2[S::kFullAhead ? p : 0] : a1[p];
                        const double a = (s & 1) ? pr.y : pr.x;
                        if (NC == 16) G16[NC == 16 ? u : 0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, sg[s], G16[NC == 16 ? u : 0], 0, 0, 0);
                        else G4[NC == 4 ? u : 0] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, sg[s], G4[NC == 4 ? u : 0], 0, 0, 0);
                        // (past the end of the stream the buffer's bounds check answers with zeros)
                        if (!S::kFullAhead && (s & 1)) a1[p] = load_at(next + p * 1024);
                    }
                if (S::kFullAhead && more) {
#pragma unroll
                    for (int i = 0; i < 2 * MT; ++i) a2[i] = load_at(next + (pairs1 + i) * 1024);
                }
            };
            // Divided rows: two tiles, t and t + kTileWaves, step by step (one wave has the SIMD to itself, and would wait for every
            // result of a single tile).  `last`: the second may not exist, one of them may be ragged.
            auto two_tiles = [&](const int t, const bool last) __attribute__((always_inline)) {
                const bool second = !last || t + kTileWaves < ta.n_tiles;
                const int my_row = 4 * ((lane >> 2) & 3) + (lane >> 4);
                bool real[2];
                double z[2], x[2], sig[2], sg[2][4];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    real[q] = !last || ta.rem_rows == 0 || t + q * kTileWaves != ta.n_tiles - 1 || my_row < ta.rem_rows;
                    z[q] = real[q] ? z0 : 0.0;
                }
                if (!S::kHoldTheta) asm volatile("" ::: "memory");
#pragma unroll
                for (int s = 0; s < 4 * MT; ++s)
                    if (s < 4 * MT - 4 || s < wa.ks1) {
                        const double b = S::kHoldTheta ? b1[S::kHoldTheta ? s : 0] : b_src[4 * s];
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const double2 pr = q ? b1_[kTwo ? s >> 1 : 0] : a1[s >> 1];
                            z[q] = __builtin_amdgcn_mfma_f64_4x4x4f64((s & 1) ? pr.y : pr.x, b, z[q], 0, 0, 0);
                        }
                        if (!S::kFullAhead && (s & 1)) ask_second_pair(t, s >> 1);
                    } else if (!S::kFullAhead && (s & 1)) {
                        ask_second_pair(t, s >> 1);
                    }
                __builtin_amdgcn_sched_barrier(0);
                if (S::kFullAhead) ask_first(t + 2 * kTileWaves);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (S::kResidual) logistic_residual(z[q], x[q], sig[q]);
                    else x[q] = __builtin_copysign(logistic_slope(z[q], sFtab), z[q]);
                }
                // rows 4s + k of the tile, which sit in quad s, for every block of the second GEMM (through LDS of the wave's own, in
                // order: six instructions where swizzles are sixteen)
#pragma unroll
                for (int q = 0; q < 2; ++q) sSpread[kTwo ? wave : 0][kTwo ? q : 0][kTwo ? lane : 0] = x[q];
                asm volatile("" ::: "memory");
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int s = 0; s < 4; ++s) sg[q][s] = sSpread[kTwo ? wave : 0][kTwo ? q : 0][kTwo ? (lane & 0x33) + 4 * s : 0];
#pragma unroll
                for (int q = 0; q < 2; ++q) {  // (in the order of row_tile)
                    if (q && !second) break;
                    if (S::kResidual) {
                        sum_abs[0] += fabs(z[q]) - z[q];
                        prod[0] *= real[q] ? sig[q] : 1.0;
                    } else {
                        const double a = fabs(z[q]);
                        sum_abs[0] = (((sum_abs[0] + a) + quad_after<1>(a)) + quad_after<2>(a)) + quad_after<3>(a);
                        prod[0] *= ((fabs(sg[q][0]) + 0.5) * (fabs(sg[q][1]) + 0.5)) * ((fabs(sg[q][2]) + 0.5) * (fabs(sg[q][3]) + 0.5));
                    }
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (q && !second) break;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int u = 0; u < MT; ++u) {
                            const int p = u * 2 + h;
                            const double2 pr = S::kFullAhead ? (q ? b2_[kTwo && S::kFullAhead ? p : 0] : a2[S::kFullAhead ? p : 0]) : (q ? b1_[kTwo ? p : 0] : a1[p]);
                            G4[NC == 4 ? u : 0] = __builtin_amdgcn_mfma_f64_4x4x4f64(pr.x, sg[q][2 * h], G4[NC == 4 ? u : 0], 0, 0, 0);
                            G4[NC == 4 ? u : 0] = __builtin_amdgcn_mfma_f64_4x4x4f64(pr.y, sg[q][2 * h + 1], G4[NC == 4 ? u : 0], 0, 0, 0);
                            if (!S::kFullAhead) (q ? b1_[kTwo ? p : 0] : a1[p]) = load_at(offset_of(t + (2 + q) * kTileWaves) + p * 1024);
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
                ask_second(t + 2 * kTileWaves);
            };
            auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < S::kQ; ++q) {
                    const double l = log_unit(prod[q], log_tab);
                    log_prod[q] += S::kResidual && prod[q] == 1.0 ? 0.0 : l;  // (log_unit(1) is off by the rounding of log 2)
                    prod[q] = 1.0;
                }
            };
            // (z0, residuals: a last tile that is not full is run after the loop, by the wave whose turn it is)
            const int n_loop = ta.rem_rows != 0 ? ta.n_tiles - 1 : ta.n_tiles;
            if constexpr (kTwo) {
                // (The first operands are waited for here, all of them: a load before the loop whose register becomes an accumulator's would
                // have the compiler wait in every turn of the loop, for operands asked for a moment ago: 6368 x 39, 49 chains 1.20 -> 1.11 ms.  Without
                // residuals it finds other registers, and the wait alone costs 0.5 %.)
                if (S::kFullAhead && S::kResidual) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
                int t = turn, left = 64;  // tiles until the products become logarithms
                for (; t + kTileWaves < n_loop; t += 2 * kTileWaves) {
                    if (left == 0) {
                        fold();
                        left = 64;
                    }
                    two_tiles(t, false);
                    left -= 2;
                }
                if (t < ta.n_tiles) {
                    if (left == 0 && t < n_loop) fold();
                    two_tiles(t, true);
                }
            }
            for (int t_chunk = kTwo ? n_loop : turn; t_chunk < n_loop; t_chunk += 64 * kTileWaves) {
                const int t_stop = min(n_loop, t_chunk + 64 * kTileWaves);
                for (int t = t_chunk; t < t_stop; t += kTileWaves) row_tile(t, false, t + kTileWaves < ta.n_tiles);
                if (t_chunk + 64 * kTileWaves < n_loop) fold();  // more follow
            }
            if (!kTwo && ta.rem_rows != 0 && turn == ((ta.n_tiles - 1) & (kTileWaves - 1))) row_tile(ta.n_tiles - 1, true, false);
            fold();
            double ll = log_prod[0] - 0.5 * sum_abs[0];
            if (S::kResidual) {  // rows 4q + k of all tiles: q = (0 + 2) + (1 + 3); with 4 chains they are in four quads
                if (NC == 16) {
                    double l[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) l[q] = log_prod[q < S::kQ ? q : 0] - 0.5 * sum_abs[q < S::kQ ? q : 0];
                    ll = (l[0] + l[2]) + (l[1] + l[3]);
                } else {
                    ll += quad_after<2>(ll);
                    ll += quad_after<1>(ll);
                }
            }
            ll = add_other_row(ll);
            ll = add_other_half(ll);
            if (lane < NC) sLL[turn][lane] = ll;
            // partial gradients to LDS: element (u, q) of the accumulators is feature 16u + 4q + lane/16 (16 chains) or
            // 16u + 4((lane/4) % 4) + lane/16 (4 chains) of chain lane % NC
            auto put = [&](double* dst, bool add) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < MT; ++u) {
                    if (NC == 16) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const double g = G16[NC == 16 ? u : 0][q];
                            dst[16 * u + 4 * q] = add ? dst[16 * u + 4 * q] + g : g;
                        }
                    } else {
                        dst[16 * u] = G4[NC == 4 ? u : 0];
                    }
                }
            };
            const int off = NC == 16 ? (lane >> 4) : 4 * ((lane >> 2) & 3) + (lane >> 4);
            if (S::kSlots == kTileWaves) {
                put(&sG[turn & (S::kSlots - 1)][lane & (NC - 1)][off], false);
            } else {  // two waves share a slot, one after the other
                if (wave < 4) put(&sG[wave & 3][lane & (NC - 1)][off], false);
                tile_lds_barrier();
                if (wave >= 4) put(&sG[wave & 3][lane & (NC - 1)][off], true);
            }
            if constexpr (kSplit) {
                // This wave's sums to the other half's wave, and that one's here.  Every 8 bytes carry the round's number beside
                // half a value, so a value that is there needs no flag and no fence; two buffers in turn, as neither half is more
                // than a round ahead of the other.
                if (!alone) {
                    // (the same for all lanes, which the compiler does not see behind the way to begin again: it would take the place for one that
                    // differs from lane to lane, and make a loop of every load and store)
                    const unsigned now_round = (unsigned)uni((int)round);
                    const int at = (((int)(now_round & 1) * S::kWaves + wave) * (MT + 1)) * kWave * 16;
                    const unsigned tag = min(now_round, last_sent);
                    auto send = [&](double v, int i) __attribute__((always_inline)) {
                        const v4u w{(unsigned)__double2loint(v), tag, (unsigned)__double2hiint(v), tag};
                        __builtin_amdgcn_raw_buffer_store_b128(w, own_rsrc, lane * 16, at + i * kWave * 16, kWideAgent);
                    };
#pragma unroll
                    for (int u = 0; u < MT; ++u) send(G4[NC == 4 ? u : 0], u);
                    send(ll, MT);
                    v4u in[MT + 1];
                    long long t0 = 0;
                    for (int looks = 1;; ++looks) {
                        asm volatile("" ::: "memory");
                        bool there = true;
#pragma unroll
                        for (int i = 0; i <= MT; ++i)
                            in[i] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(other_rsrc, lane * 16, at + i * kWave * 16, kWideAgent));
#pragma unroll
                        for (int i = 0; i <= MT; ++i) there = there && in[i][1] == now_round && in[i][3] == now_round;
                        if (__all(there)) break;
                        if (__builtin_expect((looks & 255) == 0, 0)) {
                            const long long now = wall_clock64();
                            if (t0 == 0) t0 = now;
                            if (now - t0 > (wa.apart >= 2 ? kWideMeetLimit : kWideLostLimit)) {
                                lost = true;
                                break;
                            }
                        }
                    }
                    const int theirs = (1 - half_id) * S::kWaves + wave;
#pragma unroll
                    for (int u = 0; u < MT; ++u) sG[theirs & (S::kSlots - 1)][lane & (NC - 1)][off + 16 * u] = __hiloint2double((int)in[u][2], (int)in[u][0]);
                    if (lane < NC) sLL[theirs][lane] = __hiloint2double((int)in[MT][2], (int)in[MT][0]);
                }
            }
        }
        tile_lds_barrier();
        if (kSplit && __builtin_expect(lost, 0)) sLost = 1;  // (behind the barrier: before it, a wave might not have looked at this round's)
        const long long t2 = clock64();

        // ---- 3. every chain collects its gradient and finishes its step ----
        if (at_leaf || at_init) {
            const double ll_part = (k < kTileWaves) ? sLL[k & (kTileWaves - 1)][grp] : 0.0;
            double sq = ll_part, kin = 0.0;
#pragma unroll
            for (int e = 0; e < kCpl; ++e) {
                const int i = comp(e);
                double gsum = 0.0;
                if (i < 16 * MT) {
                    if (S::kSlots == 4) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) gsum += sG[w][grp][i];
                    } else if (S::kPairs) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) gsum += sG[w][grp][i] + sG[(w + 4) & (S::kSlots - 1)][grp][i];
                    } else {
#pragma unroll
                        for (int w = 0; w < kTileWaves; ++w) gsum += sG[w & (S::kSlots - 1)][grp][i];
                    }
                }
                const double th = (double)c.tha[e];
                const double hc = !S::kResidual && i < 16 * MT ? sHalfCol[S::kResidual ? 0 : i] : 0.0;
                const T g = i < d ? (T)((S::kResidual ? gsum : hc - gsum) - th * ta.prior_prec) : (T)0;
                // |theta|^2 for the prior (not residuals: (1/2) colsum . theta = (1/2) sum z~ for the likelihood)
                if (S::kResidual) sq = fma(th, th * (-0.5 * ta.prior_prec), sq);
                else sq += fma(th, th * (-0.5 * ta.prior_prec), hc * th);
                if (at_leaf) {
                    const T r_new = c.ra[e] + half * g;
                    c.ra[e] = r_new;
                    kin = fma((double)r_new, (double)r_new, kin);
                }
                c.ga[e] = g;
            }
            if (at_leaf) {
                c.nleap += 1;
                n_leaf += 1;
                c.sub += 1;
                if (c.sub >= sa.leaf_steps) {  // otherwise the leaf is not finished: the chain stays at LEAF
                    c.sub = 0;
                    group_sum2(sq, kin);
                    const double logp = S::kResidual ? sq : ta.n_pad * 0.6931471805599453 + sq;
                    c.edge_logp = logp;
                    c.m += 1;
                    double delta = (-logp + 0.5 * kin) - c.H0;
                    if (!(fabs(delta) < INFINITY)) delta = INFINITY;
                    if (slice) {
                        const double log_slice = __shfl(c.pool_logp, kTileLanes - 1, kTileLanes);
                        c.cur_w = (log_slice <= -delta) ? 1.0 : 0.0;
                        c.cur_s = (log_slice < kDeltaMax - delta);
                    } else {
                        double e = c.log_unit_w - delta;  // logarithm of the leaf's weight in the current unit
                        if (e > 600.0) {  // the energy has fallen far: this leaf becomes the unit
                            const double shrink = exp_bounded(-e);
                            c.w_tree *= shrink;
                            if (k < 16) c.frame_w *= shrink;
                            c.log_unit_w = delta;
                            e = 0.0;
                        }
                        c.cur_w = exp_bounded(e);
                        c.cur_s = (delta <= kDeltaMax);
                    }
                    c.cur_idx = -1;  // the proposal of a one-leaf subtree is the edge itself
                    if ((c.m & 1) && c.j >= 1) {
                        const int s = (c.m == 1) ? c.j : min(__ffs(c.m - 1) - 1, c.j);
                        first_store(s, 0, c.tha);
                        first_store(s, 1, c.ra);
                    }
                    do_return();
                }
            } else {
                rest_store(kRestTopG, c.ga);
                sq = group_sum(sq);
                c.top_logp = S::kResidual ? sq : ta.n_pad * 0.6931471805599453 + sq;
                n_extra += 1;
                c.pc = kPcIterBegin;
            }
        }
        cyc_control += t1 - t0;
        cyc_grad += t2 - t1;
        cyc_post += clock64() - t2;
    }

    if (!lead) return;
    if (owns && k == 0) {
        atomicAdd(&sa.counters[kCtrUseful], n_leaf);
        atomicAdd(&sa.counters[kCtrExtra], (unsigned long long)n_extra);
    }
    if (tid == 0) {
        atomicAdd(&sa.counters[kCtrIssued], n_rounds * NC);
        atomicAdd(&sa.counters[kCtrRounds], n_rounds);
        atomicAdd(&sa.counters[kCtrCycControl], (unsigned long long)cyc_control);
        atomicAdd(&sa.counters[kCtrCycGrad], (unsigned long long)cyc_grad);
        atomicAdd(&sa.counters[kCtrCycPost], (unsigned long long)cyc_post);
    }
}

// Chains per workgroup for a launch of n_chains and `iters` iterations of n rows and d features on a chip of `cus` compute
// units (one workgroup each).  Up to 4 chains per compute unit every group of four has one to itself, and 4 is never behind
// (64 to 1024 chains, 10 to 1e6 rows x 5 to 32: 1 to 1.8 times as fast as 16).
// Up to 8, the groups beyond the first `cus` take turns with them where sixteen would all run at once.  A chain's turn of 4 takes
// between 0.45 (many rows) and 0.9 (few) of one of 16, so two turns lose in the long run; but a launch of few iterations
// lasts as long as its longest chain, and the shorter ones leave room beside it.  Time with 4 over time with 16 at 1100, 1500
// and 2048 chains, binary64, against the kernel of nuts_tile.h:
//   rows x features     1 iteration        4                 16                64                200
//   500 x 25         0.70 0.70 0.88   0.78 0.86 0.88   0.89 1.03 1.05   1.01 1.05 1.15   1.07 1.13 1.19
//   2000 x 25        0.67 0.67 0.79   0.72 0.79 0.96   0.78 0.83 0.99   0.88 0.94 0.97   0.93 0.97 1.00
//   10000 x 32       0.73 0.88 0.87   0.72 0.85 0.94   0.96 1.01 1.04   1.01 1.03 1.07   1.03 1.06 1.09
//   2000 x 16        0.78 0.62 0.91   0.64 0.79 0.93   0.88 1.00 1.11   0.99 1.05 1.13   1.06 1.10 1.13
//   8000 x 5         0.65 0.75 0.86   0.84 0.90 1.13   0.98 1.08 1.09   1.08 1.13 1.17   1.14 1.16 1.18
// (100 x 25 and 1000 x 5, 20 iterations: 1.0 to 1.36; 200 000 x 25 0.70 to 1.01 up to 16 iterations; from 700 000 x 25 on the
// stream leaves the last cache, 1.3, trajectories of one length.)  Against this kernel's own form with 16 and residuals, 4 to 20 iterations: 300 x 60
// 0.7 to 0.93, 1000 x 60 0.52 to 0.75, binary32 700 x 17 0.49 to 0.75; 100 x 40 0.86 to 1.09, binary32 100 x 5 0.86 to 1.16.
inline int wide_chains_per_block(long n_chains, int cus, long iters, long n, int d, bool residual)
{
    if (n_chains <= 4L * cus) return 4;
    if (n_chains > 8L * cus) return 16;
    if (residual) return n >= 200 ? 4 : 16;
    const long most = n < 500 || n > 200000 ? 0 : d > 16 ? (n >= 2000 ? 64 : 16) : (n >= 2000 ? 4 : 0);  // iterations
    return iters <= most ? 4 : 16;
}

// Whether the rows are divided: compute units for two workgroups of every four chains, and rows enough.  Time undivided over time
// divided, binary64, 64 and 512 chains (binary32 alike):
//   features      700 rows       1000           2000           5000           20 000
//   9             0.94 0.91      1.04 1.01      1.15 1.08      1.27 1.22      1.41 1.32
//   25            0.93 0.91      1.04 1.01      1.18 1.11      1.30 1.25      1.92 1.73
//   60            1.00 0.96      1.18 1.12      1.39 1.28      1.64 1.59      1.80 1.87
//   90            1.10 1.02      1.25 1.13      1.41 1.21      1.65 1.45
//   128           1.15 1.06      1.33 1.18      1.42 1.27      1.73 1.49
// (100 rows: 0.6 to 0.8.  One line for all numbers of features: what 700 rows of 90 and more would gain is left.)
// In a launch of one iteration (awaited iterations) the two meet for that alone, 10 us.  8 and 512 chains:
//   features               1000 rows      1500           2000           3000           5000
//   5, binary64            0.96 0.92      1.02 0.98      1.05 1.02      1.13 1.11      1.18 1.06
//   9                      0.97 0.93      1.05 1.04      1.07 1.05      1.12 1.10      1.19 1.20
//   25                     1.03 0.98      1.12 1.08      1.16 1.13      1.22 1.17      1.31 1.26
//   60 (residuals)         1.20 1.11      1.31 1.27      1.34 1.30      1.49 1.46      1.67 1.69
//   9, binary32 (same)     1.05 1.03      1.20 1.18
constexpr int kWideMaxPairs = 256;
inline bool wide_split_pays(long n_chains, int cus, long iters, long n, bool residual)
{
    return n >= (residual || iters > 1 ? 1000 : 1500) && (n_chains + 3) / 4 * 2 <= cus;
}

inline size_t wide_block_bytes(int d, int dtype_bytes, int nc, int max_depth)
{
    const int cpl = ((d + 15) / 16 * 16 + 31) / 32;
    return (size_t)nc * wide_num_vectors(max_depth) * kTileLanes * cpl * dtype_bytes;
}

// One instantiation per feature-tile count and form (each dtype in a translation unit of its own).
template <typename T, int MT>
inline void wide_launch_mt(const WideArgs& wa, const DevSample& sa, int nc, int blocks, hipStream_t stream)
{
    // (binary64 with up to 32 features: sixteen chains per workgroup are the tile kernel's)
    if constexpr (sizeof(T) == 4 || MT > 2) {
        if (nc == 16) {
            hipLaunchKernelGGL((nuts_wide_kernel<T, MT, 16, false>), dim3((unsigned)blocks), dim3(kTileThreads), 0, stream, wa, sa);
            return;
        }
    }
    if (wa.n_pairs > 0) {
        hipLaunchKernelGGL((nuts_wide_kernel<T, MT, 4, true>), dim3((unsigned)(wa.n_pairs + 7) / 8 * 16), dim3(kTileThreads / 2), 0, stream, wa, sa);
        return;
    }
    hipLaunchKernelGGL((nuts_wide_kernel<T, MT, 4, false>), dim3((unsigned)blocks), dim3(kTileThreads), 0, stream, wa, sa);
}
template <typename T>
inline void wide_launch(const WideArgs& wa, const DevSample& sa, int nc, int blocks, hipStream_t stream)
{
    switch ((wa.ta.d + 15) / 16) {
    case 1: wide_launch_mt<T, 1>(wa, sa, nc, blocks, stream); break;
    case 2: wide_launch_mt<T, 2>(wa, sa, nc, blocks, stream); break;
    case 3: wide_launch_mt<T, 3>(wa, sa, nc, blocks, stream); break;
    case 4: wide_launch_mt<T, 4>(wa, sa, nc, blocks, stream); break;
    case 5: wide_launch_mt<T, 5>(wa, sa, nc, blocks, stream); break;
    case 6: wide_launch_mt<T, 6>(wa, sa, nc, blocks, stream); break;
    case 7: wide_launch_mt<T, 7>(wa, sa, nc, blocks, stream); break;
    default: wide_launch_mt<T, 8>(wa, sa, nc, blocks, stream); break;
    }
}
void wide_launch_f64(const WideArgs& wa, const DevSample& sa, int nc, int blocks, hipStream_t stream);
void wide_launch_f32(const WideArgs& wa, const DevSample& sa, int nc, int blocks, hipStream_t stream);

}  // namespace nuts
