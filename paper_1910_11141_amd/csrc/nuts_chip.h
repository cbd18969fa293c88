// Chip kernel: logistic regression whose rows are spread over the whole chip, one persistent workgroup per compute unit (fewer
// where something else holds compute units; then a workgroup has several slices of the rows, and every chain the same bits).
//
// The chains step together, as in the wide kernel, but a round's two GEMMs  Z = X~ Theta,  G = X~' sigma(-Z)  are shared by all
// compute units, and a round is two phases of one launch that are separated by barriers over all workgroups:
//   control   every chain has a wave of its own, which keeps it in registers from the first round to the last (nuts_row.h).  Its
//             workgroup sums the row slices' partial gradients of its chains in binary64 in a fixed order; the wave
//             finishes the step, goes on to the next point that needs a gradient and publishes the position in a column of
//             Theta;
//   gradient  every workgroup has a slice of the rows, and a share of the columns where there are fewer slices than workgroups.
//             Its eight waves have tiles of 16 rows each, in LDS in one order that serves both GEMMs (and stay there
//             from round to round if a wave has only one), take groups of 16 columns through 16x16x4 matrix instructions, and
//             add their sums up in LDS in a fixed order, in binary64: one partial gradient per slice and column.
// As in the tile kernel, X~ = diag(2y - 1) X, so the labels never reach the GPU arithmetic:
// y z - log(1+e^z) = -log(1+e^{-z~}),  X'(y - sigma(z)) = X~' sigma(-z~).
//
// A chain that waits for a gradient has one of the first columns, however many have nothing to do (their trajectories
// have different lengths: on average three quarters of a short run); a column's sums do not depend on where it lies or
// on how many there are, and the split of the rows depends on the target only: a chain has the same bits in any company.
//
// What workgroups tell each other - positions, partial gradients, counters - is written through to and read from memory behind the
// L2 caches (which the eight XCDs do not share): agent scope, without fences that would empty the caches of everything else.
//
// What bounds it: with all columns busy the matrix instructions (53 of 32 ticks per 16 x 16 tile at d = 100) and the vector ones of
// the logistic functions beside them (290 ticks); with few the two barriers (1.7 us each over 256 workgroups, a counter per
// residue of the workgroup number modulo 8; flags that everybody polls: 3.1 to 5.5 us), the latency of the partial sums and of
// the chain program.  10 000 x 100: a round takes 11.5 us with one chain, 27 us with 227 columns busy (control with its barrier 7 us,
// positions 2.5, tiles 13, their sums and the second barrier 5).  1024 chains, 4 iterations of the slice sampler with four
// steps a leaf: 10.9 ms with two launches a round (nuts_grid.h) -> 8.4 (8.2 with the sums of a wave's rows in one accumulator).  185 to 238 vector registers, none in scratch memory.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "nuts_dev.h"
#include "nuts_row.h"
#include "nuts_tile_common.h"

namespace nuts {

constexpr int kChipMaxDim = 128;
constexpr int kChipWaves = 8;
constexpr int kChipThreads = kChipWaves * kWave;
constexpr int kChipOwners = 4;                 // waves of a workgroup that own a chain: 1 .. 4 (the first one waits for others)
constexpr int kChipMaxBlocks = 256;            // workgroups
constexpr int kChipMaxSlices = 128;            // row slices
constexpr int kChipRows = 16;                  // rows of a tile, columns of a group
constexpr int kChipCounters = 8;               // barrier counters (and ranges of columns)
constexpr int kChipRange = kChipMaxBlocks / kChipCounters * kChipOwners;  // columns of a range
constexpr int kChipColumns = kChipCounters * kChipRange;                  // 1024: chains resident at a time
constexpr int kChipLds = 160 * 1024, kChipStatic = 256;  // of which static variables

struct ChipData {
    float* x = nullptr;  // device: [tile][16 rows][pitch], X~ padded with zeros
    int d = 0, mt = 0, n_tiles = 0;
    long n_rows = 0;
};

template <int MT>
struct ChipShape {
    static constexpr int V = 4;                            // elements of a 16-byte access
    static constexpr int K = 16 * MT;                      // padded features
    static constexpr int P = K + V;                        // pitch of a row in LDS: an odd number of 16-byte pieces
    static constexpr int kTile = kChipRows * P;            // elements of a tile
    static constexpr int kTileBytes = kTile * 4;
    static constexpr int kLoads = (kTileBytes + 1023) / 1024;
    static constexpr int NG = 2;                           // column groups that a pass over the tiles takes at once
    static constexpr int kTheta = 2 * kChipWaves * kTileBytes;             // offsets in LDS: two tiles a wave, positions,
    static constexpr int kLl = kTheta + NG * kTileBytes;                   // log-likelihoods [wave][column] doubles,
    static constexpr int kCols = kLl + kChipWaves * kChipRows * 8;         // list of the columns in use,
    static constexpr int kTree = kCols + kChipColumns * 2;                 // tree levels of the chains
    static_assert(kChipOwners * K * 8 <= kTileBytes, "partial sums of the control phase");
    static_assert(kTree + kChipStatic <= kChipLds, "LDS");
};
constexpr int chip_pitch(int mt) { return 16 * mt + 4; }

// Whether a target's runs are the chip kernel's or those of the grid kernels (nuts_grid.h), which overlap a set of chains'
// control with another's gradient: long gradients with all columns busy are theirs.  By the target alone: a chain's
// results must not change with the batch it runs in.  Time with the grid kernels over time here (and the table below, taken with
// sums of a wave's rows that were less exact and 3 % faster): 10 000 x 100, 64 to 4096
// chains, 4 to 50 iterations 1.01 to 1.7; 3000 x 9 and 1000 x 20, 16 to 4096 chains 1.3 to 1.8; 6052 x 7, awaited iterations 2.5;
// 40 000 x 10 1.1; 15 000 x 100 1.1; 20 000 x 48 and x 64, 4096 chains 1.14 and 1.00; 100 000 x 100, 256 chains, 40 iterations 0.80;
// 50 000 x 128, 2048 chains 0.89.  With 17 to 32 features, which are one tile of 32 there: 8000 x 32 1.1, 12 000 x 25 1.00, 20 000 x 25
// 0.93, 50 000 x 25 0.82.
inline bool chip_pays(int64_t n, int64_t d) { return d <= kChipMaxDim && (d > 16 && d <= 32 ? n <= 12000 : n * d <= 1500000); }

// Into how many slices a chip with room for `blocks` workgroups divides a target's tiles (the workgroups share the columns of a slice).  Few
// slices make long passes, whose sums and positions cost less, and few partial results: better with all columns busy; many
// make the rounds short in which few chains are left.  The largest power of two (which divides the chip evenly) whose
// square is at most 2.7 times the number of tiles, up to 128.  ms with 8, 16, 32, 64, 128, 256 slices, and what the rule takes:
//   10 000 x 100, 1024 chains, 4 iterations of the slice sampler   12.3  9.5  8.5  9.3 10.7 13.8   32
//   10 000 x 100, 4096 chains, 6 iterations                        21.8 22.6 24.8 31.1 38.0 50.7   32
//   100 000 x 100, 256 chains, 4 iterations                        36.1 19.1 11.5  8.2  6.9  6.8   128 (not this kernel's)
//   16 640 x 60, 700 chains, 6 iterations                           4.8  3.9  3.5  3.6  4.3  5.4   32
//   3000 x 9, 4096 chains, 12 iterations                            7.0  7.5  8.2 10.3 15.5 24.6   16
// It depends on the target only, never on the number of chains: a chain's results must not change with the batch it runs in.
inline int chip_slices(int n_tiles, int blocks)
{
    int s = 1;
    while (s < kChipMaxSlices && 2 * s <= blocks && 4.0 * s * s <= 2.7 * n_tiles) s *= 2;
    return s;
}

// The control phase sums a chain's partial gradients in kChipMaxSlices / 16 steps: in step i the two halves of wave w take slices
// 2w + 16i and the one after it.  Which of them there are: the halves' step, and the half in it.
constexpr __host__ __device__ bool chip_step_there(int wave, int i, int n_slices) { return 2 * wave + 16 * i < n_slices; }
constexpr __host__ __device__ bool chip_half_there(int half, int n_slices) { return half < n_slices; }
constexpr bool chip_slices_taken_once()
{
    for (int n = 1; n <= kChipMaxSlices; n *= 2) {  // (what chip_slices can return)
        int taken[kChipMaxSlices] = {};
        for (int wave = 0; wave < kChipWaves; ++wave)
            for (int i = 0; i < kChipMaxSlices / 16; ++i)
                for (int half = 0; half < 2; ++half)
                    if (chip_step_there(wave, i, n) && chip_half_there(half, n)) {
                        const int s = 2 * wave + half + 16 * i;
                        if (s >= n) return false;
                        ++taken[s];
                    }
        for (int s = 0; s < n; ++s)
            if (taken[s] != 1) return false;
    }
    return true;
}
static_assert(chip_slices_taken_once(), "every slice once, and none beyond the last");

// What the workgroups share, one cache line per counter: {arrivals at the first barrier, columns handed out, arrivals at the
// second barrier, arrivals at the start}.  Line kChipCounters: {state}.
constexpr int kChipLine = 32;  // unsigned
enum : unsigned { kChipWaiting = 0, kChipRunning = 1, kChipNotStarted = 2, kChipTimedOut = 3 };

struct ChipArgs {
    const float* x;
    int d, n_tiles, n_slices, n_slots, n_blocks;
    long n_rows;
    double prior_prec;
    float* theta;    // [column][K]
    float* g_part;   // [slice][column][K]
    double* ll_part; // [slice][column]
    unsigned* shared;
    unsigned theta_bytes, g_bytes;
};

typedef float ChipPiece __attribute__((ext_vector_type(4)));  // 16 bytes of a vector, or an accumulator
// element q of an accumulator of the 16x16x4 instruction: its row (of 16) in lane group h = lane / 16
__device__ __forceinline__ int chip_acc_row(int q, int h) { return 4 * h + q; }

// Barrier of a workgroup for what it keeps in LDS.  (A fence would wait for everything under way to or from memory: tiles that
// are fetched straight into LDS make the compiler wait for all of it.)
__device__ __forceinline__ void chip_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int kAgent = 16;  // cache policy of a buffer instruction: agent scope (sc1)

// Waits (first wave of a workgroup) until word `word` of every counter's line has reached target[counter]; returns false if
// the run is over for another reason.  Every wait ends: a start that not all workgroups reach (the chip is shared with
// somebody) is given up after half a second, any other wait after 60 s.
__device__ inline bool chip_wait(const ChipArgs& ca, int lane, int word, unsigned target, bool start, v4u& seen)
{
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(ca.shared, 0, (kChipCounters + 1) * kChipLine * 4, 0x00020000);
    const long long t0 = wall_clock64(), limit = start ? 50000000ll : 6000000000ll;  // (100 MHz)
    for (;;) {
        // (lanes beyond the last line read zeros)
        seen = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * kChipLine * 4, 0, kAgent));
        const bool there = lane >= kChipCounters || (int)(seen[word] - target) >= 0;
        const unsigned state = (unsigned)__builtin_amdgcn_readlane((int)seen[0], kChipCounters);
        if (state >= kChipNotStarted) return false;
        if (__all(there)) {
            if (!start) return true;
            unsigned s = 0;
            if (lane == 0) {
                unsigned expected = kChipWaiting;
                __hip_atomic_compare_exchange_strong(&ca.shared[kChipCounters * kChipLine], &expected, (unsigned)kChipRunning, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s = expected;
            }
            return uni((int)s) < (int)kChipNotStarted;
        }
        if (wall_clock64() - t0 > limit) {
            if (lane == 0) {
                unsigned expected = start ? kChipWaiting : kChipRunning;
                __hip_atomic_compare_exchange_strong(&ca.shared[kChipCounters * kChipLine], &expected,
                                                     (unsigned)(start ? kChipNotStarted : kChipTimedOut), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
            }
            // (somebody may have started the run in between: the next look tells)
            if (!start) return false;
        }
    }
}

// kSeveral: there are fewer workgroups than slices.  (An instance of its own: the slice as a variable costs up to 28 registers, and the
// largest instances some of their state.)
template <int MT, bool kSeveral>
__global__ __launch_bounds__(kChipThreads) void nuts_chip_kernel(ChipArgs ca, DevSample sa, RowLds rl)
{
    typedef ChipShape<MT> S;
    typedef ChipPiece Piece;
    typedef ChipPiece Acc;
    auto mfma = [](float a, float b, Acc c) __attribute__((always_inline)) -> Acc { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); };
    constexpr int K = S::K, P = S::P, V = S::V, NG = S::NG;
    extern __shared__ __align__(16) unsigned char smem[];
    float* const sX = reinterpret_cast<float*>(smem);                       // [stage][wave][tile]; sums of the waves use stage 1
    double* const sPart = reinterpret_cast<double*>(smem + kChipWaves * S::kTileBytes);  // control: [wave][owner][K] (stage 1, too)
    float* const sTheta = reinterpret_cast<float*>(smem + S::kTheta);
    double* const sLl = reinterpret_cast<double*>(smem + S::kLl);
    unsigned short* const sCols = reinterpret_cast<unsigned short*>(smem + S::kCols);
    __shared__ unsigned sLive[kChipOwners], sBase, sFirst[kChipCounters], sCount[kChipCounters];
    __shared__ int sOk, sColumn[kChipOwners];

    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uni(tid >> 6);
    const int j16 = lane & 15, h = lane >> 4;
    const int my_line = blockIdx.x % kChipCounters;
    const int owner = wave - 1, slot = owner * ca.n_blocks + (int)blockIdx.x;
    const bool owns = owner >= 0 && owner < kChipOwners && slot < ca.n_slots;
    unsigned* const line = ca.shared + my_line * kChipLine;
    const unsigned on_line = lane < kChipCounters ? (unsigned)((ca.n_blocks - lane + kChipCounters - 1) / kChipCounters) : 0u;  // workgroups of counter `lane`
    auto arrive = [&](int word) __attribute__((always_inline)) {
        __hip_atomic_fetch_add(line + word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    v4u seen;
    if (tid == 0) arrive(3);
    if (wave == 0) {
        const bool ok = chip_wait(ca, lane, 3, on_line, true, seen);
        if (lane == 0) sOk = ok;
    }
    if (tid < kChipOwners) sLive[tid] = tid * ca.n_blocks + (int)blockIdx.x < ca.n_slots;
    for (int i = tid; i < NG * S::kTile; i += kChipThreads) sTheta[i] = 0.0f;
    __syncthreads();
    if (!sOk) return;

    // ---- this workgroup's rows and columns: a slice and a share of the columns, or, of fewer workgroups than slices, several slices ----
    const int share = (int)blockIdx.x / ca.n_slices, n_shares = kSeveral ? 1 : ca.n_blocks / ca.n_slices;
    const bool computes = share < n_shares;
    int slice, t_first, t_end, n_steps;
    auto take_slice = [&](int s) __attribute__((always_inline)) {
        slice = s;
        t_first = (int)((long)ca.n_tiles * s / ca.n_slices);
        t_end = (int)((long)ca.n_tiles * (s + 1) / ca.n_slices);
        n_steps = computes ? (t_end - t_first + kChipWaves - 1) / kChipWaves : 0;  // of eight tiles
    };
    take_slice((int)blockIdx.x % ca.n_slices);
    // a wave works on two of a step's tiles (four apart), for one of a pass's two groups of columns
    const int quarter = wave & 3, my_group = wave >> 2;
    const int tail_steps = (ca.d - 16 * (MT - 1) + 3) / 4;  // contraction steps of the last 16 features
    auto fetch = [&](int i) __attribute__((always_inline)) {  // this wave's tile of step i, into stage i & 1
        const int tile = t_first + i * kChipWaves + wave;
        if (tile >= t_end) return;
        const char* src = reinterpret_cast<const char*>(ca.x) + (size_t)tile * S::kTileBytes + lane * 16;
        unsigned char* dst = smem + ((i & 1) * kChipWaves + wave) * S::kTileBytes;
#pragma unroll
        for (int l = 0; l < S::kLoads; ++l)
            if (l * 1024 + lane * 16 < S::kTileBytes)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + l * 1024),
                                                 (__attribute__((address_space(3))) void*)(dst + l * 1024), 16, 0, 0);
    };
    if (n_steps > 0) fetch(0);
    bool fetching = true;  // step 0 may be on its way

    const __amdgpu_buffer_rsrc_t theta_rsrc = __builtin_amdgcn_make_buffer_rsrc(ca.theta, 0, (int)ca.theta_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t g_rsrc = __builtin_amdgcn_make_buffer_rsrc(ca.g_part, 0, (int)ca.g_bytes, 0x00020000);

    RowChain<float, 1, true, true, true> ch(sa, ca.d, lane, reinterpret_cast<float*>(sa.workspace + (size_t)(owns ? slot : 0) * sa.slot_bytes),
                                  reinterpret_cast<float*>(smem + S::kTree) + (size_t)(owns ? owner : 0) * (rl.n_first + rl.n_pool) * 2 * 128, rl);
    enum { kInit, kLeaf, kDone };
    int state = kDone, sub = 0, column = 0;
    unsigned handed_out = 0;  // lane c of the first wave: columns that range c had handed out before this round
    unsigned long long n_rounds = 0, n_issued = 0;
    long long cyc_control = 0, cyc_grad = 0;

    // which 16-byte pieces of a pass's columns this thread moves
    constexpr int kThPieces = (NG * kChipRows * (K / V) + kChipThreads - 1) / kChipThreads;
    int th_col[kThPieces], th_at[kThPieces];
#pragma unroll
    for (int q = 0; q < kThPieces; ++q) {
        th_col[q] = (tid + q * kChipThreads) / (K / V);
        th_at[q] = (tid + q * kChipThreads) % (K / V) * V;
    }

    for (unsigned epoch = 1;; ++epoch) {
        const long long t0 = clock64();
        // ---- 1. control ----
        // a column for every chain that is alive (one that ends in this round leaves its column unused)
        unsigned live[kChipOwners], n_live = 0;
#pragma unroll
        for (int o = 0; o < kChipOwners; ++o) {
            live[o] = (unsigned)uni((int)sLive[o]);
            n_live += live[o];
        }
        unsigned base = 0;
        if (tid == 0 && n_live > 0) base = __hip_atomic_fetch_add(line + 1, n_live, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool waits = epoch > 1;
        double ll = 0.0;
        if (waits && owns && live[owner & (kChipOwners - 1)]) {
            double l[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int s = lane + 64 * i;
                l[i] = 0.0;
                if (s < ca.n_slices) l[i] = __hip_atomic_load(&ca.ll_part[(size_t)s * kChipColumns + column], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            ll = l[0] + l[1];
        }
        if (waits) {
            // half a wave sums every 16th slice of a chain: slices 2 wave + half + 16 i, in that order; the loads of two chains
            // are under way together (of all four: 128 registers, and the chain's state is spilled)
            const int half = lane >> 5, piece = lane & 31;
            const unsigned row = (unsigned)(K * 4), per_slice = row * kChipColumns;
            // (lanes beyond the last feature, and the second half where there is one slice, read zeros: their own offset is past the
            // end of the buffer)
            const int lane_off = piece < K / V && chip_half_there(half, ca.n_slices) ? (int)(half * per_slice + piece * 16) : (int)0xc0000000u;
            constexpr int kMost = kChipMaxSlices / 16;
#pragma unroll
            for (int o0 = 0; o0 < kChipOwners; o0 += 2) {
                Piece p[2][kMost];
#pragma unroll
                for (int o = o0; o < o0 + 2; ++o) {
                    if (!live[o]) continue;
                    int at = (int)(2 * wave * per_slice + (unsigned)uni(sColumn[o]) * row);
#pragma unroll
                    for (int i = 0; i < kMost; ++i) {
                        if (chip_step_there(wave, i, ca.n_slices)) p[o - o0][i] = __builtin_bit_cast(Piece, __builtin_amdgcn_raw_buffer_load_b128(g_rsrc, lane_off, at, kAgent));
                        at += (int)(16 * per_slice);
                    }
                }
#pragma unroll
                for (int o = o0; o < o0 + 2; ++o) {
                    if (!live[o]) continue;
                    double a[V];
#pragma unroll
                    for (int e = 0; e < V; ++e) a[e] = 0.0;
#pragma unroll
                    for (int i = 0; i < kMost; ++i)
                        if (chip_step_there(wave, i, ca.n_slices))
#pragma unroll
                            for (int e = 0; e < V; ++e) a[e] += (double)p[o - o0][i][e];
#pragma unroll
                    for (int e = 0; e < V; ++e) a[e] = add_other_half(a[e]);
                    if (half == 0 && piece < K / V) {
#pragma unroll
                        for (int e = 0; e < V; ++e) sPart[(wave * kChipOwners + o) * K + piece * V + e] = a[e];
                    }
                }
            }
        }
        if (tid == 0) sBase = base;
        chip_barrier();
        if (owns && live[owner & (kChipOwners - 1)]) {
            double lp = 0.0;
            if (waits) {
                double ll_share = 2.0 * ll;  // (the chain program halves the sum)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 2 * lane + e;
                    double sum = 0.0;
                    const double t = (double)ch.th[e];
                    if (i < K) {
                        const double* s = sPart + (size_t)owner * K + i;
                        constexpr int st = kChipOwners * K;
                        sum = ((s[0] + s[st]) + (s[2 * st] + s[3 * st])) + ((s[4 * st] + s[5 * st]) + (s[6 * st] + s[7 * st]));
                    }
                    ch.g[e] = i < ca.d ? (float)(sum - t * ca.prior_prec) : 0.0f;
                    ll_share = fma(t * -ca.prior_prec, t, ll_share);
                }
                lp = ll_share;
            }
            bool fetch_next = !waits, begin_iter = false, begin_double = false;
            if (state == kInit) {
                ch.start_chain(lp);
                begin_iter = true;
                state = kLeaf;
            } else if (state == kLeaf) {
                ch.kick();
                if (++sub >= sa.leaf_steps) {
                    sub = 0;
                    if (!ch.finish_leaf(lp)) {
                        begin_double = ch.double_end();
                        if (!begin_double) {
                            begin_iter = ch.iter_end();
                            fetch_next = !begin_iter;
                        }
                    }
                }
            }
            if (begin_iter) ch.iter_begin();
            if (begin_iter || begin_double) ch.double_begin();
            if (fetch_next) state = ch.fetch() ? kInit : kDone;
            if (state == kLeaf) ch.kick_drift();
            // the column of this round
            unsigned rank = 0;
#pragma unroll
            for (int o = 0; o < kChipOwners; ++o) rank += o < owner ? live[o] : 0u;
            column = my_line * kChipRange + (int)(((unsigned)uni((int)sBase) - (unsigned)uni((int)sFirst[my_line]) * (epoch > 1)) + rank);
            if (state != kDone) {
                if (2 * lane < K) {
                    const unsigned off = (unsigned)(column * K + 2 * lane) * 4u;
                    typedef unsigned v2u __attribute__((ext_vector_type(2)));
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, make_float2(ch.th[0], ch.th[1])), theta_rsrc, (int)off, 0, kAgent);
                }
            }
            if (lane == 0) {
                sLive[owner] = state != kDone;
                sColumn[owner] = column;
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) arrive(0);
        if (wave == 0) {
            const bool ok = chip_wait(ca, lane, 0, epoch * on_line, false, seen);
            const unsigned now = seen[1];
            if (lane < kChipCounters) {
                sCount[lane] = now - handed_out;
                sFirst[lane] = now;  // (for the columns of the next round)
                handed_out = now;
            }
            if (lane == 0) sOk = ok;
        } else if (owns && state != kDone) {
            // while the others arrive: the random numbers of the chain's next iteration
            const int next = state == kInit ? ch.iter : ch.iter + 1;
            if (ch.ahead != next && next < sa.iter_end) ch.draw_ahead(next);
        }
        __syncthreads();
        if (!sOk) break;
        unsigned counts[kChipCounters], total = 0;
#pragma unroll
        for (int c = 0; c < kChipCounters; ++c) {
            counts[c] = (unsigned)uni((int)sCount[c]);
            total += counts[c];
        }
        if (total == 0) break;  // every chain has ended
        const long long t1 = clock64();
        n_rounds += 1;
        n_issued += (total + kChipRows - 1) / kChipRows * kChipRows;

        // ---- 2. gradient ----
        const int n_groups = (int)((total + kChipRows - 1) / kChipRows);
        if (computes && share < n_groups) {
            // the columns in use, one after the other: number k is in range c, place k minus the ranges before it
            for (int k = tid; k < (int)total; k += kChipThreads) {
                int c = 0, left = k;
#pragma unroll
                for (int i = 0; i < kChipCounters - 1; ++i)
                    if (c == i && left >= (int)counts[i]) {
                        left -= (int)counts[i];
                        c = i + 1;
                    }
                sCols[k] = (unsigned short)(c * kChipRange + left);
            }
            chip_barrier();
            Piece th_next[kThPieces];
            // positions of the groups g and g + n_shares: piece `q` of this thread
            auto ask_theta = [&](int g) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < kThPieces; ++q) {
                    const int k = (g + (th_col[q] / kChipRows) * n_shares) * kChipRows + th_col[q] % kChipRows;
                    const unsigned off = th_col[q] < NG * kChipRows && k < (int)total ? (unsigned)(sCols[k & (kChipColumns - 1)] * K + th_at[q]) * 4u : 0xffffff00u;
                    th_next[q] = __builtin_bit_cast(Piece, __builtin_amdgcn_raw_buffer_load_b128(theta_rsrc, (int)off, 0, kAgent));
                }
            };
            for (;;) {
            ask_theta(share);
            for (int g = share; g < n_groups; g += NG * n_shares) {
#pragma unroll
                for (int q = 0; q < kThPieces; ++q)
                    if (th_col[q] < NG * kChipRows) *reinterpret_cast<Piece*>(sTheta + th_col[q] * P + th_at[q]) = th_next[q];
                if (fetching) {  // (a slice of one step stays where it is)
                    __builtin_amdgcn_s_waitcnt(0);
                    fetching = false;
                }
                chip_barrier();  // positions and the first step's tiles are there, and everybody has read the last pass's sums
                const bool more = g + NG * n_shares < n_groups, busy = g + my_group * n_shares < n_groups;
                const float* const theta = sTheta + (my_group * kChipRows + j16) * P;
                Acc G[MT];
                double ll_sum = 0.0;
#pragma unroll
                for (int u = 0; u < MT; ++u) G[u] = Acc{0, 0, 0, 0};
                for (int i = 0; i < n_steps; ++i) {
                    if (i > 0) {
                        __builtin_amdgcn_s_waitcnt(0);
                        chip_barrier();  // this step's tiles are there, and the last step's have been read
                    }
                    if (i + 1 < n_steps) fetch(i + 1);
                    if (i == 0 && more) ask_theta(g + NG * n_shares);
                    const int tile0 = t_first + i * kChipWaves + quarter;
                    if (!busy || tile0 >= t_end) continue;
                    const float* const stage = sX + ((i & 1) * kChipWaves + quarter) * S::kTile;
                    // one or two tiles; every operand is asked for one block or feature tile ahead of its use (left to itself the
                    // compiler waits for each as it comes)
                    auto tiles = [&](auto count) __attribute__((always_inline)) {
                        constexpr int N = decltype(count)::value;
                        Acc z[N];
#pragma unroll
                        for (int p = 0; p < N; ++p) z[p] = Acc{0, 0, 0, 0};
                        constexpr int kBlocks = (K - 16) / (4 * V), kNext = 4 * S::kTile;  // (the second tile is four further on)
                        float x_tail[N][4], t_tail[4];
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            t_tail[s] = theta[K - 16 + 4 * s + h];
#pragma unroll
                            for (int p = 0; p < N; ++p) x_tail[p][s] = stage[p * kNext + j16 * P + K - 16 + 4 * s + h];
                        }
                        Piece xa[2][N], ta[2];
                        auto ask = [&](int b) __attribute__((always_inline)) {
                            ta[b & 1] = *reinterpret_cast<const Piece*>(theta + V * h + 4 * V * b);
#pragma unroll
                            for (int p = 0; p < N; ++p) xa[b & 1][p] = *reinterpret_cast<const Piece*>(stage + p * kNext + j16 * P + V * h + 4 * V * b);
                        };
                        if (kBlocks > 0) ask(0);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            if (s < tail_steps) {
#pragma unroll
                                for (int p = 0; p < N; ++p) z[p] = mfma(x_tail[p][s], t_tail[s], z[p]);
                            }
                        // blocks of 4 V features: 16 bytes of a row per lane, whose elements are V steps of the contraction
#pragma unroll
                        for (int b = 0; b < kBlocks; ++b) {
                            if (b + 1 < kBlocks) ask(b + 1);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int q = 0; q < V; ++q)
#pragma unroll
                                for (int p = 0; p < N; ++p) z[p] = mfma(xa[b & 1][p][q], ta[b & 1][q], z[p]);
                        }
                        float xg[2][N][4];
                        auto ask_tile = [&](int u) __attribute__((always_inline)) {
#pragma unroll
                            for (int p = 0; p < N; ++p)
#pragma unroll
                                for (int q = 0; q < 4; ++q) xg[u & 1][p][q] = stage[p * kNext + chip_acc_row(q, h) * P + 16 * u + j16];
                        };
                        ask_tile(0);
                        __builtin_amdgcn_sched_barrier(0);
                        float sg[N][4];
                        float pr = 1.0f, hinge = 0.0f;
#pragma unroll
                        for (int p = 0; p < N; ++p) {
                            const long row0 = (long)(tile0 + 4 * p) * kChipRows;
                            if (row0 + kChipRows > ca.n_rows) {
                                // rows beyond the last: a logit at which the residual and both terms of the log-likelihood are zero
#pragma unroll
                                for (int q = 0; q < 4; ++q)
                                    if (row0 + chip_acc_row(q, h) >= ca.n_rows) z[p][q] = 1e30f;
                            }
                            // log(1 + e^-z) = log(1 + e^-|z|) - min(z, 0), a lane's first terms as one logarithm of the product of
                            // their arguments (each in [1, 2]); single hardware instructions: the arguments are in their safe
                            // ranges; a NaN logit makes every result NaN
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const float zt = z[p][q];
                                const float e = __builtin_amdgcn_exp2f(fabsf(zt) * -1.44269504088896341f);
                                const float tt = 1.0f + e;
                                sg[p][q] = (zt < 0.0f ? 1.0f : e) * __builtin_amdgcn_rcpf(tt);
                                pr *= tt;
                                hinge -= __builtin_amdgcn_fmed3f(zt, -INFINITY, 0.0f);
                            }
                        }
                        ll_sum -= (double)fmaf(__builtin_amdgcn_logf(pr), 0.69314718055994531f, hinge);
                        // A tile's 16 rows are one binary32 sum; tiles are added in binary32, the four waves of a slice and the slices
                        // in binary64.  RMS error of the gradient over that of one binary32 sum per 64 rows (per 32 of fewer than 2048,
                        // per 256th of more than 16 384), emulated, 130 x 128 to 90 000 x 16: 0.28 to 0.99.  With all of a wave's rows in one
                        // binary32 sum, and the waves', it was 0.66 to 1.67 at 2.8 % less time (10 000 x 100, 1024 chains); with 32 rows a
                        // sum 0.29 to 1.19.
                        Acc t[2][N];
                        auto add = [&](int u) __attribute__((always_inline)) { G[u] += N == 2 ? t[u & 1][0] + t[u & 1][N - 1] : t[u & 1][0]; };
#pragma unroll
                        for (int u = 0; u < MT; ++u) {
                            if (u + 1 < MT) ask_tile(u + 1);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int p = 0; p < N; ++p) t[u & 1][p] = Acc{0, 0, 0, 0};
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int p = 0; p < N; ++p) t[u & 1][p] = mfma(xg[u & 1][p][q], sg[p][q], t[u & 1][p]);
                            if (u > 0) add(u - 1);
                        }
                        add(MT - 1);
                    };
                    if (tile0 + 4 < t_end) tiles(std::integral_constant<int, 2>{});
                    else tiles(std::integral_constant<int, 1>{});
                }
                // The waves' sums, through stage 1.  (Where the last step was in stage 0, nobody has read stage 1 since the
                // barrier that this step, or this pass, began with.)
                if ((n_steps & 1) == 0) chip_barrier();
                float* const sSum = sX + kChipWaves * S::kTile;
                ll_sum = add_other_half(add_other_row(ll_sum));
                if (lane < kChipRows) sLl[wave * kChipRows + lane] = ll_sum;
                float* const mine = sSum + wave * S::kTile + j16 * P;
#pragma unroll
                for (int u = 0; u < MT; ++u) *reinterpret_cast<Piece*>(mine + 16 * u + 4 * h) = G[u];
                chip_barrier();
                if (n_steps > 1 && (!kSeveral || more)) {
                    fetch(0);  // for the next pass or round
                    fetching = true;
                }
#pragma unroll
                for (int q = 0; q < kThPieces; ++q) {
                    const int k = (g + (th_col[q] / kChipRows) * n_shares) * kChipRows + th_col[q] % kChipRows;
                    if (th_col[q] < NG * kChipRows && k < (int)total) {
                        const float* const w = sSum + (th_col[q] / kChipRows) * 4 * S::kTile + (th_col[q] % kChipRows) * P + th_at[q];
                        Piece part[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) part[r] = *reinterpret_cast<const Piece*>(w + r * S::kTile);
                        Piece sum;
#pragma unroll
                        for (int e = 0; e < V; ++e) sum[e] = (float)(((double)part[0][e] + (double)part[1][e]) + ((double)part[2][e] + (double)part[3][e]));
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, sum), g_rsrc,
                                                               (int)((((unsigned)slice * kChipColumns + sCols[k]) * K + th_at[q]) * 4u), 0, kAgent);
                    }
                }
                if (tid < NG * kChipRows) {
                    const int k = (g + (tid / kChipRows) * n_shares) * kChipRows + tid % kChipRows;
                    if (k < (int)total) {
                        const double* const w = sLl + (tid / kChipRows) * 4 * kChipRows + tid % kChipRows;
                        double part[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) part[r] = w[r * kChipRows];
                        __hip_atomic_store(&ca.ll_part[(size_t)slice * kChipColumns + sCols[k]], (part[0] + part[1]) + (part[2] + part[3]),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
            }
            if constexpr (!kSeveral) break;
            // (nobody reads stage 0 since the barrier before the sums)
            const bool again = slice + ca.n_blocks < ca.n_slices;
            take_slice(again ? slice + ca.n_blocks : (int)blockIdx.x);
            fetch(0);
            fetching = true;
            if (!again) break;
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) arrive(2);
        if (wave == 0) {
            const bool ok = chip_wait(ca, lane, 2, epoch * on_line, false, seen);
            if (lane == 0) sOk = ok;
        }
        __syncthreads();
        if (!sOk) break;
        cyc_control += t1 - t0;
        cyc_grad += clock64() - t1;
    }

    if (owns && lane == 0) {
        atomicAdd(&sa.counters[kCtrUseful], ch.n_leaf);
        atomicAdd(&sa.counters[kCtrExtra], ch.n_extra);
    }
    if (blockIdx.x == 0 && tid == 0) {
        atomicAdd(&sa.counters[kCtrIssued], n_issued);
        atomicAdd(&sa.counters[kCtrRounds], n_rounds);
        atomicAdd(&sa.counters[kCtrCycControl], (unsigned long long)cyc_control);
        atomicAdd(&sa.counters[kCtrCycGrad], (unsigned long long)cyc_grad);
    }
}

// Launch shape of a run.
struct ChipPlan {
    int blocks;
    size_t lds_bytes, slot_bytes;
    RowLds rl;
};
template <int MT>
inline void chip_lds_inst(int max_depth, ChipPlan* cp)
{
    const size_t room = kChipLds - kChipStatic - ChipShape<MT>::kTree;
    cp->rl = row_lds_split(room / kChipOwners, 1, sizeof(float), max_depth, true);
    cp->lds_bytes = ChipShape<MT>::kTree + (size_t)kChipOwners * (cp->rl.n_first + cp->rl.n_pool) * row_entry_bytes(1, sizeof(float));
    cp->slot_bytes = ((size_t)row_num_vectors(max_depth) * 128 * sizeof(float) + 255) & ~(size_t)255;
}

template <int MT, bool kSeveral>
inline hipError_t chip_launch_inst(const ChipArgs& ca, const DevSample& sa, const ChipPlan& cp, hipStream_t stream)
{
    const void* fn = reinterpret_cast<const void*>(nuts_chip_kernel<MT, kSeveral>);
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)cp.lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((nuts_chip_kernel<MT, kSeveral>), dim3((unsigned)cp.blocks), dim3(kChipThreads), cp.lds_bytes, stream, ca, sa, cp.rl);
    return hipGetLastError();
}
template <int MT>
inline hipError_t chip_launch_inst(const ChipArgs& ca, const DevSample& sa, const ChipPlan& cp, hipStream_t stream)
{
    return ca.n_blocks < ca.n_slices ? chip_launch_inst<MT, true>(ca, sa, cp, stream) : chip_launch_inst<MT, false>(ca, sa, cp, stream);
}
// (in a translation unit of its own)
void chip_lds(int mt, int max_depth, ChipPlan* cp);
hipError_t chip_launch(int mt, const ChipArgs& ca, const DevSample& sa, const ChipPlan& cp, hipStream_t stream);

}  // namespace nuts
