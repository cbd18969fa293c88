// Device-side definitions shared by the sampler kernels: kernel argument
// blocks, the program-counter vocabulary of the hand-lowered NUTS recursion,
// and wavefront-level reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nuts {

constexpr int kWave = 64;
constexpr double kDeltaMax = 1000.0;  // a leaf whose energy error exceeds this is divergent

enum TargetKind : int { kStdNormal = 0, kGaussDense = 1, kGaussDiag = 2, kLogReg = 3 };

// Target data on the device, in the layouts the kernels read.
template <typename T>
struct DevTarget {
    int kind;
    int d;            // dimension
    int dstride;      // padded length of one state vector in the workspace (elements)
    int kl;           // logistic regression, wave kernel: lanes along the feature axis (power of two <= 64)
    int lds_matrix;   // dense Gaussian, wave kernel: the precision matrix is copied to LDS at kernel start
    long n;           // data rows
    const T* PT;      // dense Gaussian: transpose of the precision, [k][i]
    const T* band;    // dense Gaussian whose precision is banded (|i - k| <= kBandHalf): [row][k - i + kBandHalf],
                      // max(d, kBandRows) rows, zero outside the matrix; NULL otherwise
    const T* inv_var; // diagonal Gaussian: 1/sigma_i^2
    const T* X;       // logistic regression: [n][d]
    const T* XT;      // logistic regression: [d][n]
    const T* y;       // logistic regression: [n]
    double prior_prec;
};

// A precision matrix with at most this many off-diagonals on each side is treated as banded.
constexpr int kBandHalf = 4;
constexpr int kBandRows = 128;

// Per-call arguments.
struct DevSample {
    long n_chains;
    long first_chain;   // global id of local chain 0
    int n_iters;
    int iter_begin;     // this launch runs iterations [iter_begin, iter_end) of the n_iters
    int iter_end;
    int max_depth;
    int leaf_steps;     // leapfrog steps per tree leaf (>= 1)
    int sampler;        // kSamplerMultinomial or kSamplerSlice
    double eps;
    uint32_t key0, key1;
    void* out_states;
    int* out_depths;
    int* out_nleap;
    const void* init_states;
    char* workspace;
    size_t slot_bytes;  // workspace bytes per resident chain slot
    unsigned long long* counters;
};

// How the leaves of a trajectory are weighted.  Multinomial: leaf weight exp(H0 - H), subtrees carry
// their summed weights (general wave and grid kernels: as logarithms; the others: as numbers in a unit that moves
// when the energy falls far).  Slice (Algorithm 3 of Hoffman & Gelman, the published form):
// a height is drawn below exp(-H0) once per iteration, leaves at or above it count 1, the others 0,
// and subtrees carry their count.  The count travels in the same variables as the weight
// (an integer below 2^21 is exact in binary64).
enum : int { kSamplerMultinomial = 0, kSamplerSlice = 1 };

// counters[] slots
enum : int {
    kCtrQueue = 0, kCtrIssued = 1, kCtrUseful = 2, kCtrExtra = 3, kCtrRounds = 4,
    kCtrCycControl = 5, kCtrCycGrad = 6, kCtrCycPost = 7,  // shader-clock ticks, summed over workgroups
    kCtrSlotMax = 8,  // wave and element-wise kernels: most gradient evaluations done by one slot in this launch
    kCtrPairsMet = 9, kCtrPairsLost = 10,  // wide kernel, divided rows: groups whose workgroups met, and that one of them went on with alone
    kCtrTurns = 11,  // row kernels: chains handed over
    kCtrCount = 12
};

// Program points of one chain.  This is the NUTS recursion written in the
// vocabulary of program-counter batching (Figure 4 / Algorithm 2 of the paper):
// BUILD is the body of the recursive tree builder, AFTER_LEFT / AFTER_RIGHT are
// the return points of its two recursive calls, DOUBLE_END is the return point
// of the top-level call.  LEAF and INIT_EVAL are the points where a chain needs
// the target's gradient: the scheduler runs every chain up to such a point and
// then evaluates all waiting gradients together.  Blocks are numbered in
// program order, which is also the order the scheduler picks them in
// ("earliest block first", Section 2).
enum Pc : int {
    kPcFetch = 0,       // take the next chain from the queue, make x0
    kPcIterBegin = 1,   // draw the momentum, H0, reset the trajectory
    kPcDoubleBegin = 2, // draw the direction, call BUILD(level = j)
    kPcBuild = 3,       // level == 0 ? LEAF : call BUILD(level-1), return to AFTER_LEFT
    kPcAfterLeft = 4,   // left half done: stop early, or save its summary and call BUILD for the right half
    kPcAfterRight = 5,  // right half done: merge weights, select the proposal, U-turn test over the span
    kPcDoubleEnd = 6,   // top level: accept the new half, whole-trajectory U-turn test, loop or finish
    kPcIterEnd = 7,     // emit the iteration's outputs
    kPcInitEval = 8,    // waiting for (logp, grad) at x0
    kPcLeaf = 9,        // waiting for a leapfrog step
    kPcHalt = 10
};

// Return addresses live in a 2-bit-per-entry stack packed into 64 bits
// (depth <= max_tree_depth + 1 <= 21 entries).
enum RetCode : unsigned { kRetAfterLeft = 0, kRetAfterRight = 1, kRetDoubleEnd = 2 };

// For caches keyed by a leapfrog count: a count that no leaf has, and none a few leaves further on.
constexpr int kNoLeaf = -(1 << 30);

__device__ __forceinline__ int ret_to_pc(unsigned code)
{
    return code == kRetAfterLeft ? kPcAfterLeft : (code == kRetAfterRight ? kPcAfterRight : kPcDoubleEnd);
}

// A binary64 value moved between lanes by a DPP control word (two 32-bit moves).
template <int kCtrl>
__device__ __forceinline__ double dpp_rotate(double x)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), kCtrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), kCtrl, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double read_lane(double x, int src_lane)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), src_lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), src_lane);
    return __hiloint2double(hi, lo);
}

// Sums over the 64 lanes of a wave (all lanes active), up to four of them in one pass.  The halves of the wave change places
// first, then the rows of 16 lanes: where two sums are wanted each ends up with half of the lanes, of four each with a row, and
// what is left - rotations by 8, 4, 2, 1 inside the rows (DPP, no LDS traffic) - is done once for all of them.  A sum's terms are
// added in the same order whichever of these functions takes it, and both partners of a step add the same pair of values, so
// every lane of a row ends with the same bits.  Two sums are 24 instructions (two by rotations alone and the four row totals
// read as scalars: 48, half of them waiting for the one before), four are 29.
__device__ __forceinline__ double fold_halves(double a, double b)  // lanes 0..31: a[l] + a[l + 32]; 32..63: b[l - 32] + b[l]
{
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double fold_rows(double x, double y)  // rows: x0 + x1, y0 + y1, x2 + x3, y2 + y3
{
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(y), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double row_sum(double x)
{
    x += dpp_rotate<0x128>(x);  // row_ror:8
    x += dpp_rotate<0x124>(x);  // row_ror:4
    x += dpp_rotate<0x122>(x);  // row_ror:2
    x += dpp_rotate<0x121>(x);  // row_ror:1
    return x;
}
// a in lanes 0..31, b in lanes 32..63
__device__ __forceinline__ double wave_sum_halves(double a, double b)
{
    const double x = fold_halves(a, b);
    return row_sum(fold_rows(x, x));
}
// rows of 16 lanes: a, c, b, d
__device__ __forceinline__ double wave_sum_rows(double a, double b, double c, double d)
{
    return row_sum(fold_rows(fold_halves(a, b), fold_halves(c, d)));
}

// What lanes 0..31 hold (all the same) in every lane, and what lanes 32..63 hold.  (Not through scalar registers: an
// instruction that wants a scalar a vector instruction has just made waits some 50 ticks.)
__device__ __forceinline__ void spread_halves(double x, double& lower, double& upper)
{
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x), (unsigned)__double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(x), false, false);
    lower = __hiloint2double((int)hi[0], (int)lo[0]);
    upper = __hiloint2double((int)hi[1], (int)lo[1]);
}
// Rows 0 and 2 in both rows of their half.
__device__ __forceinline__ double spread_even_rows(double x)
{
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(x), (unsigned)__double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2hiint(x), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]);
}

__device__ __forceinline__ double wave_sum(double x) { return wave_sum_halves(x, x); }
__device__ __forceinline__ void wave_sum2(double& a, double& b) { spread_halves(wave_sum_halves(a, b), a, b); }

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
// A condition that all lanes agree on, as a scalar: what is decided by it can stay in scalar registers.
__device__ __forceinline__ bool agreed(bool x) { return __ballot(x) != 0; }

}  // namespace nuts
