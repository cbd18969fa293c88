// What the tile kernels share (nuts_tile.h: up to 32 features, binary64, 16 chains per workgroup; nuts_wide.h: up to
// 128 features, both dtypes, 16 or 4 chains): the packed operand stream, the arguments, and the reductions over the
// 32 lanes of a chain.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <vector>

#include "nuts_dev.h"

namespace nuts {

constexpr int kTileMaxDim = 32;    // of the 16-chain binary64 kernel of nuts_tile.h
constexpr int kWideMaxDim = 128;   // of the kernel of nuts_wide.h
constexpr int kTileMaxDepth = 12;
constexpr int kTileChains = 16;    // chains per workgroup = MFMA N
constexpr int kTileLanes = 32;     // lanes per chain in the control phase
constexpr int kTileWaves = 8;
constexpr int kTileThreads = kTileWaves * kWave;
constexpr int kTileRows = 16;      // data rows per MFMA tile = MFMA M of the first GEMM
constexpr int kTileLdsPool = 5;    // proposal-pool buffers 0..4 of every chain live in LDS
constexpr int kTileLdsFirst = 4;   // first-leaf slots 1..4 of every chain live in LDS (with the tables 158 KB of the 160)

struct TileData {
    double* base = nullptr;  // device: operands of every row tile, in MFMA lane order
    double* ftab = nullptr;  // device: softplus table (kFtabDoubles) followed by the logarithm table (kLogTabDoubles)
    double* colsum = nullptr;  // device: column sums of X~ (kWideMaxDim values, zero padded)
    int d = 0;
    int ks1 = 0;             // k-steps of the first GEMM  = ceil(d / 4)
    int mt = 0;              // M-tiles of the second GEMM = ceil(d / 16)
    int n_tiles = 0;         // row tiles that are run
    int n_alloc_tiles = 0;   // row tiles in the operand stream
    long n_rows = 0, n_pad = 0;
    int z0_col = -1;         // the constant column that stays out of the first GEMM, or -1
    double z0_val = 0.0;     // its value
    bool residual = false;   // laid out for the residual form of the wide kernel: no constant column, real tiles only
};

struct TileLaunch {
    int blocks = 0;
    size_t block_bytes = 0, workspace_bytes = 0;
};

struct TileArgs {
    const double* ops;
    const double* ftab;
    const double* colsum;
    int d, n_tiles;
    double prior_prec;
    double n_pad;  // zero rows appended to fill the last tiles
    unsigned ops_bytes;  // size of the operand stream
    int rem_rows;        // kZ0 kernels and residual form: real rows of the last tile if that tile is not full, else 0
    int z0_col;          // the constant column that is the accumulators' initial value (kZ0 kernels), and its value
    double z0_val;
};

// (the operand stream is read through a buffer descriptor with 32-bit offsets: 512 bytes per data row at most, so
// four million rows stay below 2 GiB)
inline bool tile_supports_shape(int64_t d, int64_t n) { return d >= 1 && d <= kTileMaxDim && n >= 1 && n <= 4000000; }
// (the wide kernel's stream takes up to 2 KB per row)
inline bool wide_supports_shape(int64_t d, int64_t n) { return d >= 1 && d <= kWideMaxDim && n >= 1 && n <= 1000000; }

// Operand stream: for every row tile t (16 rows), KS1 operands of 64 doubles for
// the first GEMM (padded to an even count) then 4*MT for the second; operand
// element l is what lane l feeds to the MFMA.  Operands are stored in pairs,
// element by element (pair p holds [2p][l], [2p+1][l] for l = 0..63), so that one
// 16-byte load per lane brings two of them.  Rows beyond n are zero, features
// beyond d are zero.
__host__ __device__ constexpr int tile_pairs_per_tile(int ks1, int mt) { return (ks1 + 1) / 2 + 2 * mt; }
inline void tile_pack_operands(const double* X, const double* y, int64_t n, int64_t d, bool residual, TileData* td,
                               std::vector<double>* out, std::vector<double>* colsum)
{
    td->residual = residual;
    colsum->assign(kWideMaxDim, 0.0);
    for (int64_t f = 0; f < d; ++f) {
        double acc = 0.0;
        for (int64_t r = 0; r < n; ++r) acc += y[r] != 0.0 ? X[r * d + f] : -X[r * d + f];
        (*colsum)[(size_t)f] = acc;
    }
    td->d = (int)d;
    td->ks1 = (int)((d + 3) / 4);
    td->mt = (int)((d + 15) / 16);
    td->z0_col = -1;
    td->z0_val = 0.0;
    if (!residual && d % 4 == 1 && d > 1) {  // one feature less is one k-step less
        for (int64_t f = 0; f < d && td->z0_col < 0; ++f) {
            bool same = X[f] != 0.0 && std::isfinite(X[f]);
            for (int64_t r = 1; r < n && same; ++r) same = X[r * d + f] == X[f];
            if (same) {
                td->z0_col = (int)f;
                td->z0_val = X[f];
                td->ks1 = (int)((d - 1) / 4);
            }
        }
    }
    const bool z0 = td->z0_col >= 0;
    const int64_t tiles = (n + kTileRows - 1) / kTileRows;
    // (the stream always holds a multiple of kTileWaves tiles: every wave asks for its first tile unconditionally)
    td->n_alloc_tiles = (int)((tiles + kTileWaves - 1) / kTileWaves * kTileWaves);
    // Rows of zeros have logit 0, which is harmless (a known constant in the log-likelihood, nothing in the gradient),
    // unless the accumulators start from the constant column's share: then only real tiles are run, and the rows that
    // fill the last one start from zero.  The residual form runs the real ones only, too, and leaves the rows beyond them out.
    td->n_tiles = z0 || residual ? (int)tiles : td->n_alloc_tiles;
    td->n_rows = (long)n;
    td->n_pad = (long)td->n_tiles * kTileRows - (long)n;
    const int pairs1 = (td->ks1 + 1) / 2;
    const int per_tile = 2 * tile_pairs_per_tile(td->ks1, td->mt);
    out->assign((size_t)td->n_alloc_tiles * per_tile * 64, 0.0);
    auto xs = [&](int64_t row, int64_t feat) -> double {
        if (row >= n || feat >= d) return 0.0;
        const double v = X[row * d + feat];
        return (z0 || y[row] != 0.0) ? v : -v;
    };
    // slot of the first GEMM's contraction -> feature: with a constant column c the last feature takes its slot
    // (the chains' lanes c and d - 1 write their positions to each other's place to match)
    auto feat1 = [&](int64_t slot) -> int64_t {
        if (!z0) return slot;
        if (slot >= d - 1) return d;  // (no feature: zero)
        return slot == td->z0_col ? d - 1 : slot;
    };
    for (int t = 0; t < td->n_alloc_tiles; ++t) {
        double* o = out->data() + (size_t)t * per_tile * 64;
        auto at = [&](int operand, int l) -> double& { return o[((operand >> 1) * 64 + l) * 2 + (operand & 1)]; };
        for (int s = 0; s < td->ks1; ++s)          // A[i][k] = X~[16t + i][4s + k], lane = i + 16k
            for (int l = 0; l < 64; ++l) at(s, l) = xs((int64_t)t * 16 + (l & 15), feat1(4 * s + (l >> 4)));
        for (int u = 0; u < td->mt; ++u)           // A[i][k] = X~[16t + 4s + k][16u + i]
            for (int s = 0; s < 4; ++s)
                for (int l = 0; l < 64; ++l)
                    at(2 * pairs1 + u * 4 + s, l) = xs((int64_t)t * 16 + 4 * s + (l >> 4), 16 * u + (l & 15));
    }
}

inline TileArgs tile_args(const TileData& td, double prior_prec)
{
    return TileArgs{td.base, td.ftab, td.colsum, td.d, td.n_tiles, prior_prec, (double)td.n_pad,
                    (unsigned)((size_t)td.n_alloc_tiles * 2 * tile_pairs_per_tile(td.ks1, td.mt) * 64 * sizeof(double)),
                    td.z0_col >= 0 || td.residual ? (int)(td.n_rows % kTileRows) : 0, td.z0_col, td.z0_val};
}

// Global-memory vectors of one chain slot, 32 doubles each (wide kernel: 32 elements per component of a lane):
//   proposal pool  2*b + c            b <= D,  c in {theta, grad}
//   first-leaf     2*(D+1) + 2*s + c  s <= D,  c in {theta, r}
__host__ __device__ inline int tile_num_vectors(int max_depth) { return 4 * (max_depth + 1); }

inline void tile_plan(const TileData&, long n_chains, int max_depth, TileLaunch* tl)
{
    long blocks = (n_chains + kTileChains - 1) / kTileChains;
    const long cap = 256L * 2;  // two resident workgroups per compute unit is the most that fits
    if (blocks > cap) blocks = cap;
    tl->blocks = (int)blocks;
    tl->block_bytes = (size_t)kTileChains * tile_num_vectors(max_depth) * kTileLanes * sizeof(double);
    tl->workspace_bytes = tl->block_bytes * (size_t)blocks;
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// ---- reductions over the 32 lanes of one chain ------------------------------
// Rotations inside each row of 16 lanes (DPP), then one exchange between the
// two rows (swizzle).  Every lane ends with the same bits: at each step the two
// partners add the same pair of values.
__device__ __forceinline__ double swap_rows(double x)  // lane ^ 16
{
    const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(x), 0x401F);
    const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(x), 0x401F);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double add_other_row(double x)  // x[lane] + x[lane ^ 16]
{
    const unsigned lo = (unsigned)__double2loint(x), hi = (unsigned)__double2hiint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}
__device__ __forceinline__ double add_other_half(double x)  // x[lane] + x[lane ^ 32]
{
    const unsigned lo = (unsigned)__double2loint(x), hi = (unsigned)__double2hiint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}
__device__ __forceinline__ double group_sum(double x)
{
    x += dpp_rotate<0x128>(x);  // row_ror:8
    x += dpp_rotate<0x124>(x);  // row_ror:4
    x += dpp_rotate<0x122>(x);  // row_ror:2
    x += dpp_rotate<0x121>(x);  // row_ror:1
    x += swap_rows(x);
    return x;
}
__device__ __forceinline__ void group_sum2(double& a, double& b)
{
    a += dpp_rotate<0x128>(a);
    b += dpp_rotate<0x128>(b);
    a += dpp_rotate<0x124>(a);
    b += dpp_rotate<0x124>(b);
    a += dpp_rotate<0x122>(a);
    b += dpp_rotate<0x122>(b);
    a += dpp_rotate<0x121>(a);
    b += dpp_rotate<0x121>(b);
    a += swap_rows(a);
    b += swap_rows(b);
}

// Two sums over the 32 lanes of one chain in one sweep, for where only their signs are wanted: the rows change halves
// first (row 0 takes a, row 1 takes b), then one set of rotations sums both.  Lanes 0..15 end with sum(a), lanes 16..31
// with sum(b).
__device__ __forceinline__ double group_sum_split(double a, double b, bool upper_row)
{
    const double keep = upper_row ? b : a, give = upper_row ? a : b;
    double x = keep + swap_rows(give);
    x += dpp_rotate<0x128>(x);
    x += dpp_rotate<0x124>(x);
    x += dpp_rotate<0x122>(x);
    x += dpp_rotate<0x121>(x);
    return x;
}
// ... and whether both are >= 0, the same answer in all 32 lanes (all of them must be running).
__device__ __forceinline__ bool group_both_nonnegative(double a, double b, int lane)
{
    const double x = group_sum_split(a, b, (lane & 16) != 0);
    const unsigned long long votes = __ballot(x >= 0.0);
    return (uint32_t)(votes >> (lane & 32)) == 0xffffffffu;
}

// Workgroup barrier that orders LDS traffic only.  The chains of a workgroup talk to each other through
// LDS alone (positions in, partial gradients out); what a lane has in flight to global memory - operands
// asked for ahead of the barrier, output samples, its own deep tree levels - nobody else in the workgroup
// reads, so the barrier need not wait for it as __syncthreads() would.
__device__ __forceinline__ void tile_lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace nuts
