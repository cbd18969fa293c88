// Block kernel: dense Gaussian targets with 128 < d <= 512, NC = 8 or 4 chains per workgroup in lock step, their
// precision-matrix products together on the binary64 matrix cores.
//
// One wavefront per chain (the chain program is that of nuts_row.h), one workgroup per compute unit.  A round: every
// chain runs to the next point that needs a gradient and publishes its position in LDS; the workgroup's eight waves
// share out the product G = P Theta (d x d times d x NC) on v_mfma_f64_4x4x4_4b, four groups of 4 rows of P against the
// same 4 chains; every chain takes its column back and goes on.  The matrix no longer fits in LDS (d = 250: 0.5 MB): it
// is streamed from L2 in operand order, once per round for all chains of the workgroup, where the general wave kernel
// reads it once per chain and step.  A wave owns one quarter of the contraction for every second row group of 16, up to
// four row groups at a time (one read of the positions for four operands), and the quarters are summed in one order.
//
// What bounds it: the operand stream, which a compute unit takes from L2 at about 45 bytes per tick (d = 256: 0.5 MB in
// 11.5 k ticks, of which the instructions of 4 chains need 4.1 k, of 8 chains 8.2 k), then the chain program (5 k ticks).
// A form with 16 chains and v_mfma_f64_16x16x4 was matrix-bound at 21 k ticks, and its 16 waves left 128 registers to
// the chain program, which then took 45 k.  (Scratch memory per lane: 36 bytes at kC = 4 in binary64, else none; with
// constants hoisted out of the loops 56, 212 and 428 at kC = 2, 3, 4 and d = 384, 2048 chains, four iterations 2.34 -> 2.75 ms.)  Binary32 targets keep binary64 sums of binary32 values, as in the wave kernel.
// d = 250, binary64, 300 chains, every iteration awaited, 10 iterations: 34.3 ms (wave kernel) -> 2.5 ms.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <vector>

#include "nuts_row.h"
#include "nuts_tile_common.h"

namespace nuts {

constexpr int kBlockMaxDim = 512;
constexpr int kBlockMaxDim8 = 384;  // of the form with 8 chains: positions and partial gradients of all chains in LDS

struct BlockData {
    double* ops = nullptr;  // device: P in MFMA operand order, see block_pack_operands
    int d = 0, n_r = 0, pq = 0;
};

struct BlockArgs {
    const double* ops;
    unsigned ops_bytes;
    int d, n_r, pq;
};

// Operand stream of P (d x d): row group R (rows 16R .. 16R + 15), column-block pair p (columns 8p .. 8p + 7), 128
// doubles: element [l][e] is P[16R + l % 16][8p + 4e + l / 16], zero beyond d.  4 pq pairs per row group, pq per quarter.
// The kernel asks for operands up to three pairs ahead, also at the end: four pairs of zeros follow.
constexpr int kBlockAheadPairs = 4;
inline size_t block_stream_doubles(int n_r, int pq) { return ((size_t)n_r * 4 * pq + kBlockAheadPairs) * 128; }
template <typename T>
inline void block_pack_operands(const T* P, int64_t d, BlockData* bd, std::vector<double>* out)
{
    bd->d = (int)d;
    bd->n_r = (int)((d + 15) / 16);
    bd->pq = (int)((d + 31) / 32);
    out->assign(block_stream_doubles(bd->n_r, bd->pq), 0.0);
    for (int64_t row = 0; row < d; ++row)
        for (int64_t col = 0; col < d; ++col) {
            const int64_t R = row / 16, p = col / 8, e = (col / 4) & 1, l = (row & 15) + 16 * (col & 3);
            (*out)[((size_t)(R * 4 * bd->pq + p) * 64 + l) * 2 + e] = (double)P[row * d + col];
        }
}

constexpr int kBlockWaves = 8;
constexpr int kBlockThreads = kBlockWaves * kWave;
constexpr int kBlockQuarters = 4;
// doubles per chain in the LDS tiles: every column of the (padded) matrix; odd: see nuts_tile.h
__host__ __device__ inline int block_pitch(int pq) { return 32 * pq + 1; }
inline size_t block_base_bytes(int nc, int pq)
{
    return (((size_t)nc * (1 + kBlockQuarters) * block_pitch(pq) * sizeof(double)) + 15) & ~(size_t)15;
}

template <typename T, int kC, int NC>
__global__ __launch_bounds__(kBlockThreads) void nuts_block_kernel(BlockArgs ba, DevSample sa, RowLds rl, int tree_off)
{
    constexpr int kSets = NC / 4;  // groups of 4 chains = columns of one matrix instruction
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int sHalted;
    double* const sTheta = reinterpret_cast<double*>(smem);  // [chain][pitch]
    const int pitch = block_pitch(ba.pq);
    double* const sG = sTheta + (size_t)NC * pitch;           // [quarter][chain][pitch]
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uni(tid >> 6);
    const bool owns = wave < NC;  // 4 chains: waves 4..7 only help with the products
    const int grp = wave & (NC - 1);
    for (int i = tid; i < NC * pitch; i += kBlockThreads) sTheta[i] = 0.0;
    if (tid == 0) sHalted = 0;
    __syncthreads();
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(ba.ops), 0, (int)ba.ops_bytes, 0x00020000);
    auto load_at = [&](int byte_off) __attribute__((always_inline)) -> double2 {
        return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, byte_off, 0));
    };
    T* const tree = reinterpret_cast<T*>(smem + tree_off) + (size_t)grp * (rl.n_first + rl.n_pool) * 2 * 128 * kC;
    const size_t slot = (size_t)blockIdx.x * NC + grp;
    RowChain<T, kC, (kC <= 2), true> ch(sa, ba.d, lane, reinterpret_cast<T*>(sa.workspace + slot * sa.slot_bytes), tree, rl);

    enum { kInit, kLeaf, kDone };
    int state = kDone, sub = 0;
    unsigned long long n_rounds = 0;
    long long cyc_control = 0, cyc_grad = 0;
    double lp = 0.0;
    const int row_bytes = 4 * ba.pq * 1024, n_pairs = ba.pq;
    const int blk_n = lane & 3, kq = lane >> 4;
    // first: the wave has not asked for a chain yet
    bool first = true;
    for (;;) {
        const long long t0 = clock64();
        // ---- 1. every chain runs to the next point that needs a gradient ----
        if (owns && (first || state != kDone)) {
            bool fetch_next = first;
            if (state == kInit) {
                ch.start_chain(lp);
                ch.iter_begin();
                ch.double_begin();
                state = kLeaf;
            } else if (state == kLeaf) {
                ch.kick();
                if (++sub >= sa.leaf_steps) {
                    sub = 0;
                    if (!ch.finish_leaf(lp)) {
                        bool begin = true;
                        if (!ch.double_end()) {
                            if (ch.iter_end()) {
                                ch.iter_begin();
                            } else {
                                begin = false;
                                fetch_next = true;
                            }
                        }
                        if (begin) ch.double_begin();
                    }
                }
            }
            if (fetch_next) {
                state = ch.fetch() ? kInit : kDone;
                if (state == kDone && lane == 0) atomicAdd(&sHalted, 1);
            }
            if (state == kLeaf) ch.kick_drift();
#pragma unroll
            for (int q = 0; q < kC; ++q)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    if (ch.elem(q, e) < pitch - 1)
                        sTheta[grp * pitch + ch.elem(q, e)] = state == kDone ? 0.0 : (double)ch.th[2 * q + e];
        }
        first = false;
        tile_lds_barrier();
        if (*const_cast<volatile int*>(&sHalted) == NC) break;  // every chain of the workgroup has halted
        n_rounds += 1;
        const long long t1 = clock64();

        // ---- 2. G = P Theta ----
        {
            const int quarter = wave & 3;
            const double* const b = sTheta + blk_n * pitch + kq + 8 * quarter * n_pairs;
            double* const g_dst = sG + (size_t)(quarter * NC + blk_n) * pitch + 4 * ((lane >> 2) & 3) + kq;
            // kR row groups R0, R0 + 2, ... at once; operands two pairs of column blocks ahead
            auto rows = [&](auto count, int R0) __attribute__((always_inline)) {
                constexpr int kR = decltype(count)::value;
                int off = R0 * row_bytes + quarter * n_pairs * 1024;
                double acc[kSets][kR];
                double2 a0[kR], a1[kR];
#pragma unroll
                for (int i = 0; i < kR; ++i) {
#pragma unroll
                    for (int c = 0; c < kSets; ++c) acc[c][i] = 0.0;
                    a0[i] = load_at(off + 2 * i * row_bytes);
                    a1[i] = load_at(off + 2 * i * row_bytes + 1024);
                }
                auto pair = [&](const double2 (&a)[kR], const double* bp) __attribute__((always_inline)) {
#pragma unroll
                    for (int c = 0; c < kSets; ++c) {
                        const double b0 = bp[4 * c * pitch], b1 = bp[4 * c * pitch + 4];
#pragma unroll
                        for (int i = 0; i < kR; ++i) acc[c][i] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[i].x, b0, acc[c][i], 0, 0, 0);
#pragma unroll
                        for (int i = 0; i < kR; ++i) acc[c][i] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[i].y, b1, acc[c][i], 0, 0, 0);
                    }
                };
                for (int p = 0; p < n_pairs; p += 2) {
                    pair(a0, b + 8 * p);
                    off += 2048;
#pragma unroll
                    for (int i = 0; i < kR; ++i) a0[i] = load_at(off + 2 * i * row_bytes);
                    if (p + 1 < n_pairs) pair(a1, b + 8 * p + 8);  // (else it is the next quarter's)
#pragma unroll
                    for (int i = 0; i < kR; ++i) a1[i] = load_at(off + 2 * i * row_bytes + 1024);
                }
#pragma unroll
                for (int c = 0; c < kSets; ++c)
#pragma unroll
                    for (int i = 0; i < kR; ++i) g_dst[4 * c * pitch + 16 * (R0 + 2 * i)] = acc[c][i];
            };
            int R = wave >> 2;
            for (; R + 6 < ba.n_r; R += 8) rows(std::integral_constant<int, 4>{}, R);
            if (R + 4 < ba.n_r) rows(std::integral_constant<int, 3>{}, R);
            else if (R + 2 < ba.n_r) rows(std::integral_constant<int, 2>{}, R);
            else if (R < ba.n_r) rows(std::integral_constant<int, 1>{}, R);
        }
        tile_lds_barrier();
        cyc_control += t1 - t0;
        cyc_grad += clock64() - t1;

        // ---- 3. every chain collects its gradient ----
        if (owns && state != kDone) {
            lp = 0.0;
#pragma unroll
            for (int q = 0; q < kC; ++q)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = ch.elem(q, e);
                    double sum = 0.0;
                    if (i < ba.d) {
                        const double* s = sG + (size_t)grp * pitch + i;
                        const size_t step = (size_t)NC * pitch;
                        sum = (s[0] + s[step]) + (s[2 * step] + s[3 * step]);
                    }
                    ch.g[2 * q + e] = (T)(-sum);
                    lp = fma((double)ch.th[2 * q + e], -sum, lp);
                }
        }
    }

    if (owns && lane == 0) {
        atomicAdd(&sa.counters[kCtrUseful], ch.n_leaf);
        atomicAdd(&sa.counters[kCtrExtra], ch.n_extra);
    }
    if (tid == 0) {
        atomicAdd(&sa.counters[kCtrIssued], n_rounds * NC);
        atomicAdd(&sa.counters[kCtrRounds], n_rounds);
        atomicAdd(&sa.counters[kCtrCycControl], (unsigned long long)cyc_control);
        atomicAdd(&sa.counters[kCtrCycGrad], (unsigned long long)cyc_grad);
    }
}

// Chains per workgroup of a run on a chip of `cus` compute units (one workgroup each).  A round of 8 chains takes 1.25 times
// as long as one of 4, so beyond 4 chains per compute unit, where the small form needs a second round, the large one wins.
inline int block_chains_per_group(int d, long n_chains, int cus) { return n_chains <= 4L * cus || d > kBlockMaxDim8 ? 4 : 8; }
inline int block_chunks(int d) { return d <= 256 ? 2 : (d <= 384 ? 3 : 4); }

// Launch shape of a run.
struct BlockPlan {
    int nc, blocks;
    size_t lds_bytes, slot_bytes;
    int tree_off;
    RowLds rl;
};

inline void block_plan(const BlockData& bd, size_t elem, long n_chains, int cus, int max_depth, int nc, BlockPlan* bp)
{
    const int kc = block_chunks(bd.d);
    bp->nc = nc;
    long blocks = (n_chains + nc - 1) / nc;
    if (blocks > cus) blocks = cus;  // one workgroup per compute unit; further chains wait in the queue
    bp->blocks = (int)blocks;
    const size_t base = block_base_bytes(nc, bd.pq), room = 158 * 1024 - base;  // (2 KB for the static variables)
    bp->rl = row_lds_split(room / nc, kc, elem, max_depth, true);
    bp->tree_off = (int)base;
    bp->lds_bytes = base + (size_t)nc * (bp->rl.n_first + bp->rl.n_pool) * row_entry_bytes(kc, elem);
    bp->slot_bytes = ((size_t)row_num_vectors(max_depth) * 128 * kc * elem + 255) & ~(size_t)255;
}

template <typename T, int kC, int NC>
inline hipError_t block_launch_inst(const BlockArgs& ba, const DevSample& sa, const BlockPlan& bp, hipStream_t stream)
{
    const void* fn = reinterpret_cast<const void*>(nuts_block_kernel<T, kC, NC>);
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bp.lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((nuts_block_kernel<T, kC, NC>), dim3((unsigned)bp.blocks), dim3(kBlockThreads), bp.lds_bytes, stream,
                       ba, sa, bp.rl, bp.tree_off);
    return hipGetLastError();
}
template <typename T>
hipError_t block_launch(const BlockData& bd, const DevSample& sa, const BlockPlan& bp, hipStream_t stream)
{
    const BlockArgs ba{bd.ops, (unsigned)(block_stream_doubles(bd.n_r, bd.pq) * sizeof(double)), bd.d, bd.n_r, bd.pq};
    switch (block_chunks(bd.d)) {
    case 2: return bp.nc == 8 ? block_launch_inst<T, 2, 8>(ba, sa, bp, stream) : block_launch_inst<T, 2, 4>(ba, sa, bp, stream);
    case 3: return bp.nc == 8 ? block_launch_inst<T, 3, 8>(ba, sa, bp, stream) : block_launch_inst<T, 3, 4>(ba, sa, bp, stream);
    default: return block_launch_inst<T, 4, 4>(ba, sa, bp, stream);
    }
}
extern template hipError_t block_launch<float>(const BlockData&, const DevSample&, const BlockPlan&, hipStream_t);  // nuts_gauss.hip
extern template hipError_t block_launch<double>(const BlockData&, const DevSample&, const BlockPlan&, hipStream_t);

}  // namespace nuts
