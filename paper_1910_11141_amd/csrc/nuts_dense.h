// Register-resident kernel for a dense Gaussian of moderate dimension (d <= 128):
// configuration 2 of the benchmark, which is chain-poor (1024 chains) and so bound by
// the latency of one chain's step, not by throughput.
//
// One wavefront per chain slot, two components of every state vector per lane (the chain program is that of
// nuts_row.h).  The precision matrix is staged once per workgroup in LDS (row pitch 128, zero padded) and a gradient is
// one pass over it: the wave publishes its position in LDS, then every lane accumulates its two rows of P theta in
// ascending column order with one 16-byte matrix read and one broadcast read per column.
#pragma once
#include "nuts_row.h"

namespace nuts {

constexpr int kDenseMaxDim = 128;
constexpr int kDensePitch = 128;  // elements per workspace vector and per matrix row in LDS
constexpr int kDenseWaves = 4;    // waves (chain slots) per workgroup

// The gradient of one chain.  kBanded: the precision matrix has at most kBandHalf off-diagonals on each side (detected
// when the target is created); a lane then keeps the 2 x 9 coefficients of its two rows in registers and a gradient
// reads ten neighbouring components of the published position instead of a pass over the matrix.  Zero entries of a
// dense row add exact zeros, so the banded sum in ascending column order has the same value.
template <typename T, bool kBanded>
struct DenseGradient {
    typedef typename RowVec<T>::type Vec;
    const int lane, d;
    const T* const mat;  // LDS: mat[k * kDensePitch + i] = P[i][k]
    T* const bcast;      // LDS: this wave's position, for the other lanes
    T band0[2 * kBandHalf + 1], band1[2 * kBandHalf + 1];  // banded: coefficients of rows 2*lane and 2*lane+1

    __device__ DenseGradient(const DevTarget<T>& tg, int lane_, const T* mat_, T* bcast_)
        : lane(lane_), d(tg.d), mat(mat_), bcast(bcast_)
    {
        if (kBanded) {
#pragma unroll
            for (int k = 0; k < 2 * kBandHalf + 1; ++k) {
                band0[k] = tg.band[(size_t)(2 * lane) * (2 * kBandHalf + 1) + k];
                band1[k] = tg.band[(size_t)(2 * lane + 1) * (2 * kBandHalf + 1) + k];
            }
        }
    }

    // g = -P theta; returns the partial sum of theta_i g_i of this lane (logp is half the wave's total).  Columns are
    // taken in ascending order with a binary64 accumulator.
    __device__ __forceinline__ double operator()(const T (&th)[2], T (&g)[2]) const
    {
        *reinterpret_cast<Vec*>(bcast + 2 * lane) = Vec{th[0], th[1]};
        __builtin_amdgcn_wave_barrier();
        double acc0 = 0.0, acc1 = 0.0;
        if (kBanded) {
            // components 2*lane - 4 .. 2*lane + 5 (the buffer has kBandHalf zeros on either side)
            T x[2 * kBandHalf + 2];
#pragma unroll
            for (int u = 0; u < kBandHalf + 1; ++u) {
                const Vec p = *reinterpret_cast<const Vec*>(bcast + 2 * lane - kBandHalf + 2 * u);
                x[2 * u] = p.x;
                x[2 * u + 1] = p.y;
            }
#pragma unroll
            for (int k = 0; k < 2 * kBandHalf + 1; ++k) {
                acc0 = fma((double)band0[k], (double)x[k], acc0);
                acc1 = fma((double)band1[k], (double)x[k + 1], acc1);
            }
            __builtin_amdgcn_wave_barrier();
            g[0] = (T)(-acc0);
            g[1] = (T)(-acc1);
            return fma((double)th[0], -acc0, (double)th[1] * -acc1);
        }
        const T* row = mat + 2 * lane;
        // columns in batches of 20 so that the LDS reads of a batch are all in flight together
        constexpr int kBatch = 20;
        int k = 0;
        for (; k + kBatch <= d; k += kBatch) {
            Vec p[kBatch];
            T t[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                p[u] = *reinterpret_cast<const Vec*>(row + (size_t)(k + u) * kDensePitch);
                t[u] = bcast[k + u];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                acc0 = fma((double)p[u].x, (double)t[u], acc0);
                acc1 = fma((double)p[u].y, (double)t[u], acc1);
            }
        }
        for (; k < d; ++k) {
            const Vec p = *reinterpret_cast<const Vec*>(row + (size_t)k * kDensePitch);
            const double t = (double)bcast[k];
            acc0 = fma((double)p.x, t, acc0);
            acc1 = fma((double)p.y, t, acc1);
        }
        __builtin_amdgcn_wave_barrier();
        g[0] = (T)(-acc0);
        g[1] = (T)(-acc1);
        return fma((double)th[0], -acc0, (double)th[1] * -acc1);
    }
};

// LDS of a workgroup ahead of its slots' tree storage: the matrix, and per wave kBandHalf zeros, the position,
// kBandHalf zeros.
constexpr int kDenseBcast = kDensePitch + 2 * kBandHalf;
__host__ __device__ inline size_t dense_base_elems(int mat_rows)
{
    return (size_t)mat_rows * kDensePitch + (size_t)kDenseWaves * kDenseBcast;
}

// kTurns: as in nuts_elem.h.
template <typename T, bool kBanded, bool kTurns>
__global__ __launch_bounds__(kDenseWaves* kWave, sizeof(T) == 8 && !kBanded ? 1 : 2) void nuts_dense_kernel(DevTarget<T> tg, DevSample sa, RowLds rl, unsigned* turns)
{
    extern __shared__ __align__(16) unsigned char smem[];
    T* mat = reinterpret_cast<T*>(smem);  // dense: d rows of kDensePitch; banded: nothing
    const int mat_rows = kBanded ? 0 : tg.d;
    const int lane = threadIdx.x & (kWave - 1), wave = uni((int)(threadIdx.x / kWave));
    T* bcast = mat + (size_t)mat_rows * kDensePitch + (size_t)wave * kDenseBcast + kBandHalf;
    for (int i = threadIdx.x; i < mat_rows * kDensePitch; i += blockDim.x) {
        const int k = i / kDensePitch, c = i % kDensePitch;
        mat[i] = c < tg.d ? tg.PT[(size_t)k * tg.d + c] : T(0);
    }
    for (int i = threadIdx.x; i < kDenseWaves * kDenseBcast; i += blockDim.x) mat[(size_t)mat_rows * kDensePitch + i] = T(0);
    __syncthreads();
    const size_t slot = (size_t)blockIdx.x * kDenseWaves + wave;
    T* tree = mat + dense_base_elems(mat_rows) + (size_t)wave * (rl.n_first + rl.n_pool) * 2 * kDensePitch;
    RowChain<T, 1, true, true, false, kTurns> ch(sa, tg.d, lane, reinterpret_cast<T*>(sa.workspace + slot * sa.slot_bytes), tree, rl, turns);
    const DenseGradient<T, kBanded> grad(tg, lane, mat, bcast);
    while (const int taken = ch.take()) {
        if (taken == kTakeFresh) ch.start_chain(grad(ch.th, ch.g));
        do {
            ch.iter_begin();
            do {
                ch.double_begin();
                double lp;
                do {
                    for (int step = 0;;) {
                        ch.kick_drift();
                        lp = grad(ch.th, ch.g);
                        ch.kick();
                        if (++step >= sa.leaf_steps) break;
                    }
                } while (ch.finish_leaf(lp));
            } while (ch.double_end());
        } while (ch.iter_end());
    }
    if (lane == 0) {
        // issued slots are charged by the host as slots x (largest count of one slot): see the wave kernel
        atomicMax(&sa.counters[kCtrSlotMax], ch.n_leaf + ch.n_extra);
        atomicAdd(&sa.counters[kCtrUseful], ch.n_leaf);
        atomicAdd(&sa.counters[kCtrExtra], ch.n_extra);
        atomicAdd(&sa.counters[kCtrRounds], ch.n_leaf + ch.n_extra);
    }
}

}  // namespace nuts
