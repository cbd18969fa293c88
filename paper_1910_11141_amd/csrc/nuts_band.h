// Banded Gaussian targets of more than 128 dimensions: at most kBandHalf off-diagonals on each side (detected when the
// target is created).  One wavefront per chain slot and the chain program of nuts_row.h; for a gradient the wave publishes
// its position in LDS and every lane takes the ten components around each of its pairs, in ascending column order with
// binary64 accumulators.  Diagonals that hold only zeros (correlation matrices of autoregressions have few others) are
// left out: they add exact zeros.  The coefficients come from L1/L2, diagonal by diagonal.
//
// What bounds it: the latency of the chain program (few chains), or the vector instructions of gradient, leaf and merge.
// Against nine entries of a row in the general wave kernel, which keeps every vector in memory: two iterations, AR(1), binary64: d = 129, 4
// chains 0.50 -> 0.14 ms; d = 1000, 1024 chains 3.3 -> 0.68 ms; d = 2000, 4096 chains 21.4 -> 14.1 ms.  Beyond 512 dimensions in
// binary64 and 1024 in binary32 the state hardly fits the registers: with constants and addresses hoisted out of the loops scratch
// memory per lane was 476 bytes at kC = 8 and 2928 at 16 in binary64, 1640 at 16 in binary32; without (nuts_gauss.hip) it is 812 at
// 16 in binary64, else none (but 40 at 4 in binary32, for two workgroups per compute unit): d = 2000, binary64, 4096 chains, six
// iterations 226 -> 118 ms, 64 chains 29.3 -> 18.8; binary32, 2048 chains 73 -> 25; d = 1000, binary64, 1024 chains 7.66 -> 6.70.
// Same outputs, bit for bit.
#pragma once
#include "nuts_row.h"

namespace nuts {

constexpr int kBandMaxDim = 2048;

template <typename T, int kC>
constexpr int band_lane_bytes() { return 2 * kC * (int)sizeof(T); }  // registers of a lane for one vector
// LDS ahead of the slots' tree storage: per wave kBandHalf zeros, the position, kBandHalf zeros.
__host__ __device__ constexpr int band_bcast(int kc) { return 128 * kc + 2 * kBandHalf; }

// diag: [2 kBandHalf + 1][128 kC], element (k, i) = P[i][i + k - kBandHalf]; bit k of `present`: diagonal k is not all zero
template <typename T, int kC>
__global__ __launch_bounds__(256, (band_lane_bytes<T, kC>() <= 32 ? 2 : 1)) void nuts_band_kernel(DevTarget<T> tg, const T* diag, int present,
                                                                                       DevSample sa, RowLds rl)
{
    typedef typename RowVec<T>::type Vec;
    constexpr int kN = 2 * kBandHalf + 1;
    extern __shared__ __align__(16) unsigned char band_smem[];
    T* const base = reinterpret_cast<T*>(band_smem);
    const int lane = threadIdx.x & (kWave - 1), wave = uni((int)(threadIdx.x / kWave));
    for (int i = threadIdx.x; i < 4 * band_bcast(kC); i += 256) base[i] = T(0);
    __syncthreads();
    T* const bcast = base + (size_t)wave * band_bcast(kC) + kBandHalf;
    T* const tree = base + 4 * (size_t)band_bcast(kC) + (size_t)wave * (rl.n_first + rl.n_pool) * 2 * 128 * kC;
    const size_t slot = (size_t)blockIdx.x * 4 + wave;
    RowChain<T, kC, (band_lane_bytes<T, kC>() <= 16), true> ch(sa, tg.d, lane, reinterpret_cast<T*>(sa.workspace + slot * sa.slot_bytes),
                                                               tree, rl);
    // g = -P theta; returns this lane's share of theta . g
    auto grad = [&]() __attribute__((always_inline)) -> double {
#pragma unroll
        for (int q = 0; q < kC; ++q) *reinterpret_cast<Vec*>(bcast + ch.elem(q, 0)) = Vec{ch.th[2 * q], ch.th[2 * q + 1]};
        __builtin_amdgcn_wave_barrier();
        double lp = 0.0;
#pragma unroll
        for (int q = 0; q < kC; ++q) {
            T x[kN + 1];
#pragma unroll
            for (int u = 0; u < kBandHalf + 1; ++u) {
                const Vec p = *reinterpret_cast<const Vec*>(bcast + ch.elem(q, 0) - kBandHalf + 2 * u);
                x[2 * u] = p.x;
                x[2 * u + 1] = p.y;
            }
            double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
            for (int k = 0; k < kN; ++k)
                if ((present >> k) & 1) {
                    const Vec c = *reinterpret_cast<const Vec*>(diag + (size_t)k * (128 * kC) + ch.elem(q, 0));
                    acc0 = fma((double)c.x, (double)x[k], acc0);
                    acc1 = fma((double)c.y, (double)x[k + 1], acc1);
                }
            ch.g[2 * q] = (T)(-acc0);
            ch.g[2 * q + 1] = (T)(-acc1);
            lp = fma((double)ch.th[2 * q], -acc0, lp);
            lp = fma((double)ch.th[2 * q + 1], -acc1, lp);
        }
        __builtin_amdgcn_wave_barrier();
        return lp;
    };
    while (ch.fetch()) {
        ch.start_chain(grad());
        do {
            ch.iter_begin();
            do {
                ch.double_begin();
                double lp;
                do {
                    for (int step = 0;;) {
                        ch.kick_drift();
                        lp = grad();
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

// Instances with the compiler flags of nuts_gauss.hip: those whose state does not fit the registers beside hoisted constants.  The
// others are 3 to 6 % faster without (kC = 4 in binary64 only up to four chains per compute unit: beyond, the flags would give it
// a second wave per SIMD and 1.4 to 1.5 times the speed).
#define NUTS_BAND_INSTANCE(T, kC) template __global__ void nuts_band_kernel<T, kC>(DevTarget<T>, const T*, int, DevSample, RowLds);
#define NUTS_BAND_INSTANCES(pre) pre NUTS_BAND_INSTANCE(float, 16) pre NUTS_BAND_INSTANCE(double, 8) pre NUTS_BAND_INSTANCE(double, 16)
NUTS_BAND_INSTANCES(extern)

}  // namespace nuts
