// Register-resident kernel for element-wise targets (standard normal, diagonal Gaussian).
//
// One wavefront per chain slot and the chain program of nuts_row.h.  The end of the trajectory that is being extended -
// position and momentum - stays in registers, and the gradient -theta_i / sigma_i^2 is recomputed from the position
// instead of being stored: a leapfrog step moves no memory at all.  What is left is the tree's own traffic: the first leaf
// of a subtree of four or more leaves is written once and read by the merges it takes part in, from LDS as far as that
// reaches; the proposal of such a subtree is written once if it is a left half; a change of direction swaps the register
// end with the other one (in registers too while a vector takes up to 32 bytes of a lane, else in memory).
//
// What bounds it: with few chains or dimensions the latency of the chain program, with many the vector instructions of
// leaf and merge (the energies, kinetic terms and U-turn sums are binary64 sums of the elements): d = 1000 in binary32 459
// vector instructions a step, one every 4.5 cycles of a SIMD, 3.4 KB of HBM traffic a step.  Scratch memory per lane: 124 bytes
// at 16 in binary64 (644 with constants hoisted out of the loops; d = 2000, 8192 chains, six iterations 12.5 -> 7.5 ms, 256 chains
// 1.13 -> 0.78), none elsewhere.
// Against the kernel before it (weights as logarithms through a table, 53 KB of LDS for that table, the random numbers
// of a doubling drawn one by one, first leaves and both ends in memory), the same outputs bit for bit: d = 2 binary64, 4
// chains, 100 iterations 1170 -> 670 us; d = 500 binary32 standard normal, 16384 chains, 20 iterations 10.0 -> 4.3 ms; d = 1000 binary32
// diagonal, 16384 chains, 8 iterations 95 -> 52 ms (now 42.9: sums in one pass, chains that take turns, nuts_row.h).
#pragma once
#include "nuts_row.h"

namespace nuts {

// Registers of a lane for one vector.
template <typename T, int kC>
constexpr int elem_lane_bytes() { return 2 * kC * (int)sizeof(T); }

// Workgroups are four waves; LDS: 1 / sigma^2 (unless it is held in registers), then the slots' tree storage.
// kTurns: the call's last chains take turns.  An instance of its own: with the code for turns a step takes 1.02 to 1.03 times
// as long where its latency counts (d = 2 and 100, one wave per SIMD or less).
template <typename T, int kC, bool kTurns>
__global__ __launch_bounds__(256, (elem_lane_bytes<T, kC>() <= 64 ? 2 : 1)) void nuts_elem_kernel(DevTarget<T> tg, DevSample sa, RowLds rl, unsigned* turns)
{
    typedef typename RowVec<T>::type Vec;
    constexpr int kVpl = 2 * kC;
    constexpr bool kHeld = elem_lane_bytes<T, kC>() <= 32;
    extern __shared__ __align__(16) unsigned char elem_smem[];
    T* const s_w = reinterpret_cast<T*>(elem_smem);
    const int lane = threadIdx.x & (kWave - 1), wave = uni((int)(threadIdx.x / kWave));
    const size_t slot = (size_t)blockIdx.x * 4 + wave;
    T* const tree = s_w + (kHeld ? 0 : 128 * kC) + (size_t)wave * (rl.n_first + rl.n_pool) * 2 * 128 * kC;
    RowChain<T, kC, kHeld, false, false, kTurns> ch(sa, tg.d, lane, reinterpret_cast<T*>(sa.workspace + slot * sa.slot_bytes), tree, rl, turns);
    // 1 / sigma^2, zero beyond d
    auto weight = [&](int i) -> T { return i < tg.d ? (tg.kind == kGaussDiag ? tg.inv_var[i] : T(1)) : T(0); };
    T w_reg[kHeld ? kVpl : 1];
    if constexpr (kHeld) {
#pragma unroll
        for (int i = 0; i < kVpl; ++i) w_reg[i] = weight(ch.elem(i / 2, i & 1));
    } else {
        for (int i = threadIdx.x; i < 128 * kC; i += 256) s_w[i] = weight(i);
        __syncthreads();
    }
    auto pair_weight = [&](int q, T (&w)[2]) __attribute__((always_inline)) {
        if constexpr (kHeld) {
            w[0] = w_reg[kHeld ? 2 * q : 0];
            w[1] = w_reg[kHeld ? 2 * q + 1 : 0];
        } else {
            const Vec x = *reinterpret_cast<const Vec*>(s_w + ch.elem(q, 0));
            w[0] = x.x;
            w[1] = x.y;
        }
    };
    // one leapfrog step; returns this lane's share of theta . gradient
    auto leapfrog = [&]() __attribute__((always_inline)) -> double {
        const T half = (T)(0.5 * (ch.v * sa.eps)), full = (T)(ch.v * sa.eps);
        double lp = 0.0;
#pragma unroll
        for (int q = 0; q < kC; ++q) {
            T w[2];
            pair_weight(q, w);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int i = 2 * q + e;
                const T g0 = -(ch.th[i] * w[e]);
                const T rh = ch.r[i] + half * g0;
                const T tn = ch.th[i] + full * rh;
                const T g1 = -(tn * w[e]);
                ch.th[i] = tn;
                ch.r[i] = rh + half * g1;
                lp = fma((double)tn, (double)g1, lp);
            }
        }
        return lp;
    };
    while (const int taken = ch.take()) {
        double lp = 0.0;
        if (taken == kTakeFresh) {
#pragma unroll
            for (int q = 0; q < kC; ++q) {
                T w[2];
                pair_weight(q, w);
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const T g = -(ch.th[2 * q + e] * w[e]);
                    lp = fma((double)ch.th[2 * q + e], (double)g, lp);
                }
            }
            ch.start_chain(lp);
        }
        do {
            ch.iter_begin();
            do {
                ch.double_begin();
                do {
                    for (int step = 0;;) {
                        lp = leapfrog();
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

// The instance with the compiler flags of nuts_gauss.hip; with them d = 1000 takes 1.03 (binary32) to 1.06 times as long.
#define NUTS_ELEM_INSTANCE(T, kC, kTurns) template __global__ void nuts_elem_kernel<T, kC, kTurns>(DevTarget<T>, DevSample, RowLds, unsigned*);
extern NUTS_ELEM_INSTANCE(double, 16, false)

}  // namespace nuts
