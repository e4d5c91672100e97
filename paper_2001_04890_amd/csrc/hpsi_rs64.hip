// Register-streamed FP64 sector GEMMs of Eq. dgemm (Section 2.2.1) for gfx950, on
// v_mfma_f64_16x16x4f64 with FP64 accumulation.
//
// One wavefront owns one 16-row tile of a target psi block of at most 128 columns and runs over a range
// of its tasks Y += f * A . X . B^T; there is no LDS and no barrier. A task is cut into steps, one per
// 16-wide column tile jc of the source, and per step:
//   GEMM1  T'(rt, jc)^T = X^T(jc, :) . A(rt, :)^T   A's row tile stays in registers for the task
//   GEMM2  Y(rt, :)   += f T'(rt, jc) . B(:, jc)^T  GEMM1's result layout is GEMM2's A-operand layout
// The X^T and B tiles stream from the caches into register rings that are refilled as soon as a tile has
// been used, up to a whole GEMM ahead of their next use (every load is unconditional: a tile outside
// the block re-reads its first one, so that the compiler knows how many loads are in flight and never
// waits for the newest). MFMAs run only on the 4-wide k steps that hold data.
//
// Why: an FP64 16x16x4 MFMA takes 64 cycles, so one wavefront needs 2 KB per 256 cycles, half of what a
// CU's vector cache delivers to four of them; what small sectors lack is work in flight. A workgroup of
// seven wavefronts per target that steps behind barriers (hpsi_lds64.hip) leaves six of them idle on a
// target of up to 16 rows.
//
// Tile format (internal.h, hpsi_big64.hip): a 16 x 16 tile holds M[16 rt + li][16 kt + 4 v + g] in
// lane (li, g) = (l % 16, l / 16), value v.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace dmrg {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kTileD = 256;   // doubles per 16 x 16 tile

// 32 bytes per lane at a wave-uniform address
__device__ __forceinline__ f64x4 ld4(const double* p, uint32_t lane_bytes) {
    return *reinterpret_cast<const f64x4*>(reinterpret_cast<const char*>(p) + lane_bytes);
}
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double unid(double v) {
    return __builtin_bit_cast(double, uni64(__builtin_bit_cast(int64_t, v)));
}

// Task descriptor in scalar registers (offsets in doubles; pa16 / pd16: tile strides of the source's
// rows / columns; ka4 / kd4: the 4-wide k steps of them that hold data).
struct TD { int64_t x, a, b; double f; int pa16, pd16, ka4, kd4; };
__device__ __forceinline__ TD load_td(const LTask64* __restrict__ p) {
    TD d;
    d.x = uni64(p->x_off);
    d.a = uni64(p->a_off);
    d.b = uni64(p->b_off);
    d.f = unid(p->f);
    d.pa16 = uni(p->pa16);
    d.pd16 = uni(p->pd16);
    d.ka4 = uni(p->ka4);
    d.kd4 = uni(p->kd4);
    return d;
}

// keeps the loads before it from sinking to their uses and those after it from rising
__device__ __forceinline__ void fence() { asm volatile("" ::: "memory"); }

template <int KT, int QT>
__device__ __forceinline__ void rs_item(const Item* __restrict__ ip, const LTask64* __restrict__ tasks,
                                        const double* __restrict__ pool_t, const double* __restrict__ xt,
                                        double* __restrict__ y, double* __restrict__ part, int lane) {
    constexpr int RX = KT == 8 ? 4 : KT, RB = QT == 8 ? 4 : QT;   // ring sizes (divisors of KT, QT)
    const int rt = uni(ip->r0) >> 4, m_dp = uni(ip->m_dp);
    const int tq = (m_dp + 15) >> 4;
    const int t_begin = uni(ip->t_begin), t_end = uni(ip->t_end);
    const uint32_t lb = (uint32_t)lane * 32;

    f64x4 acc[QT], ar[KT], xr[RX], br[RB];
#pragma unroll
    for (int q = 0; q < QT; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};

    auto load_a = [&](const TD& T) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
            ar[kt] = ld4(pool_t + T.a + (int64_t)(rt * T.pa16 + (4 * kt < T.ka4 ? kt : 0)) * kTileD, lb);
    };
    auto x_tile = [&](const TD& T, int jc, int kt) {
        return ld4(xt + T.x + (int64_t)(jc * T.pa16 + (4 * kt < T.ka4 ? kt : 0)) * kTileD, lb);
    };
    auto b_tile = [&](const TD& T, int jc, int q) {
        return ld4(pool_t + T.b + (int64_t)((q < tq ? q : 0) * T.pd16 + jc) * kTileD, lb);
    };

    int t = t_begin, jc = 0;
    TD T = load_td(tasks + t);
    TD Tnext = load_td(tasks + min(t + 1, t_end - 1));   // the following task, one ahead
    load_a(T);
#pragma unroll
    for (int i = 0; i < RX; ++i) xr[i] = x_tile(T, 0, i);
#pragma unroll
    for (int i = 0; i < RB; ++i) br[i] = b_tile(T, 0, i);
    fence();
    for (;;) {
        const bool more_cols = 4 * (jc + 1) < T.kd4;
        const bool new_task = !more_cols && t + 1 < t_end;
        // the next step (the last step's successor is its own task's first step: loaded, never used)
        const int njc = more_cols ? jc + 1 : 0;
        const TD N = new_task ? Tnext : T;
        f64x4 tt = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (4 * kt + v < T.ka4)
                    tt = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[kt % RX][v], ar[kt][v], tt, 0, 0, 0);
            fence();
            xr[kt % RX] = kt + RX < KT ? x_tile(T, jc, kt + RX) : x_tile(N, njc, kt + RX - KT);
            fence();
        }
        // tt[v] = T'[16 rt + li][16 jc + 4 v + g] (unscaled); the A rows are free now
        if (new_task) {
            fence();
            load_a(Tnext);
            fence();
        }
        tt *= T.f;
        const int kd = T.kd4 - 4 * jc;   // k steps of this column tile that hold data (4 or the rest)
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            if (q < tq) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (v < kd) acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(tt[v], br[q % RB][v], acc[q], 0, 0, 0);
            }
            fence();
            br[q % RB] = q + RB < QT ? b_tile(T, jc, q + RB) : b_tile(N, njc, q + RB - QT);
            fence();
        }
        if (!more_cols && !new_task) break;
        jc = njc;
        if (new_task) {
            ++t;
            T = Tnext;
            Tnext = load_td(tasks + min(t + 1, t_end - 1));
        }
    }
    // store: lane (li, g) holds Y[16 rt + g + 4 v][16 q + li]
    const int64_t y_off = uni64(ip->y_off), part_off = uni64(ip->part_off);
    const int m_ap = uni(ip->m_ap), tn = 16 * tq;
    const int li = lane & 15, g = lane >> 4;
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        if (q >= tq) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * rt + g + 4 * v, col = 16 * q + li;
            if (part_off < 0) {
                if (row < m_ap && col < m_dp) y[y_off + (int64_t)row * m_dp + col] += acc[q][v];
            } else {
                part[part_off + (int64_t)row * tn + col] = acc[q][v];
            }
        }
    }
}

}  // namespace

// Group G runs the classes (KT, QT) of its register budget: 0: up to 2 x 2 tiles, 1: up to 3 x 3,
// 2: up to 8 x 8. Item.c0 holds the class, kRsSizes indices 8 * k + q.
template <int G, int MINW>
__global__ __launch_bounds__(kRsWaves * 64, MINW) void k_hpsi_rs64(const Item* __restrict__ items, int n_items,
                                                                const LTask64* __restrict__ tasks,
                                                                const double* __restrict__ pool_t,
                                                                const double* __restrict__ xt,
                                                                double* __restrict__ y, double* __restrict__ part,
                                                                const int32_t* __restrict__ mask) {
    const int w = uni((int)(blockIdx.x * kRsWaves + (threadIdx.x >> 6)));
    if (w >= n_items) return;
    const Item* ip = items + w;
    if (uni(ip->t_begin) >= uni(ip->t_end)) return;              // filler of a workgroup
    if (mask && mask[uni(ip->part)] != kPartActive) return;
    const int lane = threadIdx.x & 63;
#define DMRG_RS(K_, Q_, KT_, QT_) \
    case 8 * K_ + Q_: rs_item<KT_, QT_>(ip, tasks, pool_t, xt, y, part, lane); break;
    const int cls = uni(ip->c0);
    if constexpr (G == 0) {
        switch (cls) {
            DMRG_RS(0, 0, 1, 1) DMRG_RS(0, 1, 1, 2) DMRG_RS(1, 0, 2, 1)
            default: rs_item<2, 2>(ip, tasks, pool_t, xt, y, part, lane); break;
        }
    } else if constexpr (G == 1) {
        switch (cls) {
            DMRG_RS(0, 2, 1, 3) DMRG_RS(1, 2, 2, 3) DMRG_RS(2, 0, 3, 1) DMRG_RS(2, 1, 3, 2)
            default: rs_item<3, 3>(ip, tasks, pool_t, xt, y, part, lane); break;
        }
    } else {
        switch (cls) {
            DMRG_RS(0, 3, 1, 4) DMRG_RS(0, 4, 1, 6) DMRG_RS(0, 5, 1, 8)
            DMRG_RS(1, 3, 2, 4) DMRG_RS(1, 4, 2, 6) DMRG_RS(1, 5, 2, 8)
            DMRG_RS(2, 3, 3, 4) DMRG_RS(2, 4, 3, 6) DMRG_RS(2, 5, 3, 8)
            DMRG_RS(3, 0, 4, 1) DMRG_RS(3, 1, 4, 2) DMRG_RS(3, 2, 4, 3) DMRG_RS(3, 3, 4, 4) DMRG_RS(3, 4, 4, 6) DMRG_RS(3, 5, 4, 8)
            DMRG_RS(4, 0, 6, 1) DMRG_RS(4, 1, 6, 2) DMRG_RS(4, 2, 6, 3) DMRG_RS(4, 3, 6, 4) DMRG_RS(4, 4, 6, 6) DMRG_RS(4, 5, 6, 8)
            DMRG_RS(5, 0, 8, 1) DMRG_RS(5, 1, 8, 2) DMRG_RS(5, 2, 8, 3) DMRG_RS(5, 3, 8, 4) DMRG_RS(5, 4, 8, 6)
            default: rs_item<8, 8>(ip, tasks, pool_t, xt, y, part, lane); break;
        }
    }
#undef DMRG_RS
}

hipError_t launch_hpsi_rs64(const RsPlan64& P, const LTask64* tasks, const double* pool_t, const double* xt, double* y,
                            double* partial, hipStream_t s, const int32_t* active) {
    for (int g = kRsGroups - 1; g >= 0; --g) {   // the longest items first
        const int b = P.begin[g], n = P.begin[g + 1] - b;
        if (n <= 0) continue;
        const dim3 grid((n + kRsWaves - 1) / kRsWaves), block(kRsWaves * 64);
        if (g == 0) hipLaunchKernelGGL((k_hpsi_rs64<0, 4>), grid, block, 0, s, P.items + b, n, tasks, pool_t, xt, y, partial, active);
        else if (g == 1) hipLaunchKernelGGL((k_hpsi_rs64<1, 3>), grid, block, 0, s, P.items + b, n, tasks, pool_t, xt, y, partial, active);
        else hipLaunchKernelGGL((k_hpsi_rs64<2, 2>), grid, block, 0, s, P.items + b, n, tasks, pool_t, xt, y, partial, active);
    }
    return hipGetLastError();
}

}  // namespace dmrg
