// Register-streamed FP64 sector GEMMs of Eq. dgemm (Section 2.2.1) for gfx950, on
// v_mfma_f64_16x16x4f64 with FP64 accumulation.
//
// One wavefront owns one 16-row tile of a target psi block of at most 128 columns and runs over a range
// of its tasks Y += f * A . X . B^T; there is no LDS and no barrier. A task is cut into steps, one per
// 16-wide column tile jc of the source, and per step:
//   GEMM1  T'(rt, jc)^T = X^T(jc, :) . A(rt, :)^T   A's row tile stays in registers for the task
//   GEMM2  Y(rt, :)   += f T'(rt, jc) . B(:, jc)^T  GEMM1's result layout is GEMM2's A-operand layout
// X^T and B stream from the caches into register rings that are refilled as soon as an operand has been
// used, up to a whole GEMM ahead of its next use (every load is unconditional: what lies outside the block
// re-reads a part of it, so that the compiler knows how many loads are in flight and never waits for the
// newest). MFMAs run only on the 4-wide k steps that hold data. Operands are read in the compact form of
// internal.h, 16 bytes per lane and two k steps.
//
// What bounds it: an FP64 16x16x4 MFMA takes 64 cycles, so a wavefront needs 2 KB per 256 cycles, half of
// what a CU's vector cache delivers to four of them: the matrix cores and the traffic between the L2s
// and memory bound large sectors, latency (hidden by 8 .. 16 wavefronts per CU) and launches the small.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace dmrg {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double unid(double v) {
    return __builtin_bit_cast(double, uni64(__builtin_bit_cast(int64_t, v)));
}

// 16 bytes per lane, lane_bytes after a wave-uniform address
__device__ __forceinline__ f64x2 ld2(const double* p, uint32_t lane_bytes) {
    return *reinterpret_cast<const f64x2*>(reinterpret_cast<const char*>(p) + lane_bytes);
}

// Task descriptor in scalar registers.
struct TD { int64_t x, a, b; double f; int ka4, kd4; };
__device__ __forceinline__ TD load_td(const LTask64* __restrict__ p) {
    TD d;
    d.x = uni64(p->x_off);
    d.a = uni64(p->a_off);
    d.b = uni64(p->b_off);
    d.f = unid(p->f);
    d.ka4 = uni(p->ka4);
    d.kd4 = uni(p->kd4);
    return d;
}

// keeps the loads before it from sinking to their uses and those after it from rising
__device__ __forceinline__ void fence() { asm volatile("" ::: "memory"); }

// KP: column groups (two k steps each) of the A row tile; QT: column tiles of the target; JP: column
// groups of a source column tile that are read (1: every source has at most 8 columns).
template <int KP, int QT, int JP>
__device__ __forceinline__ void rs_item(const Item* __restrict__ ip, const LTask64* __restrict__ tasks,
                                        const double* __restrict__ ops, const double* __restrict__ xt,
                                        double* __restrict__ y, double* __restrict__ part, int lane) {
    constexpr int RX = KP == 16 ? 8 : KP, RB = QT == 8 ? 4 : QT;   // ring sizes (divisors of KP, QT)
    const int rt = uni(ip->r0) >> 4, m_ap = uni(ip->m_ap), m_dp = uni(ip->m_dp);
    const int ra4 = (m_ap + 3) >> 2, rb4 = (m_dp + 3) >> 2, tq = (m_dp + 15) >> 4;
    const int t_begin = uni(ip->t_begin), t_end = uni(ip->t_end);
    const uint32_t li = lane & 15, g = lane >> 4;
    // byte offset of the lane in row tile t of an operand of r4 4-row groups (rows past the end of a
    // ragged last tile read its last row)
    auto lane_at = [&](int t, int r4) {
        const uint32_t w = min(16, 4 * (r4 - 4 * t));
        return (uint32_t)t * 1024u + (g * w + min(li, w - 1)) * 16u;
    };
    const uint32_t a_lane = lane_at(rt, ra4), b_full = (uint32_t)lane * 16u, b_last = lane_at(tq - 1, rb4);

    f64x4 acc[QT];
    f64x2 ar[KP], xr[RX], br[RB][JP];
#pragma unroll
    for (int q = 0; q < QT; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};

    auto load_a = [&](const TD& T) {
#pragma unroll
        for (int p = 0; p < KP; ++p) ar[p] = ld2(ops + T.a + (int64_t)((2 * p < T.ka4 ? p : 0) * ra4) * 32, a_lane);
    };
    auto x_pair = [&](const TD& T, uint32_t x_lane, int p) {
        return ld2(xt + T.x + (int64_t)((2 * p < T.ka4 ? p : 0) * T.kd4) * 32, x_lane);
    };
    auto b_tile = [&](const TD& T, int jc, int q, f64x2 (&b)[JP]) {
        const uint32_t at = q < tq - 1 ? (uint32_t)q * 1024u + b_full : b_last;
#pragma unroll
        for (int h = 0; h < JP; ++h) {
            const int p = 2 * jc + (4 * jc + 2 * h < T.kd4 ? h : 0);
            b[h] = ld2(ops + T.b + (int64_t)(p * rb4) * 32, at);
        }
    };

    int t = t_begin, jc = 0;
    TD T = load_td(tasks + t);
    TD Tnext = load_td(tasks + min(t + 1, t_end - 1));   // the following task, one ahead
    load_a(T);
    uint32_t xl = lane_at(0, T.kd4);                      // the lane's place in X^T's row tile jc
#pragma unroll
    for (int i = 0; i < RX; ++i) xr[i] = x_pair(T, xl, i);
#pragma unroll
    for (int i = 0; i < RB; ++i) b_tile(T, 0, i, br[i]);
    fence();
    for (;;) {
        const bool more_cols = 4 * (jc + 1) < T.kd4;
        const bool new_task = !more_cols && t + 1 < t_end;
        // the next step (the last step's successor is its own task's first step: loaded, never used)
        const int njc = more_cols ? jc + 1 : 0;
        const TD N = new_task ? Tnext : T;
        const uint32_t nxl = lane_at(njc, N.kd4);
        f64x4 tt = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int p = 0; p < KP; ++p) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (2 * p + u < T.ka4) tt = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[p % RX][u], ar[p][u], tt, 0, 0, 0);
            fence();
            xr[p % RX] = p + RX < KP ? x_pair(T, xl, p + RX) : x_pair(N, nxl, p + RX - KP);
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
                for (int v = 0; v < 2 * JP; ++v)
                    if (v < kd) acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(tt[v], br[q % RB][v >> 1][v & 1], acc[q], 0, 0, 0);
            }
            fence();
            if (q + RB < QT) b_tile(T, jc, q + RB, br[q % RB]);
            else b_tile(N, njc, q + RB - QT, br[q % RB]);
            fence();
        }
        if (!more_cols && !new_task) break;
        jc = njc;
        xl = nxl;
        if (new_task) {
            ++t;
            T = Tnext;
            Tnext = load_td(tasks + min(t + 1, t_end - 1));
        }
    }
    // store: lane (li, g) holds Y[16 rt + g + 4 v][16 q + li]
    const int64_t y_off = uni64(ip->y_off), part_off = uni64(ip->part_off);
    const int tn = 16 * tq;
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

template <int G, int K, int Q>
__device__ __forceinline__ bool rs_try(int cls, const Item* __restrict__ ip, const LTask64* __restrict__ tasks,
                                       const double* __restrict__ ops, const double* __restrict__ xt, double* __restrict__ y,
                                       double* __restrict__ part, int lane) {
    if constexpr (rs_group(K, Q) == G) {
        if (cls == 8 * K + Q) {
            rs_item<K == 0 ? 1 : 2 * kRsK[K], kRsQ[Q], K == 0 ? 1 : 2>(ip, tasks, ops, xt, y, part, lane);
            return true;
        }
    }
    return false;
}

template <int G, int K>
__device__ __forceinline__ void rs_try_k(int cls, const Item* __restrict__ ip, const LTask64* __restrict__ tasks,
                                         const double* __restrict__ ops, const double* __restrict__ xt, double* __restrict__ y,
                                         double* __restrict__ part, int lane) {
    if ((cls >> 3) != K) return;
    (void)(rs_try<G, K, 0>(cls, ip, tasks, ops, xt, y, part, lane) || rs_try<G, K, 1>(cls, ip, tasks, ops, xt, y, part, lane) ||
           rs_try<G, K, 2>(cls, ip, tasks, ops, xt, y, part, lane) || rs_try<G, K, 3>(cls, ip, tasks, ops, xt, y, part, lane) ||
           rs_try<G, K, 4>(cls, ip, tasks, ops, xt, y, part, lane) || rs_try<G, K, 5>(cls, ip, tasks, ops, xt, y, part, lane));
}

}  // namespace

// Group G runs the classes of its register budget (rs_group).
template <int G, int MINW>
__global__ __launch_bounds__(kRsWaves * 64, MINW) void k_hpsi_rs64(const Item* __restrict__ items, int n_items,
                                                                const LTask64* __restrict__ tasks,
                                                                const double* __restrict__ ops,
                                                                const double* __restrict__ xt,
                                                                double* __restrict__ y, double* __restrict__ part,
                                                                const int32_t* __restrict__ mask) {
    const int w = uni((int)(blockIdx.x * kRsWaves + (threadIdx.x >> 6)));
    if (w >= n_items) return;
    const Item* ip = items + w;
    if (uni(ip->t_begin) >= uni(ip->t_end)) return;              // filler of a workgroup
    if (mask && mask[uni(ip->part)] != kPartActive) return;
    const int lane = threadIdx.x & 63, cls = uni(ip->c0);
    rs_try_k<G, 0>(cls, ip, tasks, ops, xt, y, part, lane);
    rs_try_k<G, 1>(cls, ip, tasks, ops, xt, y, part, lane);
    rs_try_k<G, 2>(cls, ip, tasks, ops, xt, y, part, lane);
    rs_try_k<G, 3>(cls, ip, tasks, ops, xt, y, part, lane);
    rs_try_k<G, 4>(cls, ip, tasks, ops, xt, y, part, lane);
    rs_try_k<G, 5>(cls, ip, tasks, ops, xt, y, part, lane);
    rs_try_k<G, 6>(cls, ip, tasks, ops, xt, y, part, lane);
}

hipError_t launch_hpsi_rs64(const RsPlan64& P, const double* ops, const double* xt, double* y, hipStream_t s,
                            const int32_t* active) {
    if (P.n_items == 0) return hipSuccess;
    for (int g = kRsGroups - 1; g >= 0; --g) {   // the longest items first
        const int b = P.begin[g], n = P.begin[g + 1] - b;
        if (n <= 0) continue;
        const dim3 grid((n + kRsWaves - 1) / kRsWaves), block(kRsWaves * 64);
        const Item* it = P.items + b;
        if (g == 0) hipLaunchKernelGGL((k_hpsi_rs64<0, 4>), grid, block, 0, s, it, n, P.tasks, ops, xt, y, P.partial, active);
        else if (g == 1) hipLaunchKernelGGL((k_hpsi_rs64<1, 3>), grid, block, 0, s, it, n, P.tasks, ops, xt, y, P.partial, active);
        else hipLaunchKernelGGL((k_hpsi_rs64<2, 2>), grid, block, 0, s, it, n, P.tasks, ops, xt, y, P.partial, active);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || P.n_reduces <= 0) return e;
    return launch_reduce_partials(P.reduces, P.n_reduces, P.red_chunks, P.partial, y, s, active);
}

}  // namespace dmrg
