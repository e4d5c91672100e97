// Register-streamed FP64 sector GEMMs of Eq. dgemm (Section 2.2.1) for gfx950, on
// v_mfma_f64_16x16x4f64 with FP64 accumulation.
//
// One wavefront owns one 16-row tile of a target psi block of at most 128 columns and runs over a range
// of its tasks Y += f * A . X . B^T; there is no LDS and no barrier. A task is cut into steps, one per
// 16-wide column tile jc of the source, and per step:
//   GEMM1  T'(rt, jc)^T = X^T(jc, :) . A(rt, :)^T   A's row tile stays in registers for the task
//   GEMM2  Y(rt, :)   += f T'(rt, jc) . B(:, jc)^T  GEMM1's result layout is GEMM2's A-operand layout
// X^T and B stream from the caches into register rings that are refilled as soon as an operand has been
// used, up to a whole GEMM ahead of its next use. Every load is unconditional, so that the compiler knows how
// many are in flight and never waits for the newest; being a buffer load with the operand's size, it moves
// nothing past the operand's end and takes its address from scalar registers. MFMAs run only on the 4-wide k
// steps that hold data. Operands are read in the compact form of internal.h, 16 bytes per lane and two k steps.
//
// What bounds it: an FP64 16x16x4 MFMA takes 64 cycles, so a wavefront needs 2 KB per 256 cycles, half of
// what a CU's vector cache delivers to four of them: the matrix cores and the traffic between the L2s
// and memory bound large sectors, latency (hidden by 8 .. 32 wavefronts per CU) and launches the small. 24 orbitals
// at bond dimension 1024 read 29 GB, and the matrix cores are busy 86, 86 and 74% of the three launches. One
// matvec of 24 orbitals at bond dimension 1024 takes 5.1 .. 5.3 ms (3.6 ms of MFMAs; 6.5 ms with pointer loads and
// the accumulators copied around conditional MFMAs), of 17 orbitals at 333 states 228 us (278 us with the
// smallest classes at 4 wavefronts per SIMD instead of 8), of a batch of 12 problems with sectors of up to some
// 30 states 782 us (1.0 ms).
#include "device.h"
#include "internal.h"

namespace dmrg {

namespace {

// 16 bytes per lane at byte `at` (wave-uniform) + lane_bytes of an operand; zero past its end
__device__ __forceinline__ f64x2 ld2(__amdgpu_buffer_rsrc_t op, uint32_t lane_bytes, uint32_t at) {
    return __builtin_bit_cast(f64x2, ld16(op, lane_bytes, at));
}
// An operand of r4 4-row groups and k4 k steps in the compact form.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand(const double* p, int r4, int k4) {
    return buf(p, ((k4 + 1) >> 1) * r4 * 256);
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
    each<QT>([&](auto q) { acc[q] = f64x4{0.0, 0.0, 0.0, 0.0}; });

    // a load past an operand's last column group gives zeros and moves nothing
    auto load_a = [&](const TD& T) {
        const __amdgpu_buffer_rsrc_t op = operand(ops + T.a, ra4, T.ka4);
        each<KP>([&](auto p) { ar[p] = ld2(op, a_lane, (uint32_t)(p * ra4) * 256u); });
    };
    auto x_op = [&](const TD& T) { return operand(xt + T.x, T.kd4, T.ka4); };
    auto b_op = [&](const TD& T) { return operand(ops + T.b, rb4, T.kd4); };
    auto x_pair = [&](__amdgpu_buffer_rsrc_t op, int kd4, uint32_t x_lane, int p) {
        return ld2(op, x_lane, (uint32_t)(p * kd4) * 256u);
    };
    auto b_tile = [&](__amdgpu_buffer_rsrc_t op, int jc, int q, f64x2 (&b)[JP]) {
        const uint32_t lane_off = q < tq - 1 ? b_full : b_last;
        each<JP>([&](auto h) {
            b[h] = ld2(op, lane_off, (uint32_t)((2 * jc + h) * rb4) * 256u + (q < tq - 1 ? (uint32_t)q * 1024u : 0u));
        });
    };

    int t = t_begin, jc = 0;
    TD T = load_td(tasks + t);
    TD Tnext = load_td(tasks + min(t + 1, t_end - 1));   // the following task, one ahead
    load_a(T);
    uint32_t xl = lane_at(0, T.kd4);                      // the lane's place in X^T's row tile jc
    __amdgpu_buffer_rsrc_t xo = x_op(T), bo = b_op(T);
    each<RX>([&](auto i) { xr[i] = x_pair(xo, T.kd4, xl, i); });
    each<RB>([&](auto i) { b_tile(bo, 0, i, br[i]); });
    fence();
    for (;;) {
        const bool more_cols = 4 * (jc + 1) < T.kd4;
        const bool new_task = !more_cols && t + 1 < t_end;
        // the next step (the last step's successor is its own task's first step: loaded, never used)
        const int njc = more_cols ? jc + 1 : 0;
        const TD N = new_task ? Tnext : T;
        const uint32_t nxl = lane_at(njc, N.kd4);
        const __amdgpu_buffer_rsrc_t nxo = x_op(N), nbo = b_op(N);
        f64x4 tt = f64x4{0.0, 0.0, 0.0, 0.0};
        each<KP>([&](auto p) {
            constexpr int P = p;
            each<2>([&](auto u) {
                constexpr int U = u;
                if (2 * P + U < T.ka4) tt = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[P % RX][U], ar[P][U], tt, 0, 0, 0);
            });
            fence();
            xr[P % RX] = P + RX < KP ? x_pair(xo, T.kd4, xl, P + RX) : x_pair(nxo, N.kd4, nxl, P + RX - KP);
            fence();
        });
        // tt[v] = T'[16 rt + li][16 jc + 4 v + g] (unscaled); the A rows are free now
        if (new_task) {
            fence();
            load_a(Tnext);
            fence();
        }
        tt *= T.f;
        const int kd = T.kd4 - 4 * jc;   // k steps of this column tile that hold data (4 or the rest)
        each<QT>([&](auto q) {
            constexpr int Q = q;
            if (Q < tq) {
                each<2 * JP>([&](auto v) {
                    constexpr int V = v;
                    if (V < kd) acc[Q] = __builtin_amdgcn_mfma_f64_16x16x4f64(tt[V], br[Q % RB][V >> 1][V & 1], acc[Q], 0, 0, 0);
                });
            }
            fence();
            if constexpr (Q + RB < QT) b_tile(bo, jc, Q + RB, br[Q % RB]);
            else b_tile(nbo, njc, Q + RB - QT, br[Q % RB]);
            fence();
        });
        if (!more_cols && !new_task) break;
        jc = njc;
        xl = nxl;
        xo = nxo;
        bo = nbo;
        if (new_task) {
            ++t;
            T = Tnext;
            Tnext = load_td(tasks + min(t + 1, t_end - 1));
        }
    }
    // store: lane (li, g) holds Y[16 rt + g + 4 v][16 q + li]
    const int64_t y_off = uni64(ip->y_off), part_off = uni64(ip->part_off);
    if (part_off >= 0) {
        const __amdgpu_buffer_rsrc_t op = buf(part + part_off + (int64_t)rt * 256 * tq, 2048 * tq);
        const int at = (int)((g * 16 * tq + li) * 8);
        each<QT>([&](auto q) {
            if (q < tq) each<4>([&](auto i) {
                constexpr int v = i;
                const double a = acc[q][v];
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, a), op, at, (64 * v * tq + 16 * q) * 8, 0);
            });
        });
    } else {
        // the loads of four column tiles are in flight at once; what lies outside the block is neither read nor written
        const __amdgpu_buffer_rsrc_t op = buf(y + y_off + (int64_t)rt * 16 * m_dp, min(16, m_ap - 16 * rt) * m_dp * 8);
        auto at = [&](int q, int v) { return (int)(16 * q + li < (uint32_t)m_dp ? ((g + 4 * v) * m_dp + 16 * q + li) * 8u : kNowhere); };
        each<(QT + 3) / 4>([&](auto h) {
            constexpr int q0 = 4 * h, nq = QT - q0 < 4 ? QT - q0 : 4;
            f64x4 old[nq];
            each<nq>([&](auto q) {
                if (q0 + q < tq) each<4>([&](auto i) {
                    constexpr int v = i;
                    old[q][v] = __builtin_bit_cast(double, (i32x2)__builtin_amdgcn_raw_buffer_load_b64(op, at(q0 + q, v), 0, 0));
                });
            });
            each<nq>([&](auto q) {
                if (q0 + q < tq) each<4>([&](auto i) {
                    constexpr int v = i;
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, old[q][v] + acc[q0 + q][v]), op, at(q0 + q, v), 0, 0);
                });
            });
        });
    }
}

template <int G, int K, int Q>
__device__ __forceinline__ bool rs_try(int cls, const Item* __restrict__ ip, const LTask64* __restrict__ tasks,
                                       const double* __restrict__ ops, const double* __restrict__ xt, double* __restrict__ y,
                                       double* __restrict__ part, int lane) {
    if constexpr (rs_group(K, Q) <= G) {
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

// Group G runs the classes within its register budget (rs_group and below).
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
#define DMRG_RS(G, W) hipLaunchKernelGGL((k_hpsi_rs64<G, W>), grid, block, 0, s, it, n, P.tasks, ops, xt, y, P.partial, active)
        switch (g) {
            case 0: DMRG_RS(0, 8); break;
            case 1: DMRG_RS(1, 5); break;
            case 2: DMRG_RS(2, 4); break;
            case 3: DMRG_RS(3, 3); break;
            default: DMRG_RS(4, 2); break;
        }
#undef DMRG_RS
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || P.n_reduces <= 0) return e;
    return launch_reduce_partials(P.reduces, P.n_reduces, P.red_chunks, P.partial, y, s, active);
}

}  // namespace dmrg
