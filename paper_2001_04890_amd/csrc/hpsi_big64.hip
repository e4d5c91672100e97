// FP64 sector GEMMs of Eq. dgemm (Section 2.2.1) for large sector blocks (gfx950), the FP64
// counterpart of hpsi_big.hip: pass 1 T'^T = X^T A^T per task, pass 2 Y += sum_tasks T B^T per
// 128 x 128 target tile, on v_mfma_f64_16x16x4f64.
//
// Operands are in the FP64 operand form of internal.h: of a 16 x 16 tile, lane l = (li, g) = (l % 16, l / 16)
// takes M[16 rt + li][16 kt + 4 v + g], v = 0..3, as two 16-byte halves (v = 0, 1 and v = 2, 3), each half
// 1 KB in lane order where all 16 rows are there. Value v is the lane's operand of the v-th 16x16x4 MFMA
// over that tile (A operand M[i = li][k = g], or B operand M^T[k = g][n = li]). The MFMA result layout
// (lane holds D[g + 4 v][li]) of a 16 x 16 tile of T'^T = X^T A^T is exactly this order for T
// (rows r = li, k = j = 4 v + g), so pass 1 stores its accumulators as T tiles (2 KB, two halves) without
// a shuffle. Stages hold 16 tiles (32 KB) of both operands for one 16-wide k tile, copied with
// global_load_lds_dwordx4 one stage ahead (two stages); what lies outside a block is copied from inside it
// and never used. Accumulation is FP64 throughout.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace dmrg {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int kTileD = 256;                  // doubles per tile
constexpr int kStageTiles = 16;
constexpr int kStageD = kStageTiles * kTileD;

// a lane's four values of a staged tile: p = the lane's 16 bytes of the first half
__device__ __forceinline__ f64x4 lds4(const double* p) {
    const f64x2 a = *reinterpret_cast<const f64x2*>(p), b = *reinterpret_cast<const f64x2*>(p + kTileD / 2);
    return f64x4{a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Copy half h of row tile rt, k tile kt of an operand of r4 4-row groups and k4 k steps to dst (1 KB, lane
// order). Rows past the operand's last 4-row group repeat the last row; a half past the last k step is
// taken from `zeros` (at least 1 KB of them).
__device__ __forceinline__ void copy_half(const double* __restrict__ op, int r4, int k4, int rt, int kt, int h,
                                          const double* __restrict__ zeros, double* dst, int lane) {
    const int w = min(16, 4 * (r4 - 4 * rt));
    const int at = (lane >> 4) * w + min(lane & 15, w - 1);
    const double* src = 4 * kt + 2 * h < k4 ? op + (int64_t)(2 * kt + h) * r4 * 32 + rt * 128 : zeros;
    __builtin_amdgcn_global_load_lds((const void*)(src + at * 2), (lds_ptr_t)dst, 16, 0, 0);
}

}  // namespace

// ------------------------------------------------------------------ FP64 operand form
// element (row, k) of 16-byte unit e of an operand of r4 4-row groups (u = 0; u = 1 is k + 4)
__device__ __forceinline__ void op64_unit(int e, int r4, int& row, int& k) {
    const int per = r4 * 16, p = e / per, in = e - p * per, rt = in >> 6;
    const int w = min(16, 4 * (r4 - 4 * rt)), q = in - 64 * rt, g = q / w;
    row = 16 * rt + q - g * w;
    k = 8 * p + g;
}

// pool block (row-major, zero-padded to 16 rows and ld columns) -> operand form
__global__ void k_op64(const double* __restrict__ pool, const OpBlock64* __restrict__ blocks, double* __restrict__ ops) {
    const OpBlock64 B = blocks[blockIdx.x];
    const int r4 = (B.rows + 3) / 4, n = r4 * ((B.cols + 7) / 8) * 16;
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        int row, k;
        op64_unit(e, r4, row, k);
        const double* src = pool + B.src + (int64_t)row * B.ld + k;
        *reinterpret_cast<f64x2*>(ops + B.dst + (int64_t)e * 2) = f64x2{src[0], src[4]};
    }
}

hipError_t launch_op64(const double* pool, const OpBlock64* blocks, int n_blocks, double* ops, hipStream_t s) {
    if (n_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_op64, dim3(n_blocks), dim3(256), 0, s, pool, blocks, ops);
    return hipGetLastError();
}

// psi block X (m_a x m_d) -> X^T in operand form (m_d rows, m_a columns) at dst_off
__global__ void k_pack_xt64(const PackBlock* __restrict__ packs, const double* __restrict__ x, double* __restrict__ xt) {
    const PackBlock P = packs[blockIdx.x];
    const int r4 = (P.m_d + 3) / 4, n = r4 * ((P.m_a + 7) / 8) * 16;
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        int j, k;
        op64_unit(e, r4, j, k);
        const double* src = x + P.src_off + (int64_t)k * P.m_d + j;
        f64x2 v;
        v[0] = j < P.m_d && k < P.m_a ? src[0] : 0.0;
        v[1] = j < P.m_d && k + 4 < P.m_a ? src[4 * (int64_t)P.m_d] : 0.0;
        *reinterpret_cast<f64x2*>(xt + P.dst_off + (int64_t)e * 2) = v;
    }
}

// ------------------------------------------------------------------ pass 1: T = f A X per task
// Group: one task, T rows [16 rb, 16 rb + 128) (8 row tiles), T columns [16 jb, 16 jb + 128) (8 j
// tiles). The k loop stops at the last k step that holds data, and T tiles past the source's columns are
// neither copied nor stored.
// Wave (wj, wr): j tiles jb + 4 wj + {0..3}, row tiles rb + 4 wr + {0..3}: 16 accumulator tiles.
__global__ __launch_bounds__(256) void k_big64_t(const BigT1* __restrict__ work, const int32_t* __restrict__ ranges,
                                                 const double* __restrict__ ops, const double* __restrict__ xt,
                                                 double* __restrict__ tbuf, int64_t zeros,
                                                 const int32_t* __restrict__ mask) {
    __shared__ __attribute__((aligned(16))) double lds[2 * kStageD];
    const int g_begin = uni(ranges[blockIdx.x]), g_end = uni(ranges[blockIdx.x + 1]);
    if (mask && mask[work[g_begin].part] != kPartActive) return;   // a workgroup's groups share one part
    const int wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wj = wave & 1, wr = wave >> 1;
    struct G { int64_t x, a, t; double f; int ka16, pd, ra4, rb, jb, ka4, kd4; };
    auto load_g = [&](int i) {
        const BigT1* wp = work + i;
        G d;
        d.x = uni64(wp->xt); d.a = uni64(wp->a); d.t = uni64(wp->t);
        d.f = __builtin_bit_cast(double, uni64(__builtin_bit_cast(int64_t, wp->f)));
        d.ka16 = uni(wp->pa32); d.pd = uni(wp->pd32); d.ra4 = uni(wp->nrt); d.rb = uni(wp->rb); d.jb = uni(wp->jb);
        d.ka4 = uni(wp->ka); d.kd4 = uni(wp->kd);
        return d;
    };
    auto stage = [&](const G& d, int kt, double* to) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int hh = wave * 8 + k, tile = hh >> 1, h = hh & 1;   // waves 0, 1: X^T, waves 2, 3: A
            const bool isx = tile < 8;
            const int rt = isx ? d.jb + tile : d.rb + tile - 8, r4 = isx ? d.kd4 : d.ra4;
            if (4 * rt < r4)
                copy_half(isx ? xt + d.x : ops + d.a, r4, d.ka4, rt, kt, h, ops + zeros, to + tile * kTileD + h * 128, lane);
        }
    };
    f64x4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
        }
    auto store = [&](const G d) {
        int ln = lane;   // opaque copy: keep the store addresses out of the main loop
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int jt = d.jb + 4 * wj + jj, rt = d.rb + 4 * wr + rr;
                if (4 * jt < d.kd4 && 4 * rt < d.ra4) {
                    // acc[jj][rr][v] = T'^T[j 16 jt + g + 4 v][r 16 rt + li] = T tile (rt, jt), lane value v
                    const f64x4 v = acc[jj][rr] * d.f;
                    double* to = tbuf + d.t + (int64_t)(rt * d.pd + jt) * kTileD + ln * 2;
                    *reinterpret_cast<f64x2*>(to) = f64x2{v[0], v[1]};
                    *reinterpret_cast<f64x2*>(to + kTileD / 2) = f64x2{v[2], v[3]};
                }
                acc[jj][rr] = f64x4{0.0, 0.0, 0.0, 0.0};
            }
    };

    int gi = g_begin, kt = 0;
    G cur = load_g(gi);
    stage(cur, 0, lds);
    wait_vm();
    __syncthreads();
    int st = 0;
    for (;;) {
        int ngi = gi, nkt = kt + 1;
        if (nkt == cur.ka16) { ngi = gi + 1; nkt = 0; }
        const bool has_next = ngi < g_end;
        G nxt = cur;
        if (has_next) {
            if (ngi != gi) nxt = load_g(ngi);
            stage(nxt, nkt, lds + (st ^ 1) * kStageD);
        }
        const double* sp = lds + st * kStageD + lane * 2;
        f64x4 p[4], q[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) p[jj] = lds4(sp + (4 * wj + jj) * kTileD);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) q[rr] = lds4(sp + (8 + 4 * wr + rr) * kTileD);
        // consecutive MFMAs accumulate into the same registers (the fast path of the matrix core); every
        // tile and k step runs (skipping those outside the block costs this kernel its second workgroup
        // per CU)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[jj][rr] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[jj][v], q[rr][v], acc[jj][rr], 0, 0, 0);
        if (ngi != gi) store(cur);
        wait_vm();
        __syncthreads();
        if (!has_next) break;
        gi = ngi; kt = nkt; cur = nxt;
        st ^= 1;
    }
}

// ------------------------------------------------------------------ pass 2: Y += sum T B^T per tile
// The k loop runs over the T tiles and k steps that hold data; a wave runs the MFMAs of its output tiles
// inside the target only.
__global__ __launch_bounds__(256) void k_big64_y(const Item* __restrict__ items, const BigT2* __restrict__ tasks,
                                                 const double* __restrict__ ops, const double* __restrict__ tbuf,
                                                 double* __restrict__ y, double* __restrict__ part, int64_t zeros,
                                                 const int32_t* __restrict__ mask) {
    __shared__ __attribute__((aligned(16))) double lds[2 * kStageD];
    const Item* ip = items + blockIdx.x;
    if (mask && mask[ip->part] != kPartActive) return;
    const int64_t y_off = uni64(ip->y_off), part_off = uni64(ip->part_off);
    const int m_ap = uni(ip->m_ap), m_dp = uni(ip->m_dp), r0 = uni(ip->r0), c0 = uni(ip->c0);
    const int t_begin = uni(ip->t_begin), t_end = uni(ip->t_end);
    const int wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wr = wave >> 1, wq = wave & 1;
    const int rb = r0 >> 4, qb = c0 >> 4;
    const int nrt = (m_ap + 15) >> 4, nq = (m_dp + 15) >> 4;
    const int tn = 16 * min(8, nq - qb);

    const int rb4 = (m_dp + 3) >> 2;
    auto stage = [&](int64_t t_t, int64_t t_b, int pd, int kd4, int jt, double* to) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int hh = wave * 8 + k, tile = hh >> 1, h = hh & 1;   // waves 0, 1: T, waves 2, 3: B
            double* dst = to + tile * kTileD + h * 128;
            if (tile < 8) {
                const int rt = rb + tile;
                if (rt < nrt)
                    __builtin_amdgcn_global_load_lds((const void*)(tbuf + t_t + (int64_t)(rt * pd + jt) * kTileD + h * 128 + lane * 2),
                                                     (lds_ptr_t)dst, 16, 0, 0);
            } else {
                const int q = qb + tile - 8;
                if (q < nq) copy_half(ops + t_b, rb4, kd4, q, jt, h, ops + zeros, dst, lane);
            }
        }
    };
    f64x4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
            asm volatile("" : "+a"(acc[a][b]));   // accumulators live in AGPRs across the loop
        }

    // this wave's output tiles inside the target (wave-uniform counts)
    const int nr = min(4, max(0, nrt - rb - 4 * wr)), nqw = min(4, max(0, nq - qb - 4 * wq));
    int t = t_begin, jt = 0;
    int64_t T_t = uni64(tasks[t].t), T_b = uni64(tasks[t].b);
    int T_pd = uni(tasks[t].pd32), T_kd = uni(tasks[t].kd);
    stage(T_t, T_b, T_pd, T_kd, 0, lds);
    wait_vm();
    __syncthreads();
    int st = 0;
    for (;;) {
        int nt = t, njt = jt + 1;
        if (njt == T_pd) { nt = t + 1; njt = 0; }
        const bool has_next = nt < t_end;
        int64_t N_t = T_t, N_b = T_b;
        int N_pd = T_pd, N_kd = T_kd;
        if (has_next) {
            if (nt != t) {
                N_t = uni64(tasks[nt].t); N_b = uni64(tasks[nt].b);
                N_pd = uni(tasks[nt].pd32); N_kd = uni(tasks[nt].kd);
            }
            stage(N_t, N_b, N_pd, N_kd, njt, lds + (st ^ 1) * kStageD);
        }
        const double* sp = lds + st * kStageD + lane * 2;
        f64x4 p[4], q[4];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) p[rr] = lds4(sp + (4 * wr + rr) * kTileD);
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) q[qq] = lds4(sp + (8 + 4 * wq + qq) * kTileD);
        const int kleft = T_kd - 4 * jt;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
#pragma unroll
            for (int qq = 0; qq < 4; ++qq)
                if (rr < nr && qq < nqw) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (v < kleft)
                            acc[rr][qq] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[rr][v], q[qq][v], acc[rr][qq], 0, 0, 0);
                }
        wait_vm();
        __syncthreads();
        if (!has_next) break;
        t = nt; jt = njt; T_t = N_t; T_b = N_b; T_pd = N_pd; T_kd = N_kd;
        st ^= 1;
    }
    // pin the accumulators to AGPRs at the loop exit (else the allocator copies them to VGPRs on every
    // iteration, for the epilogue's sake)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) asm volatile("" : "+a"(acc[rr][qq]));
    // acc[rr][qq][v] = Y[16 rt + g + 4 v][16 q + li]
    int ln = lane;   // opaque copy: keep the store addresses out of the main loop
    asm volatile("" : "+v"(ln));
    const int li = ln & 15, g = ln >> 4;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
            const int rt = rb + 4 * wr + rr, q = qb + 4 * wq + qq;
            if (rt >= nrt || q >= nq) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * rt + g + 4 * v, col = 16 * q + li;
                if (part_off < 0) {
                    if (row < m_ap && col < m_dp) y[y_off + (int64_t)row * m_dp + col] += acc[rr][qq][v];
                } else {
                    part[part_off + (int64_t)(row - r0) * tn + (col - c0)] = acc[rr][qq][v];
                }
            }
            if (qq == 3) asm volatile("" ::: "memory");   // at most 16 read-modify-writes of y in flight
        }
}

__global__ void k_reduce_big64(const Reduce* __restrict__ red, const double* __restrict__ part, double* __restrict__ y,
                               const int32_t* __restrict__ mask) {
    const Reduce R = red[blockIdx.x];
    if (mask && mask[R.part] != kPartActive) return;
    const int n = R.tm * R.tn;
    const int e = blockIdx.y * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int rr = e / R.tn, cc = e - (e / R.tn) * R.tn;
    const int row = R.r0 + rr, col = R.c0 + cc;
    if (row >= R.m_ap || col >= R.m_dp) return;
    double s = 0.0;
    for (int k = 0; k < R.n_parts; ++k) s += part[R.part_off + (int64_t)k * n + e];
    y[R.y_off + (int64_t)row * R.m_dp + col] += s;
}

hipError_t launch_pack_xt64(const PackBlock* packs, int n_packs, const double* x, double* xt, hipStream_t s) {
    if (n_packs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_xt64, dim3(n_packs), dim3(256), 0, s, packs, x, xt);
    return hipGetLastError();
}

hipError_t launch_hpsi_big64(const BigPlan& P, const double* ops, const double* xt, double* y, hipStream_t s,
                             const int32_t* active) {
    if (P.n_chunks == 0) return hipSuccess;
    const double* tb = reinterpret_cast<const double*>(P.tbuf);
    for (int c = 0; c < P.n_chunks; ++c) {
        const BigChunk& C = P.chunks[c];
        if (C.t1_end > C.t1_begin)
            hipLaunchKernelGGL(k_big64_t, dim3(C.t1_end - C.t1_begin), dim3(256), 0, s, P.t1, P.t1_ranges + C.t1_begin,
                               ops, xt, reinterpret_cast<double*>(P.tbuf), P.zeros, active);
        if (C.item_end > C.item_begin)
            hipLaunchKernelGGL(k_big64_y, dim3(C.item_end - C.item_begin), dim3(256), 0, s, P.items + C.item_begin, P.t2,
                               ops, tb, y, P.partial, P.zeros, active);
        if (C.red_end > C.red_begin)
            hipLaunchKernelGGL(k_reduce_big64, dim3(C.red_end - C.red_begin, P.red_chunks), dim3(256), 0, s,
                               P.reduces + C.red_begin, P.partial, y, active);
    }
    return hipGetLastError();
}

}  // namespace dmrg
