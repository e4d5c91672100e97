// FP64 sector GEMMs of Eq. dgemm (Section 2.2.1) for large sector blocks (gfx950), the FP64
// counterpart of hpsi_big.hip: pass 1 T'^T = X^T A^T per task, pass 2 Y += sum_tasks T B^T, on
// v_mfma_f64_16x16x4f64 with FP64 accumulation.
//
// A wavefront by itself owns up to 4 x 4 tiles of T or of Y (128 accumulator registers) and reads both
// operands, one 8-wide column group at a time, straight into registers; there is no LDS and no barrier. A
// column group is 8 loads of 1 KB and 32 MFMAs (2048 cycles); two of them are in flight, and every register
// is loaded again, for the group after next, as soon as its last MFMA has been issued. All loads are
// unconditional buffer loads (what lies outside the block or past the last group moves nothing), so the
// compiler knows how many are in flight. Only tiles and 4-wide k steps that hold data are multiplied.
//
// Operands are in the FP64 operand form of internal.h: of a 16 x 16 tile, lane l = (li, g) = (l % 16, l / 16)
// takes M[16 rt + li][16 kt + 4 v + g], v = 0..3, as two 16-byte halves (v = 0, 1 and v = 2, 3: one column
// group each). The MFMA result layout (lane holds D[g + 4 v][li]) of a 16 x 16 tile of T'^T = X^T A^T is
// exactly this order for T (rows r = li, k = j = 4 v + g), so pass 1 stores its accumulators as T tiles
// (2 KB, two halves) without a shuffle.
//
// What bounds it: the MFMAs, which keep the matrix cores busy 82% of the time a CU has work (64 cycles each; the
// rest is the start and end of a wavefront's work and the ends of the launches). 76 orbitals at bond dimension
// 6000, one share: 25.3 ms, of which 18.6 ms are MFMAs; 42.4 ms with 128 x 128 tiles of four wavefronts staged
// through LDS, whose stages waited at a barrier and which multiplied whole tiles at the blocks' edges.
#include "device.h"
#include "internal.h"

namespace dmrg {

namespace {

constexpr int kTileD = 256;                  // doubles per tile

__device__ __forceinline__ f64x2 ld2(__amdgpu_buffer_rsrc_t b, uint32_t at) { return __builtin_bit_cast(f64x2, ld16(b, at, 0)); }

// The lane's byte offset in row tile `tile` of a column group of an operand of r4 4-row groups (rows past the
// operand's last group repeat its last row)
__device__ __forceinline__ uint32_t lane_at(int tile, int r4, int lane) {
    const int w = min(16, 4 * (r4 - 4 * tile));
    return (uint32_t)tile * 1024u + (uint32_t)((lane >> 4) * w + min(lane & 15, w - 1)) * 16u;
}

// One column group of both operands: P's tiles at byte po[i], Q's at qo[i]; n = k steps that hold data (0: past
// the last group)
struct Group { __amdgpu_buffer_rsrc_t p, q; int n; };

// acc[i][j] += P tile i . Q tile j^T over the column groups that next(po, qo) gives, for i < np and j < nq
template <class Next>
__device__ __forceinline__ void multiply(f64x4 (&acc)[4][4], int np, int nq, uint32_t (&po)[4], uint32_t (&qo)[4], Next&& next) {
    f64x2 p[2][4], q[2][4];
    int n[2];
    each<2>([&](auto b) {
        const Group G = next();
        each<4>([&](auto i) { p[b][i] = ld2(G.p, po[i]); });
        each<4>([&](auto i) { q[b][i] = ld2(G.q, qo[i]); });
        n[b] = G.n;
        fence();
    });
    for (;;) {
        bool more = true;
        each<2>([&](auto bb) {
            constexpr int b = bb;
            if (!more) return;
            if (n[b] == 0) {
                more = false;
                return;
            }
            const Group G = next();
            each<4>([&](auto ii) {
                constexpr int i = ii;
                each<4>([&](auto jj) {
                    constexpr int j = jj;
                    // consecutive MFMAs accumulate into the same registers (the fast path of the matrix core)
                    if (i < np && j < nq) {
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[b][i][0], q[b][j][0], acc[i][j], 0, 0, 0);
                        if (n[b] > 1) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[b][i][1], q[b][j][1], acc[i][j], 0, 0, 0);
                    }
                    if constexpr (i == 3) {
                        fence();
                        q[b][j] = ld2(G.q, qo[j]);
                        fence();
                    }
                });
                fence();
                p[b][i] = ld2(G.p, po[i]);
                fence();
            });
            n[b] = G.n;
        });
        if (!more) break;
    }
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

// psi block X (m_a x m_d) -> X^T in operand form (m_d rows, m_a columns) at dst_off; clears the block of y (a
// launch of its own took a tenth of the smallest matvecs)
__global__ void k_pack_xt64(const PackBlock* __restrict__ packs, const double* __restrict__ x, double* __restrict__ xt,
                            double* __restrict__ y) {
    const PackBlock P = packs[blockIdx.x];
    if (y) {
        const int64_t len = (int64_t)P.m_a * P.m_d;
        for (int64_t e = threadIdx.x; e < len; e += blockDim.x) y[P.src_off + e] = 0.0;
    }
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
__global__ __launch_bounds__(64, 2) void k_big64_t(const BigT* __restrict__ work, const double* __restrict__ ops,
                                                   const double* __restrict__ xt, double* __restrict__ tbuf,
                                                   const int32_t* __restrict__ mask) {
    const BigT* wp = work + blockIdx.x;
    const int ka4 = uni(wp->ka), kd4 = uni(wp->kd), ra4 = uni(wp->ra), pd = uni(wp->pd);
    if (ka4 == 0) return;                                      // filler
    if (mask && mask[uni(wp->part)] != kPartActive) return;
    const int rb = uni(wp->rb), nr = uni(wp->nr), jb = uni(wp->jb), nj = uni(wp->nj);
    const int lane = threadIdx.x;
    const double* x = xt + uni64(wp->xt);
    const double* a = ops + uni64(wp->a);
    f64x4 acc[4][4];
    uint32_t xo[4], ao[4];
    each<4>([&](auto i) {
        each<4>([&](auto j) { acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0}; });
        xo[i] = i < nj ? lane_at(jb + i, kd4, lane) : kNowhere;
        ao[i] = i < nr ? lane_at(rb + i, ra4, lane) : kNowhere;
    });
    int left = ka4;                                            // k steps from the next group on
    multiply(acc, nj, nr, xo, ao, [&]() {
        const Group G{buf(x, left > 0 ? kd4 * 256 : 0), buf(a, left > 0 ? ra4 * 256 : 0), max(0, min(2, left))};
        x += (int64_t)kd4 * 32;
        a += (int64_t)ra4 * 32;
        left -= 2;
        return G;
    });
    // acc[jj][rr][v] = T'^T[j 16 jt + g + 4 v][r 16 rt + li] = T tile (rt, jt), lane value v
    const double f = unid(wp->f);
    double* to = tbuf + uni64(wp->t) + ((int64_t)rb * pd + jb) * kTileD + lane * 2;
    each<4>([&](auto jj) {
        each<4>([&](auto rr) {
            if (jj < nj && rr < nr) {
                const f64x4 v = acc[jj][rr] * f;
                double* tile = to + (int64_t)(rr * pd + jj) * kTileD;
                *reinterpret_cast<f64x2*>(tile) = f64x2{v[0], v[1]};
                *reinterpret_cast<f64x2*>(tile + kTileD / 2) = f64x2{v[2], v[3]};
            }
        });
    });
}

// ------------------------------------------------------------------ pass 2: Y += sum T B^T
__global__ __launch_bounds__(64, 2) void k_big64_y(const Item* __restrict__ items, const BigT2* __restrict__ tasks,
                                                   const double* __restrict__ ops, const double* __restrict__ tbuf,
                                                   double* __restrict__ y, double* __restrict__ part,
                                                   const int32_t* __restrict__ mask) {
    const Item* ip = items + blockIdx.x;
    int task = uni(ip->t_begin);
    const int t_end = uni(ip->t_end);
    if (task >= t_end) return;                                 // filler
    if (mask && mask[uni(ip->part)] != kPartActive) return;
    const int m_ap = uni(ip->m_ap), m_dp = uni(ip->m_dp), rb = uni(ip->r0) >> 4, qb = uni(ip->c0) >> 4;
    const int nr = part_len((m_ap + 15) >> 4, rb, 4), nq = part_len((m_dp + 15) >> 4, qb, 4), rb4 = (m_dp + 3) >> 2;
    const int lane = threadIdx.x;
    f64x4 acc[4][4];
    uint32_t to[4], bo[4];
    each<4>([&](auto i) {
        each<4>([&](auto j) { acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0}; });
        bo[i] = i < nq ? lane_at(qb + i, rb4, lane) : kNowhere;
    });
    const double *t = nullptr, *b = nullptr;
    int left = 0;                                              // k steps of the task from the next group on
    multiply(acc, nr, nq, to, bo, [&]() {
        if (left <= 0 && task < t_end) {
            const BigT2* tp = tasks + task++;
            const int pd = uni(tp->pd32);
            left = uni(tp->kd);
            t = tbuf + uni64(tp->t) + (int64_t)rb * pd * kTileD;
            b = ops + uni64(tp->b);
            each<4>([&](auto i) { to[i] = i < nr ? (uint32_t)(i * pd) * 2048u + (uint32_t)lane * 16u : kNowhere; });
        }
        const Group G{buf(t, left > 0 ? 0x7fffffff : 0), buf(b, left > 0 ? rb4 * 256 : 0), max(0, min(2, left))};
        t += kTileD / 2;
        b += (int64_t)rb4 * 32;
        left -= 2;
        return G;
    });
    // acc[rr][qq][v] = Y[16 rt + g + 4 v][16 q + li]
    const int64_t y_off = uni64(ip->y_off), part_off = uni64(ip->part_off);
    const int li = lane & 15, g = lane >> 4, tn = 16 * nq;
    if (part_off >= 0) {
        double* dst = part + part_off + g * tn + li;
        each<4>([&](auto rr) {
            each<4>([&](auto qq) {
                if (rr < nr && qq < nq) each<4>([&](auto i) { constexpr int v = i; dst[(16 * rr + 4 * v) * tn + 16 * qq] = acc[rr][qq][v]; });
            });
        });
        return;
    }
    each<4>([&](auto rr) {
        if (rr >= nr) return;
        // one row tile of Y: what lies outside the block is neither read nor written
        const int rt = rb + rr;
        const __amdgpu_buffer_rsrc_t out = buf(y + y_off + (int64_t)rt * 16 * m_dp, min(16, m_ap - 16 * rt) * m_dp * 8);
        auto at = [&](int q, int v) { return (int)(16 * q + li < m_dp ? (uint32_t)((g + 4 * v) * m_dp + 16 * q + li) * 8u : kNowhere); };
        f64x4 old[4];
        each<4>([&](auto qq) {
            if (qq < nq) each<4>([&](auto i) {
                constexpr int v = i;
                old[qq][v] = __builtin_bit_cast(double, (i32x2)__builtin_amdgcn_raw_buffer_load_b64(out, at(qb + qq, v), 0, 0));
            });
        });
        each<4>([&](auto qq) {
            if (qq < nq) each<4>([&](auto i) {
                constexpr int v = i;
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, old[qq][v] + acc[rr][qq][v]), out, at(qb + qq, v), 0, 0);
            });
        });
    });
}

hipError_t launch_pack_xt64(const PackBlock* packs, int n_packs, const double* x, double* xt, double* y, hipStream_t s) {
    if (n_packs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_xt64, dim3(n_packs), dim3(256), 0, s, packs, x, xt, y);
    return hipGetLastError();
}

hipError_t launch_hpsi_big64(const BigPlan& P, const double* ops, const double* xt, double* y, hipStream_t s,
                             const int32_t* active) {
    if (P.n_chunks == 0) return hipSuccess;
    const double* tb = reinterpret_cast<const double*>(P.tbuf);
    for (int c = 0; c < P.n_chunks; ++c) {
        const BigChunk& C = P.chunks[c];
        if (C.t1_end > C.t1_begin)
            hipLaunchKernelGGL(k_big64_t, dim3(C.t1_end - C.t1_begin), dim3(64), 0, s, P.t1 + C.t1_begin, ops, xt,
                               reinterpret_cast<double*>(P.tbuf), active);
        if (C.item_end > C.item_begin)
            hipLaunchKernelGGL(k_big64_y, dim3(C.item_end - C.item_begin), dim3(64), 0, s, P.items + C.item_begin, P.t2,
                               ops, tb, y, P.partial, active);
        const hipError_t e = launch_reduce_partials(P.reduces + C.red_begin, C.red_end - C.red_begin, P.red_chunks,
                                                    P.partial, y, s, active);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

}  // namespace dmrg
