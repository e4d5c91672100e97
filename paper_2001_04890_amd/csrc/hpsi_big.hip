// Split-BF16 sector GEMMs of Eq. dgemm (Section 2.2.1) for sector blocks above the row-mode kernel's classes
// (gfx950): pass 1 T'^T = X^T A^T per task, pass 2 Y += sum_tasks T B^T.
//
// A wavefront by itself owns up to 4 x 4 tiles of T'^T or of Y and reads both operands, one 32-wide k tile at a
// time, straight into registers; there is no LDS and no barrier. A k tile is 16 loads of 1 KB and 48 MFMAs
// (768 cycles); two of them are in flight, and every register is loaded again, for the k tile after next, as
// soon as its last MFMA has been issued. All loads are unconditional buffer loads (what lies outside the block
// or past the last k tile moves nothing), so the compiler knows how many are in flight.
//
// Operands are stored pre-tiled in fragment order (internal.h: 16 rows x 32 columns, hi and lo, 2 KB). The
// MFMA result layout of T'^T = X^T A^T is the A-operand layout of pass 2, so pass 1 stores its tiles of T
// without a shuffle.
//
// What bounds it: the traffic between the L2s and the last-level cache and the vector cache (16 KB per 768
// cycles and wavefront, 85 B per clock of the 64 a CU's cache delivers were the matrix cores always busy). In
// the matvec of 24 orbitals at bond dimension 1024 the path takes 1.2 ms, 1.7 ms with 128 x 128 tiles of four
// wavefronts staged through LDS, which multiplied whole tiles at the blocks' edges.
//
// Precision: each product a.b is a_hi b_hi + a_hi b_lo + a_lo b_hi on v_mfma_f32_16x16x32_bf16 with FP32
// accumulation; T is scaled by f and re-split; the results of at most kFlushBig tasks are accumulated in FP32
// and then added in FP64.
#include "device.h"
#include "internal.h"

namespace dmrg {

namespace {

constexpr int kFlushBig = 8;
constexpr int kTileBytes = 2 * kTileU16;

// One k tile of both operands: P's tiles at byte po[i], Q's at qo[i]. use: 0 past the last k tile, 1 inside a
// task, 2 a task's last k tile, 3 the last of all
struct Step { __amdgpu_buffer_rsrc_t p, q; int use; };

// acc[i][j] += P tile i . Q tile j^T over the k tiles that next() gives, for i < np and j < nq; after(use)
// follows each k tile
template <class Next, class After>
__device__ __forceinline__ void multiply(f32x4 (&acc)[4][4], int np, int nq, uint32_t (&po)[4], uint32_t (&qo)[4], Next&& next,
                                         After&& after) {
    Frag p[2][4], q[2][4];
    int use[2];
    each<2>([&](auto b) {
        const Step S = next();
        each<4>([&](auto i) { p[b][i] = ld_frag(S.p, po[i]); });
        each<4>([&](auto i) { q[b][i] = ld_frag(S.q, qo[i]); });
        use[b] = S.use;
        fence();
    });
    for (bool more = true; more;) {
        each<2>([&](auto bb) {
            constexpr int b = bb;
            if (!more) return;
            if (use[b] == 0) {
                more = false;
                return;
            }
            const Step S = next();
            each<4>([&](auto ii) {
                constexpr int i = ii;
                if (i < np) each<3>([&](auto w) {
                    // the chains of the different accumulators alternate: an MFMA's result is not needed by the next
                    each<4>([&](auto jj) {
                        constexpr int j = jj, W = decltype(w)::value;
                        if (j < nq) acc[i][j] = mma<W>(p[b][i], q[b][j], acc[i][j]);
                    });
                });
                fence();
                p[b][i] = ld_frag(S.p, po[i]);
                fence();
            });
            each<4>([&](auto j) { q[b][j] = ld_frag(S.q, qo[j]); });
            fence();
            after(use[b]);
            use[b] = S.use;
        });
    }
}

}  // namespace

// ------------------------------------------------------------------ pass 1: T = f A X per task
__global__ __launch_bounds__(64, 2) void k_big_t(const BigT* __restrict__ work, const uint16_t* __restrict__ pool_t,
                                                 const uint16_t* __restrict__ xt, uint16_t* __restrict__ tbuf,
                                                 const int32_t* __restrict__ mask) {
    const BigT* wp = work + blockIdx.x;
    const int ka = uni(wp->ka), pd = uni(wp->pd);
    if (ka == 0) return;                                       // filler
    if (mask && mask[uni(wp->part)] != kPartActive) return;
    const int rb = uni(wp->rb), nr = uni(wp->nr), jb = uni(wp->jb), nj = uni(wp->nj);
    const int lane = threadIdx.x;
    const uint16_t* x = xt + uni64(wp->xt) + (int64_t)(2 * jb) * ka * kTileU16;
    const uint16_t* a = pool_t + uni64(wp->a) + (int64_t)rb * ka * kTileU16;
    f32x4 acc[4][4];                                           // [column chunk half][row tile]
    uint32_t xo[4], ao[4];
    each<4>([&](auto i) {
        each<4>([&](auto j) { acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f}; });
        xo[i] = i < 2 * nj ? (uint32_t)(i * ka) * kTileBytes + (uint32_t)lane * 16u : kNowhere;
        ao[i] = i < nr ? (uint32_t)(i * ka) * kTileBytes + (uint32_t)lane * 16u : kNowhere;
    });
    int left = ka;                                             // k tiles from the next one on
    multiply(acc, 2 * nj, nr, xo, ao,
             [&]() {
                 const int bytes = left > 0 ? 0x7fffffff : 0;
                 const Step S{buf(x, bytes), buf(a, bytes), left > 0};
                 x += kTileU16;
                 a += kTileU16;
                 --left;
                 return S;
             },
             [](int) {});
    // acc[2 jj + h2][rr][v] = T'[row 16 rt + li][col 32 jc + 8 g + 4 h2 + v]
    const float f = (float)unid(wp->f);
    uint16_t* to = tbuf + uni64(wp->t) + ((int64_t)rb * pd + jb) * kTileU16 + lane * 8;
    each<2>([&](auto jj) {
        each<4>([&](auto rr) {
            if (jj < nj && rr < nr) {
                float v[8];
                each<8>([&](auto i) {
                    constexpr int u = i;
                    v[u] = acc[2 * jj + (u >> 2)][rr][u & 3];
                });
                const Frag t = split8(f, v);
                uint16_t* dst = to + (int64_t)(rr * pd + jj) * kTileU16;
                *reinterpret_cast<u16x8*>(dst) = t.h;
                *reinterpret_cast<u16x8*>(dst + 512) = t.l;
            }
        });
    });
}

// ------------------------------------------------------------------ pass 2: Y += sum T B^T
__global__ __launch_bounds__(64, 2) void k_big_y(const Item* __restrict__ items, const BigT2* __restrict__ tasks,
                                                 const uint16_t* __restrict__ pool_t, const uint16_t* __restrict__ tbuf,
                                                 double* __restrict__ y, double* __restrict__ part,
                                                 const int32_t* __restrict__ mask) {
    const Item* ip = items + blockIdx.x;
    int task = uni(ip->t_begin);
    const int t_end = uni(ip->t_end);
    if (task >= t_end) return;                                 // filler
    if (mask && mask[uni(ip->part)] != kPartActive) return;
    const int m_ap = uni(ip->m_ap), m_dp = uni(ip->m_dp), rb = uni(ip->r0) >> 4, qb = uni(ip->c0) >> 4;
    const int nr = part_len((m_ap + 15) >> 4, rb, 4), nq = part_len((m_dp + 15) >> 4, qb, 4);
    const int64_t y_off = uni64(ip->y_off), part_off = uni64(ip->part_off);
    const int lane = threadIdx.x;
    f32x4 acc[4][4];
    uint32_t to[4], bo[4];
    each<4>([&](auto i) { each<4>([&](auto j) { acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f}; }); });
    const uint16_t *t = nullptr, *b = nullptr;
    int left = 0, since_flush = 0;                             // k tiles of the task from the next one on; tasks since
    bool first = true;
    multiply(acc, nr, nq, to, bo,
             [&]() {
                 if (left <= 0 && task < t_end) {
                     const BigT2* tp = tasks + task++;
                     const int pd = uni(tp->pd32);
                     left = pd;
                     t = tbuf + uni64(tp->t) + (int64_t)rb * pd * kTileU16;
                     b = pool_t + uni64(tp->b) + (int64_t)qb * pd * kTileU16;
                     each<4>([&](auto i) {
                         const uint32_t at = (uint32_t)(i * pd) * kTileBytes + (uint32_t)lane * 16u;
                         to[i] = i < nr ? at : kNowhere;
                         bo[i] = i < nq ? at : kNowhere;
                     });
                 }
                 const int bytes = left > 0 ? 0x7fffffff : 0;
                 const Step S{buf(t, bytes), buf(b, bytes), left <= 0 ? 0 : left > 1 ? 1 : task < t_end ? 2 : 3};
                 t += kTileU16;
                 b += kTileU16;
                 --left;
                 return S;
             },
             [&](int use) __attribute__((always_inline)) {
                 if (use < 2 || (++since_flush < kFlushBig && use != 3)) return;
                 since_flush = 0;
                 // addresses from an opaque copy of the lane id, so that they are not held through the main loop
                 int ln = lane;
                 asm volatile("" : "+v"(ln));
                 const int li = ln & 15, g = ln >> 4, tn = 16 * nq;
                 each<4>([&](auto rr) {
                     each<4>([&](auto qq) {
                         if (rr < nr && qq < nq) {
                             each<4>([&](auto i) {
                                 constexpr int v = i;
                                 const int r = 16 * rr + 4 * g + v, c = 16 * qq + li;
                                 if (part_off < 0) {
                                     const int row = 16 * rb + r, col = 16 * qb + c;
                                     if (row < m_ap && col < m_dp) y[y_off + (int64_t)row * m_dp + col] += (double)acc[rr][qq][v];
                                 } else {
                                     double* d = part + part_off + r * tn + c;
                                     *d = first ? (double)acc[rr][qq][v] : *d + (double)acc[rr][qq][v];
                                 }
                             });
                             fence();   // the read-modify-writes of one tile stay together (bounded register use)
                         }
                         acc[rr][qq] = f32x4{0.f, 0.f, 0.f, 0.f};
                     });
                 });
                 first = false;
             });
}

hipError_t launch_hpsi_big(const BigPlan& P, const uint16_t* pool_t, const uint16_t* xt, double* y, hipStream_t s,
                           const int32_t* active) {
    for (int c = 0; c < P.n_chunks; ++c) {
        const BigChunk& C = P.chunks[c];
        if (C.t1_end > C.t1_begin)
            hipLaunchKernelGGL(k_big_t, dim3(C.t1_end - C.t1_begin), dim3(64), 0, s, P.t1 + C.t1_begin, pool_t, xt, P.tbuf,
                               active);
        if (C.item_end > C.item_begin)
            hipLaunchKernelGGL(k_big_y, dim3(C.item_end - C.item_begin), dim3(64), 0, s, P.items + C.item_begin, P.t2,
                               pool_t, P.tbuf, y, P.partial, active);
        const hipError_t e = launch_reduce_partials(P.reduces + C.red_begin, C.red_end - C.red_begin, P.red_chunks,
                                                    P.partial, y, s, active);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

}  // namespace dmrg
