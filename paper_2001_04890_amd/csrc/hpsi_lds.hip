// Split-BF16 sector GEMMs of Eq. dgemm (Section 2.2.1) for sectors within 96 x 96 (gfx950).
//
// Row-mode kernel: a workgroup owns a range of the tasks Y += f * A . X . B^T of a target psi block (every
// column), sorted by source block; each of its two or three wavefronts owns two row tiles and runs the range by
// itself. A task is cut into steps, one per 32-wide column chunk jc of the source, and per step:
//   GEMM1  T'^T(:, jc) = X^T(jc, :) . A(rows)^T   A's rows stay in registers for the task
//   GEMM2  Y          += T'(:, jc) . B(:, jc)^T   GEMM1's result layout is GEMM2's A-operand layout
// X^T and B stream from the caches into registers that are loaded again, for the next step, as soon as their
// last MFMA has been issued: every load is an unconditional buffer load a whole step (up to 1152 cycles of
// MFMAs) ahead of its use. There is no barrier; the wavefronts of a workgroup read the same X^T and B and find
// them in the vector cache. LDS holds the FP64 sums, which leaves the registers to the operands.
// Operands are stored pre-tiled in fragment order (internal.h): every load is a contiguous 1 KB.
//
// What bounds it: the traffic between the L2s and the memory behind them (24 orbitals at bond dimension 1024: 10 GB
// read in the row-mode launches, 6.0 .. 6.4 TB/s in three of the four; an operator block is read once per target
// that uses it), with the 1.5 (S = 96) to 2.5 (S = 64) wavefronts per SIMD that the sums in LDS leave room for.
// That problem's matvec takes 3.63 ms; 4.55 ms when the X^T and B of one workgroup per CU were staged in LDS, with
// a barrier per task and the matrix cores busy 13 .. 21% of the time.
//
// Precision: each product a.b is a_hi b_hi + a_hi b_lo + a_lo b_hi on v_mfma_f32_16x16x32_bf16 with
// FP32 accumulation; T' is scaled by f and re-split; task results are accumulated in FP32 over at
// most kFlush tasks and then added into FP64 accumulators.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.h"
#include "internal.h"

namespace dmrg {

namespace {

constexpr int kFlush = 8;   // tasks accumulated in FP32 before the FP64 update

__device__ __forceinline__ unsigned short bf16_rne(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_f32(unsigned short h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }
// Wave-uniform values in scalar registers.
__device__ __forceinline__ float unif(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// Task descriptor held in scalar registers.
struct TD { int64_t x, a, b; float f; int pa32, pd32; };
__device__ __forceinline__ TD load_td(const LTask* __restrict__ p) {
    TD d;
    d.x = uni64(p->x_off);
    d.a = uni64(p->a_off);
    d.b = uni64(p->b_off);
    d.f = unif(p->f);
    d.pa32 = uni(p->pa32);
    d.pd32 = uni(p->pd32);
    return d;
}
struct ID { int64_t y_off, part_off; int m_ap, m_dp, r0, c0, t_begin, t_end; };
__device__ __forceinline__ ID load_item(const Item* __restrict__ p) {
    ID d;
    d.y_off = uni64(p->y_off);
    d.part_off = uni64(p->part_off);
    d.m_ap = uni(p->m_ap);
    d.m_dp = uni(p->m_dp);
    d.r0 = uni(p->r0);
    d.c0 = uni(p->c0);
    d.t_begin = uni(p->t_begin);
    d.t_end = uni(p->t_end);
    return d;
}

}  // namespace

// ------------------------------------------------------------------ operator pool -> tiled hi/lo
__global__ void k_split_tiled(const double* __restrict__ pool, const PoolBlock* __restrict__ blocks,
                              uint16_t* __restrict__ tiled) {
    const PoolBlock B = blocks[blockIdx.x];
    const int ld = B.k32 * 32;
    const int n = B.r16 * B.k32 * 64;   // lane slots
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        const int tile = e >> 6, lane = e & 63;
        const int rt = tile / B.k32, kt = tile - (tile / B.k32) * B.k32;
        const int row = rt * 16 + (lane & 15), col = kt * 32 + 8 * (lane >> 4);
        const double* src = pool + B.off + (int64_t)row * ld + col;
        u16x8 h, l;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double x = src[u];
            const unsigned short hh = bf16_rne((float)x);
            h[u] = hh;
            l[u] = bf16_rne((float)(x - (double)bf16_f32(hh)));
        }
        uint16_t* dst = tiled + 2 * B.off + (int64_t)tile * kTileU16 + lane * 8;
        *reinterpret_cast<u16x8*>(dst) = h;
        *reinterpret_cast<u16x8*>(dst + 512) = l;
    }
}

hipError_t launch_split_tiled(const double* pool, const PoolBlock* blocks, int n_blocks, uint16_t* tiled,
                              hipStream_t s) {
    if (n_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_tiled, dim3(n_blocks), dim3(256), 0, s, pool, blocks, tiled);
    return hipGetLastError();
}

// ------------------------------------------------------------------ psi -> tiled X^T (per matvec)
// Source block X (m_a x m_d, row-major in the caller's vector) -> X^T tiles: 32-row chunk jc of X^T
// (rows j = columns of X), half h2, k tile kt: lane l = (li, g) holds X^T[j][k] with
// j = 32 jc + 8 (li / 4) + li % 4 + 4 h2, k = 32 kt + 8 g + u. With this row order the GEMM1 result
// lane layout is the GEMM2 A-operand layout (see the kernel).
__global__ void k_pack_xt(const PackBlock* __restrict__ packs, const double* __restrict__ xall, int64_t n_coeff,
                          int64_t xt_size, uint16_t* __restrict__ xtall, double* __restrict__ yall) {
    const PackBlock P = packs[blockIdx.x];
    if (yall) {   // clears the block of y
        double* __restrict__ y = yall + (int64_t)blockIdx.y * n_coeff + P.src_off;
        for (int64_t e = threadIdx.x; e < (int64_t)P.m_a * P.m_d; e += blockDim.x) y[e] = 0.0;
    }
    const double* __restrict__ x = xall + (int64_t)blockIdx.y * n_coeff + P.src_off;
    uint16_t* __restrict__ xt = xtall + (int64_t)blockIdx.y * xt_size + 2 * P.dst_off;
    const int pa32 = P.pa / 32, pd32 = P.pd / 32;
    const int n = pd32 * 2 * pa32 * 64;
    for (int e = threadIdx.x; e < n; e += blockDim.x) {
        const int tile = e >> 6, lane = e & 63;
        const int kt = tile % pa32, jh = tile / pa32;
        const int jc = jh >> 1, h2 = jh & 1;
        const int li = lane & 15, g = lane >> 4;
        const int j = 32 * jc + 8 * (li >> 2) + (li & 3) + 4 * h2;
        const int k0 = 32 * kt + 8 * g;
        u16x8 h, l;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = k0 + u;
            const double v = (j < P.m_d && k < P.m_a) ? x[(int64_t)k * P.m_d + j] : 0.0;
            const unsigned short hh = bf16_rne((float)v);
            h[u] = hh;
            l[u] = bf16_rne((float)(v - (double)bf16_f32(hh)));
        }
        uint16_t* dst = xt + (int64_t)tile * kTileU16 + lane * 8;
        *reinterpret_cast<u16x8*>(dst) = h;
        *reinterpret_cast<u16x8*>(dst + 512) = l;
    }
}

// ------------------------------------------------------------------ row-mode kernel
// NR row tiles of one wavefront (see the head of the file). sum: the wavefront's FP64 sums in LDS, one
// double per lane and accumulator register.
template <int S, int NR>
__device__ __forceinline__ void rows_item(const ID& I, const LTask* __restrict__ tasks, const uint16_t* __restrict__ pool_t,
                                          const uint16_t* __restrict__ xt, double* __restrict__ y,
                                          double* __restrict__ part, int rt0, int nrt, double* sum, int lane) {
    constexpr int KS = S / 32, QS = S / 16;     // k tiles (and column chunks) of a source, column tiles of a target
    const int tq = (I.m_dp + 15) >> 4;
    const uint32_t at = (uint32_t)lane * 16u;
    auto tile = [&](__amdgpu_buffer_rsrc_t op, int byte) { return ld_frag(op, at, (uint32_t)byte); };
    auto a_op = [&](const TD& T) { return buf(pool_t + T.a, nrt * T.pa32 * 2048); };
    auto x_op = [&](const TD& T) { return buf(xt + T.x, T.pd32 * T.pa32 * 4096); };
    auto b_op = [&](const TD& T) { return buf(pool_t + T.b, tq * T.pd32 * 2048); };
    Frag a[NR][KS], x[2 * KS], b[QS];
    f32x4 c32[NR][QS];
    auto load_a = [&](const TD& T) {
        const __amdgpu_buffer_rsrc_t op = a_op(T);
        each<NR>([&](auto p) {
            each<KS>([&](auto kt) { a[p][kt] = tile(op, (kt < T.pa32 ? (rt0 + p) * T.pa32 + kt : nrt * T.pa32) * 2048); });
        });
    };
    // X^T tile (half i % 2 of column chunk jc, k tile i / 2)
    auto x_tile = [&](__amdgpu_buffer_rsrc_t op, const TD& T, int jc, int i) {
        return tile(op, ((i >> 1) < T.pa32 ? (2 * jc + (i & 1)) * T.pa32 + (i >> 1) : 2 * T.pd32 * T.pa32) * 2048);
    };
    each<NR>([&](auto p) { each<QS>([&](auto q) { c32[p][q] = f32x4{0.f, 0.f, 0.f, 0.f}; }); });

    int t = I.t_begin, jc = 0, since_flush = 0;
    bool first = true;
    TD T = load_td(tasks + t);
    TD Tn = load_td(tasks + min(t + 1, I.t_end - 1));    // the following task, one ahead
    load_a(T);
    {
        const __amdgpu_buffer_rsrc_t xo = x_op(T), bo = b_op(T);
        each<2 * KS>([&](auto i) { x[i] = x_tile(xo, T, 0, i); });
        each<QS>([&](auto q) { b[q] = tile(bo, q * T.pd32 * 2048); });
    }
    fence();
    for (;;) {
        const bool more_cols = jc + 1 < T.pd32;
        const bool new_task = !more_cols && t + 1 < I.t_end;
        // the next step (the last step's successor is its own task's first step: loaded, never used)
        const int njc = more_cols ? jc + 1 : 0;
        const TD N = new_task ? Tn : T;
        const __amdgpu_buffer_rsrc_t nxo = x_op(N), nbo = b_op(N);
        // the chains of the different accumulators alternate: an MFMA's result is not needed by the next
        f32x4 tt[2][NR];
        each<2>([&](auto h2) { each<NR>([&](auto p) { tt[h2][p] = f32x4{0.f, 0.f, 0.f, 0.f}; }); });
        each<KS>([&](auto k) {
            constexpr int kt = k;
            if (kt < T.pa32) {
                each<3>([&](auto w) {
                    constexpr int W = w;
                    each<2>([&](auto h) {
                        constexpr int h2 = h;
                        each<NR>([&](auto p) {
                            tt[h2][p] = mma<W>(x[2 * kt + h2], a[p][kt], tt[h2][p]);
                        });
                    });
                });
            }
            fence();
            each<2>([&](auto h2) { x[2 * kt + h2] = x_tile(nxo, N, njc, 2 * kt + h2); });
            fence();
        });
        // tt[h2][p][v] = T'[row 16 (rt0 + p) + li][col 32 jc + 8 g + 4 h2 + v] (unscaled); A is free now
        if (new_task) {
            fence();
            load_a(Tn);
            fence();
        }
        Frag tf[NR];
        each<NR>([&](auto p) {
            float v[8];
            each<8>([&](auto i) {
                constexpr int u = i;
                v[u] = tt[u >> 2][p][u & 3];
            });
            tf[p] = split8(T.f, v);
        });
        each<QS / 2>([&](auto qq) {
            auto gemm2 = [&](auto nq) {
                each<3>([&](auto w) {
                    constexpr int W = w;
                    each<decltype(nq)::value>([&](auto i) {
                        constexpr int q = 2 * decltype(qq)::value + i;
                        each<NR>([&](auto p) {
                            c32[p][q] = mma<W>(tf[p], b[q], c32[p][q]);
                        });
                    });
                });
            };
            if (2 * qq + 1 < tq) gemm2(std::integral_constant<int, 2>{});
            else if (2 * qq < tq) gemm2(std::integral_constant<int, 1>{});
            fence();
            each<2>([&](auto i) {
                constexpr int q = 2 * decltype(qq)::value + i;
                b[q] = tile(nbo, (q * N.pd32 + njc) * 2048);
            });
            fence();
        });
        if (!more_cols && (++since_flush == kFlush || !new_task)) {
            since_flush = 0;
            each<NR>([&](auto p) {
                each<QS>([&](auto q) {
                    each<4>([&](auto i) {
                        constexpr int v = i;
                        double* const at = sum + ((p * QS + q) * 4 + v) * 64 + lane;
                        *at = (first ? 0.0 : *at) + (double)c32[p][q][v];
                    });
                    c32[p][q] = f32x4{0.f, 0.f, 0.f, 0.f};
                });
            });
            first = false;
        }
        if (!more_cols && !new_task) break;
        jc = njc;
        if (new_task) {
            ++t;
            T = Tn;
            Tn = load_td(tasks + min(t + 1, I.t_end - 1));
        }
    }
    // store: lane (li, g) holds Y[16 (rt0 + p) + 4 g + v][16 q + li]
    const int li = lane & 15, g = lane >> 4, tn = 16 * tq;
    each<NR>([&](auto p) {
        each<QS>([&](auto q) {
            if (q < tq) each<4>([&](auto v) {
                const int row = 16 * (rt0 + p) + 4 * g + v, col = 16 * q + li;
                const double s = sum[((p * QS + q) * 4 + v) * 64 + lane];
                if (I.part_off < 0) {
                    if (row < I.m_ap && col < I.m_dp) y[I.y_off + (int64_t)row * I.m_dp + col] += s;
                } else {
                    part[I.part_off + (int64_t)row * tn + col] = s;
                }
            });
        });
    });
}

// S: largest padded dimension of the class; NW wavefronts of two row tiles
template <int S, int NW>
__global__ __launch_bounds__(NW * 64, 2) void k_hpsi_rows(const Item* __restrict__ items, const LTask* __restrict__ tasks,
                                                          const uint16_t* __restrict__ pool_t,
                                                          const uint16_t* __restrict__ xtall, double* __restrict__ yall,
                                                          double* __restrict__ partall, int64_t n_coeff, int64_t xt_size,
                                                          int64_t slot_stride, const int32_t* __restrict__ mask) {
    constexpr int kSums = 2 * (S / 16) * 4 * 64;
    __shared__ double sums[NW * kSums];
    if (mask && mask[items[blockIdx.x].part] != kPartActive) return;
    const ID I = load_item(items + blockIdx.x);
    const uint16_t* __restrict__ xt = xtall + (int64_t)blockIdx.y * xt_size;
    double* __restrict__ y = yall + (int64_t)blockIdx.y * n_coeff;
    double* __restrict__ part = partall + (int64_t)blockIdx.y * slot_stride;
    const int wave = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nrt = (I.m_ap + 15) >> 4, rt0 = 2 * wave;
    if (rt0 >= nrt) return;
    if (rt0 + 1 < nrt) rows_item<S, 2>(I, tasks, pool_t, xt, y, part, rt0, nrt, sums + wave * kSums, lane);
    else rows_item<S, 1>(I, tasks, pool_t, xt, y, part, rt0, nrt, sums + wave * kSums, lane);
}

// ------------------------------------------------------------------ task-mode kernel (small sources)
// For tasks whose source block fits one 32 x 32 tile (pa32 = pd32 = 1). One wavefront owns a row
// block of NR row tiles (every column, tq <= NQ column tiles) of a target and runs its tasks in
// order with every operand fragment read straight from global memory (1 KB coalesced per wave
// instruction); the fragments of tasks t+1 and t+2 are in flight while task t computes, and many
// independent wavefronts per CU hide the remaining latency. Results are accumulated in FP32 over kFlushT tasks
// and added into the FP64 output (y, or the item's partial tile) by read-modify-write: the item
// is the only writer of those elements in its launch.
constexpr int kFlushT = 32;

template <int NR, int NQ>
__global__ __launch_bounds__(64) void k_hpsi_small(const Item* __restrict__ items, const LTask* __restrict__ tasks,
                                                   const uint16_t* __restrict__ pool_t,
                                                   const uint16_t* __restrict__ xtall, double* __restrict__ yall,
                                                   double* __restrict__ partall, int64_t n_coeff, int64_t xt_size,
                                                   int64_t slot_stride, const int32_t* __restrict__ mask) {
    if (mask && mask[items[blockIdx.x].part] != kPartActive) return;
    const ID I = load_item(items + blockIdx.x);
    const uint16_t* __restrict__ xt = xtall + (int64_t)blockIdx.y * xt_size;
    double* __restrict__ y = yall + (int64_t)blockIdx.y * n_coeff;
    double* __restrict__ part = partall + (int64_t)blockIdx.y * slot_stride;
    const int lane = threadIdx.x & 63;
    const int rt0 = I.r0 >> 4, qt0 = I.c0 >> 4;
    const int nr = min(NR, ((I.m_ap + 15) >> 4) - rt0);
    const int tq = min(NQ, ((I.m_dp - I.c0) + 15) >> 4);
    const int tn = 16 * tq;

    // operand fragments of two tasks: A rows, X^T (two halves), B rows; row tiles past the target and column
    // tiles past tq are outside the operand, so their loads move nothing
    const uint32_t at = (uint32_t)lane * 16u;
    const int a_bytes = ((I.m_ap + 15) >> 4) * 2048, b_bytes = ((I.m_dp + 15) >> 4) * 2048;
    auto tile = [&](__amdgpu_buffer_rsrc_t op, int n) { return ld_frag(op, at, (uint32_t)n * 2048u); };
    Frag a[2][NR], x[2][2], b[2][NQ];
    auto load_ax = [&](const TD& T, Frag (&fa)[NR], Frag (&fx)[2]) {
        const __amdgpu_buffer_rsrc_t ao = buf(pool_t + T.a, a_bytes), xo = buf(xt + T.x, 4096);
        each<2>([&](auto h2) { fx[h2] = tile(xo, h2); });
        each<NR>([&](auto p) { fa[p] = tile(ao, rt0 + p); });
    };
    auto b_op = [&](const TD& T) { return buf(pool_t + T.b, b_bytes); };

    f32x4 c32[NR][NQ];
    each<NR>([&](auto p) { each<NQ>([&](auto q) { c32[p][q] = f32x4{0.f, 0.f, 0.f, 0.f}; }); });
    bool first_flush = true;
    auto flush = [&]() __attribute__((always_inline)) {
        // addresses from an opaque copy of the lane id, so they are not hoisted into the main loop
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int fli = ln & 15, fg = ln >> 4;
        each<NR>([&](auto p) {
            each<NQ>([&](auto q) {
                if (p < nr && q < tq) {
                    each<4>([&](auto i) {
                        constexpr int v = i;
                        const int row = 16 * (rt0 + p) + 4 * fg + v, col = 16 * (qt0 + q) + fli;
                        if (I.part_off < 0) {
                            if (row < I.m_ap && col < I.m_dp)
                                y[I.y_off + (int64_t)row * I.m_dp + col] += (double)c32[p][q][v];
                        } else {
                            double* d = part + I.part_off + (int64_t)(row - I.r0) * tn + (col - I.c0);
                            *d = first_flush ? (double)c32[p][q][v] : *d + (double)c32[p][q][v];
                        }
                    });
                    // keep the read-modify-writes of one tile together (bounded register use)
                    asm volatile("" ::: "memory");
                }
                c32[p][q] = f32x4{0.f, 0.f, 0.f, 0.f};
            });
        });
        first_flush = false;
    };

    int t = I.t_begin;
    const int last = I.t_end - 1;
    float f[2];
    each<2>([&](auto n) {
        const TD T = load_td(tasks + min(t + n, last));
        f[n] = T.f;
        load_ax(T, a[n], x[n]);
        const __amdgpu_buffer_rsrc_t bo = b_op(T);
        each<NQ>([&](auto q) { b[n][q] = tile(bo, qt0 + q); });
        fence();
    });
    TD N = load_td(tasks + min(t + 2, last));            // the task after next, one task ahead of its loads
    int since_flush = 0;
    for (bool more = true; more;) {
        each<2>([&](auto nn) {
            constexpr int n = nn;
            if (!more) return;
            const bool ends = t == last;
            // GEMM1: T'^T (32 x 16 per row tile) = X^T A(rows)^T, one k step (K = 32); the chains alternate
            f32x4 tt[2][NR];
            each<2>([&](auto h2) { each<NR>([&](auto p) { tt[h2][p] = f32x4{0.f, 0.f, 0.f, 0.f}; }); });
            each<3>([&](auto w) {
                constexpr int W = w;
                each<2>([&](auto h) {
                    constexpr int h2 = h;
                    each<NR>([&](auto p) {
                        tt[h2][p] = mma<W>(x[n][h2], a[n][p], tt[h2][p]);
                    });
                });
            });
            fence();
            load_ax(N, a[n], x[n]);
            fence();
            Frag tf[NR];
            each<NR>([&](auto p) {
                float v[8];
                each<8>([&](auto i) {
                    constexpr int u = i;
                    v[u] = tt[u >> 2][p][u & 3];
                });
                tf[p] = split8(f[n], v);
            });
            // GEMM2: Y += T' B^T
            const __amdgpu_buffer_rsrc_t bo = b_op(N);
            each<NQ / 2>([&](auto qq) {
                each<3>([&](auto w) {
                    constexpr int W = w;
                    each<2>([&](auto i) {
                        constexpr int q = 2 * decltype(qq)::value + i;
                        if (q < tq) each<NR>([&](auto p) {
                            c32[p][q] = mma<W>(tf[p], b[n][q], c32[p][q]);
                        });
                    });
                });
                fence();
                each<2>([&](auto i) {
                    constexpr int q = 2 * decltype(qq)::value + i;
                    b[n][q] = tile(bo, qt0 + q);
                });
                fence();
            });
            f[n] = N.f;
            N = load_td(tasks + min(t + 3, last));
            if (++since_flush == kFlushT || ends) {
                since_flush = 0;
                flush();
            }
            if (ends) more = false;
            ++t;
        });
    }
}

// y_tile += sum of its partial tiles, in item order; block (record, 256-element chunk), one element
// per thread. Bound by the latency of its loads: 16 of them are in flight at a time (issued one after
// another, a target of 100 partials waited 100 times).
__global__ void k_reduce_lds(const Reduce* __restrict__ red, const double* __restrict__ partall,
                             double* __restrict__ yall, int64_t n_coeff, int64_t part_stride,
                             const int32_t* __restrict__ mask) {
    constexpr int B = 16;
    const Reduce R = red[blockIdx.x];
    if (mask && mask[R.part] != kPartActive) return;
    const int n = R.tm * R.tn;
    const int e = blockIdx.z * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int rr = e / R.tn, cc = e - (e / R.tn) * R.tn;
    const int row = R.r0 + rr, col = R.c0 + cc;
    if (row >= R.m_ap || col >= R.m_dp) return;
    const double* __restrict__ part = partall + (int64_t)blockIdx.y * part_stride + R.part_off + e;
    double* const y = yall + (int64_t)blockIdx.y * n_coeff + R.y_off + (int64_t)row * R.m_dp + col;
    const double y0 = *y;
    double s = 0.0;
    for (int k = 0; k < R.n_parts; k += B) {
        double v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) v[u] = part[(int64_t)min(k + u, R.n_parts - 1) * n];
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (k + u < R.n_parts) s += v[u];
    }
    *y = y0 + s;
}

hipError_t launch_reduce_partials(const Reduce* reduces, int n, int chunks, const double* partial, double* y,
                                  hipStream_t s, const int32_t* active) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_lds, dim3(n, 1, chunks), dim3(256), 0, s, reduces, partial, y, (int64_t)0, (int64_t)0,
                       active);
    return hipGetLastError();
}

hipError_t launch_hpsi_lds(const LdsPlan& P, const uint16_t* pool_t, const double* x, double* y, int64_t n_coeff,
                           int nvec, bool zero_y, hipStream_t s, const int32_t* active) {
    if (P.n_packs == 0) return hipGetLastError();
    hipLaunchKernelGGL(k_pack_xt, dim3(P.n_packs, nvec), dim3(256), 0, s, P.packs, x, n_coeff, P.xt_size, P.xt,
                       zero_y ? y : nullptr);
    const int64_t ss = P.partial_size;
    for (int c = 0; c < kLdsClasses; ++c) {
        const int b = P.cls_begin[c], n = P.cls_begin[c + 1] - b;
        if (n <= 0) continue;
        const dim3 grid(n, nvec);
#define DMRG_ROWS(S, NW) hipLaunchKernelGGL((k_hpsi_rows<S, NW>), grid, dim3(NW * 64), 0, s, P.items + b, P.tasks, pool_t, \
                                            P.xt, y, P.partial, n_coeff, P.xt_size, ss, active)
        switch (c) {
            case 0: DMRG_ROWS(64, 2); break;
            case 1: DMRG_ROWS(64, 3); break;
            case 2: DMRG_ROWS(96, 2); break;
            default: DMRG_ROWS(96, 3); break;
        }
#undef DMRG_ROWS
    }
    for (int c = 0; c < kSmallClasses; ++c) {
        const int b = P.small_begin[c], n = P.small_begin[c + 1] - b;
        if (n <= 0) continue;
        const dim3 grid(n, nvec), block(64);
#define DMRG_SMALL(NR, NQ) hipLaunchKernelGGL((k_hpsi_small<NR, NQ>), grid, block, 0, s, P.items + b, P.tasks, pool_t, \
                                              P.xt, y, P.partial, n_coeff, P.xt_size, ss, active)
        switch (c) {
            case 0: DMRG_SMALL(1, 2); break;
            case 1: DMRG_SMALL(2, 2); break;
            default: DMRG_SMALL(1, 4); break;
        }
#undef DMRG_SMALL
    }
    // one launch per record kind: the records of one launch touch disjoint parts of y
    for (int k = 0; k < kReduceKinds; ++k) {
        const int nr = P.red_begin[k + 1] - P.red_begin[k];
        if (nr > 0)
            hipLaunchKernelGGL(k_reduce_lds, dim3(nr, nvec, P.red_chunks[k]), dim3(256), 0, s, P.reduces + P.red_begin[k],
                               P.partial, y, n_coeff, P.partial_size, active);
    }
    return hipGetLastError();
}

}  // namespace dmrg
