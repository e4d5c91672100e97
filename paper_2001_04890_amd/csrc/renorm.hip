// Density matrices of the enlarged blocks and Eq. renorm_mat per sector block (Section 2.1; Section
// 2.2.2) on v_mfma_f64_16x16x4f64, FP64 throughout, every element summed in a fixed order.
//
// Operands are read from the caller's row-major, unpadded arrays; what lies outside a block is read
// inside it (clamped) and made zero where it would enter a sum. Every element is the same chain of fused
// multiply-adds in ascending order as a scalar loop: a 16x16x4 FP64 MFMA adds its four products one after
// another, so the v-th MFMA of a 16-wide k tile takes k = 16 b + 4 v + g in lane (li, g).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "internal.h"

namespace dmrg {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4 mfma(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Elements k, k + 4, k + 8, k + 12 of a row of n doubles, zero outside it. (Reading four consecutive
// elements per lane and transposing between the 16-lane rows halves the cache lines touched, but its
// permutes wait for the loads at once: 139 us against 99 in k_renorm.)
__device__ __forceinline__ f64x4 row4(const double* __restrict__ row, int k, int n) {
    f64x4 r;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double x = row[min(k + 4 * v, n - 1)];
        r[v] = k + 4 * v < n ? x : 0.0;
    }
    return r;
}

// Elements (k, j), (k + 4, j), .. of an n x ld row-major matrix, zero from row n on.
__device__ __forceinline__ f64x4 col4(const double* __restrict__ m, int k, int n, int64_t ld, int j) {
    f64x4 r;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double x = m[(int64_t)min(k + 4 * v, n - 1) * ld + j];
        r[v] = k + 4 * v < n ? x : 0.0;
    }
    return r;
}

constexpr int kRdmWaves = 4;   // 32 x 32 tiles (wavefronts) per workgroup

}  // namespace

// rho of one unit: a 32 x 32 tile (2 x 2 MFMA tiles) of one item, one wavefront each. RIGHT: the psi blocks
// are contracted over their rows.
// 4096 x 4096 states in 77 sectors are ~1e8 flops over 2 MB of psi: bound by launch and load latency, so the
// units are exact (a grid padded to the widest item spends its time dispatching empty workgroups) and the
// next k tile is loaded while one is multiplied.
template <bool RIGHT>
__global__ __launch_bounds__(kRdmWaves * 64) void k_rdm(const RdmItem* __restrict__ items, const RdmUnit* __restrict__ units,
                                                        int n_units, const int64_t* __restrict__ gblk,
                                                        const int32_t* __restrict__ inner, const double* __restrict__ psi,
                                                        double* __restrict__ rho) {
    const int u = (int)(blockIdx.x * kRdmWaves + (threadIdx.x >> 6));
    if (u >= n_units) return;
    const RdmItem it = items[units[u].item];
    const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
    const int nt2 = (it.ma2 + 31) / 32, r0 = units[u].tile / nt2 * 32, c0 = units[u].tile % nt2 * 32;
    const bool r2 = r0 + 16 < it.ma, c2 = c0 + 16 < it.ma2;       // the second row / column of tiles holds data
    const int ra = min(r0 + li, it.ma - 1), rb = min(r0 + 16 + li, it.ma - 1);
    const int ca = min(c0 + li, it.ma2 - 1), cb = min(c0 + 16 + li, it.ma2 - 1);
    f64x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i][0] = acc[i][1] = f64x4{0.0, 0.0, 0.0, 0.0};
    // (k, b): column group and 16-wide k tile
    int k = 0, b = 0, n = 0;
    const double *x = psi, *y = psi;
    auto group = [&]() {
        n = inner[it.cd + k];
        x = psi + gblk[it.g + k];
        y = psi + gblk[it.g2 + k];
    };
    struct Tile { f64x4 p[2], q[2]; };
    auto load = [&](Tile& t) {
        if constexpr (RIGHT) {
            t.p[0] = col4(x, b + g, n, it.ma, ra);
            t.p[1] = col4(x, b + g, n, it.ma, rb);
            t.q[0] = col4(y, b + g, n, it.ma2, ca);
            t.q[1] = col4(y, b + g, n, it.ma2, cb);
        } else {
            t.p[0] = row4(x + (int64_t)ra * n, b + g, n);
            t.p[1] = row4(x + (int64_t)rb * n, b + g, n);
            t.q[0] = row4(y + (int64_t)ca * n, b + g, n);
            t.q[1] = row4(y + (int64_t)cb * n, b + g, n);
        }
    };
    if (it.n_cd > 0) {
        Tile cur, nxt;
        group();
        load(cur);
        for (;;) {
            b += 16;
            if (b >= n) {
                b = 0;
                if (++k < it.n_cd) group();
            }
            const bool more = k < it.n_cd;
            nxt = cur;
            if (more) load(nxt);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc[0][0] = mfma(cur.p[0][v], cur.q[0][v], acc[0][0]);
                if (c2) acc[0][1] = mfma(cur.p[0][v], cur.q[1][v], acc[0][1]);
                if (r2) acc[1][0] = mfma(cur.p[1][v], cur.q[0][v], acc[1][0]);
                if (r2 && c2) acc[1][1] = mfma(cur.p[1][v], cur.q[1][v], acc[1][1]);
            }
            if (!more) break;
            cur = nxt;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = r0 + 16 * i + g + 4 * v, col = c0 + 16 * j + li;
                if (row < it.ma && col < it.ma2) rho[it.rho_off + (int64_t)row * it.ld + col] = acc[i][j][v];
            }
}

hipError_t launch_rdm(bool right, const RdmItem* items, const RdmUnit* units, int n_units, const int64_t* gblk,
                      const int32_t* inner, const double* psi, double* rho, hipStream_t s) {
    if (n_units <= 0) return hipSuccess;
    const dim3 grid((unsigned)((n_units + kRdmWaves - 1) / kRdmWaves)), block(kRdmWaves * 64);
    if (right) hipLaunchKernelGGL(k_rdm<true>, grid, block, 0, s, items, units, n_units, gblk, inner, psi, rho);
    else hipLaunchKernelGGL(k_rdm<false>, grid, block, 0, s, items, units, n_units, gblk, inner, psi, rho);
    return hipGetLastError();
}

// out = O_out^T A O_in of one block, for 32 columns of O_in and up to 256 of O_out per workgroup of four
// wavefronts. The rows of A go by in chunks of 128: T = A O_in of the chunk (2 x 2 tiles a wavefront) goes to
// LDS, and out += O_out(chunk)^T T adds to the accumulators (4 x 2 tiles a wavefront). No intermediate goes
// to memory (allocating and freeing 10 MB for one takes 65 us, and two passes with exact tile lists took
// 54 us beside it), and A is read once per 32 columns. The next 16 of the reduction index are loaded while
// the last are multiplied; a wavefront's chain of loads through the largest block bounds it. 8 and 16
// wavefronts for taller blocks, as launches of their own, took 174 us for 12 operators of 4096 states; one
// thread per element took 700.
__global__ __launch_bounds__(256) void k_renorm(const RenormItem* __restrict__ items, const double* __restrict__ A,
                                                const double* __restrict__ O, double* __restrict__ out) {
    constexpr int W = 4, TILES = 4;         // wavefronts; row tiles of the output per wavefront
    constexpr int ROWS = 32 * W, LD = 36;   // LDS row stride in doubles (rows g, g + 1 land 8 banks apart)
    __shared__ double t[ROWS * LD];
    const RenormItem it = items[blockIdx.x];
    const int c0 = (int)blockIdx.y * 32, o0 = (int)blockIdx.z * 16 * TILES * W;
    if (c0 >= it.k_in || o0 >= it.k_out) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
    const double *a = A + it.a_off, *oi = O + it.oi_off, *oo = O + it.oo_off;
    const int j0 = min(c0 + li, it.k_in - 1), j1 = min(c0 + 16 + li, it.k_in - 1);
    f64x4 acc[TILES][2];
#pragma unroll
    for (int q = 0; q < TILES; ++q) acc[q][0] = acc[q][1] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int rc = 0; rc < it.rows; rc += ROWS) {
        const int ra = rc + 32 * wave;      // the wavefront's 32 rows of T
        f64x4 tt[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) tt[q][0] = tt[q][1] = f64x4{0.0, 0.0, 0.0, 0.0};
        if (ra < it.rows) {
            const double* a0 = a + (int64_t)min(ra + li, it.rows - 1) * it.cols;
            const double* a1 = a + (int64_t)min(ra + 16 + li, it.rows - 1) * it.cols;
            struct Tile { f64x4 x0, x1, y0, y1; } cur, nxt;
            auto load = [&](int b, Tile& s) {   // past the last column: reads inside the block
                s.x0 = row4(a0, b + g, it.cols);
                s.x1 = row4(a1, b + g, it.cols);
                s.y0 = col4(oi, b + g, it.cols, it.k_in, j0);
                s.y1 = col4(oi, b + g, it.cols, it.k_in, j1);
            };
            load(0, cur);
            for (int b = 0; b < it.cols; b += 16) {
                load(b + 16, nxt);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    tt[0][0] = mfma(cur.x0[v], cur.y0[v], tt[0][0]);
                    tt[0][1] = mfma(cur.x0[v], cur.y1[v], tt[0][1]);
                    tt[1][0] = mfma(cur.x1[v], cur.y0[v], tt[1][0]);
                    tt[1][1] = mfma(cur.x1[v], cur.y1[v], tt[1][1]);
                }
                cur = nxt;
            }
        }
        if (rc > 0) __syncthreads();        // the previous chunk has been read
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 32 * wave + 16 * q + g + 4 * v;
                const bool in = rc + row < it.rows;   // rows past the block enter the second product as zeros
                t[row * LD + li] = in ? tt[q][0][v] : 0.0;
                t[row * LD + 16 + li] = in ? tt[q][1][v] : 0.0;
            }
        __syncthreads();
        const int rows = min(ROWS, it.rows - rc);
        if (o0 + 16 * wave < it.k_out) {
            for (int b = 0; b < rows; b += 16) {
                f64x4 t0, t1;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    t0[v] = t[(b + 4 * v + g) * LD + li];
                    t1[v] = t[(b + 4 * v + g) * LD + 16 + li];
                }
#pragma unroll
                for (int q = 0; q < TILES; ++q) {
                    const int o = o0 + 16 * (wave + W * q);
                    if (o < it.k_out) {
                        const f64x4 x = col4(oo, rc + b + g, it.rows, it.k_out, min(o + li, it.k_out - 1));
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            acc[q][0] = mfma(x[v], t0[v], acc[q][0]);
                            acc[q][1] = mfma(x[v], t1[v], acc[q][1]);
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < TILES; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = o0 + 16 * (wave + W * q) + g + 4 * v;
            if (row < it.k_out) {
                double* to = out + it.out_off + (int64_t)row * it.k_in;
                if (c0 + li < it.k_in) to[c0 + li] = acc[q][0][v];
                if (c0 + 16 + li < it.k_in) to[c0 + 16 + li] = acc[q][1][v];
            }
        }
}

// The same for a block of at most 32 rows and 32 kept states, by one wavefront: T stays in the registers in which
// the first product leaves it, which are the second one's operand, so there is no LDS and no barrier, and 16 blocks
// run on a CU, 2 of k_renorm. The sums are those of k_renorm. Bound by the latency of each block's loads (operators
// of a few dozen states are thousands of such blocks): 20,000 blocks of 9 -> 5 states take 19 us, 133 us when each had
// a workgroup of k_renorm.
__global__ __launch_bounds__(256) void k_renorm_small(const RenormItem* __restrict__ items, int n_items,
                                                      const double* __restrict__ A, const double* __restrict__ O,
                                                      double* __restrict__ out) {
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (w >= n_items) return;
    const RenormItem it = items[w];
    const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
    const double *a = A + it.a_off, *oi = O + it.oi_off, *oo = O + it.oo_off;
    const bool r2 = it.rows > 16, c2 = it.k_in > 16;           // the second tile of rows / columns holds data
    const double* a0 = a + (int64_t)min(li, it.rows - 1) * it.cols;
    const double* a1 = a + (int64_t)min(16 + li, it.rows - 1) * it.cols;
    const int j0 = min(li, it.k_in - 1), j1 = min(16 + li, it.k_in - 1);
    const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
    f64x4 tt[2][2] = {{zero, zero}, {zero, zero}};
    for (int b = 0; b < it.cols; b += 16) {
        const f64x4 x0 = row4(a0, b + g, it.cols), x1 = r2 ? row4(a1, b + g, it.cols) : zero;
        const f64x4 y0 = col4(oi, b + g, it.cols, it.k_in, j0), y1 = c2 ? col4(oi, b + g, it.cols, it.k_in, j1) : zero;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            tt[0][0] = mfma(x0[v], y0[v], tt[0][0]);
            if (c2) tt[0][1] = mfma(x0[v], y1[v], tt[0][1]);
            if (r2) tt[1][0] = mfma(x1[v], y0[v], tt[1][0]);
            if (r2 && c2) tt[1][1] = mfma(x1[v], y1[v], tt[1][1]);
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool in = 16 * q + g + 4 * v < it.rows;      // rows past the block enter the second product as zeros
            tt[q][0][v] = in ? tt[q][0][v] : 0.0;
            tt[q][1][v] = in ? tt[q][1][v] : 0.0;
        }
    for (int o = 0; o < it.k_out; o += 16) {
        const int i = min(o + li, it.k_out - 1);
        f64x4 acc[2] = {zero, zero};
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (q == 0 || r2) {
                const f64x4 x = col4(oo, 16 * q + g, it.rows, it.k_out, i);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    acc[0] = mfma(x[v], tt[q][0][v], acc[0]);
                    if (c2) acc[1] = mfma(x[v], tt[q][1][v], acc[1]);
                }
            }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = o + g + 4 * v;
            if (row < it.k_out) {
                double* to = out + it.out_off + (int64_t)row * it.k_in;
                if (li < it.k_in) to[li] = acc[0][v];
                if (16 + li < it.k_in) to[16 + li] = acc[1][v];
            }
        }
    }
}

hipError_t launch_renormalize(const RenormItem* items, int n_large, int n_small, int max_in, int max_out, const double* A,
                              const double* O, double* out, hipStream_t s) {
    if (n_large > 0) {
        const dim3 grid((unsigned)n_large, (unsigned)((max_in + 31) / 32), (unsigned)((max_out + 255) / 256));
        hipLaunchKernelGGL(k_renorm, grid, dim3(256), 0, s, items, A, O, out);
    }
    if (n_small > 0)
        hipLaunchKernelGGL(k_renorm_small, dim3((unsigned)((n_small + 3) / 4)), dim3(256), 0, s, items + n_large, n_small, A, O, out);
    return hipGetLastError();
}

}  // namespace dmrg
