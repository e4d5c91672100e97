// Learned Davidson preconditioner: kernels of the per-coefficient MLP (HIP, gfx950).
//
// Network (one MLP shared by all psi coefficients, 16 features per coefficient, see k_mlp_features):
//   h1 = relu(x W1 + b1)   W1 16 x 256
//   h2 = relu(h1 W2 + b2)  W2 256 x 256
//   m  = h2 . w3 + b3
// and the correction of Davidson's method becomes t_i = t_diag_i (1 + m_i), with t_diag the
// diagonal correction r / (theta - D) (Sections 2.1, 2.2.1). A network with w3 = b3 = 0 is exactly
// the diagonal preconditioner.
//
// Precision. The master parameters are FP32 (Adam state too). Inference and training use BF16
// copies of W1 and W2 on the matrix cores with FP32 accumulation (k_mlp_fwd_mfma); a debug mode runs
// the same network from the FP32 parameters on the vector units (k_mlp_fwd_f32).
//
// MFMA forward. One wavefront owns 64 rows (4 row tiles of 16). Both layers are computed transposed,
// H^T = W^T X^T, so the rows of the data are the N dimension of v_mfma_f32_16x16x32_bf16: after
// layer 1 lane l holds units 16u + 4(l/16) + v (v = 0..3) of row l%16 of every row tile, which is
// the B-operand layout of layer 2 once layer 2's reduction index is permuted the same way
// (slot s of lane group g in k-step q <-> unit 32q + 16(s/4) + 4g + s%4). W1 and W2 are stored
// pre-permuted (k_mlp_pack) so every A fragment is one 16-byte load, and layer 1's output never
// leaves the registers.
#include <hip/hip_runtime.h>
#include <stdint.h>


#include "mlp.h"

namespace dmrg {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// float -> bf16, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2(float a, float b) {   // (one v_cvt_pk_bf16_f32, nearest even)
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                  0, 0);
}

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

unsigned grid_of(int64_t n, int per) {
    int64_t b = (n + per - 1) / per;
    if (b > 16384) b = 16384;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

// ------------------------------------------------------------------ features
// Per chunk of one psi block: sum r^2 and u^2 (deterministic tree reduction).
__global__ __launch_bounds__(256) void k_mlp_block_sums(const MlpChunk* __restrict__ chunks, const double* __restrict__ r,
                                                        const double* __restrict__ u, double* __restrict__ part) {
    __shared__ double s0[256], s1[256];
    const MlpChunk C = chunks[blockIdx.x];
    double sr = 0.0, su = 0.0;
    for (int64_t i = C.begin + threadIdx.x; i < C.end; i += blockDim.x) {
        sr += r[i] * r[i];
        su += u[i] * u[i];
    }
    s0[threadIdx.x] = sr;
    s1[threadIdx.x] = su;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            s0[threadIdx.x] += s0[threadIdx.x + w];
            s1[threadIdx.x] += s1[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = s0[0];
        part[2 * blockIdx.x + 1] = s1[0];
    }
}

// Features of every coefficient of one chunk (layout in mlp.h).
__global__ __launch_bounds__(256) void k_mlp_features(const MlpChunk* __restrict__ chunks,
                                                      const MlpBlockInfo* __restrict__ blocks,
                                                      const double* __restrict__ part, const double* __restrict__ r,
                                                      const double* __restrict__ t, const double* __restrict__ u,
                                                      const double* __restrict__ d, double theta, MlpScales sc,
                                                      float* __restrict__ feat) {
    const MlpChunk C = chunks[blockIdx.x];
    const MlpBlockInfo B = blocks[C.block];
    double sr = 0.0, su = 0.0;
    for (int k = B.chunk_begin; k < B.chunk_end; ++k) {
        sr += part[2 * k];
        su += part[2 * k + 1];
    }
    const double cnt = (double)B.m_a * (double)B.m_d;
    const float f12 = (float)asinh(sqrt(sr / cnt) * sc.inv_r);
    const float f13 = (float)asinh(sqrt(su / cnt) * sc.inv_u);
    float oh[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        oh[k] = B.b == k ? 1.f : 0.f;
        oh[4 + k] = B.c == k ? 1.f : 0.f;
    }
    for (int64_t i = C.begin + threadIdx.x; i < C.end; i += blockDim.x) {
        float4* f = reinterpret_cast<float4*>(feat + i * kMlpIn);
        f[0] = make_float4((float)asinh(r[i] * sc.inv_r), (float)asinh(t[i] * sc.inv_t), (float)asinh(u[i] * sc.inv_u),
                           (float)asinh((d[i] - theta) * sc.inv_dt));
        f[1] = make_float4(oh[0], oh[1], oh[2], oh[3]);
        f[2] = make_float4(oh[4], oh[5], oh[6], oh[7]);
        f[3] = make_float4(f12, f13, B.lma, B.lmd);
    }
}

// out[k][:] = in[idx[k]][:] (cols floats per row)
__global__ void k_mlp_gather(const float* __restrict__ in, const int64_t* __restrict__ idx, int64_t n, int cols,
                             float* __restrict__ out) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n * cols; k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = k / cols, c = k - row * cols;
        out[k] = in[idx[row] * cols + c];
    }
}

// Training pairs of one recorded iteration at sampled coefficients i = idx[k]: a = sa t_i, b = sb v_i,
// weight w.
__global__ void k_mlp_pairs(const double* __restrict__ t, const double* __restrict__ v, const int64_t* __restrict__ idx,
                            int64_t n, double sa, double sb, float w, float* __restrict__ aux) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = idx[k];
        aux[3 * k] = (float)(sa * t[i]);
        aux[3 * k + 1] = (float)(sb * v[i]);
        aux[3 * k + 2] = w;
    }
}

// ------------------------------------------------------------------ weights
// BF16 copies: W1p / W2p in the MFMA fragment order described at the top, w2 row-major.
__global__ void k_mlp_pack(const float* __restrict__ p, uint16_t* __restrict__ w1p, uint16_t* __restrict__ w2p,
                           uint16_t* __restrict__ w2) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e < kMlpHidden * kMlpHidden) {
        // W2p[((o*8 + q)*64 + l)*8 + s] = W2[32q + 16(s/4) + 4(l/16) + s%4][16o + l%16]
        const int s = (int)(e & 7), l = (int)((e >> 3) & 63), q = (int)((e >> 9) & 7), o = (int)(e >> 12);
        const int g = l >> 4, c = l & 15;
        const int kin = 32 * q + 16 * (s >> 2) + 4 * g + (s & 3);
        w2p[e] = f32_to_bf16_bits(p[kOffW2 + kin * kMlpHidden + 16 * o + c]);
        w2[e] = f32_to_bf16_bits(p[kOffW2 + e]);
    }
    if (e < 16 * 64 * 8) {
        // W1p[(u*64 + l)*8 + s] = W1[8(l/16) + s][16u + l%16] for l/16 < 2, else 0 (K padded to 32)
        const int s = (int)(e & 7), l = (int)((e >> 3) & 63), uu = (int)(e >> 9);
        const int g = l >> 4, c = l & 15;
        w1p[e] = g < 2 ? f32_to_bf16_bits(p[(8 * g + s) * kMlpHidden + 16 * uu + c]) : (uint16_t)0;
    }
}

// ------------------------------------------------------------------ forward (BF16, matrix cores)
// m of rows row0 .. row0 + 16 RT - 1 by one wavefront, weights in LDS.
template <int RT>
__device__ __forceinline__ void mlp_rows(const u32x4* w1p, const u32x4* w2p, const float4* b1v, const float4* b2v,
                                         const float4* w3v, float b3, const float* __restrict__ feat, int64_t n, int64_t row0,
                                         int l, float* __restrict__ out, double* __restrict__ t_apply) {
    asm volatile("" ::: "memory");   // keeps the weights' reads here (the registers hold h1)
    const int g = l >> 4, c = l & 15;
    // layer-1 B operand (X^T, K padded to 32): lane holds X[row][8g .. 8g+7] for g < 2
    u32x4 xb[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int64_t row = row0 + 16 * rt + c;
        xb[rt] = u32x4{0u, 0u, 0u, 0u};
        if (g < 2 && row < n) {
            const float4* src = reinterpret_cast<const float4*>(feat + row * kMlpIn + 8 * g);
            const float4 a = src[0], b = src[1];
            xb[rt] = u32x4{pack2(a.x, a.y), pack2(a.z, a.w), pack2(b.x, b.y), pack2(b.z, b.w)};
        }
    }
    // layer 1 -> h1 as BF16 pairs: hb[u / 2][rt], halves u % 2 = units 16u + 4g + {0,1 | 2,3} of row 16rt + c
    u32x4 hb[8][RT];
#pragma unroll
    for (int uu = 0; uu < 16; ++uu) {
        const u32x4 a = w1p[uu * 64 + l];
        const float4 bb = b1v[4 * uu + g];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const f32x4 acc = mfma_bf16(a, xb[rt], f32x4{0.f, 0.f, 0.f, 0.f});
            hb[uu >> 1][rt][2 * (uu & 1)] = pack2(fmaxf(acc[0] + bb.x, 0.f), fmaxf(acc[1] + bb.y, 0.f));
            hb[uu >> 1][rt][2 * (uu & 1) + 1] = pack2(fmaxf(acc[2] + bb.z, 0.f), fmaxf(acc[3] + bb.w, 0.f));
        }
    }
    // layer 2 and the output dot product
    float part[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) part[rt] = 0.f;
#pragma unroll 1
    for (int o = 0; o < 16; ++o) {
        f32x4 acc[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const u32x4 a = w2p[(o * 8 + q) * 64 + l];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt] = mfma_bf16(a, hb[q][rt], acc[rt]);
        }
        const float4 bb = b2v[4 * o + g];
        const float4 ww = w3v[4 * o + g];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const float h0 = fmaxf(acc[rt][0] + bb.x, 0.f), h1 = fmaxf(acc[rt][1] + bb.y, 0.f);
            const float h2 = fmaxf(acc[rt][2] + bb.z, 0.f), h3 = fmaxf(acc[rt][3] + bb.w, 0.f);
            part[rt] += h0 * ww.x + h1 * ww.y + h2 * ww.z + h3 * ww.w;
        }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        float v = part[rt];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        const int64_t row = row0 + 16 * rt + c;
        if (g == 0 && row < n) {
            const float m = v + b3;
            if (out) out[row] = m;
            if (t_apply) t_apply[row] *= 1.0 + (double)m;
        }
    }
}

// Inference over many rows: one workgroup of eight wavefronts per CU keeps the weights (147 KB, W1 and W2 in
// fragment order) in LDS and takes 64 rows per wavefront at a time. 64 rows are 512 MFMAs of 16 cycles and about as many
// cycles of vector work, against 128 KB of W2: from the L2s that traffic bound the kernel (660,770 rows in
// 116 us with a wavefront per workgroup).
constexpr int kFwdWaves = 8, kFwdLds = (16 * 64 + 16 * 8 * 64) * 16 + 3 * kMlpHidden * 4;   // bytes: W1, W2, b1, b2, w3
__global__ __launch_bounds__(kFwdWaves * 64, 2) void k_mlp_fwd_mfma(const MlpDev W, const float* __restrict__ feat, int64_t n,
                                                                 float* __restrict__ out, double* __restrict__ t_apply) {
    extern __shared__ u32x4 wl[];
    u32x4 *w1p = wl, *w2p = wl + 16 * 64;
    float4 *b1v = reinterpret_cast<float4*>(w2p + 16 * 8 * 64), *b2v = b1v + kMlpHidden / 4, *w3v = b2v + kMlpHidden / 4;
    const int j = (int)threadIdx.x;
    for (int i = j; i < 16 * 64; i += kFwdWaves * 64) w1p[i] = reinterpret_cast<const u32x4*>(W.w1p)[i];
#pragma unroll 4
    for (int i = j; i < 16 * 8 * 64; i += kFwdWaves * 64) w2p[i] = reinterpret_cast<const u32x4*>(W.w2p)[i];
    if (j < kMlpHidden / 4) {
        b1v[j] = reinterpret_cast<const float4*>(W.p + kOffB1)[j];
        b2v[j] = reinterpret_cast<const float4*>(W.p + kOffB2)[j];
        w3v[j] = reinterpret_cast<const float4*>(W.p + kOffW3)[j];
    }
    const int l = j & 63;
    const float b3 = W.p[kOffB3];
    __syncthreads();
    // whole rounds of 64 rows per wavefront, then what is left in pieces of 16 (a round of few 64-row chunks
    // would take as long as a full one)
    const int64_t stride = (int64_t)gridDim.x * kFwdWaves, first = (int64_t)(j >> 6) * gridDim.x + blockIdx.x;
    const int64_t rounds = n / (64 * stride);
    for (int64_t k = 0; k < rounds; ++k)
        mlp_rows<4>(w1p, w2p, b1v, b2v, w3v, b3, feat, n, 64 * (first + k * stride), l, out, t_apply);
    for (int64_t row0 = 64 * stride * rounds + 16 * first; row0 < n; row0 += 16 * stride)
        mlp_rows<1>(w1p, w2p, b1v, b2v, w3v, b3, feat, n, row0, l, out, t_apply);
}

// Minibatches (TRAIN: keeping the hidden activations) and small inference calls: 16 rows per workgroup of four
// wavefronts, which each compute layer 1 for themselves and a quarter of layer 2's units; the output's terms
// meet in LDS and are added in unit order, so m is that of k_mlp_fwd_mfma bit for bit. 4096 rows are 256
// workgroups here; as 64 wavefronts of 64 rows, each walking all of W2 alone, they took 38 us.
template <bool TRAIN>
__global__ __launch_bounds__(256) void k_mlp_fwd_rows(const MlpDev W, const float* __restrict__ feat, int64_t n,
                                                      float* __restrict__ out, float* __restrict__ h1o,
                                                      float* __restrict__ h2o, double* __restrict__ t_apply) {
    __shared__ float terms[16][64];
    const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, c = l & 15;
    const int64_t row = (int64_t)blockIdx.x * 16 + c;
    const u32x4* w1p = reinterpret_cast<const u32x4*>(W.w1p);
    const u32x4* w2p = reinterpret_cast<const u32x4*>(W.w2p);
    const float4* b1v = reinterpret_cast<const float4*>(W.p + kOffB1);
    const float4* b2v = reinterpret_cast<const float4*>(W.p + kOffB2);
    const float4* w3v = reinterpret_cast<const float4*>(W.p + kOffW3);
    u32x4 w2f[4][8];                                   // the wavefront's quarter of W2
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 8; ++q) w2f[i][q] = w2p[((4 * wave + i) * 8 + q) * 64 + l];
    u32x4 xb = u32x4{0u, 0u, 0u, 0u};
    if (g < 2 && row < n) {
        const float4* src = reinterpret_cast<const float4*>(feat + row * kMlpIn + 8 * g);
        const float4 a = src[0], b = src[1];
        xb = u32x4{pack2(a.x, a.y), pack2(a.z, a.w), pack2(b.x, b.y), pack2(b.z, b.w)};
    }
    uint32_t h1p[16][2];
#pragma unroll
    for (int uu = 0; uu < 16; ++uu) {
        const float4 bb = b1v[4 * uu + g];
        const f32x4 acc = mfma_bf16(w1p[uu * 64 + l], xb, f32x4{0.f, 0.f, 0.f, 0.f});
        const float h0 = fmaxf(acc[0] + bb.x, 0.f), h1 = fmaxf(acc[1] + bb.y, 0.f);
        const float h2 = fmaxf(acc[2] + bb.z, 0.f), h3 = fmaxf(acc[3] + bb.w, 0.f);
        h1p[uu][0] = pack2(h0, h1);
        h1p[uu][1] = pack2(h2, h3);
        if (TRAIN && (uu >> 2) == wave && row < n)
            *reinterpret_cast<float4*>(h1o + row * kMlpHidden + 16 * uu + 4 * g) = make_float4(h0, h1, h2, h3);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int o = 4 * wave + i;
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 8; ++q)
            acc = mfma_bf16(w2f[i][q], u32x4{h1p[2 * q][0], h1p[2 * q][1], h1p[2 * q + 1][0], h1p[2 * q + 1][1]}, acc);
        const float4 bb = b2v[4 * o + g];
        const float4 ww = w3v[4 * o + g];
        const float h0 = fmaxf(acc[0] + bb.x, 0.f), h1 = fmaxf(acc[1] + bb.y, 0.f);
        const float h2 = fmaxf(acc[2] + bb.z, 0.f), h3 = fmaxf(acc[3] + bb.w, 0.f);
        terms[o][l] = h0 * ww.x + h1 * ww.y + h2 * ww.z + h3 * ww.w;
        if (TRAIN && row < n) *reinterpret_cast<float4*>(h2o + row * kMlpHidden + 16 * o + 4 * g) = make_float4(h0, h1, h2, h3);
    }
    __syncthreads();
    if (wave > 0) return;
    float v = 0.f;
#pragma unroll
    for (int o = 0; o < 16; ++o) v += terms[o][l];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (g == 0 && row < n) {
        const float m = v + W.p[kOffB3];
        if (out) out[row] = m;
        if (t_apply) t_apply[row] *= 1.0 + (double)m;
    }
}

// ------------------------------------------------------------------ forward (FP32 debug mode)
// 64 rows per workgroup of 256 threads; thread j owns hidden unit j of both layers.
constexpr int kRows = 64;

template <bool TRAIN>
__global__ __launch_bounds__(256) void k_mlp_fwd_f32(const MlpDev W, const float* __restrict__ feat, int64_t n,
                                                     float* __restrict__ out, float* __restrict__ h1o,
                                                     float* __restrict__ h2o, double* __restrict__ t_apply) {
    __shared__ float X[kRows][kMlpIn + 1];
    __shared__ float H1[kRows][kMlpHidden + 1];
    __shared__ float R[kRows][4];
    const int j = threadIdx.x;
    const int64_t row0 = (int64_t)blockIdx.x * kRows;
    for (int e = j; e < kRows * kMlpIn; e += blockDim.x) {
        const int r = e / kMlpIn, c = e % kMlpIn;
        X[r][c] = row0 + r < n ? feat[(row0 + r) * kMlpIn + c] : 0.f;
    }
    float w1[kMlpIn];
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) w1[k] = W.p[k * kMlpHidden + j];
    const float b1 = W.p[kOffB1 + j], b2 = W.p[kOffB2 + j], w3 = W.p[kOffW3 + j];
    __syncthreads();
    for (int r = 0; r < kRows; ++r) {
        float z = b1;
#pragma unroll
        for (int k = 0; k < kMlpIn; ++k) z += X[r][k] * w1[k];
        const float h = fmaxf(z, 0.f);
        H1[r][j] = h;
        if (TRAIN && row0 + r < n) h1o[(row0 + r) * kMlpHidden + j] = h;
    }
    __syncthreads();
    const int wave = j >> 6, lane = j & 63;
    for (int r = 0; r < kRows; ++r) {
        float z = b2;
        for (int k = 0; k < kMlpHidden; ++k) z += H1[r][k] * W.p[kOffW2 + k * kMlpHidden + j];
        const float h = fmaxf(z, 0.f);
        if (TRAIN && row0 + r < n) h2o[(row0 + r) * kMlpHidden + j] = h;
        float v = h * w3;
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) R[r][wave] = v;
    }
    __syncthreads();
    if (j < kRows && row0 + j < n) {
        const float m = W.p[kOffB3] + R[j][0] + R[j][1] + R[j][2] + R[j][3];
        if (out) out[row0 + j] = m;
        if (t_apply) t_apply[row0 + j] *= 1.0 + (double)m;
    }
}

// ------------------------------------------------------------------ backward
// loss = (1/B) sum_r w_r (a_r (1 + m_r) - b_r)^2 over the B rows of the minibatch.
// Per row: g = dloss/dm, d2 = g w3 [h2 > 0], d1 = (d2 W2^T) [h1 > 0].
// The contractions run on v_mfma_f32_16x16x4_f32 (FP32 throughout), which adds its four products one after
// another, so every sum is the same chain of fused multiply-adds as a scalar loop over its index.
//
// Workgroup: 64 rows (four wavefronts of 16) and 64 of layer 1's units (blockIdx.y; the first column writes
// g and the loss). D2 and the units' rows of W2 are staged in LDS as FP32.
__global__ __launch_bounds__(256) void k_mlp_backward(const MlpDev W, const float* __restrict__ aux,
                                                      const float* __restrict__ m, const float* __restrict__ h1,
                                                      const float* __restrict__ h2, int64_t n, float inv_b,
                                                      float* __restrict__ g_out, float* __restrict__ d1,
                                                      float* __restrict__ d2, float* __restrict__ loss_part) {
    __shared__ float D2[kRows][kMlpHidden + 1];
    __shared__ float W2[64][kMlpHidden + 1];
    __shared__ float G[kRows];
    __shared__ float Lp[kRows];
    const int j = threadIdx.x, cg = (int)blockIdx.y;
    const int64_t row0 = (int64_t)blockIdx.x * kRows;
    if (j < kRows) {
        float gg = 0.f, ll = 0.f;
        if (row0 + j < n) {
            const float a = aux[3 * (row0 + j)], b = aux[3 * (row0 + j) + 1], w = aux[3 * (row0 + j) + 2];
            const float e = a * (1.f + m[row0 + j]) - b;
            gg = 2.f * inv_b * w * a * e;
            ll = inv_b * w * e * e;
            if (cg == 0) g_out[row0 + j] = gg;
        }
        G[j] = gg;
        Lp[j] = ll;
    }
    const float w3 = W.p[kOffW3 + j];
    if (W.fp32) {
#pragma unroll 16
        for (int u = 0; u < 64; ++u) W2[u][j] = W.p[kOffW2 + (64 * cg + u) * kMlpHidden + j];
    } else {
#pragma unroll 32
        for (int u = 0; u < 64; ++u) W2[u][j] = bf16_bits_to_f32(W.w2[(64 * cg + u) * kMlpHidden + j]);
    }
    __syncthreads();
#pragma unroll 32
    for (int r = 0; r < kRows; ++r) {
        const int64_t row = row0 + r, rc = row < n ? row : n - 1;
        D2[r][j] = h2[rc * kMlpHidden + j];
    }
#pragma unroll 8
    for (int r = 0; r < kRows; ++r) {
        const int64_t row = row0 + r;
        const float v = row < n && D2[r][j] > 0.f ? G[r] * w3 : 0.f;
        if (row < n && (j >> 6) == cg) d2[row * kMlpHidden + j] = v;
        D2[r][j] = v;
    }
    __syncthreads();
    const int wave = j >> 6, l = j & 63, li = l & 15, g = l >> 4;
    f32x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int q = 0; q < kMlpHidden; q += 4) {
        const float a = D2[16 * wave + li][q + g];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = mfma_f32(a, W2[16 * t + li][q + g], acc[t]);
    }
    // acc[t][v] = d1 before its mask at row 16 wave + 4 g + v, unit 64 cg + 16 t + li
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t row = row0 + 16 * wave + 4 * g + v, at = row * kMlpHidden + 64 * cg + 16 * t + li;
            if (row < n) d1[at] = h1[at] > 0.f ? acc[t][v] : 0.f;
        }
    if (j == 0 && cg == 0) {
        float s = 0.f;
        for (int r = 0; r < kRows; ++r) s += Lp[r];
        loss_part[blockIdx.x] = s;
    }
}

// Parameter gradients, each a sum over the minibatch rows in row order:
//   dW1[k][j] = sum_r x[r][k] d1[r][j], db1 = sum d1, dW2[k][j] = sum_r h1[r][k] d2[r][j], db2 = sum d2,
//   dw3[j] = sum_r g[r] h2[r][j], db3 = sum g,
// and the loss, the sum of its workgroup parts. Workgroup: a 32 x 32 tile of a product left^T right over the
// rows (2 x 2 MFMA tiles, one a wavefront), where left is h1, [x | 1], 1 or g and right d2, d1, h2, g or the
// parts. Bound by the chain of n / 4 MFMAs of 32 cycles (14 us at n = 4096), if the rows arrive in time: only
// some 90 of the CUs have a workgroup, so each keeps four stages of 128 rows in flight in its registers (loads
// of single k steps left 274 us, one thread per parameter took 1.0 ms).
constexpr int kWgStage = 128, kWgLd = 80, kWgAhead = 4;   // rows a stage; LDS row stride (rows g: 16 banks apart)
constexpr int kWgW2 = 64, kWgUnits = kWgW2 + 8 + 8 + 8 + 2;
struct WgIn {
    const float *x, *h1, *h2, *d1, *d2, *g, *loss_part;
    int64_t n;
    int n_part;
};

// KIND: 0 dW2, 1 dW1 and db1, 2 db2, 3 dw3, 4 db3, 5 the loss; k0, j0: first row and column of the tile.
// Loads go straight to registers (vectors, or the scalars g and parts); constants, zeros and the end of the
// rows come in on the way to LDS, so that nothing waits for a load before its stage.
template <int KIND>
__device__ __forceinline__ void wgrad_tile(const WgIn& in, int k0, int j0, float (*lds)[kWgStage * kWgLd],
                                           float* __restrict__ grad, float* __restrict__ loss) {
    constexpr bool VEC = KIND < 4, SCALAR = KIND >= 3;
    const int j = (int)threadIdx.x;
    const int64_t rows = KIND == 5 ? in.n_part : in.n;
    // thread j stages columns c4 .. c4 + 3 (left factor 0 .. 31, right 32 .. 63) of rows r0 + 16 i
    const int c4 = 4 * (j & 15), r0 = j >> 4;
    const bool is_left = c4 < 32, is_x = KIND == 1 && c4 < kMlpIn;
    const float* right = KIND == 1 ? in.d1 : KIND == 3 ? in.h2 : in.d2;
    const float* vec = is_x ? in.x + c4 : KIND == 0 && is_left ? in.h1 + k0 + c4 : right + j0 + (is_left ? 0 : c4 - 32);
    const int ld = is_x ? kMlpIn : kMlpHidden;
    const float* sc = KIND == 5 ? in.loss_part : in.g;
    const float one = c4 == (KIND == 1 ? kMlpIn : 0) ? 1.f : 0.f;
    constexpr int kLoads = kWgStage / 16;
    float4 vb[kWgAhead][kLoads];
    float sb[kWgAhead][kLoads];
    auto load = [&](int64_t stage, float4 (&v)[kLoads], float (&f)[kLoads]) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int64_t row = stage * kWgStage + r0 + 16 * i, r = row < rows ? row : rows - 1;
            if constexpr (VEC) v[i] = *reinterpret_cast<const float4*>(vec + r * ld);
            if constexpr (SCALAR) f[i] = sc[r];
        }
    };
    auto value = [&](int64_t row, const float4& v, float f) {
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row >= rows) return t;
        if constexpr (KIND == 0) return v;
        if constexpr (KIND == 1) { if (is_x || !is_left) return v; t.x = one; }
        if constexpr (KIND == 2) { if (!is_left) return v; t.x = one; }
        if constexpr (KIND == 3) { if (!is_left) return v; t.x = c4 == 0 ? f : 0.f; }
        if constexpr (KIND >= 4) t.x = is_left ? one : c4 == 32 ? f : 0.f;
        return t;
    };
    const int wave = j >> 6, l = j & 63, li = l & 15, g = l >> 4, ti = wave >> 1, tj = wave & 1;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const int64_t stages = (rows + kWgStage - 1) / kWgStage;
#pragma unroll
    for (int s = 0; s < kWgAhead; ++s) load(s, vb[s], sb[s]);
    for (int64_t s0 = 0; s0 < stages; s0 += kWgAhead) {
#pragma unroll
        for (int k = 0; k < kWgAhead; ++k) {       // past the last stage: zeros
            float* t = lds[k & 1];
#pragma unroll
            for (int i = 0; i < kLoads; ++i)
                *reinterpret_cast<float4*>(t + (r0 + 16 * i) * kWgLd + c4) = value((s0 + k) * kWgStage + r0 + 16 * i, vb[k][i], sb[k][i]);
            load(s0 + kWgAhead + k, vb[k], sb[k]);
            __syncthreads();                       // (the other half is read until the next barrier)
            const float *pa = t + g * kWgLd + 16 * ti + li, *pb = t + g * kWgLd + 32 + 16 * tj + li;
#pragma unroll
            for (int q = 0; q < kWgStage / 4; ++q) acc = mfma_f32(pa[4 * q * kWgLd], pb[4 * q * kWgLd], acc);
        }
    }
    // acc[v] = row 16 ti + 4 g + v, column 16 tj + li of the workgroup's tile
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = 16 * ti + 4 * g + v, col = j0 + 16 * tj + li;
        if (KIND == 0) grad[kOffW2 + (k0 + row) * kMlpHidden + col] = acc[v];
        else if (KIND == 1 && row < kMlpIn) grad[row * kMlpHidden + col] = acc[v];
        else if (KIND == 1 && row == kMlpIn) grad[kOffB1 + col] = acc[v];
        else if (KIND == 2 && row == 0) grad[kOffB2 + col] = acc[v];
        else if (KIND == 3 && row == 0) grad[kOffW3 + col] = acc[v];
        else if (KIND >= 4 && row == 0 && col == 0) *(KIND == 4 ? grad + kOffB3 : loss) = acc[v];
    }
}

__global__ __launch_bounds__(256) void k_mlp_wgrad(const WgIn in, float* __restrict__ grad, float* __restrict__ loss) {
    __shared__ __attribute__((aligned(16))) float lds[2][kWgStage * kWgLd];
    const int u = (int)blockIdx.x, j0 = 32 * (u & 7);
    if (u < kWgW2) wgrad_tile<0>(in, 32 * (u >> 3), j0, lds, grad, loss);
    else if (u < kWgW2 + 8) wgrad_tile<1>(in, 0, j0, lds, grad, loss);
    else if (u < kWgW2 + 16) wgrad_tile<2>(in, 0, j0, lds, grad, loss);
    else if (u < kWgW2 + 24) wgrad_tile<3>(in, 0, j0, lds, grad, loss);
    else if (u == kWgUnits - 2) wgrad_tile<4>(in, 0, 0, lds, grad, loss);
    else wgrad_tile<5>(in, 0, 0, lds, grad, loss);
}

// Adam (bias-corrected moments) on the FP32 parameters.
__global__ void k_mlp_adam(float* __restrict__ p, const float* __restrict__ grad, float* __restrict__ m1,
                           float* __restrict__ m2, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= kMlpParams) return;
    const float gg = grad[i];
    const float a = b1 * m1[i] + (1.f - b1) * gg;
    const float v = b2 * m2[i] + (1.f - b2) * gg * gg;
    m1[i] = a;
    m2[i] = v;
    p[i] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
}

// ------------------------------------------------------------------ launchers
hipError_t launch_mlp_features(const MlpChunk* chunks, int n_chunks, const MlpBlockInfo* blocks, double* part,
                               const double* r, const double* t, const double* u, const double* d, double theta,
                               const MlpScales& sc, float* feat, hipStream_t s) {
    if (n_chunks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_block_sums, dim3(n_chunks), dim3(256), 0, s, chunks, r, u, part);
    hipLaunchKernelGGL(k_mlp_features, dim3(n_chunks), dim3(256), 0, s, chunks, blocks, part, r, t, u, d, theta, sc,
                       feat);
    return hipGetLastError();
}

hipError_t launch_mlp_gather(const float* in, const int64_t* idx, int64_t n, int cols, float* out, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_gather, dim3(grid_of(n * cols, 256)), dim3(256), 0, s, in, idx, n, cols, out);
    return hipGetLastError();
}

hipError_t launch_mlp_pairs(const double* t, const double* v, const int64_t* idx, int64_t n, double sa, double sb,
                            float w, float* aux, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_pairs, dim3(grid_of(n, 256)), dim3(256), 0, s, t, v, idx, n, sa, sb, w, aux);
    return hipGetLastError();
}

hipError_t launch_mlp_pack(const float* p, uint16_t* w1p, uint16_t* w2p, uint16_t* w2, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_pack, dim3(kMlpHidden * kMlpHidden / 256), dim3(256), 0, s, p, w1p, w2p, w2);
    return hipGetLastError();
}

constexpr int kCus = 256;
// From here on inference keeps the weights in LDS: filling 147 KB costs 12 us, below 11 us the row kernel is
// done (700 rows: 4.5 us against 11.9; 16,384: 11.3 against 12.5; 32,768: 20.1 against 12.8).
constexpr int64_t kLdsRows = 18000;

hipError_t launch_mlp_forward(const MlpDev& W, const float* feat, int64_t n, float* out, float* h1, float* h2,
                              double* t_apply, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const bool train = h1 != nullptr;
    if (W.fp32) {
        const unsigned nb = (unsigned)((n + kRows - 1) / kRows);
        if (train)
            hipLaunchKernelGGL(k_mlp_fwd_f32<true>, dim3(nb), dim3(256), 0, s, W, feat, n, out, h1, h2, t_apply);
        else
            hipLaunchKernelGGL(k_mlp_fwd_f32<false>, dim3(nb), dim3(256), 0, s, W, feat, n, out, h1, h2, t_apply);
    } else {
        // the row kernel reads W2 once per 16 rows from the L2s, the other fills 144 KB of LDS first
        const unsigned nr = (unsigned)((n + 15) / 16);
        if (train) {
            hipLaunchKernelGGL(k_mlp_fwd_rows<true>, dim3(nr), dim3(256), 0, s, W, feat, n, out, h1, h2, t_apply);
        } else if (n < kLdsRows) {
            hipLaunchKernelGGL(k_mlp_fwd_rows<false>, dim3(nr), dim3(256), 0, s, W, feat, n, out, nullptr, nullptr, t_apply);
        } else {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_mlp_fwd_mfma),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kFwdLds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_mlp_fwd_mfma, dim3(kCus), dim3(kFwdWaves * 64), kFwdLds, s, W, feat, n, out, t_apply);
        }
    }
    return hipGetLastError();
}

int mlp_loss_parts(int64_t n) { return (int)((n + kRows - 1) / kRows); }

hipError_t launch_mlp_backward(const MlpDev& W, const float* aux, const float* m, const float* h1, const float* h2,
                               int64_t n, float* g, float* d1, float* d2, float* loss_part, hipStream_t s) {
    if (n <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mlp_backward, dim3((unsigned)mlp_loss_parts(n), kMlpHidden / 64), dim3(256), 0, s, W, aux, m, h1, h2, n,
                       1.f / (float)n, g, d1, d2, loss_part);
    return hipGetLastError();
}

hipError_t launch_mlp_wgrad(const float* x, const float* h1, const float* h2, const float* d1, const float* d2,
                            const float* g, int64_t n, const float* loss_part, float* grad, float* loss, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(kWgUnits), dim3(256), 0, s, WgIn{x, h1, h2, d1, d2, g, loss_part, n, mlp_loss_parts(n)},
                       grad, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_adam(float* p, const float* grad, float* m1, float* m2, float lr, int step, hipStream_t s) {
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_mlp_adam, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, p, grad, m1, m2, lr, b1, b2, 1e-8f,
                       c1, c2);
    return hipGetLastError();
}

}  // namespace dmrg

namespace dmrg {

// Sums of squares of r, u, t and D - theta (FP64, fixed-order reduction): part[4 * block + k], then
// out[k] = sum over blocks.
__global__ __launch_bounds__(256) void k_mlp_norms(const double* __restrict__ r, const double* __restrict__ u,
                                                   const double* __restrict__ t, const double* __restrict__ d,
                                                   double theta, int64_t n, double* __restrict__ part) {
    __shared__ double red[4][4];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double dd = d[i] - theta;
        s[0] += r[i] * r[i];
        s[1] += u[i] * u[i];
        s[2] += t[i] * t[i];
        s[3] += dd * dd;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double v = s[k];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        part[4 * blockIdx.x + k] = red[k][0] + red[k][1] + red[k][2] + red[k][3];
    }
}

__global__ void k_mlp_norms_finish(const double* __restrict__ part, int nb, double* __restrict__ out) {
    if (threadIdx.x < 4) {
        double s = 0.0;
        for (int b = 0; b < nb; ++b) s += part[4 * b + threadIdx.x];
        out[threadIdx.x] = s;
    }
}

// Loss of rows (a, b, w) at outputs m (NULL: m = 0, the diagonal preconditioner): part[block] =
// sum of w (a (1 + m) - b)^2 over the block's rows (FP64, fixed order).
__global__ __launch_bounds__(256) void k_mlp_loss(const float* __restrict__ aux, const float* __restrict__ m, int64_t n,
                                                  double* __restrict__ part) {
    __shared__ double red[4];
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double mm = m ? (double)m[i] : 0.0;
        const double e = (double)aux[3 * i] * (1.0 + mm) - (double)aux[3 * i + 1];
        s += (double)aux[3 * i + 2] * e * e;
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ void k_mlp_sum_f64(const double* __restrict__ part, int nb, double* __restrict__ out) {
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int b = 0; b < nb; ++b) s += part[b];
        out[0] = s;
    }
}

int mlp_reduce_blocks(int64_t n) {
    int64_t b = (n + 4095) / 4096;
    if (b < 1) b = 1;
    if (b > 1024) b = 1024;
    return (int)b;
}

hipError_t launch_mlp_norms(const double* r, const double* u, const double* t, const double* d, double theta,
                            int64_t n, double* part, double* out, hipStream_t s) {
    const int nb = mlp_reduce_blocks(n);
    hipLaunchKernelGGL(k_mlp_norms, dim3(nb), dim3(256), 0, s, r, u, t, d, theta, n, part);
    hipLaunchKernelGGL(k_mlp_norms_finish, dim3(1), dim3(64), 0, s, part, nb, out);
    return hipGetLastError();
}

hipError_t launch_mlp_loss(const float* aux, const float* m, int64_t n, double* part, double* out, hipStream_t s) {
    const int nb = mlp_reduce_blocks(n);
    hipLaunchKernelGGL(k_mlp_loss, dim3(nb), dim3(256), 0, s, aux, m, n, part);
    hipLaunchKernelGGL(k_mlp_sum_f64, dim3(1), dim3(64), 0, s, part, nb, out);
    return hipGetLastError();
}

}  // namespace dmrg
