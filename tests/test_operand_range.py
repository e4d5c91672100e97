"""Addresses of the register-streamed H.psi kernels (hpsi_rs64.hip, hpsi_lds.hip), checked on the CPU.

The kernels are compiled for the host with stand-ins for the HIP names and for the buffer builtins, and run
lane by lane over work items whose tasks differ in size: every operand in turn is the last one of its array.
A buffer load is taken two ways, as the hardware checks it (lane offset + scalar offset against the buffer's
size) and as the intrinsic promises it (the lane offset alone): by both, every byte that it may touch has to
lie in the array or in the kOperandSlack bytes that the library allocates behind it. Buffer stores, and the
loads of the result, must stay inside their own buffer by both, word by word
with offsets of 32 bits. Values play no part: matrix products return their accumulator.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2001_04890_amd", "csrc")

SHIM = r"""
#pragma once
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <algorithm>
#include <type_traits>
#include <utility>
#include <vector>
#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __shared__ static
#define __launch_bounds__(...)
#define asm
#define volatile(...)
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
inline dim3 blockIdx, blockDim, threadIdx;
typedef int hipError_t;
typedef void* hipStream_t;
constexpr int hipSuccess = 0, hipErrorInvalidValue = 1;
inline hipError_t hipGetLastError() { return hipSuccess; }
template <class T> T min(T a, T b) { return a < b ? a : b; }
template <class T> T max(T a, T b) { return a > b ? a : b; }
template <class K, class... A> void launch(K k, dim3 grid, dim3 block, A... a) {
    blockDim = block;
    for (unsigned z = 0; z < grid.z; ++z) for (unsigned y = 0; y < grid.y; ++y) for (unsigned x = 0; x < grid.x; ++x)
        for (unsigned t = 0; t < block.x; ++t) { blockIdx = dim3(x, y, z); threadIdx = dim3(t, 0, 0); k(a...); }
}
#define hipLaunchKernelGGL(k, grid, block, lds, stream, ...) launch(k, grid, block, __VA_ARGS__)

struct Range { const char *begin, *end; };
inline std::vector<Range> arrays;            // operand arrays with their slack
inline long checked = 0, beyond = 0, furthest = 0;
inline void touch(const char* p, int n) {    // an operand read: inside one of the arrays
    ++checked;
    for (const Range& r : arrays) if (p >= r.begin && p + n <= r.end) return;
    ++beyond;
    for (const Range& r : arrays) if (p >= r.begin && p < r.end + (1 << 24)) furthest = std::max(furthest, (long)(p + n - r.end));
}
struct Rsrc { const char* base; uint32_t num; };
#define __amdgpu_buffer_rsrc_t Rsrc
inline Rsrc __builtin_amdgcn_make_buffer_rsrc(void* p, short, int num, int) { return Rsrc{(const char*)p, (uint32_t)num}; }
inline int __builtin_amdgcn_readfirstlane(int v) { return v; }
typedef uint32_t B128 __attribute__((ext_vector_type(4)));
typedef uint32_t B64 __attribute__((ext_vector_type(2)));
inline B128 __builtin_amdgcn_raw_buffer_load_b128(Rsrc b, int lane, int scalar, int) {
    const uint64_t sum = (uint64_t)(uint32_t)lane + (uint32_t)scalar;
    if (sum < b.num || (uint32_t)lane < b.num) touch(b.base + sum, 16);
    return B128{0, 0, 0, 0};
}
inline void word(Rsrc b, uint32_t lane, uint32_t scalar, int n) {   // n bytes of the result
    ++checked;
    const uint64_t sum = (uint64_t)lane + scalar;
    if ((sum < b.num || lane < b.num) && (sum + n > b.num || (sum & 3))) ++beyond;
}
inline B64 __builtin_amdgcn_raw_buffer_load_b64(Rsrc b, int lane, int scalar, int) {
    word(b, lane, scalar, 4);
    word(b, (uint32_t)lane + 4u, scalar, 4);
    return B64{0, 0};
}
template <class V> void __builtin_amdgcn_raw_buffer_store_b64(V, Rsrc b, int lane, int scalar, int) {
    (void)__builtin_amdgcn_raw_buffer_load_b64(b, lane, scalar, 0);
}
template <class A, class C> C __builtin_amdgcn_mfma_f64_16x16x4f64(A, A, C c, int, int, int) { return c; }
template <class A, class C> C __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, A, C c, int, int, int) { return c; }
"""

MAIN = r"""
#include "%(kernel)s"
%(more)s
#include <random>
using namespace dmrg;
static std::mt19937 rng(5);
template <class V> const typename V::value_type& pick(const V& v) { return v[rng() %% v.size()]; }
static char* const kOps = (char*)(1ull << 40);       // operands are never dereferenced
static char* const kXt = (char*)(2ull << 40);
// an operand of `bytes` bytes that ends its array, whose end is at byte `end`
static int64_t place(int64_t end, int64_t bytes) { return end - bytes; }
int main() {
    const int64_t end = 1 << 26;
    arrays = {{kOps, kOps + end + kOperandSlack}, {kXt, kXt + end + kOperandSlack}};
    const std::vector<int> sizes = {%(sizes)s};
    std::vector<double> y(256 * 256), part(256 * 256);
    for (int n = 0; n < %(items)d; ++n) {
        const int ma = pick(sizes), md = pick(sizes);
%(body)s
    }
    printf("checked %%ld beyond %%ld furthest %%ld\n", checked, beyond, furthest);
    return beyond ? 1 : 0;
}
"""

REDUCE = r"""
namespace dmrg {   // defined in hpsi_lds.hip; not reached, as no item is cut
hipError_t launch_reduce_partials(const Reduce*, int, int, const double*, double*, hipStream_t, const int32_t*) { return 0; }
}
"""

RS64 = r"""
        std::vector<LTask64> tasks;
        int ka4 = 0, kd4 = 0;
        const bool small = n % 4 == 0;                    // the class of sources within 8 x 8, too
        for (int t = 0; t < 3; ++t) {
            const int sa = small ? 1 + rng() % 8 : pick(sizes), sd = small ? 1 + rng() % 8 : pick(sizes);
            LTask64 L{};
            L.ka4 = k4_of(sa);
            L.kd4 = k4_of(sd);
            L.f = 1.0;
            L.x_off = place(end, 8 * op64_size(sd, sa)) / 8;
            L.a_off = place(end, 8 * op64_size(ma, sa)) / 8;
            L.b_off = place(end, 8 * op64_size(md, sd)) / 8;
            ka4 = std::max(ka4, L.ka4);
            kd4 = std::max(kd4, L.kd4);
            tasks.push_back(L);
        }
        const int tq = (md + 15) / 16, nrt = (ma + 15) / 16, k = rs_kclass(ka4, kd4), q = rs_qclass(tq);
        std::vector<Item> items;
        for (int rt = 0; rt < nrt; ++rt) items.push_back({0, n % 2 ? 0 : -1, ma, md, 16 * rt, 8 * k + q, 0, (int)tasks.size()});
        RsPlan64 P;
        P.items = items.data();
        P.tasks = tasks.data();
        P.partial = part.data();
        P.n_items = 1;
        const int g = std::min(rs_group(k, q) + (int)(rng() % 2), kRsGroups - 1);   // its group or the next
        for (int i = 0; i <= kRsGroups; ++i) P.begin[i] = i > g ? (int)items.size() : 0;
        launch_hpsi_rs64(P, (const double*)kOps, (const double*)kXt, y.data(), nullptr);
"""

SPLIT = r"""
        std::vector<LTask> tasks;
        const bool task_mode = n % 3 == 0;                // sources of one 32 x 32 tile
        int widest = (md + 31) / 32;
        for (int t = 0; t < 3; ++t) {
            const int sa = task_mode ? 1 + rng() % 32 : pick(sizes), sd = task_mode ? 1 + rng() % 32 : pick(sizes);
            LTask L{};
            L.pa32 = (sa + 31) / 32;
            L.pd32 = (sd + 31) / 32;
            L.f = 1.f;
            const int nrt = (ma + 15) / 16, tq = (md + 15) / 16;
            L.x_off = place(end, 4096ll * L.pa32 * L.pd32) / 2;
            L.a_off = place(end, 2048ll * nrt * L.pa32) / 2;
            L.b_off = place(end, 2048ll * tq * L.pd32) / 2;
            widest = std::max({widest, (int)L.pa32, (int)L.pd32});
            tasks.push_back(L);
        }
        const int nrt = (ma + 15) / 16, tq = (md + 15) / 16;
        std::vector<Item> items;
        LdsPlan P;
        PackBlock none{0, 0, 0, 0, 0, 0};
        static uint16_t* const xt = (uint16_t*)kXt;
        P.packs = &none;
        P.n_packs = 1;
        P.xt = xt;
        P.tasks = tasks.data();
        P.partial = part.data();
        const int64_t part_off = n % 2 ? 0 : -1;
        if (task_mode) {
            const int NQ = tq <= 2 ? 2 : 4, NR = NQ == 2 && nrt > 1 ? 2 : 1, cls = NQ == 4 ? 2 : NR - 1;
            for (int r = 0; r < nrt; r += NR)
                for (int c = 0; c < tq; c += NQ) items.push_back({0, part_off, ma, md, 16 * r, 16 * c, 0, (int)tasks.size()});
            for (int i = cls + 1; i <= kSmallClasses; ++i) P.small_begin[i] = (int)items.size();
        } else {
            const int cls = (widest <= 2 && tq <= 4 ? 0 : 2) + (nrt > kLdsRows ? 1 : 0);
            items.push_back({0, part_off, ma, md, 0, 0, 0, (int)tasks.size()});
            for (int i = cls + 1; i <= kLdsClasses; ++i) P.cls_begin[i] = 1;
        }
        P.items = items.data();
        launch_hpsi_lds(P, (const uint16_t*)kOps, y.data(), y.data(), 0, 1, false, nullptr);
"""

EDGES = (1, 3, 4, 5, 8, 9, 12, 13, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96)


CASES = {
    "hpsi_rs64.hip": (REDUCE, RS64, EDGES + (97, 111, 112, 113, 127, 128)),
    "hpsi_lds.hip": ("", SPLIT, EDGES),
}


@pytest.mark.parametrize("kernel", sorted(CASES))
def test_operand_loads_stay_in_their_arrays(tmp_path, kernel):
    more, body, sizes = CASES[kernel]
    cxx = "/opt/rocm/bin/amdclang++"
    if not os.path.exists(cxx):
        cxx = shutil.which("amdclang++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no clang (the sources use its vector types)")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(SHIM)
    src = tmp_path / "main.cpp"
    src.write_text('#include <hip/hip_runtime.h>\n' + MAIN % {
        "kernel": os.path.join(CSRC, kernel), "sizes": ", ".join(map(str, sizes)), "more": more, "items": 400, "body": body})
    exe = tmp_path / "main"
    subprocess.run([cxx, "-x", "c++", "-std=c++17", "-O0", "-w", "-I", str(tmp_path), "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, timeout=300)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(kernel, run.stdout.strip(), flush=True)
    assert run.returncode == 0, run.stdout
    assert int(run.stdout.split()[1]) > 100000
