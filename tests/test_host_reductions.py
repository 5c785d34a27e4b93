"""The workgroup reductions of csrc/exact_sum.h on the host: every lane a thread, a
workgroup's shared memory static, lanes exchanging through their wave's barrier, built
with g++ under the thread sanitizer.  Two sums of a kernel may follow each other with
nothing between (a leading reduce_partials, then write_partial), so no wave may reach
memory that another one still reads.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1802_02854_amd", "csrc")

# what exact_sum.h uses of the device language, a thread per lane
HIP_STUB = r"""
#pragma once
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <pthread.h>
#define __device__
#define __forceinline__ inline
#define __shared__ static
typedef struct stub_stream *hipStream_t;
struct double2 { double x, y; };
inline double2 make_double2(double x, double y) { return double2{x, y}; }
struct uint3_t { unsigned x, y, z; };
extern thread_local uint3_t threadIdx, blockIdx, gridDim;
extern pthread_barrier_t group_bar, wave_bar[16];
extern int lanes[1024], lanes2[1024];
inline void __syncthreads() { pthread_barrier_wait(&group_bar); }
inline void wave_sync() { pthread_barrier_wait(&wave_bar[threadIdx.x >> 6]); }
inline void __builtin_amdgcn_fence(int, const char *, const char *) {}
inline void __builtin_amdgcn_s_barrier() { __syncthreads(); }
inline int exchange(int x, unsigned from)
{
    lanes[threadIdx.x] = x;
    wave_sync();
    const int r = lanes[(threadIdx.x & ~63u) | from];
    wave_sync();
    return r;
}
inline int __builtin_amdgcn_readfirstlane(int x) { return exchange(x, 0); }
inline int __builtin_amdgcn_update_dpp(int, int x, int ctrl, int, int, bool)
{
    const unsigned l = threadIdx.x & 63u;
    const unsigned from = ctrl == 0xB1 ? l ^ 1u : ctrl == 0x4E ? l ^ 2u : ctrl == 0x141 ? l ^ 7u : l ^ 15u;
    return exchange(x, from);
}
struct two_t { int v[2]; int operator[](int i) const { return v[i]; } };
inline two_t swap_rows(int a, int b, unsigned row)
{
    const unsigned l = threadIdx.x & 63u;
    lanes[threadIdx.x] = a;
    lanes2[threadIdx.x] = b;
    wave_sync();
    const unsigned w = threadIdx.x & ~63u;
    two_t r;
    r.v[0] = l & row ? lanes2[w | (l ^ row)] : lanes[w | l];
    r.v[1] = l & row ? lanes2[w | l] : lanes[w | (l ^ row)];
    wave_sync();
    return r;
}
inline two_t __builtin_amdgcn_permlane16_swap(int a, int b, bool, bool) { return swap_rows(a, b, 16); }
inline two_t __builtin_amdgcn_permlane32_swap(int a, int b, bool, bool) { return swap_rows(a, b, 32); }
inline double __shfl_xor(double, int, int) { return 0.0; }
"""

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#include "exact_sum.h"
thread_local uint3_t threadIdx, blockIdx, gridDim;
pthread_barrier_t group_bar, wave_bar[16];
int lanes[1024], lanes2[1024];
using namespace ftk;

constexpr int T = THREADS;

int main()
{
    pthread_barrier_init(&group_bar, nullptr, T);
    for (int w = 0; w < T / 64; ++w) pthread_barrier_init(&wave_bar[w], nullptr, 64);
    const int nparts = T + 37;
    std::vector<double> in(2 * nparts), out(2), seen(T);
    double want = 0;
    for (int i = 0; i < nparts; ++i) in[2 * i] = i + 1, in[2 * i + 1] = 0, want += i + 1;
    std::vector<std::thread> ts;
    for (int t = 0; t < T; ++t)
        ts.emplace_back([&, t] {
            threadIdx = {(unsigned)t, 0, 0};
            blockIdx = {0, 0, 0};
            // as k_lanczos_b and the last pass of a step do: a leading sum, then the
            // workgroup's own partial sum, nothing between
            seen[t] = reduce_partials<T>(in.data(), nparts);
            write_partial<T>(out.data(), t + 1.0, 0.0);
        });
    for (auto &t : ts) t.join();
    int bad = out[0] + out[1] != 0.5 * T * (T + 1);
    for (double s : seen) bad += s != want;
    std::printf(bad ? "WRONG\n" : "OK\n");
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("block", [64, 256, 512])
def test_consecutive_sums_share_no_memory(tmp_path, block):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_STUB)
    src = tmp_path / "drv.cpp"
    src.write_text(DRIVER)
    exe = tmp_path / "drv"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-w", "-fsanitize=thread", f"-DTHREADS={block}", "-I", str(tmp_path),
                    "-I", CSRC, str(src), "-o", str(exe), "-pthread"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert "data race" not in out.stderr, out.stderr[:4000]
    assert out.returncode == 0 and out.stdout.strip() == "OK", out.stdout + out.stderr[:4000]
