"""The exact sums of csrc/exact_sum.h on the host.

Reductions: every lane a thread, a workgroup's shared memory static, lanes exchanging
through their wave's barrier, built with g++ under the thread sanitizer.  Two sums of a
kernel may follow each other with nothing between (a leading reduce_partials, then
write_partial), so no wave may reach memory that another one still reads.

Accuracy: a thread's running sum and the sums of whole waves against double-double.
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
            Sum s;
            s.product(t + 1.0, 1.0);
            write_partial<T>(out.data(), s);
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
    if "unexpected memory mapping" in out.stderr:  # the sanitizer's shadow wants a fixed layout
        out = subprocess.run(["setarch", "-R", str(exe)], capture_output=True, text=True, timeout=120)
    assert "data race" not in out.stderr, out.stderr[:4000]
    assert out.returncode == 0 and out.stdout.strip() == "OK", out.stdout + out.stderr[:4000]


ACCURACY = r"""
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>
#include "exact_sum.h"
thread_local uint3_t threadIdx, blockIdx, gridDim;
pthread_barrier_t group_bar, wave_bar[16];
int lanes[1024], lanes2[1024];
using namespace ftk;
typedef __float128 Q;

// double-double with the products' errors summed apart, one renormalisation a product
struct Ref {
    double hi = 0, lo = 0, err = 0;
    static double two(double &a, double b)
    {
        const double s = a + b, bb = s - a, e = (a - (s - bb)) + (b - bb);
        a = s;
        return e;
    }
    void fast(double e)
    {
        const double s = hi + e;
        lo = e - (s - hi);
        hi = s;
    }
    void product(double a, double b)
    {
        const double p = a * b;
        err += std::fma(a, b, -p);
        const double e = two(hi, p) + lo;
        fast(e);
    }
    void end()
    {
        const double e = two(hi, err) + lo;
        fast(e);
    }
    void add(const Ref &o)
    {
        double e = two(hi, o.hi), t = lo;
        const double f = two(t, o.lo);
        fast(e + t);
        lo += f;
        fast(lo);
    }
};

int main()
{
    std::mt19937_64 g(11);
    std::normal_distribution<double> N01;
    int bad = 0;
    const int per[] = {1, 4, 16, 64, 1024, 4096};  // complex elements of a thread
    for (int n : per) {
        const int T = n > 64 ? 8 : 64, trials = 60;
        double worst = 0, worst_ref = 0;
        for (int trial = 0; trial < trials; ++trial) {
            std::vector<Sum> s(T);
            std::vector<Ref> r(T);
            Q exact = 0, scale = 0;
            for (int t = 0; t < T; ++t) {
                for (int i = 0; i < n; ++i) {
                    const double a = N01(g), b = N01(g), c = trial % 2 ? a : N01(g), d = trial % 2 ? b : N01(g);
                    s[t].product(a, c);
                    s[t].product(b, d);
                    if (i % 8 == 7) s[t].normalise();
                    r[t].product(a, c);
                    r[t].product(b, d);
                    exact += (Q)a * c + (Q)b * d;
                    scale += (Q)std::fabs(a * c) + (Q)std::fabs(b * d);
                }
                s[t].normalise();
                r[t].end();
            }
            for (int m = T / 2; m > 0; m /= 2)
                for (int t = 0; t < m; ++t) s[t].add(s[t + m].hi, s[t + m].lo, s[t + m].er), r[t].add(r[t + m]);
            const double l = s[0].low();
            worst = std::max(worst, std::fabs((double)(((Q)s[0].hi + l - exact) / scale)));
            worst_ref = std::max(worst_ref, std::fabs((double)(((Q)r[0].hi + r[0].lo - exact) / scale)));
        }
        std::printf("%d threads of %d elements: 2^%.1f, double-double 2^%.1f\n", T, n, std::log2(worst), std::log2(worst_ref));
        bad += !(worst <= 1.5 * worst_ref);
    }
    std::printf(bad ? "WRONG\n" : "OK\n");
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_sums_are_as_accurate_as_double_double(tmp_path):
    """The unrounded sum of a wave's threads with up to 4096 elements each (a thread's share at 30
    sites), normalised every eight as the pass kernels do, against renormalised double-double: the same
    rounding of the pair at the end, which alone is up to 2^-106, so no more than half as much again
    in the worst of 60."""
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_STUB)
    src = tmp_path / "acc.cpp"
    src.write_text(ACCURACY)
    exe = tmp_path / "acc"
    subprocess.run(["g++", "-std=gnu++17", "-O1", "-w", "-ffp-contract=off", "-I", str(tmp_path), "-I", CSRC, str(src), "-o",
                    str(exe), "-pthread"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip().endswith("OK"), out.stdout + out.stderr
