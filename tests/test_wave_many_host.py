"""wave_sum_many on the host: the kernel's own source, its 64 lanes as 64
threads that meet at every exchange. For every number of values, each index
is returned only by lanes that hold that value's sum, and every value has one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <pthread.h>
#include <cstdio>
#include <thread>
#include <utility>
#include <vector>

#define __device__
#define __forceinline__ inline

namespace spx {
static thread_local int t_lane;
static double s_lanes[64];
static pthread_barrier_t s_all;
inline int lane_id() { return t_lane; }

// the partners of the device exchange: mirrored lanes at strides 8 and 4
template <int Stride, typename T>
T exchange(T v)
{
    const int partner = Stride == 8 ? t_lane ^ 15 : (Stride == 4 ? t_lane ^ 7 : t_lane ^ Stride);
    s_lanes[t_lane] = v;
    pthread_barrier_wait(&s_all);
    const T r = s_lanes[partner];
    pthread_barrier_wait(&s_all);
    return r;
}
}  // namespace spx

#include "wave_many.hpp"

// lane l holds 2^(i % 32) (l + 1) + i as value i: every sum differs
static double value(int i, int lane) { return (double)(1ll << (i % 32)) * (lane + 1) + i; }

static double s_sum[65][64];
static int s_index[65][64];

template <int K>
void lane_run()
{
    double v[K];
    for (int i = 0; i < K; ++i) v[i] = value(i, spx::t_lane);
    int k = 0;
    s_sum[K][spx::t_lane] = spx::wave_sum_many<K>(v, &k);
    s_index[K][spx::t_lane] = k;
}

template <int... I>
void all(std::integer_sequence<int, I...>)
{
    (lane_run<I + 1>(), ...);
}

int main()
{
    pthread_barrier_init(&spx::s_all, nullptr, 64);
    std::vector<std::thread> lanes;
    for (int l = 0; l < 64; ++l)
        lanes.emplace_back([l] {
            spx::t_lane = l;
            all(std::make_integer_sequence<int, 64>());
        });
    for (auto &t : lanes) t.join();
    int bad = 0;
    for (int K = 1; K <= 64; ++K) {
        bool seen[64] = {};
        for (int l = 0; l < 64; ++l) {
            const int k = s_index[K][l];
            if (k >= K) continue;
            double want = 0.0;
            for (int q = 0; q < 64; ++q) want += value(k, q);
            seen[k] = true;
            if (s_sum[K][l] != want && ++bad <= 20)
                std::printf("K=%d lane %d: index %d, sum %.17g, wanted %.17g\n", K, l, k, s_sum[K][l], want);
        }
        for (int k = 0; k < K; ++k)
            if (!seen[k] && ++bad <= 20) std::printf("K=%d: no lane has value %d\n", K, k);
    }
    std::printf("%d wrong\n", bad);
    return bad != 0;
}
"""


def test_every_index_has_one_value(tmp_path):
    src, exe = tmp_path / "wave_many.cpp", tmp_path / "wave_many"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-pthread",
                    "-I" + os.path.join(ROOT, "paper_2006_14290_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
