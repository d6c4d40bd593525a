"""Stages in LDS that a workgroup fills with atomics and empties together: the device functions themselves, taken from the kernel
source and compiled for the CPU, one host thread per wave.  Barriers are real ones, and after each of them one wave (every wave
in turn) is held up, as a scheduler may do on the GPU: a decision that is taken from a counter other waves already move on
then differs from wave to wave, the waves part, and keys are lost or the barriers never meet.  No GPU."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2312_17530_amd", "csrc", "rsdgc_kernels.hip")

_SHIM = r"""
#include <pthread.h>
#include <unistd.h>
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>
#define __device__
#define __forceinline__ inline
#define __restrict__
using std::min;
constexpr int kWaves = 4;
struct Dim { uint32_t x; };
static thread_local Dim threadIdx;
static int lagging;                      // the wave that is held up after every barrier
static pthread_barrier_t barrier;
static void __syncthreads() {
    pthread_barrier_wait(&barrier);
    if (static_cast<int>(threadIdx.x) == lagging) usleep(2000);
}
static uint32_t atomicAdd(uint32_t *p, uint32_t v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
struct uint2 { uint32_t x, y; };
static uint2 make_uint2(uint32_t x, uint32_t y) { return uint2{x, y}; }
"""

_MAIN = r"""
static void *body(void *p) {
    threadIdx.x = static_cast<uint32_t>(reinterpret_cast<intptr_t>(p));
    wave();
    return nullptr;
}
int main() {
    alarm(60);                           // (waves that have parted wait for each other for good)
    for (lagging = 0; lagging < kWaves; ++lagging) {
        reset();
        pthread_barrier_init(&barrier, nullptr, kWaves);
        pthread_t t[kWaves];
        for (intptr_t w = 0; w < kWaves; ++w) pthread_create(&t[w], nullptr, body, reinterpret_cast<void *>(w));
        for (int w = 0; w < kWaves; ++w) pthread_join(t[w], nullptr);
        pthread_barrier_destroy(&barrier);
        if (!complete()) { std::printf("wave %d held up: keys lost or doubled\n", lagging); return 1; }
    }
    std::printf("ok\n");
}
"""

# rounds of appends as k_gather makes them: room for 1024 keys first, then the keys of every wave
_GATHER = r"""
constexpr int kStage = 2048;
struct GatherShared { unsigned long long ent[kStage + 4096]; uint32_t n, base; };
struct GatherList { uint32_t *cnt; unsigned long long *ent; uint32_t cap; };
%s
constexpr uint32_t kRounds = 12;
static GatherShared sh;
static uint32_t count;
static std::vector<unsigned long long> out;
static GatherList list;
static void reset() {
    sh.n = count = 0;
    out.assign(4 * 1024 * kRounds, ~0ull);
    list = GatherList{&count, out.data(), static_cast<uint32_t>(out.size())};
}
static uint32_t keys_of(uint32_t round, uint32_t w) { return round %% 3 == 2 ? 40 + w : 256; }
static void wave() {
    for (uint32_t r = 0; r < kRounds; ++r) {
        gather_make_room(sh, list);
        for (uint32_t i = 0; i < keys_of(r, threadIdx.x); ++i)
            sh.ent[atomicAdd(&sh.n, 1u)] = (r * kWaves + threadIdx.x) * 1024u + i;
    }
    gather_flush_keys(sh, list);
}
static bool complete() {
    std::vector<unsigned long long> want, got(out.begin(), out.begin() + min<size_t>(count, out.size()));
    for (uint32_t r = 0; r < kRounds; ++r)
        for (uint32_t w = 0; w < kWaves; ++w)
            for (uint32_t i = 0; i < keys_of(r, w); ++i) want.push_back((r * kWaves + w) * 1024u + i);
    std::sort(want.begin(), want.end());
    std::sort(got.begin(), got.end());
    return want == got;
}
"""

# the chunks of k_dyn_split: some within half of the stage, some that fill it, some that go past its end
_DYN = r"""
constexpr uint32_t kDynStage = 1024;
struct DynSplit { uint32_t n_list; };
struct DynSplitArgs { DynSplit *state; uint2 *list; uint32_t list_cap; };
%s
constexpr uint32_t kChunks = 24;
static DynStage sh;
static DynSplit state;
static std::vector<uint2> out;
static DynSplitArgs args;
static void reset() {
    sh.n = state.n_list = 0;
    out.assign(4 * 1024 * kChunks, uint2{~0u, 0u});
    args = DynSplitArgs{&state, out.data(), static_cast<uint32_t>(out.size())};
}
static uint32_t keys_of(uint32_t chunk, uint32_t w) {
    static const uint32_t n[6] = {100, 20, 0, 128, 300, 7};
    return n[chunk %% 6] + (chunk %% 2) * w;
}
static void wave() {
    for (uint32_t c = 0; c < kChunks; ++c) {
        for (uint32_t i = 0; i < keys_of(c, threadIdx.x); ++i)
            dyn_stage_key(sh, args, make_uint2((c * kWaves + threadIdx.x) * 1024u + i, c));
        dyn_make_room(sh, args);
    }
    dyn_flush_stage(sh, args);
}
static bool complete() {
    std::vector<uint32_t> want, got;
    for (uint32_t i = 0; i < min<size_t>(state.n_list, out.size()); ++i) got.push_back(out[i].x);
    for (uint32_t c = 0; c < kChunks; ++c)
        for (uint32_t w = 0; w < kWaves; ++w)
            for (uint32_t i = 0; i < keys_of(c, w); ++i) want.push_back((c * kWaves + w) * 1024u + i);
    std::sort(want.begin(), want.end());
    std::sort(got.begin(), got.end());
    return want == got;
}
"""


def _functions(names):
    """The definitions of these device functions, with the workgroup's 256 threads replaced by one per wave."""
    src, out = open(SOURCE).read(), []
    for name in names:
        m = re.search(r"^(struct %s \{.*?^};|__device__ __forceinline__ [^\n]*\b%s\(.*?^})\n" % (name, name), src, re.S | re.M)
        assert m, name
        out.append(m.group(0))
    return "\n".join(out).replace("i += 256", "i += kWaves")


def _run(tmp_path, program):
    src, exe = tmp_path / "stage.cpp", tmp_path / "stage"
    src.write_text(_SHIM + program + _MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", str(src), "-o", str(exe)])
    return subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=120)


STAGES = [("gather", _GATHER, ["staged_more_than", "gather_flush_keys", "gather_make_room"]),
          ("dynamic_ratios", _DYN, ["staged_more_than", "DynStage", "dyn_stage_key", "dyn_flush_stage", "dyn_make_room"])]


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("name, program, functions", STAGES, ids=[s[0] for s in STAGES])
def test_no_key_is_lost_whichever_wave_is_held_up(tmp_path, name, program, functions):
    proc = _run(tmp_path, program % _functions(functions))
    assert proc.returncode == 0 and proc.stdout == "ok\n", (proc.returncode, proc.stdout)
