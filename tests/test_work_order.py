"""The order in which the key side of the backward pass takes its key blocks (csrc/work_order.h), on the CPU: the header itself, compiled
for the host with a thread per lane, against what it states - every key block of every head once, on its XCD, long lists first, then
group by group and longest first.  And that the shapes of the GPU tests over groups of heads fall into the groups that they claim."""
import os
import random
import shutil
import subprocess

import pytest

from test_gpu_backward_tiles import GROUPED

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_12675_amd", "csrc", "work_order.h")
XCDS, KEY_BLOCKS, UNSET = 8, 2048, -7

# what work_order.h takes from common.h and from the device, for 256 threads of a workgroup
COMMON = """#pragma once
#include <algorithm>
#include <atomic>
#include <barrier>
#include <cstdint>
#include <cstdio>
#include <thread>
#include <vector>
#define __device__
#define __forceinline__ inline
using std::max; using std::min;
struct Index { int x; };
inline thread_local Index threadIdx;
inline std::barrier<> whole(256);
inline std::barrier<> wave[4] = {std::barrier<>(64), std::barrier<>(64), std::barrier<>(64), std::barrier<>(64)};
inline int lanes[256];
inline void __syncthreads() { whole.arrive_and_wait(); }
inline int atomicAdd(int* p, int x) { return std::atomic_ref<int>(*p).fetch_add(x); }
inline int __shfl_up(int x, int o) {
  std::barrier<>& b = wave[threadIdx.x / 64];
  lanes[threadIdx.x] = x;
  b.arrive_and_wait();
  const int y = lanes[threadIdx.x % 64 >= o ? threadIdx.x - o : threadIdx.x];
  b.arrive_and_wait();
  return y;
}
namespace sla2 {
constexpr int kWave = 64, kXcds = XCDS, kMaxKeyBlocks = KEY_BLOCKS;
struct Shape { int BH, N, d, Tm, Tn, k; bool bf16; };
struct BwdArgs { int32_t* col_cnt; int32_t* order; };
}
""".replace("XCDS", str(XCDS)).replace("KEY_BLOCKS", str(KEY_BLOCKS))
MAIN = """#include "work_order.h"
using namespace sla2;
int main() {      // per line: BH N d Tm Tn k bf16, with_order, then BH Tn list lengths -> groups, heads a group, long list, the order
  Shape s; int bf16, with_order;
  while (scanf("%d %d %d %d %d %d %d %d", &s.BH, &s.N, &s.d, &s.Tm, &s.Tn, &s.k, &bf16, &with_order) == 8) {
    s.bf16 = bf16;
    std::vector<int32_t> counts(with_order ? s.BH * s.Tn : 0), order(with_order ? s.BH * kXcds * ((s.Tn + kXcds - 1) / kXcds) : 0, UNSET);
    for (int32_t& c : counts) if (scanf("%d", &c) != 1) return 1;
    const WorkOrder o = make_order(s, BwdArgs{counts.data(), order.data()});
    printf("%d %d %d", o.groups, o.heads_per_group, o.long_list);
    for (int id = 0; with_order && id <= o.groups; id++) {
      std::vector<int> hist(kXcds * 256), at(2 * kXcds);
      std::vector<std::thread> block;
      for (int t = 0; t < 256; t++) block.emplace_back([&, t] { threadIdx.x = t; order_job(o, id, hist.data(), at.data()); });
      for (std::thread& t : block) t.join();
    }
    for (int32_t x : order) printf(" %d", x);
    printf("\\n");
  }
}
""".replace("UNSET", str(UNSET))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    folder = tmp_path_factory.mktemp("order")
    shutil.copy(HEADER, folder / "work_order.h")
    (folder / "common.h").write_text(COMMON)
    (folder / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-o", "order", "main.cpp"], cwd=folder, check=True)
    return str(folder / "order")


def ask(program, N, d, block_q, BH, k, bf16, lengths=None):
    Tm, Tn = -(-N // block_q), -(-N // 64)
    line = [BH, N, d, Tm, Tn, k, int(bf16), int(lengths is not None)] + (lengths or [])
    got = subprocess.run([program], input=" ".join(map(str, line)) + "\n", capture_output=True, text=True, check=True, timeout=60).stdout.split()
    return int(got[0]), int(got[1]), int(got[2]), [int(x) for x in got[3:]]


@pytest.mark.parametrize("w,groups,heads", [x[:3] for x in GROUPED], ids=lambda x: x.name if hasattr(x, "name") else str(x))
def test_groups_of_the_gpu_tests(program, w, groups, heads):
    assert ask(program, w.N, w.d, w.block_q, w.B * w.H, w.k, w.dtype == "bf16")[:2] == (groups, heads)


@pytest.mark.parametrize("N,d,block_q,BH,k,bf16", [
    (4000, 128, 128, 64, 3, True),       # three groups, a short last run
    (4096, 128, 128, 50, 6, True),       # two groups, runs of equal length
    (32700, 128, 128, 9, 15, True),      # groups of two heads
    (75600, 128, 128, 3, 35, True),      # groups of one
    (4096, 64, 64, 32, 6, True),         # one group
    (1500, 64, 64, 90, 2, True),         # 24 key blocks: three a run
    (460, 64, 64, 300, 1, True),         # one a run, seven runs
    (600, 64, 64, 300, 1, True),         # ten key blocks: five runs of two, three XCDs without one of a head
    (200, 128, 128, 5, 1, False),
    (9000, 64, 64, 40, 9, False),
    (64, 64, 64, 700, 1, True),          # one key block a head
])
@pytest.mark.parametrize("longest", [0, 40, 2000])
def test_every_key_block_once(program, N, d, block_q, BH, k, bf16, longest):
    """longest: the length of a tenth of the lists, past the line of a long one and past the 255 that are told apart"""
    rng = random.Random(N + longest)
    Tn = -(-N // 64)
    lengths = [longest if longest and rng.random() < 0.1 else rng.randint(0, 2 * k) for _ in range(BH * Tn)]
    groups, heads, long_list, order = ask(program, N, d, block_q, BH, k, bf16, lengths)
    assert UNSET not in order and sorted(x for x in order if x >= 0) == [bh * KEY_BLOCKS + j for bh in range(BH) for j in range(Tn)]
    per_head = -(-Tn // XCDS)
    for x in range(XCDS):
        run = order[x::XCDS]
        taken = [(e // KEY_BLOCKS, e % KEY_BLOCKS) for e in run if e >= 0]
        assert all(e == -1 for e in run[len(taken):])                           # empty places are the last ones
        assert all((j // per_head + (bh if groups > 1 else 0)) % XCDS == x for bh, j in taken)
        place = []
        for bh, j in taken:
            n = lengths[bh * Tn + j]
            is_long = groups > 1 and n > long_list
            place.append((0 if is_long else 1 + min(bh // heads, groups - 1), -min(n, 255)))
        assert place == sorted(place)
