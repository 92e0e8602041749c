"""Warm re-plans around the size of the scratch array that holds the partial states of the allocation-free call (CPU).

A batch whose fastest plan writes more states than the array holds gets a plan of larger units where that one fits. A
warm re-plan keeps such a choice only while it is the right one: it goes back to the fastest plan when the batch has
shrunk, and takes larger units when it has grown. The library re-plans only beside a GPU, so a small program compiled
here drives the planner itself.
"""

import subprocess

import pytest

from paper_2509_00195_amd.build import CSRC

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "tts_meta.h"
using namespace tts;
// n requests of 64 beams: a prompt of 12 blocks, groups of 8 beams (40 blocks), pairs (4), 3 private blocks.
static HostMeta batch(int n) {
  std::vector<int32_t> tab(n * 64 * 59, -1), len, off{0};
  int32_t nxt = 0, prompt[12], mid[40], pair[4];
  for (int r = 0; r < n; ++r) {
    for (auto& x : prompt) x = nxt++;
    for (int b = 0; b < 64; ++b) {
      if (b % 8 == 0) for (auto& x : mid) x = nxt++;
      if (b % 2 == 0) for (auto& x : pair) x = nxt++;
      int32_t* row = tab.data() + (r * 64 + b) * 59;
      std::memcpy(row, prompt, sizeof prompt);
      std::memcpy(row + 12, mid, sizeof mid);
      std::memcpy(row + 52, pair, sizeof pair);
      for (int k = 56; k < 59; ++k) row[k] = nxt++;
      len.push_back(16 * 59 - 5);
    }
    off.push_back((r + 1) * 64);
  }
  MetaInput in;
  in.num_reqs = n, in.req_seq_offsets = off.data(), in.num_seqs = 64 * n, in.block_tables = tab.data();
  in.max_blocks = 59, in.seq_lens = len.data(), in.num_blocks = nxt;
  HostMeta m;
  std::string err;
  if (build_host_meta(in, &m, &err)) std::abort();
  return m;
}
int main(int argc, char** argv) {
  const PlanShape shape{28, 4, 128, 2, 256};
  WorkPlan last;
  for (int i = 1; i < argc; ++i) {
    const HostMeta m = batch(std::atoi(argv[i]));
    WorkPlan cold, warm;
    build_work_plan(m, shape, &cold);
    build_work_plan(m, shape, &warm, i > 1 ? &last : nullptr);
    std::printf("%d %d %d %d\n", cold.few_states, cold.rows_per_head, warm.few_states, warm.rows_per_head);
    last = warm;
  }
}
"""

ROW_BYTES = 4 * (2 * 128 + 16)  # KV heads x (fp16 elements + m, l, z, pad)
LIMIT = 64 << 20


@pytest.fixture(scope="module")
def replan(tmp_path_factory):
    d = tmp_path_factory.mktemp("replan")
    (d / "replan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", f"-I{CSRC}", str(d / "replan.cpp"), f"{CSRC}/tts_meta.cpp",
                    f"{CSRC}/tts_plan.cpp", "-o", str(d / "replan")], check=True)

    def run(*requests):
        r = subprocess.run([str(d / "replan"), *map(str, requests)], check=True, capture_output=True, text=True)
        return [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]

    return run


def test_grown_and_shrunk_batches(replan):
    steps = replan(30, 48, 47, 30, 48)
    for cold_few, cold_rows, few, rows in steps:
        assert rows * ROW_BYTES <= LIMIT and few == cold_few
    assert [s[2] for s in steps] == [0, 1, 1, 0, 1]
    assert steps[3][3] == steps[3][1]  # the shrunk batch has the plan of a cold search


def test_batch_that_shrank_from_beyond_any_plan(replan):
    beyond, smaller = replan(100, 60)
    assert beyond[1] * ROW_BYTES > LIMIT and beyond[3] == beyond[1] and beyond[2] == 0
    assert smaller[0] == smaller[2] == 1 and smaller[3] * ROW_BYTES <= LIMIT


def test_batch_beyond_any_plan_stays_warm(replan):
    first, again = replan(100, 99)
    assert first[2] == again[2] == 0 and again[3] * ROW_BYTES > LIMIT
