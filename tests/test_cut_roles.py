"""Who runs what in a launch of bf16 passes that cuts some chains in two (CPU: the kernel's own arithmetic, compiled
for the host).  Workgroups are started in several orders, the reverse of their ids among them."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP = "/opt/rocm/include"

PROGRAM = r"""
#include "ltn_kernels.h"
#include <algorithm>
#include <cstdio>
#include <map>
#include <numeric>
#include <random>
#include <tuple>
#include <vector>

#define CHECK(c) do { if (!(c)) { std::printf("%s: chains %d count %d slices %d cut %d order %d\n", #c, pb.chains, pb.count, NS, pb.cut_chains, order); return 1; } } while (0)

template <int NS>
int launch(int chains, int count, int cut_chains, int order) {
    ltn::PassBatch pb{};
    pb.chains = chains;
    pb.count = count;
    pb.cut_chains = cut_chains;
    const int grid = ltn::cut_launch_ids(pb, NS), xcd = (chains & 7) == 0;
    CHECK(grid > 0 && pb.cut_ids[2] % 8 == 0);
    std::vector<int> ids(grid);
    std::iota(ids.begin(), ids.end(), 0);
    std::mt19937 rng(chains * 8 + count);
    if (order == 1) std::reverse(ids.begin(), ids.end());
    if (order == 2) std::shuffle(ids.begin(), ids.end(), rng);
    if (order == 3) std::rotate(ids.begin(), ids.begin() + pb.cut_ids[0], ids.end());
    int drawn[8] = {};
    std::map<std::tuple<int, int, int, int>, int> runs;      // pass, chain, split, part -> when it started
    for (int i = 0; i < grid; ++i) {
        const int wg = ids[i], c = wg & 7;
        const bool draws = ltn::cut_draws(pb, wg);
        const ltn::CutRole r = ltn::cut_role<NS>(pb, xcd, draws ? ltn::cut_id(pb, wg, drawn[c]++) : wg);
        if (r.chain >= chains) continue;                     // a padding workgroup
        CHECK(r.chain >= 0 && r.split >= 0 && r.split < NS && r.pass >= 0 && r.pass < count);
        CHECK(runs.emplace(std::make_tuple(r.pass, r.chain, r.split, r.part), i).second);
        CHECK(draws == (r.part != 0));
        if (r.part == 2) CHECK(runs.count(std::make_tuple(r.pass, r.chain, r.split, 1)));      // started before
        if (r.part == 2 && drawn[c] == 2 * ltn::cut_parts_of(pb, c)) {       // the last to draw: its rows hold the counter
            int chain, split;
            ltn::cut_part<NS>(ltn::cut_last_part(pb, c), xcd, chain, split);
            CHECK(chain == r.chain && split == r.split);
            drawn[c] += 1 << 20;                             // nobody draws after it
        }
    }
    for (int c = 0; c < 8; ++c) CHECK(drawn[c] == (ltn::cut_parts_of(pb, c) ? 2 * ltn::cut_parts_of(pb, c) + (1 << 20) : 0));
    for (int p = 0; p < count; ++p)
        for (int v = 0; v < chains; ++v)
            for (int s = 0; s < NS; ++s) {
                const bool cut = p == count - 1 && v < cut_chains;
                for (int part = 0; part < 3; ++part) CHECK(runs.count(std::make_tuple(p, v, s, part)) == (cut ? part != 0 : part == 0));
            }
    return 0;
}

int main() {
    int n = 0;
    for (int order = 0; order < 4; ++order)
        for (int chains = 1; chains <= 400; chains += chains < 40 ? 1 : 13 + (chains & 3))
            for (int count = 1; count <= 3; ++count)
                for (int step = 0; step < 4; ++step) {
                    int cut = std::max(1, step == 0 ? 1 : chains * step / 3);
                    if ((chains & 7) == 0) cut = (cut + 7) / 8 * 8;
                    if (launch<1>(chains, count, cut, order) || launch<2>(chains, count, cut, order) ||
                        launch<4>(chains, count, cut, order)) return 1;
                    n += 3;
                }
    std::printf("%d launches\n", n);
    return 0;
}
"""


def test_every_part_is_run_once_and_second_parts_after_their_first(tmp_path):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if not cxx or not os.path.isdir(HIP):
        pytest.skip("no host compiler or HIP headers")
    src, exe = tmp_path / "roles.cpp", str(tmp_path / "roles")
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__=1", "-isystem", HIP,
                    "-I", os.path.join(ROOT, "paper_2307_14995_amd", "csrc"), str(src), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "launches" in r.stdout, r.stdout[-2000:] + r.stderr[-2000:]
