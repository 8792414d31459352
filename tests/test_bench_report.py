"""Host-side arithmetic of bench.py's report (CPU only): traffic records keep the kernel variants of one
workload apart, and fp32 FLOP counts are those of the tiles and launches that run."""
import json
import os
import re

import bench
from paper_2307_14995_amd import build

NAME = "void ltn::(anonymous namespace)::pass_f32_kernel<{}>(ltn::PassBatch, int, int)"


def test_traffic_record_keeps_the_fp32_variants_apart(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "traffic_profile_path", lambda w: str(tmp_path / f"{w}.json"))
    rows = {NAME.format("128, 128, 32, 1, 128, 0"): 30.0, NAME.format("128, 128, 32, 1, 128, 2"): 20.0,
            NAME.format("128, 64, 32, 2, 64, 0"): 10.0, "__amd_rocclr_copyBuffer": float(1 << 20)}
    paths = []
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        paths.append(tmp_path / f"{counter}.csv")
        paths[-1].write_text("Kernel_Name,Counter_Name,Counter_Value\n" +
                             "".join(f'"{n}",{counter},{v}\n' for n, v in rows.items()))
    assert bench.write_traffic_profile("w", *map(str, paths)) == 0
    kernels = json.loads((tmp_path / "w.json").read_text())["kernels"]
    assert {k: v["read_bytes_per_launch"] for k, v in kernels.items()} == {
        "pass_f32_kernel<128,128,32>": 30 * 1024, "pass_f32_kernel<128,128,32> mode 2": 20 * 1024,
        "pass_f32_kernel<128,64,32> DC 64": 10 * 1024}


BF16 = "void ltn::(anonymous namespace)::pass_bf16_kernel<{}>(ltn::PassBatch, int)"


def test_traffic_record_of_launches_with_chains_in_two_parts(tmp_path, monkeypatch):
    """They count under the name of the pass they are, averaged with its launches in whole chains (a step whose
    forward is whole and whose backward is cut has both at one width)."""
    monkeypatch.setattr(bench, "traffic_profile_path", lambda w: str(tmp_path / f"{w}.json"))
    rows = [(BF16.format("128, 128, 0, 128, 128"), 10.0), (BF16.format("128, 128, 5, 128, 128"), 30.0),
            (BF16.format("128, 128, 5, 128, 128"), 32.0), (BF16.format("128, 128, 6, 128, 128"), 7.0),
            (BF16.format("128, 128, 1, 128, 128"), 9.0), (BF16.format("128, 96, 8, 96, 96"), 4.0),
            (BF16.format("64, 64, 9, 64, 64"), 5.0), (BF16.format("128, 128, 2, 128, 128"), 3.0),
            ("__amd_rocclr_copyBuffer", float(1 << 20))]
    for order in (rows, rows[::-1]):
        paths = []
        for counter in ("FETCH_SIZE", "WRITE_SIZE"):
            paths.append(tmp_path / f"{counter}.csv")
            paths[-1].write_text("Kernel_Name,Counter_Name,Counter_Value\n" +
                                 "".join(f'"{n}",{counter},{v}\n' for n, v in order))
        assert bench.write_traffic_profile("w", *map(str, paths)) == 0
        kernels = json.loads((tmp_path / "w.json").read_text())["kernels"]
        assert {k: (v["launches"], v["read_bytes_per_launch"]) for k, v in kernels.items()} == {
            "pass_bf16_kernel<128,128>": (3, 24 * 1024), "pass_bf16_kernel<128,128> mode 1": (2, 8 * 1024),
            "pass_bf16_kernel<128,96> mode 3": (1, 4 * 1024), "pass_bf16_kernel<64,64> mode 4": (1, 5 * 1024),
            "pass_bf16_kernel<128,128> mode 2": (1, 3 * 1024)}


def test_fp32_flops_are_those_of_the_tiles_and_launches_that_run():
    # a block of 64 tokens is two tiles of 32: 24 keys a token on average, whatever the block
    whole = bench.f32_issued_flops_per_token_head(64, 64, 64, 1, 0)
    assert whole == bench.f32_issued_flops_per_token_head(64, 32, 64, 1, 0) == 2 * 24 * 64 * 2 + 4 * 64 * 64
    # chains cut into segments: one state update more for each sweep, of which a backward has two or three
    assert bench.f32_issued_flops_per_token_head(64, 64, 64, 1, 1) == whole + 2 * 64 * 64
    assert bench.f32_issued_flops_per_token_head(64, 64, 64, 3, 2) == 3 * whole + 2 * 2 * 64 * 64


def test_sweeps_of_a_segmented_backward_count_as_often_as_they_run():
    def exec_(*plans):
        return bench.flops_per_token_head(256, 64, *plans)["F_exec"]

    whole = exec_((64, 1), (64, 1))
    assert exec_((64, 4), (64, 1)) == whole + 2 * 256 * 256
    assert exec_((64, 1), (64, 4), 2) == whole + 2 * 2 * 256 * 256
    assert exec_((64, 4), (64, 4), 3) == whole + 4 * 2 * 256 * 256


def test_a_traffic_record_goes_stale_with_every_source_it_depends_on(monkeypatch):
    included = {name for src in bench.TIMED_SOURCES for name in
                re.findall(r'#include "(ltn_\S+)"', open(os.path.join(build.CSRC, src)).read())}
    assert included <= set(bench.TIMED_SOURCES)
    for src in ("ltn_scan.hip", "ltn_cache.h"):
        assert src in bench.TIMED_SOURCES
    before = bench.kernel_source_hash()
    monkeypatch.setattr(build, "HIPCC_FLAGS", build.HIPCC_FLAGS + ["-O2"])
    assert bench.kernel_source_hash() != before
