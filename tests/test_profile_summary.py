"""The summaries of profiles, on a few lines of what the profiler writes for the kernels as they are named now."""
import csv
import re
import sys

import pytest

from paper_2509_06980_amd import profile_summary as ps

GRID = 128 * 8 * 256                   # decode launches of 128 trajectories and 8 kv heads
KERNELS = ["void attention_mfma_kernel<false, %d>(unsigned short const*, char*)" % form for form in (0, 1, 2)]
COPY = ("__amd_rocclr_copyBuffer", 1024)


def _counters(path, counter, rows):
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Grid_Size", "Counter_Name", "Counter_Value"])
        for name, grid, value in rows:
            w.writerow([name, grid, counter, value])
    return str(path)


def _trace(path, rows):
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Grid_Size_X", "Start_Timestamp", "End_Timestamp"])
        w.writerows(rows)
    return str(path)


def test_hbm_traffic_of_every_form_of_the_decode_attention(tmp_path, monkeypatch, capsys):
    copied = 151936 * 2560 * 2 / 1024                  # KiB, both factors 1
    other = ("void attention_mfma_kernel<true, 0>(char*)", GRID, 9e9)
    fetch = _counters(tmp_path / "f.csv", "FETCH_SIZE", [(*COPY, copied), (KERNELS[0], GRID, 3000.0), (KERNELS[0], GRID, 5000.0),
                                                         (KERNELS[1], GRID, 1000.0), (KERNELS[1], 512, 7e7), other])
    write = _counters(tmp_path / "w.csv", "WRITE_SIZE", [(*COPY, copied), (KERNELS[0], GRID, 30.0), (KERNELS[1], GRID, 10.0), other])
    monkeypatch.setattr(sys, "argv", ["profile_summary", fetch, write])
    ps.main()
    out = capsys.readouterr().out
    assert "(grid 262144 threads): 3 with FETCH_SIZE, 2 with WRITE_SIZE" in out
    assert f"traffic_bytes_per_launch: {(3000 + 20) * 1024}" in out
    assert "- norm, RoPE and cache write before: 2 launches, 4.1 MB fetched, 0.0 MB written" in out and "inside: 1 launches, 1.0 MB fetched" in out
    assert re.search(r"kernel_source_sha256_16: " + ps.kernel_source_hash(), out)


def test_no_decode_launch_is_an_error_that_says_so(tmp_path, monkeypatch):
    empty = _counters(tmp_path / "f.csv", "FETCH_SIZE", [(*COPY, 1.0), ("void attention_mfma_kernel<true, 0>(char*)", GRID, 1.0)])
    monkeypatch.setattr(sys, "argv", ["profile_summary", empty, empty])
    with pytest.raises(SystemExit, match="no decode launch"):
        ps.main()
    with pytest.raises(SystemExit, match="no launch"):
        ps.trace_summary(_trace(tmp_path / "t.csv", [("void other(int)", 1, 0, 1)]))


def test_trace_keeps_the_forms_apart(tmp_path, capsys):
    rows = [(KERNELS[0], GRID, 0, 140000), (KERNELS[0], GRID, 0, 150000), (KERNELS[1], GRID, 0, 35000), (KERNELS[2], GRID, 0, 36000)]
    ps.trace_summary(_trace(tmp_path / "t.csv", rows))
    lines = capsys.readouterr().out.splitlines()
    assert "| 262144 | before | 2 | 145.00 |" in lines
    assert "| 262144 | inside | 1 | 35.00 |" in lines and "| 262144 | inside, rows divided by their rms there | 1 | 36.00 |" in lines


def test_hash_covers_every_file_of_the_decode_attention(tmp_path, monkeypatch):
    before = ps.kernel_source_hash()
    assert [p.rsplit("/", 1)[1] for p in ps.KERNEL_SRC] == ["kernels_mfma.hip", "qkrope.h"]
    changed = tmp_path / "qkrope.h"
    changed.write_bytes(open(ps.KERNEL_SRC[1], "rb").read() + b"\n")
    monkeypatch.setattr(ps, "KERNEL_SRC", [ps.KERNEL_SRC[0], str(changed)])
    assert ps.kernel_source_hash() != before


def test_products_of_a_decode_step_are_named_as_in_the_library(tmp_path, capsys):
    # what a product has to move stands beside what it moved: the table's names are those of kernels that are there
    from test_kernel_resources import _kernels

    import paper_2509_06980_amd as rl
    there = {f"{name}<{', '.join(map(str, args))}>" for name, args in _kernels(rl.LIB_PATH)}
    expect = ps.decode_products()
    assert {re.match(r"\w+: ", what.replace("lm-head", "head")).group(0) for what in expect.values()} == {"head: ", "qkv: ", "o: ", "gate_up: ", "down: "}
    for kernel, _ in expect:
        assert kernel.replace("false", "0") in there, kernel
    (kernel, grid), what = next(iter(expect.items()))
    rows = [(*COPY, 151936 * 2560 * 2 / 1024)] + [(f"void {kernel}(float*)", grid, 1000.0)] * 100
    ps.decode_step_table(_counters(tmp_path / "f.csv", "FETCH_SIZE", rows), _counters(tmp_path / "w.csv", "WRITE_SIZE", rows))
    assert f"| {kernel} | {grid} | 100 | 1.02 | 1.02 | {what} |" in capsys.readouterr().out
