"""The traffic record: told apart by what a launch writes where one kernel serves two problems, and reported only for the
kernel that is launched (CPU)."""
import json

import pytest

import bench
from paper_2412_20386_amd import profile_summary

KERNEL = "void (anonymous namespace)::linear_mfma_persistent<ptq4vm::mfma::Int8Path, true, false, 8>(ptq4vm::mfma::LinearArgs)"


def counters(directory, name, values):
    directory.mkdir()
    lines = ["Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value,Grid_Size,LDS_Block_Size"]
    for i, v in enumerate(values):  # a dispatch's value is the sum of its rows
        lines += [f'{i},"{KERNEL}",{name},{v / 4},131072,0', f'{i},"{KERNEL}",{name},{v * 3 / 4},131072,0']
        lines.append(f'{1000 + i},"void other_kernel()",{name},{1e6},256,0')
    (directory / "p_counter_collection.csv").write_text("\n".join(lines) + "\n")
    return str(directory)


def test_reads_of_the_launches_that_write_the_most(tmp_path):
    reads = counters(tmp_path / "f", "FETCH_SIZE", [300, 500, 301, 501, 302, 502, 303, 503, 304, 504])
    writes = counters(tmp_path / "w", "WRITE_SIZE", [3000, 700, 3000, 701, 3001, 702, 3000, 700, 3002, 700])
    got = profile_summary.dominant_readings(reads, writes, "linear_mfma_persistent<int8>")
    assert got == ([300, 301, 302, 303, 304], [3000, 3000, 3001, 3000, 3002])
    fewer = counters(tmp_path / "f2", "FETCH_SIZE", [300, 500])
    assert profile_summary.dominant_readings(fewer, writes, "linear_mfma_persistent<int8>") == ([], [])


@pytest.mark.parametrize("launched,traffic", [("linear_mfma_persistent<int8>", 7.0), ("linear_mfma_tile<int8 128x128>", None), (None, None)])
def test_traffic_of_the_kernel_that_is_launched(tmp_path, monkeypatch, launched, traffic):
    record = tmp_path / "traffic.json"
    record.write_text(json.dumps(dict(config=3, kernel="linear_mfma_persistent<int8>", traffic_bytes=7)))
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(record))
    monkeypatch.setattr(bench, "dominant_kernel_name", lambda *_: launched)
    assert bench.dominant_traffic(3, None, None) == traffic
    assert bench.dominant_traffic(2, None, None) is None
