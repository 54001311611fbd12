"""Host-side logic of bench.py and of the counter summaries it reads (no GPU)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2602_03839_amd import traffic  # noqa: E402


def test_counter_bound_reproduces_its_two_streams():
    # a launch that moves exactly the read stream's bytes takes fetch / read rate
    cb = bench.counter_bound((6.0e9, 0.0), 6000.0, 4000.0, 1.0)
    assert cb["bound_ms"] == pytest.approx(1.0)
    assert cb["frac"] == pytest.approx(1.0)
    # a launch with the read-modify-write stream's mix (8 B read, 4 B written
    # per element) runs at that stream's rate
    n = 1.0e9
    cb = bench.counter_bound((8.0 * n, 4.0 * n), 6000.0, 4000.0, 3.0)
    assert cb["bound_ms"] == pytest.approx(12.0 * n / 4000e9 * 1e3)
    # written bytes cost more than read ones whenever the rmw stream is slower
    assert cb["write_marginal_GBps"] < 6000.0


def test_traffic_summary_split_and_source_hash(tmp_path):
    good = tmp_path / "good.txt"
    good.write_text(f"# header: with a colon\nsource_hash: {traffic.kernel_source_hash()}\n"
                    "fetch_bytes_per_launch: 100\nwrite_bytes_per_launch: 23\n")
    assert traffic.read_summary_split(str(good)) == (100.0, 23.0)
    assert traffic.read_summary(str(good)) == 123.0
    stale = tmp_path / "stale.txt"
    stale.write_text("source_hash: 0000000000000000\nfetch_bytes_per_launch: 1\nwrite_bytes_per_launch: 1\n")
    assert traffic.read_summary_split(str(stale)) is None
    assert traffic.read_summary(str(tmp_path / "missing.txt")) is None


def test_kernel_labels():
    assert traffic.kernel_label("void pulse::(anonymous namespace)::outer_kernel(pulse::OuterParams)") == \
        "outer_kernel"
    assert traffic.kernel_label("void pulse::encode_kernel<15, 2, true>(pulse::EncodeParams)") == \
        "encode_kernel<15, 2, true>"


# encode_kernel<waves, groups, refresh, table>: the refresh forms with and without the
# table, the plain ones, the one-tile form and another kernel
REFRESH_FORMS = [("void pulse::encode_kernel<15, 2, true, false>(pulse::EncodeParams)", True),
                 ("void pulse::encode_kernel<15, 2, true, true>(pulse::EncodeParams)", True),
                 ("void pulse::encode_kernel<15, 2, false, true>(pulse::EncodeParams)", False),
                 ("void pulse::encode_kernel<15, 2, false, false>(pulse::EncodeParams)", False),
                 ("void pulse::encode_one_kernel<4, true, true>(pulse::EncodeParams)", False),
                 ("void pulse::loco_kernel<15, 1, 1, true>(pulse::LocoParams)", False)]


def test_counter_summary_takes_the_refresh_launches(tmp_path):
    rows = [("void at::native::bitwise_not_kernel(int)", 1 << 20)]
    rows += [(name, 1000 + i) for i, (name, _) in enumerate(REFRESH_FORMS)]
    lines = ["Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value"]
    lines += [f'{i},"{name}",FETCH_SIZE,{v}' for i, (name, v) in enumerate(rows)]
    (tmp_path / "run_counter_collection.csv").write_text("\n".join(lines) + "\n")
    scale, total, values = traffic._measure(str(tmp_path), "FETCH_SIZE", 2)
    assert scale == 1.0 and values == [1000.0, 1001.0] and total == 2001.0 * 1024
    with pytest.raises(SystemExit):  # a third refresh launch is not there
        traffic._measure(str(tmp_path), "FETCH_SIZE", 3)


def test_stats_summary_finds_the_timed_refresh_launches(tmp_path):
    names = [n for n, refresh in REFRESH_FORMS if refresh] * 2
    trace = ["Dispatch_Id,Kernel_Name,Start_Timestamp,End_Timestamp"]
    for i, (name, _) in enumerate(REFRESH_FORMS):
        trace.append(f'{i},"{name}",0,{1000000 * (i + 1)}')
    (tmp_path / "t.csv").write_text("\n".join(trace) + "\n")
    (tmp_path / "s.csv").write_text("Name,Calls,AverageNs,MinNs,MaxNs,TotalDurationNs\n" +
                                    "".join(f'"{n}",1,1e6,1e6,1e6,1e6\n' for n in names))
    (tmp_path / "b.json").write_text('{"ms_per_step": 1.5, "steps": 2, "warmup": 0, "config": {"launches_per_step": 1},'
                                     ' "roofline": {"avg_launch_ms": 1.5, "achieved": 1.0, "frac": 0.1}}\n')
    out = tmp_path / "o.md"
    traffic.stats_main(["--stats-csv", str(tmp_path / "s.csv"), "--bench-json", str(tmp_path / "b.json"), "--out", str(out),
                        "--trace-csv", str(tmp_path / "t.csv")])
    assert "average 1.5000 ms, 0.0% from the events' 1.5000 ms" in out.read_text()


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)
