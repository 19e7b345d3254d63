"""Host-side helpers of bench.py (no GPU): the committed counter summary feeds
the traffic fields only of the workload it was measured on, its dedup phase
only for the dedup it was measured with, and only while the kernel sources it
names are unchanged."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
import synth  # noqa: E402


def _workload_line(name):
    w = synth.workload(name)
    return f"{w.name}: {w.description}"


def test_counter_traffic_only_for_the_measured_workload():
    c3 = bench.counter_traffic(_workload_line("c3"), "emb_unique_ids")
    assert set(c3) == set(bench.PHASE_SOURCES)
    for name in ("c1", "c2", "c4", "c5"):
        other = bench.counter_traffic(_workload_line(name), "emb_unique_ids")
        assert other == {phase: None for phase in bench.PHASE_SOURCES}, name


def test_counter_traffic_follows_the_source_hashes(tmp_path, monkeypatch):
    wl = _workload_line("c3")
    src = tmp_path / "k.hip"
    src.write_text("kernel source\n")
    counters = tmp_path / "counters.txt"
    counters.write_text(f"Workload: {wl}\nDedup: emb_unique_ids_batched, groups of 4\n\nhbm_bytes_fwd = 123\n"
                        f"hbm_bytes_dedup = 45\nsha_k.hip = {bench.file_sha(str(src))}\n")
    monkeypatch.setattr(bench, "COUNTERS", str(counters))
    monkeypatch.setattr(bench, "PHASE_SOURCES", {"fwd": [str(src)], "dedup": [str(src)]})
    assert bench.counter_traffic(wl, "emb_unique_ids_batched, groups of 4") == {"fwd": 123.0, "dedup": 45.0}
    # the dedup phase only for the dedup the counters were taken with
    assert bench.counter_traffic(wl, "emb_unique_ids_batched, groups of 8") == {"fwd": 123.0, "dedup": None}
    assert bench.counter_traffic(wl, "emb_unique_ids") == {"fwd": 123.0, "dedup": None}
    src.write_text("kernel source, changed\n")
    assert bench.counter_traffic(wl, "emb_unique_ids_batched, groups of 4") == {"fwd": None, "dedup": None}


def test_phase_sources_are_all_that_the_kernels_are_compiled_from():
    """Every kernel the counters list, in whichever source it is defined, and
    every header of that source (headers of headers too): an edit of any of
    them makes the phase's recorded bytes stale."""
    csrc = os.path.join(ROOT, "paper_2112_02752_amd", "csrc")
    text = {n: open(os.path.join(csrc, n)).read() for n in os.listdir(csrc)}
    listed = {os.path.basename(f) for src in bench.PHASE_SOURCES.values() for f in src}
    kernels = re.findall(r"^\| (k_\w+) \|", open(bench.COUNTERS).read(), re.M)
    assert kernels
    for k in kernels:
        homes = [n for n, t in text.items() if re.search(r"\b__global__\b[^;{]*\b%s\(" % k, t)]
        assert homes and set(homes) <= listed, (k, homes)
    for phase, src in bench.PHASE_SOURCES.items():
        names = {os.path.basename(f) for f in src}
        for n in names:
            missing = set(re.findall(r'#include "([^"]+)"', text[n])) & set(text) - names
            assert not missing, (phase, n, missing)
    # both forms of the reduce and of the dedup, whichever of them the counters were taken with
    assert {"reduce.hip", "reduce_wave.hip"} <= {os.path.basename(f) for f in bench.PHASE_SOURCES["bwd_update"]}
    assert {"dedup.hip", "dedup_small.hip"} <= {os.path.basename(f) for f in bench.PHASE_SOURCES["dedup"]}
