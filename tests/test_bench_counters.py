"""bench_counters.py takes a summary's numbers only from runs of the present sources, one result file per run, and only where the
cycles of a counter run fit the time of the trace (no GPU)."""
import pytest

import bench_counters as bc


def _run(base, name, files=("a_counter_collection.csv",)):
    bc.stamp(str(base / name))
    for f in files:
        (base / name / f).write_text("Dispatch_Id,Kernel_Name,Counter_Name,Counter_Value\n1,k,C,2\n1,k,C,3\n")


def test_a_run_of_the_present_sources_is_read(tmp_path):
    _run(tmp_path, "sq1")
    assert bc.dispatches("sq1", str(tmp_path)) == [("k", {"C": 5.0})]


def test_what_an_older_run_left_is_refused(tmp_path):
    _run(tmp_path, "sq1", ("a_counter_collection.csv", "b_counter_collection.csv"))
    _run(tmp_path, "sq2")
    (tmp_path / "sq2" / "sources").write_text("0" * 16)
    _run(tmp_path, "sq3")
    (tmp_path / "sq3" / "sources").unlink()
    _run(tmp_path, "kt", ())
    for name in ("sq1", "sq2", "sq3", "kt", "none"):
        with pytest.raises(SystemExit):
            bc.dispatches(name, str(tmp_path))
    with pytest.raises(FileExistsError):   # a folder is stamped once
        bc.stamp(str(tmp_path / "sq1"))


def test_cycles_and_times_of_different_work_are_refused():
    assert abs(bc.clock(2.0e6, 1.0, "k") - 2.0) < 1e-12
    with pytest.raises(SystemExit):
        bc.clock(1.367e6, 0.468, "k_est_sums")


def test_a_kernel_figure_is_of_all_its_sources(monkeypatch, tmp_path):
    """A change of any file that the attention kernel is compiled from changes the hash that its stored figures go by."""
    import os
    import shutil

    import bench
    files = sorted(os.path.relpath(f, bench.ROOT) for f in bench.kernel_sources())
    assert {os.path.basename(f) for f in files} == {"vs_attn.hip", "vs_attn_short.h", "vs_common.h", "vs_decode_walk.h", "vs.h"}
    for f in files:
        os.makedirs(tmp_path / os.path.dirname(f), exist_ok=True)
        shutil.copy(os.path.join(bench.ROOT, f), tmp_path / f)
    here = bench.kernel_source_hash()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_source_hash() == here
    seen = {here}
    for f in files:
        with open(tmp_path / f, "a") as g:
            g.write("// changed\n")
        seen.add(bench.kernel_source_hash())
    assert len(seen) == 1 + len(files)
