"""bench.py --traffic-from: HBM bytes per launch out of rocprofv3's counter tables,
here made up. A decoder step is everything from one window build to the next, a
verification all of its kernels (draft statistics, rows, finalize, drafting); the
kernels it looks for are kernels of the library."""
import argparse
import csv
import os

import pytest

import bench

COPY = "__amd_rocclr_copyBuffer"


def _write(path, counter, dispatches):
    os.makedirs(path)
    with open(os.path.join(path, "1_counter_collection.csv"), "w", newline="") as fh:
        w = csv.DictWriter(fh, ["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
        w.writeheader()
        for i, (name, kib) in enumerate(dispatches):
            w.writerow(dict(Dispatch_Id=i, Kernel_Name=name, Counter_Name=counter, Counter_Value=kib))


STEP = [("void sjd::k_window_in(WindowIn)", 7.0), ("void sjd::k_gemm<4, 1, 4, false>(GemmArgs)", 100.0),
        ("void sjd::k_verify_rows<1024, 16, false>(VerifyArgs)", 20.0), ("sjd::k_verify_finalize(VerifyArgs)", 2.0),
        ("sjd::k_step_end(DevState*)", 1.0)]
VERIFY = [("void sjd::k_draft_stats<512, 8>(VerifyArgs)", 80.0), ("void sjd::k_verify_rows<512, 8, false>(VerifyArgs)", 90.0),
          ("sjd::k_verify_finalize(VerifyArgs)", 3.0), ("void sjd::k_verify_pd<512, 8>(VerifyArgs)", 10.0)]


@pytest.mark.parametrize("workload,launch,per", [("7b", STEP, 130.0), ("verify", VERIFY, 183.0),
                                                 ("verify", VERIFY[1:], 103.0)])
def test_traffic_per_launch(tmp_path, monkeypatch, workload, launch, per):
    calib = bench.CALIB_BYTES / 1024.0
    # the counter reads half of the bytes; set-up launches come before the copy
    runs = launch + [(COPY, calib / 2)] + 3 * launch + launch[:1] * (workload == "7b")
    for counter in ("FETCH_SIZE", "WRITE_SIZE"):
        _write(tmp_path / counter, counter, runs)
    monkeypatch.setattr(bench, "traffic_file", lambda w: str(tmp_path / f"traffic_{w}.txt"))
    bench.traffic_from(argparse.Namespace(workload=workload,
                                          traffic_from=[str(tmp_path / "FETCH_SIZE"), str(tmp_path / "WRITE_SIZE")]))
    assert bench.recorded_traffic(workload) == pytest.approx(2 * 2 * per * 1024.0, rel=1e-9)


def test_the_kernels_that_mark_launches_are_the_library_s():
    csrc = os.path.join(bench.ROOT, "paper_2603_18599_amd", "csrc")
    text = "".join(open(os.path.join(csrc, f)).read() for f in os.listdir(csrc) if f.endswith(".hip"))
    for start, own in bench.LAUNCH_KERNELS:
        assert f"void {start}(" in text or f"void\n{start}(" in text
        for k in own:
            assert f" {k}" in text or f"\n{k}" in text or f"void {k}" in text
