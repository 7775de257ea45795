"""Host-side checks of bench.py and of the byte models its figures rest on (no GPU)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2302_08545_amd import workloads as wl  # noqa: E402


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "one GPU" in r.stderr
    assert r.stdout.strip() == ""


@pytest.mark.parametrize("w,want", [(wl.C1, 26.0), (wl.C2, 110.0), (wl.C3, 46.0), (wl.C4_B4, 88.0), (wl.C4_B2, 78.0),
                                    (wl.C5, 360.0)], ids=lambda x: getattr(x, "name", str(x)))
def test_compulsory_bytes_per_coordinate(w, want):
    # every datum once: n (in + [EF 4 + 4] + b/8) + (n b/8 + w/8) + (w/8 + 4), written out per workload by hand
    assert wl.bytes_per_coord(w) == want


@pytest.mark.parametrize("w,want", [(wl.C3, 8 * 12.5 + 5 + 13), (wl.C4_B4, 16 * 12.5 + 10 + 14),
                                    (wl.C2, 8 * (12 + 4.5 + 4.5 + 16) + 5 + 13),
                                    (wl.replace(wl.C2, block=1 << 26, d=1 << 26),
                                     8 * (12 + 8 + 4.5 + 4.5 + 8 + 16) + 5 + (1 + 4 + 8 + 8)),
                                    (wl.replace(wl.C3, block=1 << 13), 8 * (4 + 4.5) + 5 + 5),
                                    (wl.replace(wl.C2, block=1 << 14), 8 * (8 + 12.5) + 5 + 5),
                                    (wl.replace(wl.C3, block=1 << 15), 8 * 12.5 + 5 + 5),
                                    (wl.replace(wl.C2, block=1 << 15), 8 * (12 + 4.5 + 12.5) + 5 + 5)],
                         ids=lambda x: f"{x.name}-{x.block}" if isinstance(x, wl.Workload) else str(x))
def test_moved_bytes_per_coordinate_of_the_pass_structure(w, want):
    # two passes (three above 2^25), each reading and writing the vector once; up to 2^15 one pass back, and up to 2^14 one
    # pass forward behind one that reads for the norms
    assert wl.moved_bytes_per_coord(w) == want
    again = 0 if w.block <= 1 << 14 else w.n * (4 + (4 if w.ef else 0))
    assert wl.moved_bytes_per_coord(w, "each") == want + again


def test_the_kernels_that_the_roofline_names_are_those_that_run():
    small, ef15 = wl.replace(wl.C3, block=1 << 14), wl.replace(wl.C2, block=1 << 15)
    assert "k_whole" in bench.forward_kernels(small, "all", False) and "k_fwd_hi_quant" not in bench.forward_kernels(small, "all", False)
    assert "one inverse pass" in bench.forward_kernels(ef15, "all", False)
    assert "inverse passes" in bench.forward_kernels(wl.C2, "all", False) and "inverse" not in bench.forward_kernels(wl.C3, "all", False)
    assert "k_pipe_forward" in bench.forward_kernels(wl.C3, "all", True)
    assert "k_whole" in bench.forward_kernels(small, "all", True)
    assert bench.forward_kernels(wl.C3, "each", False) == "thc_prepare_range + n x thc_compress"


def test_counted_traffic_of_the_default_workload_is_read_from_the_tracked_profile():
    t = bench.measured_traffic("c3_vgg16")
    assert t is not None
    # the forward sweep moves 12.5 bytes per worker-coordinate through the L2s (and 16 MiB of partial sums)
    assert 0.99 < t / (8 * 2 ** 28 * 12.5) < 1.02
    assert bench.measured_traffic("no_such_workload") is None


def test_the_largest_kernel_of_the_default_workload_is_read_from_the_tracked_profile():
    name, per_round, avg_us = bench.profiled_kernel("c3_vgg16", "k_fwd_lo")
    # the default walk takes groups of 2^27 worker-coordinates, 512 MB read and written each: 128 us at 8 TB/s, 300 at 3.6
    assert name.startswith("k_fwd_lo<13") and per_round == 8 * 2 ** 28 // 2 ** 27 and 128 < avg_us < 300
    assert bench.profiled_kernel("no_such_workload", "k_fwd_lo") is None
