"""Host-side rules of the benchmark (CPU): the KV copies it rotates keep both
each call's cache bytes and each draft's gathered rows out of the 256 MB
Infinity Cache, so that its figures are HBM figures."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2607_27735_amd.workloads import CONFIGS, make_config  # noqa: E402

MIB = 1 << 20


@pytest.mark.parametrize("n", sorted(CONFIGS))
def test_rotation_keeps_cache_and_gathers_cold(n):
    w = make_config(n)
    kv_bytes = w.k.size * 2 * 2          # K and V, bf16
    draft = bench.algorithmic_bytes(w, out_bytes=2)[0]["draft"]
    c = bench.kv_copies(w, kv_bytes)
    assert 2 <= c <= 256
    # between two uses of one copy, the other copies' bytes (and their
    # drafts' gathered rows) exceed 512 MiB, unless the cap of 256 copies
    # binds first
    assert (c - 1) * kv_bytes > 512 * MIB
    assert (c - 1) * draft > 512 * MIB or c == 256


def test_algorithmic_bytes_of_the_32k_workload():
    """Verify: K and V once (8 heads x 32768 keys x 256 B each), the scores
    and the query / output rows; draft: the gathered K and V rows and their
    indices; select: the scores and the index list."""
    w = make_config(2)
    nb, n_idx = bench.algorithmic_bytes(w, out_bytes=2)
    assert nb["verify"] == 8 * 32768 * 128 * 2 * 2 + 8 * 32768 * 4 + 7 * 32 * 128 * 2 * 2
    assert n_idx == [2048]
    assert nb["draft"] == 8 * 2048 * (128 * 2 * 2 + 4) + 32 * 128 * 4
    assert nb["select"] == 8 * 32768 * 4 + 8 * 2048 * 4 + 4


@pytest.mark.parametrize("short,paged", [
    ("verify_stream_kernel<true, false, false>", True), ("verify_stream_kernel<false, true, true>", False),
    ("verify_fused_kernel<2, true, true, false>", True), ("verify_fused_kernel<2, true, false, true>", False),
    ("verify_main_kernel<2, true, false>", True), ("verify_main_kernel<2, false, true>", False),
    ("verify_stats_kernel<4, true>", True), ("draft_kernel<3, 1>", True), ("draft_kernel<0, 1>", False),
    ("verify_combine_kernel", False)])
def test_paged_instances_are_told_apart(short, paged):
    assert bench.is_paged(short) is paged


def test_kernel_list_names_every_kernel_of_the_library():
    """Each __global__ function of the sources is in the benchmark's list."""
    import re
    csrc = os.path.join(ROOT, "paper_2607_27735_amd", "csrc")
    text = "".join(open(os.path.join(csrc, f)).read() for f in os.listdir(csrc))
    names = set(re.findall(r"__global__[^;{]*?\b(\w+_kernel)\(", text))
    names.discard("take_status_kernel")   # reads the exchange status, no part of a call
    assert names and names == set(bench.OUR_KERNELS)


def test_select_schedule_names():
    assert bench.select_schedule(True, 32768, 8) == "one kernel"
    assert bench.select_schedule(False, 65536, 30) == "workgroup per unit"
    assert bench.select_schedule(False, 65536, 29) == "three kernels"
    assert bench.select_schedule(False, 65537, 64) == "three kernels"
