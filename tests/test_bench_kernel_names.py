"""The kernel names bench.py reports follow the library's choice of form."""
import ctypes
import json

import bench
import paper_1205_0752_amd as gf
from paper_1205_0752_amd.workloads import CONFIGS, Params, Propagators, Quadrature


def test_groups_follow_the_library():
    lib = gf.load()
    count = lib._ZN2gf11group_countEi  # the library's own rule
    count.argtypes, count.restype = [ctypes.c_int], ctypes.c_int
    for n in list(range(1, 600)) + [1023, 1024, 4097, 8191, 8192]:
        assert bench.angular_groups(n) == count(n), n


def test_both_fp64_forms_have_their_names():
    legs = (((1.0, 1.0),), ((1.0, 1.0),))
    q = Quadrature(256, 128, 16)
    assert bench.scan_kernel_name(Params(), q, 1) == "scan_kernel_fp64<1, false, false, false>"
    assert bench.scan_kernel_name(Params(), q, 1, Propagators(*legs)) == \
        "scan_kernel_fp64<1, true, false, true>"
    assert bench.scan_kernel_name(Params(), q, 1, Propagators(*legs, ((0, 0, 1.0),))) == \
        "scan_kernel_fp64_pairs<1, true, false, true>"
    assert bench.scan_kernel_name(Params(), Quadrature(64, 32, 16), 64) == \
        "scan_kernel_fp64_pairs<64, false, false, false>"


def test_counters_are_used_only_for_the_sources_they_were_taken_on():
    p, _, q = CONFIGS["c1_fp64_1024sq"]
    name = bench.scan_kernel_name(p, q, 1)
    with open(bench.COUNTERS_FILE) as f:
        rec = json.load(f)
    got = bench.launch_counters(name)
    if rec["kernels_source_sha256"] == bench.kernel_source_sha256():
        assert got == rec["kernels"][name] and got["traffic_bytes"] >= 16 << 20
    else:
        assert got is None
    assert bench.launch_counters("scan_kernel_fp64<2, false, false, false>") is None
