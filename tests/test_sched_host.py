"""The workgroup -> work item mapping of the attention launches, checked on the host:
tests/sched_check.hip is compiled for the host only and enumerates every hardware
workgroup id for a set of head lists and block counts."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_work_item_is_mapped_exactly_once():
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "sched_check")
        cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wno-unused-command-line-argument",
               "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2407_02490_amd", "csrc"),
               os.path.join(ROOT, "tests", "sched_check.hip"), "-o", exe]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
        assert "FAIL" not in r.stdout and r.stdout.count("ok heads") == 57 and r.stdout.count("ok mixed") == 15
        assert r.stdout.count("ok wide") == 30 and r.stdout.count("ok order") == 82


def test_shared_tile_vertical_slash_schedule_covers_every_run_key_once():
    """tests/vs_ring_check.cpp (host only): the four waves of a workgroup yield equally many
    steps, followers read exactly the rows their leader fetched, and the attended keys of every
    wave equal the brute-force cover of the slash runs (App. C.4.2), each key once."""
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, "vs_ring_check")
        cmd = ["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2407_02490_amd", "csrc"),
               os.path.join(ROOT, "tests", "vs_ring_check.cpp"), "-o", exe]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout.startswith("ok cases"), r.stdout[-2000:] + r.stderr[-2000:]


def run_host_check(name):
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, name)
        cmd = ["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2407_02490_amd", "csrc"),
               os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        r = subprocess.run([exe], capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout[-2000:] + r.stderr[-2000:]


def test_selection_ranges_keep_exactly_k_keys():
    """tests/key_range_check.cpp (host only): the range passes of the register selection on rows with
    ties, infinities and NaN scores and with places that hold no element."""
    run_host_check("key_range_check")


def test_kernel_rules_take_the_faster_kernel_at_measured_sizes():
    """tests/dispatch_check.cpp (host only): the rules of dispatch.h at sizes where both kernels
    were timed."""
    run_host_check("dispatch_check")


def test_outputs_of_a_batch_that_the_rule_calls_apart_are_apart():
    """tests/batch_rule_check.cpp (host only): batch_rule.h against the places of drawn and of ordinary layouts."""
    run_host_check("batch_rule_check")
