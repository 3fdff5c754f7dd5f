"""The host side of the library under AddressSanitizer and UBSan, on the CPU: the attention planner (counts, the lists
of the host twin of the device builder), the workspace layouts, the split-K plane sizes and the validators, over the
five benchmark shapes and 4000 seeded random batches (csrc/host_check.cpp states the properties checked).  The host
arithmetic checked here is what turns into device addresses, so an off-by-one in it would be an out-of-bounds access
on the GPU."""
import os
import re
import subprocess

from paper_2602_18447_amd import build as B


def test_host_planner_and_layouts_under_asan_ubsan():
    exe = B.HOST_CHECK
    srcs = [os.path.join(B.CSRC, f) for f in os.listdir(B.CSRC)]
    if not os.path.exists(exe) or os.path.getmtime(exe) < max(os.path.getmtime(f) for f in srcs):
        exe = B.build_host_check(verbose=False)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-4000:]
    assert "host_check: ok" in r.stdout
    assert "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr


def test_planner_loses_no_more_than_stated_on_measured_batches():
    """The planner's picks on batches that its constants were not fitted to, against the fastest plan of each as measured (csrc/attn_plan.cpp
    quotes the figures): a change of its model shows here without a GPU."""
    test_host_planner_and_layouts_under_asan_ubsan()          # builds the checker if need be
    table = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles", "attention_plans_of_random_batches.txt")
    r = subprocess.run([B.HOST_CHECK, table], capture_output=True, text=True, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"), timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    got = {m[1]: (int(m[2]), float(m[3]), float(m[4])) for m in re.finditer(r"(\S+): (\d+) batches, mean loss (\S+), worst (\S+)", r.stdout)}
    assert got["all"][0] == 200 and got["all"][1] <= 0.030 and got["all"][2] <= 0.178, r.stdout
    assert got["12/2"][1] <= 0.018 and got["40/8"][1] <= 0.022, r.stdout
