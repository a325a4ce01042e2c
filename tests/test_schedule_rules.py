"""The work list's scheduling rules: host functions of the library's internal
header, compiled into a small program by the host compiler and run on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2504_16083_amd", "csrc", "internal.hpp")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    """run(body) -> integers of the lines that a C++ body prints with out(...)."""
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no host compiler or HIP headers")
    d = tmp_path_factory.mktemp("rules")

    def go(body):
        src, exe = str(d / "t.cpp"), str(d / "t")
        with open(src, "w") as f:
            f.write(f'#include "{HEADER}"\n#include <cstdio>\nusing namespace mmi;\n'
                    'template <typename... T> void out(T... x) { ((printf("%lld ", (long long)x)), ...); puts(""); }\n'
                    f"int main() {{\n{body}\n}}\n")
        subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", src, "-o", exe],
                       check=True, capture_output=True, text=True)
        r = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60)
        return [[int(x) for x in line.split()] for line in r.stdout.splitlines()]
    return go


@pytest.mark.parametrize("cus", [256, 64, 8])
def test_few_workgroups_wait_for_their_first_item(run, cus):
    """The entries of a list that start side by side leave at most an eighth of an XCD's workgroups without an item;
    where they are a run, the entry behind it waits for all of them but the slack."""
    wgs = cus // 8
    rows = run("for (long long n : {1ll, 63ll, 64ll, 500ll, 1024ll, 1300ll, 1791ll, 1792ll, 2047ll, 2048ll, 4096ll, 131073ll}) {"
               f" const MapShape m = map_shape(n); const int side = side_by_side(m.run, {cus});"
               f" int wait = 0; for (int k = 0; k < {wgs}; ++k) wait += lead_need(k, side) > 0;"
               " out(n, m.run, wait, lead_need(m.run, side)); }")
    assert len(rows) == 12
    for n, r, wait, after in rows:
        assert wait <= wgs / 8, n
        assert after == (r - 2 if r * 8 >= wgs * 7 else -2), n


@pytest.mark.parametrize("S,R,steps,staged,computed,lead", [
    (1 << 19, 4, 256, 4000, 4000, True), (1 << 19, 4, 255, 4000, 16000, False),            # 8192 key blocks, any union
    ((1 << 19) - 64, 4, 1023, 4000, 16000, False), ((1 << 19) - 64, 4, 1024, 4000, 4000, True),
    (294912, 4, 1024, 4000, 4000, True), (294912 - 64, 4, 1024, 4000, 4000, False),        # 4608
    (294912 - 64, 4, 1024, 4000, 15600, True), (294912 - 64, 4, 1024, 4000, 15599, False),  # every member selects it
    (294912 - 64, 1, 1024, 4000, 4000, True), (294912 - 64, 2, 1024, 4000, 4000, False),
    (1 << 18, 4, 1024, 1024, 4090, True), ((1 << 18) - 64, 4, 1024, 4000, 16000, False),   # 4096
    ((1 << 18) - 63, 4, 1024, 4000, 16000, True), (4096, 4, 64, 64, 256, False)])
def test_items_that_start_side_by_side(run, S, R, steps, staged, computed, lead):
    """The rule counts a head's keys once, whatever its key layouts, and long walks of fewer keys."""
    assert run(f"out(lead_steps({S}, {R}, {steps}, {staged}, {computed}));") == [[steps if lead else 0]]
