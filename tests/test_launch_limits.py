"""Launch rules of the search that the host computes, at the limits of the
launch settings a caller may give (no GPU: compiled with the host compiler)."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT


def run_cxx(tmp_path, body):
    cxx = shutil.which("g++") or shutil.which("c++")
    inc = "/opt/rocm/include"
    if cxx is None or not os.path.isdir(inc):
        pytest.skip("no host C++ compiler or no HIP headers")
    src = tmp_path / "rule.cpp"
    src.write_text('#include <cstdio>\n#include "comine.h"\nint main() {\n%s\nreturn 0;\n}\n' % body)
    exe = tmp_path / "rule"
    subprocess.run([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + inc,
                    "-I" + os.path.join(ROOT, "paper_2507_14813_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()


def test_hand_on_limit_for_any_number_of_waves(tmp_path):
    """No division by the waves of 2^30 workgroups (2^32 of them: 0 in 32 bits),
    and the same limits as the rule gives in whole numbers."""
    waves = [1, 64, 4096, 8192, 2 ** 31, 2 ** 32, 2 ** 33, 0]
    roots = [0, 131_072, 300_000, 20_000_000, 2 ** 31 - 1]
    body = "".join('printf("%%u %%u\\n", mg::hand_on_limit(%dull, %dull, false), '
                   'mg::hand_on_limit(%dull, %dull, true));\n' % (r, w, r, w) for r in roots for w in waves)
    want = []
    for r in roots:
        for w in waves:
            share = r // max(w, 1)
            want += [min(8192, max(512, 2 * share)) & ~63, min(2048, max(256, share // 4)) & ~63]
    assert [int(x) for x in run_cxx(tmp_path, body)] == want
