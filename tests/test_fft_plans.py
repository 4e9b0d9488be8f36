"""Every run-time FFT plan uses only radices that the stage lists of the line
transform hold: a radix missing there would fall to another one's case."""

import os
import re
import subprocess

import pytest

import stub_common

CSRC = os.path.join(stub_common.ROOT, "paper_1512_07295_amd", "csrc")

PROGRAM = '''
#include <hip/hip_runtime.h>
#include <cstdio>
#include "fft_line.hpp"
int main() {
  for (int L = 2; L <= 1024; ++L) {
    fsest::RtLine p;
    if (!fsest::make_rt_line(L, &p)) continue;
    printf("%d %d", p.L, p.tpl);
    for (int i = 0; i < p.nst; ++i) printf(" %d", p.radix[i]);
    printf("\\n");
  }
}
'''


def _lists():
    text = open(os.path.join(CSRC, "fft_line.hpp")).read()
    text = text[text.index("void line_fft_rt_io("):text.index("// Plan for length L")]
    found = {}
    for kind in ("FIRST", "MID", "LAST"):
        found[kind] = {int(r) for r in re.findall(r"FSEST_RT_%s\((\d+)\)" % kind, text)}
    assert "case 16: break;" in text and "case 16: rt_stage16" in text
    found["FIRST"].add(16)  # by way of LDS, as a middle stage
    found["MID"].add(16)
    return found


def test_plans_and_stage_lists(tmp_path):
    src, exe = tmp_path / "plans.hip", tmp_path / "plans"
    src.write_text(PROGRAM)
    hipcc = next((p for p in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc") if p and os.path.exists(p)), None)
    if hipcc is None:
        pytest.skip("no hipcc")
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True,
                   capture_output=True)
    lists, seen, lengths = _lists(), {"FIRST": set(), "MID": set(), "LAST": set()}, set()
    for line in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines():
        length, tpl, *radices = map(int, line.split())
        product = 1
        for r in radices:
            product *= r
        assert product == length and tpl == -(-length // 16)
        lengths.add(length)
        for i, r in enumerate(radices):
            # a line left in LDS ends with a middle stage too
            kinds = ["FIRST"] if i == 0 else (["MID", "LAST"] if i == len(radices) - 1 else ["MID"])
            for kind in kinds:
                assert r in lists[kind], (length, radices, kind)
                seen[kind].add(r)
    # every length of a grid axis or packed row that has no compile-time line has a plan
    for n in range(8, 1025, 4):
        for length in (n, n // 2):
            rest = length
            for p in (2, 3, 5):
                while rest % p == 0:
                    rest //= p
            if rest == 1 and length & (length - 1):
                assert length in lengths, length
    for kind in lists:  # and no list holds a radix that no plan has there, 2, 4 and 8 of short lines apart
        assert lists[kind] - seen[kind] <= {2, 4, 8}, kind
