"""Which of two kernels a short launch takes, by its tiles and by the slices that hold something: the rule of the header,
compiled for the CPU, against launches at which both were measured (GPU time, context-free calls and models without a list of slices)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2006_15704_amd", "csrc")

# (replicas, bytes of an element, staged, tiles, slices that hold something): slices took so much less (-) or more time than tiles, %
MEASURED = {
    (9, 4, False, 160, 668): -16, (9, 4, False, 190, 400): -5, (9, 4, False, 200, 397): 9, (9, 4, False, 205, 388): 6,
    (12, 4, False, 167, 940): -10, (12, 4, False, 190, 784): -13, (12, 4, False, 273, 933): 7,
    (16, 4, False, 190, 784): -13, (16, 4, False, 240, 956): 4, (16, 4, False, 273, 933): 15,
    (17, 4, False, 160, 668): -19, (17, 4, False, 200, 397): 22, (17, 4, False, 200, 680): 12,
    (24, 4, False, 140, 757): -24, (24, 4, False, 190, 400): -7, (24, 4, False, 200, 680): 14, (24, 4, False, 213, 923): 5,
    (24, 4, False, 273, 933): 11, (32, 4, False, 200, 680): 13, (64, 4, False, 140, 361): 9,
    (9, 2, False, 200, 680): -15, (9, 2, False, 234, 1291): -16, (12, 2, False, 262, 1433): 10, (12, 2, False, 288, 1412): 15,
    (16, 2, False, 212, 391): -11, (16, 2, False, 262, 1433): 4, (17, 2, False, 200, 398): 7, (17, 2, False, 320, 1403): 8,
    (20, 2, False, 212, 391): 7, (24, 2, False, 410, 1432): 25, (24, 2, False, 320, 1403): 11,
    (8, 4, True, 339, 1913): -12, (8, 4, True, 547, 1906): 16, (12, 4, True, 350, 1910): -9, (12, 4, True, 547, 1906): 15,
    (16, 4, True, 307, 1925): -16, (16, 4, True, 547, 1906): 17, (17, 4, True, 427, 1876): 9, (24, 4, True, 322, 1848): 6,
    (24, 4, True, 350, 1910): 8, (24, 4, True, 547, 1906): 16, (5, 2, True, 307, 1925): -10, (5, 2, True, 427, 1877): 14,
    (5, 2, True, 547, 1906): 34, (8, 2, True, 322, 1848): -12, (8, 2, True, 480, 1877): 12, (12, 2, True, 350, 1910): -9,
    (16, 2, True, 350, 1910): -10, (16, 2, True, 547, 1906): 22, (17, 2, True, 322, 1848): -8, (24, 2, True, 307, 1925): -7,
    (24, 2, True, 480, 1877): 4, (32, 2, True, 547, 1906): 19,
}


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_launches_without_a_list_take_slices_where_they_are_faster(tmp_path):
    points = list(MEASURED)
    rows = ",\n".join("{%d, %d, %s, %d, %d}" % (r, e, str(s).lower(), t, k) for r, e, s, t, k in points)
    source = tmp_path / "rules.cpp"
    source.write_text('#include "ddp_kernels.h"\n#include <cstdio>\nstruct P { int R, es; bool staged; long tiles, slices; };\n'
                      "int main() {\n    const P all[] = {\n" + rows + "};\n"
                      '    for (const P& p : all) std::printf("%d\\n", ddp::takes_slices(p.R, p.es, p.staged, p.tiles, p.slices, false) ? 1 : 0);\n}\n')
    exe = str(tmp_path / "rules")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    build = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-isystem", os.path.join(rocm, "include"),
                            "-o", exe, str(source)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout
    taken = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60).stdout.split()
    wrong = [(p, MEASURED[p]) for p, t in zip(points, taken) if int(t) != (MEASURED[p] < 0)]
    assert len(taken) == len(points) and not wrong, wrong
