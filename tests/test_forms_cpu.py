"""Which shapes run in the Gram form (csrc/ocd_forms.h), compiled for the host: the benchmark's
copy of the rule is the library's, and the gradients' rule takes part of detection's."""

import os
import shutil
import subprocess

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [(B, U, W, S, K) for B in (16, 24, 64, 128, 200, 256, 257, 512) for U in (1, 4, 5, 8, 9, 10, 12, 16, 17, 24, 32)
          for W in (1, 256, 300, 513, 2049, 5000) for S in (1, 2, 3, 4, 5, 8, 9, 16, 17, 33) for K in (1, 2, 3, 4, 6, 20)]

PROGRAM = r"""
#include <cstdio>
#include "ocd_forms.h"
int main()
{
    int B, U, W, S, K;
    while (std::scanf("%d %d %d %d %d", &B, &U, &W, &S, &K) == 5)
        if (U == 0) std::printf("%ld\n", ocd::groups_per_launch(B, W));   // blocks, -, threads
        else std::printf("%d %d\n", (int)ocd::gram_form(B, U, W, S, K), (int)ocd::gram_gradient(B, U, W, S, K));
}
"""


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("forms")
    (d / "forms.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-I" + os.path.join(ROOT, "paper_1611_08779_amd", "csrc"),
                    str(d / "forms.cpp"), "-o", str(d / "forms")], check=True)

    def run(shapes):
        text = "\n".join(" ".join(map(str, s)) for s in shapes)
        out = subprocess.run([str(d / "forms")], input=text, capture_output=True, text=True, check=True)
        return [tuple(int(x) for x in line.split()) for line in out.stdout.splitlines()]
    return run


def test_the_benchmarks_rule_is_the_librarys(forms):
    for shape, (det, _) in zip(SHAPES, forms(SHAPES)):
        assert bench.gram_form(*shape) == bool(det), shape


def test_gradients_are_in_the_gram_form_on_fewer_shapes(forms):
    few = forms([(B, U, 1, S, K) for B, U, _, S, K in SHAPES])
    for shape, (_, grad), (base, _) in zip(SHAPES, forms(SHAPES), few):
        assert base or not grad, shape


@pytest.mark.parametrize("shape,det,grad", [
    # B, U, W, S, K: either side of the lines, by what was measured at them
    ((128, 8, 1200, 14, 3), True, True), ((128, 16, 2048, 4, 4), True, True),
    ((64, 8, 300, 14, 3), True, True), ((64, 8, 1000, 14, 2), True, False),
    ((100, 12, 585, 14, 2), True, False), ((100, 12, 500, 14, 2), True, True),
    ((32, 8, 1000, 17, 2), True, False), ((128, 24, 988, 17, 2), False, False),
    ((128, 24, 123, 17, 2), True, True), ((256, 32, 988, 17, 4), True, True),
    ((64, 9, 5600, 3, 4), False, False), ((64, 9, 2300, 3, 4), True, True),
    ((32, 8, 6000, 4, 4), True, False), ((128, 8, 6000, 4, 4), True, True),
    ((64, 8, 230000, 3, 4), True, False), ((64, 16, 230000, 2, 4), True, True), ((512, 20, 150, 14, 1), False, False),
])
def test_shapes_beside_the_lines(forms, shape, det, grad):
    assert forms([shape]) == [(det, grad)]


@pytest.mark.parametrize("blocks", [1, 2, 3, 63, 1 << 20])
@pytest.mark.parametrize("threads", [64, 128, 256])
def test_a_launch_stays_below_2_to_the_32_threads(forms, blocks, threads):
    (groups,), = forms([(blocks, 0, threads, 0, 0)])
    assert groups * blocks * threads < 2**32 <= (groups + 1) * blocks * threads
