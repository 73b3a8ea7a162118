"""The rule that chooses the kernel and the shape of an fp32 attention launch (csrc/attend_f32_choice.hpp, the code the dispatch runs) built
for the CPU: which form each launch of the GPU tests takes, that every form that is built is taken by some launch, and that none is
taken that is not built."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "attend_f32_choice.hpp"
int main() {
  int d, q, k;
  long long bh;
  float scale;
  while (std::scanf("%d %lld %d %d %f", &d, &bh, &q, &k, &scale) == 5) {
    const amskv::F32Choice c = amskv::choose_f32(d, bh, q, k, scale);
    std::printf("%d %d %d\n", c.parts, c.qt, c.split);
  }
}
"""
# (head dim, row groups of the kernel in parts or 0, rows of a unit, slices)
BUILT = {(64, 0, 16, 1), (64, 0, 16, 2), (64, 0, 16, 4), (64, 0, 16, 8), (64, 0, 32, 2), (64, 0, 32, 4), (64, 0, 32, 8),
         (64, 4, 32, 1), (64, 4, 32, 2), (64, 8, 32, 1),
         (128, 0, 16, 1), (128, 0, 16, 2), (128, 0, 16, 4), (128, 0, 16, 8), (128, 4, 32, 1)}


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("choice")
    src, exe = str(d / "choice.cpp"), str(d / "choice")
    with open(src, "w") as f:
        f.write(PROGRAM)
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-I" + os.path.join(ROOT, "paper_2511_16047_amd", "csrc"), src, "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert b.returncode == 0, b.stdout[-4000:]

    def ask(launches, scale=0.125):
        r = subprocess.run([exe], input="".join("%d %d %d %d %r\n" % (*x, scale) for x in launches), stdout=subprocess.PIPE, text=True,
                           timeout=120, check=True)
        return [(x[0],) + tuple(int(y) for y in line.split()) for x, line in zip(launches, r.stdout.splitlines())]

    return ask


def test_every_form_that_is_built_and_no_other(choose):
    launches = [(d, bh, q, q + more) for d in (64, 128) for bh in (1, 2, 3, 7, 16, 24, 48, 100, 256, 480, 1000, 4000)
                for q in (1, 9, 16, 17, 25, 32, 33, 64, 65, 100, 169, 256, 400, 576, 676, 1024, 1302, 2500) for more in (0, 1, 60, 300, 3000, 12000)]
    forms = choose(launches)
    assert set(forms) == BUILT
    for (d, bh, q, k), f in zip(launches, forms):
        assert f != (64, 0, 16, 1) or q <= 64      # that one has a workgroup per (b,h)
        assert f[1] == 0 or q > 32
    assert all(f[1] == 0 for f in choose(launches, 2.0 ** 31))


# head dim, (b,h), queries, keys of test_gpu_f32_parts.py (magnitudes, tiny beside ordinary, token-major) and of the cases of
# test_gpu_f32_precision.py that are there for the kernel in parts
@pytest.mark.parametrize("launch,form", [
    ((64, 256, 255, 321), (8, 32, 1)), ((64, 300, 127, 128), (4, 32, 1)), ((64, 304, 127, 128), (4, 32, 1)), ((64, 48, 577, 579), (4, 32, 2)),
    ((128, 256, 200, 263), (4, 32, 1)),
    ((64, 256, 255, 258), (8, 32, 1)), ((64, 256, 65, 131), (8, 32, 1)), ((64, 64, 257, 457), (4, 32, 2)), ((128, 256, 255, 258), (4, 32, 1)),
    ((128, 48, 577, 579), (4, 32, 1)), ((128, 64, 257, 457), (4, 32, 1)), ((128, 256, 65, 131), (4, 32, 1)),
    ((64, 16, 257, 457), (0, 16, 8)), ((128, 16, 257, 457), (0, 16, 4))])
def test_launches_of_the_gpu_tests(choose, launch, form):
    assert choose([launch]) == [(launch[0],) + form]


def test_steps_of_the_gpu_test_of_forms(choose):
    """test_forms of test_gpu_f32_parts.py, its layer that keeps everything: every shape of the kernel in parts, several times."""
    taken = choose([(d, bh, t, sum(tokens[: s + 1])) for d in (64, 128) for bh in (104, 152, 304, 259)
                    for tokens in ((31, 97, 129, 64, 256, 255, 33, 160, 1), (127, 65, 225, 257, 63)) for s, t in enumerate(tokens)])
    assert all(taken.count(f) >= 4 for f in BUILT if f[1])
