"""The launch choices made from tuning records (csrc/tuning.h, compiled here
with the host compiler)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2103_10765_amd", "csrc")

MAIN = """
#include <cstdio>
#include <cstring>
#include "tuning.h"
// commands: "ht K search class shape", "bm K search class method split" (records),
// "shape K search tiles batch", "method K search tiles" (questions)
int main() {
  gbm3d::Tuning t;
  char tag[16];
  int a, b, c, d, e;
  while (std::scanf("%15s %d %d %d", tag, &a, &b, &c) == 4) {
    if (!std::strcmp(tag, "ht") && std::scanf("%d", &d) == 1) t.shapes[{a, b, c}] = {d, 0.1f};
    else if (!std::strcmp(tag, "bm") && std::scanf("%d %d", &d, &e) == 2) t.matching[{a, b, c}] = {d, e, 0.1f};
    else if (!std::strcmp(tag, "shape") && std::scanf("%d", &d) == 1) std::printf("%d\\n", gbm3d::choose_shape(t, a, b, c, d != 0));
    else if (!std::strcmp(tag, "method")) std::printf("%d\\n", gbm3d::choose_bm(t, 0, 0, b, c, a).method);
  }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "rules")], check=True)

    def run(*lines):
        r = subprocess.run([str(d / "rules")], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        return [int(x) for x in r.stdout.split()]
    return run


def test_shape_records_of_small_images_stay_with_them(ask):
    """A small image's shape 0 is a smaller tile than a batch's or a large
    image's: its record answers for single images of its class alone."""
    small = "ht 16 39 7 1"  # 128 .. 255 tiles of 4 x 4 references
    assert ask(small, "shape 16 39 200 0") == [1]
    assert ask(small, "shape 16 39 200 1", "shape 16 39 900 0", "shape 16 39 100000 0", "shape 16 39 100000 1") == [0] * 4
    large = "ht 16 39 12 1"
    assert ask(large, "shape 16 39 5000 0", "shape 16 39 5000 1", "shape 16 39 100000 0", "shape 16 39 200 1") == [1] * 4
    assert ask(large, "shape 16 39 200 0", "shape 16 21 5000 0", "shape 8 39 5000 0") == [0] * 3
    # the nearest of the records that may answer
    assert ask("ht 16 39 11 0", "ht 16 39 14 1", small, "shape 16 39 2500 1", "shape 16 39 40000 1", "shape 16 39 130 1") == [0, 1, 0]


def test_matching_method_without_records(ask):
    """The shift-wise kernel (1) for small windows on large images, else the
    correlation kernel (2); a record of the group size and window decides."""
    assert ask("method 16 39 30000", "method 8 13 30000", "method 8 11 3000", "method 8 5 1000") == [2] * 4
    assert ask("method 8 11 3001", "method 8 5 1001", "method 2 3 30000") == [1] * 3
    assert ask("bm 8 5 14 2 1", "method 8 5 20000", "method 8 5 500", "method 16 5 20000") == [2, 2, 1]
