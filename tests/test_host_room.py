"""The rule that shares out the backward workspace (csrc/room.h), with an allocator that refuses sizes above a limit: what
is refused once is not asked for again, and a workspace that graphs hold addresses in is replaced only where it
has to be."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2304_14698_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "room.h"
// limit, then per call: fixed least most stay; prints per call: status, room, workspace's size, times it was replaced
int main(int argc, char **argv) {
  const size_t limit = strtoull(argv[1], nullptr, 10);
  size_t have = 0, room = 0;
  bool refused = false;
  for (int i = 2; i + 3 < argc; i += 4) {
    int replaced = 0;
    auto grow = [&](size_t bytes) -> int {
      if (bytes <= have) return 0;
      ++replaced;
      have = 0;
      if (bytes > limit) return -8;
      have = bytes;
      return 0;
    };
    const int rc = fit_room(have, strtoull(argv[i], nullptr, 10), strtoull(argv[i + 1], nullptr, 10), strtoull(argv[i + 2], nullptr, 10),
                            atoi(argv[i + 3]) != 0, -8, &refused, &room, grow);
    printf("%d %zu %zu %d\n", rc, room, have, replaced);
  }
}
"""


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    d = tmp_path_factory.mktemp("room")
    (d / "room.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(d / "room"), str(d / "room.cpp")], check=True)

    def run(limit, *c):
        out = subprocess.run([str(d / "room"), str(limit)] + [str(x) for call in c for x in call], check=True, capture_output=True, text=True)
        return [tuple(int(x) for x in line.split()) for line in out.stdout.splitlines()]
    return run


A = (1024, 512, 8192, 0)       # a batch whose room does not fit ...
B = (512, 256, 1 << 20, 0)     # ... a smaller one, whose room would not either, and a larger one
C = (4096, 1024, 1 << 20, 0)


def test_refused_room_is_not_asked_for_again(calls):
    first, second, smaller, again = calls(6000, A, A, B, A)
    assert first == (0, 512, 1536, 2)
    assert second == (0, 512, 1536, 0)
    assert smaller == (0, 1024, 1536, 0)                      # all that is there
    assert again == (0, 512, 1536, 0)


def test_larger_batch_after_a_refusal_grows_to_what_it_needs(calls):
    assert calls(6000, A, C, C, A) == [(0, 512, 1536, 2), (0, 1024, 5120, 1), (0, 1024, 5120, 0), (0, 4096, 5120, 0)]
    assert calls(4000, A, C)[1][0] == -8                      # not even the least


def test_workspace_of_graphs_stays(calls):
    stay = lambda c: c[:3] + (1,)
    assert calls(1 << 30, A, stay(B), stay(A)) == [(0, 8192, 9216, 1), (0, 8704, 9216, 0), (0, 8192, 9216, 0)]
    assert calls(1 << 30, A, stay(C))[1] == (0, 5120, 9216, 0)
    assert calls(1 << 30, B, C, A) == [(0, 1 << 20, (1 << 20) + 512, 1), (0, 1 << 20, (1 << 20) + 4096, 1), (0, 8192, (1 << 20) + 4096, 0)]


def test_exact_room(calls):
    assert calls(1 << 20, (1000, 300, 300, 1), (1000, 300, 300, 1)) == [(0, 300, 1300, 1), (0, 300, 1300, 0)]
    assert calls(1000, (1000, 300, 300, 0)) == [(-8, 300, 0, 1)]
