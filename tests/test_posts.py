"""The words that control kernels post checks to, as the host reads them (compiled here; no GPU)."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_01596_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "posts.hpp"
using ffcz::PostWords;

static unsigned long long word(unsigned long long tag, int done, unsigned checks) {
  return (tag << 40) | ((unsigned long long)done << 32) | checks;
}
#define CHECK(c) \
  if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; }

int main() {
  unsigned long long mem[8] = {0};
  PostWords w;
  w.p = mem;
  w.n = 8;
  w.begin(8);
  CHECK(w.tag == 1);
  CHECK(w.read(7).checks == 0 && !w.read(7).done);
  for (int i = 0; i < 8; ++i) mem[i] = word(w.tag, i & 1, 3u + i);
  CHECK(w.read(2).checks == 5 && !w.read(2).done);
  CHECK(w.read(7).checks == 10 && w.read(7).done);
  mem[0] = word(w.tag, 1, 0xffffffffu >> 1);
  CHECK(w.read(0).checks == 0x7fffffff && w.read(0).done);
  // small calls until the tag of the batch of eight comes round again: the words that only the
  // batch used must not read as this call's
  for (int k = 0; k < 0xffffff - 1; ++k) {
    w.begin(1);
    mem[0] = word(w.tag, 1, 1);
  }
  CHECK(w.tag == 0xffffff);
  w.begin(8);
  CHECK(w.tag == 1);
  for (int i = 0; i < 8; ++i) CHECK(w.read(i).checks == 0 && !w.read(i).done);
  // a late post of a call before (another tag) does not count either
  mem[3] = word(0xffffff, 1, 9);
  CHECK(w.read(3).checks == 0 && !w.read(3).done);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_words_of_earlier_calls_are_never_taken_for_this_ones(tmp_path):
    src, exe = tmp_path / "posts.cpp", tmp_path / "posts"
    src.write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=100)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout
