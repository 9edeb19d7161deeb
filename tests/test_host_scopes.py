"""CPU: the scopes that the solver sets state for are left as they were found, also by an exception (a
failed launch while sweeps are timed).  Compiled from the library's own header."""

import os
import subprocess

import pytest

from paper_2604_26518_amd import build as b

PROGRAM = r"""
#include <cstdio>
#include "common.h"
using namespace gmt;
static int bad = 0;
static void expect(bool ok, const char* what) {
  if (!ok) std::printf("%s\n", what), bad = 1;
}
int main() {
  Hier h;
  int cb = 0, xcd = 1;
  try {
    const Solving timing(h);
    const Trial trial(cb, xcd);
    cb = 5, xcd = 0;
    throw 1;
  } catch (int) {
  }
  expect(!h.solving, "a failure outside a solve leaves `solving` set");
  expect(cb == 0 && xcd == 1, "a failure keeps the shape that was being timed");
  {
    const Solving solve(h);
    { const Solving timing(h); }
    expect(h.solving, "timing inside a solve ends it");
  }
  expect(!h.solving, "a solve leaves `solving` set");
  return bad;
}
"""


def test_scopes_restore_what_they_set(tmp_path):
    try:
        cc = b.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    src = tmp_path / "scopes.hip"
    src.write_text(PROGRAM)
    exe = tmp_path / "scopes"
    subprocess.run([cc, "-std=c++17", "-O1", "--cuda-host-only", "-I", os.path.join(b.ROOT, "include"), "-I", b.CSRC,
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
