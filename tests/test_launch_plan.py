"""The host's choice of launch sequences (gsi_launch_plan.h), compiled by itself and run against a
model of the device: an iteration that needs the full sequence makes a short one hold, and the
launches behind a hold return at once."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_10379_amd", "csrc")

DRIVER = r"""
#include "gsi_launch_plan.h"
using namespace gsi;
// needs[i]: iteration i asks for an explicit A X or takes no step. Returns the launched sequences.
extern "C" int run(const unsigned char* needs, int n, int every, int short_ok, int* full, int* polls) {
  LaunchPlan plan(every, short_ok != 0);
  int k = 0, launched = 0;
  *full = *polls = 0;
  bool lead_due = true;  // the gradient is not current
  while (k < n) {
    const Batch b = plan.next(n - k);
    bool held = false;
    if (b.count < 1 || b.count > n - k) return -1;
    for (int j = 0; j < b.count; ++j) {
      const Sequence q = j ? b.rest : b.first;
      ++launched;
      *full += q != SEQ_LEAN;
      if (held) continue;
      if (q == SEQ_LEAN && lead_due) return -2;  // a short sequence from a state that it cannot take
      lead_due = needs[k] != 0;
      if (lead_due && q != SEQ_FULL) held = true;
      ++k;
    }
    ++*polls;
    plan.ran(b, held);
  }
  return launched;
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Werror", "-I", CSRC,
                           str(d / "driver.cpp"), "-o", str(d / "driver.so")])
    lib = ctypes.CDLL(str(d / "driver.so"))

    def go(needs, every, short_ok=True):
        full, polls = ctypes.c_int(), ctypes.c_int()
        n = lib.run(bytes(needs), len(needs), every, int(short_ok), ctypes.byref(full), ctypes.byref(polls))
        return n, full.value, polls.value

    return go


@pytest.mark.parametrize("every", [1, 3, 25])
@pytest.mark.parametrize("n", [1, 7, 25, 26, 400])
def test_no_hold_launches_one_full_sequence(run, n, every):
    assert run([0] * n, every) == (n, 1, -(-n // every))
    assert run([0] * n, every, short_ok=False) == (n, n, -(-n // every))


@pytest.mark.parametrize("every", [1, 3, 25])
def test_holds_in_every_iteration_waste_a_logarithmic_number_of_launches(run, every):
    n = 4000
    launched, _, polls = run([1] * n, every)
    doublings = (n // every).bit_length()
    assert launched <= n + every * (doublings + 1)
    assert polls <= n // every + 3 * (doublings + 1)


@pytest.mark.parametrize("every", [1, 3, 25])
@pytest.mark.parametrize("at", [0, 10, 24, 25, 30, 60])
def test_single_hold(run, at, every):
    """The launches behind the hold, and one batch of full sequences after it."""
    n = 400
    needs = [0] * n
    needs[at] = 1
    launched, full, _ = run(needs, every)
    assert launched <= n + every - 1
    assert full <= 1 + 1 + every


def test_holds_now_and_then(run):
    """One in 200 iterations: the short sequence stays the rule."""
    n = 10000
    launched, full, _ = run([int(i % 200 == 199) for i in range(n)], 25)
    assert launched <= n + 24 * (n // 200)
    assert full <= n // 4
