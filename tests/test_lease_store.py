"""The store of host objects that batched runs take their streams and
page-locked memory from (csrc/lease.h), compiled with the host compiler: calls
from many short-lived threads leave a bounded number of objects, calls at the
same time never share one, and a call gets only an object that fits it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1304_4334_amd", "csrc")

HARNESS = r"""
#include <atomic>
#include <stdio.h>
#include <thread>
#include "lease.h"
struct Obj { int kind; std::atomic<int> users{0}; };
static std::atomic<int> made{0}, live{0}, most{0}, shared{0}, misfit{0};
static smc::LeaseStore<Obj> store(4);
static void call(int kind) {
  Obj *x = store.take([&](const Obj &o) { return o.kind == kind; });
  if (!x) {
    x = new Obj;
    x->kind = kind;
    ++made;
    const int n = ++live;
    int m = most;
    while (n > m && !most.compare_exchange_weak(m, n)) {}
  }
  if (x->users++ != 0) ++shared;
  if (x->kind != kind) ++misfit;
  std::this_thread::yield();
  --x->users;
  if (Obj *out = store.give(x)) { delete out; --live; }
}
int main() {
  for (int i = 0; i < 200; ++i) std::thread([] { call(0); }).join();
  printf("%d %d ", made.load(), live.load());
  std::thread t[8];
  for (int k = 0; k < 8; ++k)
    t[k] = std::thread([k] { for (int i = 0; i < 20000; ++i) call((k + i) % 6); });
  for (auto &x : t) x.join();
  printf("%d %d %d %d\n", live.load(), most.load(), shared.load(), misfit.load());
  return 0;
}
"""


def test_store_is_bounded_and_never_shares(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    cpp, exe = tmp_path / "l.cpp", tmp_path / "l"
    cpp.write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", CSRC, "-o", str(exe), str(cpp)],
                   check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    made, live, left, most, shared, misfit = map(int, out.split())
    assert made == 1 and live == 1     # 200 threads, one call at a time
    assert left <= 4                   # idle ones kept
    assert most <= 8 + 4 + 8           # calls at a time, idle ones, ones on their way out
    assert shared == 0 and misfit == 0
