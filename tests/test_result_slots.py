"""The slots of host memory that the reductions' results take (one per call
in flight, result_slots.h), built for the host."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r'''
#include "paper_1909_01580_amd/csrc/result_slots.h"
#include <atomic>
#include <cstdio>
#include <set>
#include <thread>
#include <vector>
static double block[64 * 8];
static int allocated = 0;
static double* some() { ++allocated; return block; }
static double* none() { return nullptr; }
static hgks::ResultSlots<some> slots;
static hgks::ResultSlots<none> empty;
static std::atomic<int> owner[64];
int main() {
  // any number of calls one after another
  for (int i = 0; i < 1000; ++i) {
    double* p = slots.take();
    if (!p) return 1;
    slots.give(p);
  }
  // 64 at a time, each its own; none is left for the next, and one given back is
  std::set<double*> held;
  for (int i = 0; i < 64; ++i) held.insert(slots.take());
  if (held.size() != 64 || held.count(nullptr) || slots.take()) return 2;
  for (double* p : held)
    if (p < block || p >= block + 64 * 8 || (p - block) % 8) return 3;
  slots.give(block + 8 * 17);
  if (slots.take() != block + 8 * 17 || slots.take()) return 4;
  for (double* p : held) slots.give(p);
  // no block: no slots, and nothing to give back
  if (empty.take()) return 5;
  empty.give(nullptr);
  slots.give(nullptr);
  // threads never share one
  std::atomic<int> bad{0};
  std::vector<std::thread> t;
  for (int k = 1; k <= 16; ++k)
    t.emplace_back([&, k] {
      for (int i = 0; i < 20000; ++i) {
        double* p = slots.take();
        if (!p) { ++bad; continue; }
        auto& o = owner[(p - block) / 8];
        int free = 0;
        if (!o.compare_exchange_strong(free, k)) ++bad;
        o = 0;
        slots.give(p);
      }
    });
  for (auto& x : t) x.join();
  if (bad || allocated != 1) return 6;
  printf("ok\n");
  return 0;
}
'''


def test_slots(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    src = tmp_path / "slots.cpp"
    src.write_text(HARNESS)
    exe = str(tmp_path / "slots")
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", "-I", ROOT, "-o", exe, str(src)], check=True,
                   capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", (out.returncode, out.stdout)
