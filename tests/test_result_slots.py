"""The pool of pinned result slots (csrc/result_slots.h), compiled for the host
with an allocator of its own: no slot is handed out twice, a slot whose stream
could not be waited for is never handed out again, and a failed allocation is
tried again by the next call."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2206_11297_amd", "csrc")

DRIVER = r"""
#include "result_slots.h"
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <thread>
#include <vector>
using namespace rsz;
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s, line %d\n", #x, __LINE__); return 1; } } while (0)
static int allocs = 0, refuse = 1;
static void *page(size_t n) {
  ++allocs;
  if (refuse > 0) { --refuse; return nullptr; }
  return std::calloc(1, n);
}
int main() {
  ResultSlots slots(page);
  { Result r(slots); CHECK(!r.slot && allocs == 1); }          // refused: no slot
  { Result r(slots); CHECK(r.slot && allocs == 2); }           // and asked for again
  std::vector<std::unique_ptr<Result>> held;
  for (int i = 0; i < ResultSlots::kSlots; ++i) {
    held.emplace_back(new Result(slots));
    CHECK(held.back()->slot);
    for (int j = 0; j < i; ++j) CHECK(held[j]->slot != held[i]->slot);
  }
  CHECK(allocs == 2);
  { Result r(slots); CHECK(!r.slot); }                         // all taken
  ResultSlot *lost = held[5]->slot, *given = held[9]->slot;
  held[5]->abandon();                                          // still the device's
  held[5].reset();
  { Result r(slots); CHECK(!r.slot); }
  held[9].reset();
  { Result r(slots); CHECK(r.slot == given); }
  held.clear();
  for (int i = 0; i + 1 < ResultSlots::kSlots; ++i) {
    held.emplace_back(new Result(slots));
    CHECK(held.back()->slot && held.back()->slot != lost);
  }
  { Result r(slots); CHECK(!r.slot); }
  held.clear();
  std::atomic<int> bad{0};
  std::vector<std::thread> threads;
  for (int t = 0; t < 40; ++t)
    threads.emplace_back([&, t] {
      for (int k = 0; k < 2000; ++k) {
        Result r(slots);
        if (!r.slot) continue;
        r.slot->status = t;
        r.slot->bytes = (uint64_t)k;
        if (r.slot == lost || r.slot->status != t || r.slot->bytes != (uint64_t)k) ++bad;
      }
    });
  for (auto &t : threads) t.join();
  CHECK(bad == 0);
  std::puts("ok");
  return 0;
}
"""


def test_slots(tmp_path):
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-pthread",
                    "-fsanitize=thread", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
