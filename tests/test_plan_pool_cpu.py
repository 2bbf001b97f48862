"""The memory that compression plans hand on to one another (csrc/plan_pool.h).  When it counts as free, on queues simulated on the CPU: never before all
work that was marked as reading it has run, also where two queues answer to one handle: the per-thread handle in two
threads, and the handle of a destroyed stream that comes back for a new one.  And which block a plan takes: plans of changing sizes settle on blocks of their
own instead of replacing each other's."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_04802_amd", "csrc")
MODEL = r"""
#include <cstdint>
#include <memory>
#include <random>
#include <vector>
#include "plan_pool.h"
// A queue is a row of operations, each with what it waits for; an event is one operation of one queue.  Handle 0 is the
// per-thread queue, the others name whatever queue they were last bound to.
struct Queue;
struct Op { Queue *q = nullptr; size_t at = 0; };
struct Queue { std::vector<Op> needs; size_t ran = 0; };
static std::vector<std::unique_ptr<Queue>> queues;
static Queue *bound[8];
static Queue *fresh() { queues.emplace_back(new Queue); return queues.back().get(); }
struct PerThread { Queue *q; PerThread() : q(fresh()) {} };
static Queue *of(int st) {
  if (st) return bound[st];
  thread_local PerThread own;
  return own.q;
}
static Op launch(int st, Op needs = {}) { Queue *q = of(st); q->needs.push_back(needs); return {q, q->needs.size()}; }
static bool ran(const Op &o) { return !o.q || o.q->ran >= o.at; }
static bool step(Queue *q) {                       // the next operation, if there is one and it waits for nothing
  if (q->ran == q->needs.size() || !ran(q->needs[q->ran])) return false;
  ++q->ran;
  return true;
}
struct Gpu {
  struct Event { bool made = false; Op op; bool operator!() const { return !made; } };
  typedef int Stream;
  static bool per_thread(int st) { return st == 0; }
  static bool create(Event *e) { e->made = true; return true; }
  static bool wait(int st, const Event &e) { launch(st, e.op); return true; }
  static bool record(Event &e, int st) { e.op = launch(st); return true; }
  static bool done(const Event &e) { return ran(e.op); }
};
// random programs: launch a reader and mark it, rebind a handle, run a random queue; a new thread for every piece of the
// program.  0, or 1: free while a reader has not run, 2: not free though every operation has run
extern "C" int random_programs(int seed, int handles) {
  std::mt19937 r(seed);
  for (int trial = 0; trial < 300; ++trial) {
    queues.clear();
    for (Queue *&b : bound) b = fresh();
    reslim::UseMarks<Gpu> marks;
    std::vector<Op> readers;
    int bad = 0;
    bool kept = true;
    auto piece = [&]() {
      for (int i = 0; i < 8 && kept && !bad; ++i) {
        const int st = r() % handles, what = r() % 8;
        if (what < 3) {
          readers.push_back(launch(st));
          kept = marks.add(st);
        } else if (what < 4 && st) {
          bound[st] = fresh();
        } else {
          step(queues[r() % queues.size()].get());
        }
        bool all = true;
        for (const Op &o : readers) all = all && ran(o);
        if (kept && marks.done() && !all) bad = 1;
      }
    };
    for (int k = 0; k < 4; ++k) std::thread(piece).join();      // one after the other: a thread's id may be the last one's
    std::thread a([&] { piece(); std::thread(piece).join(); piece(); });
    a.join();
    if (bad) return bad;
    for (bool any = true; any;) {
      any = false;
      for (auto &q : queues) any = step(q.get()) || any;
    }
    if (kept && !marks.done()) return 2;
  }
  return 0;
}
// one queue that marks often takes one mark; as many queues as there are marks can be told apart, one more is refused
extern "C" int bounded() {
  queues.clear();
  for (Queue *&b : bound) b = fresh();
  reslim::UseMarks<Gpu> marks;
  for (int i = 0; i < 100; ++i)
    if (!marks.add(1) || marks.n != 1) return 1;
  for (int st = 2; st <= marks.kMost; ++st)
    if (!marks.add(st) || marks.n != st) return 2;
  if (marks.add(marks.kMost + 1)) return 3;
  return marks.add(2) && marks.n == marks.kMost ? 0 : 4;
}
// plans of sizes[0 .. n) in turn, each given back before the next is made; blocks allocated in the second half of the run
extern "C" int allocations(const int *sizes, int n, int passes, int busy_every) {
  constexpr int kMost = 4;
  std::vector<reslim::KeptBlock> kept;
  int made = 0;
  for (int i = 0; i < n * passes; ++i) {
    const size_t bytes = sizes[i % n];
    for (size_t k = 0; k < kept.size(); ++k) kept[k].done = !busy_every || (i + k) % busy_every != 0;
    const int c = reslim::choose_block(kept.data(), static_cast<int>(kept.size()), kMost, bytes);
    if (c < -1 || c >= static_cast<int>(kept.size()) || (c < 0 && kept.size() == kMost)) return -1;
    reslim::KeptBlock b{0, true};
    if (c >= 0) {
      b = kept[c];
      for (const auto &o : kept)      // a finished block that fits is never passed over for a worse one
        if (o.done && o.cap >= bytes && (!b.done || b.cap < bytes || b.cap > o.cap)) return -2;
      kept.erase(kept.begin() + c);
    } else {
      for (const auto &o : kept)
        if (o.done && o.cap >= bytes) return -3;
    }
    if (b.cap < bytes) {
      b.cap = bytes + bytes / 4;
      made += i >= n * passes / 2;
    }
    if (kept.size() == kMost) return -4;
    kept.push_back(b);
  }
  return made;
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("marks")
    src, so = d / "marks.cpp", d / "marks.so"
    src.write_text(MODEL)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", "-I", CSRC, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("handles", [1, 2, 4])
@pytest.mark.parametrize("seed", range(4))
def test_a_block_is_free_only_when_its_readers_have_run(model, seed, handles):
    assert model.random_programs(seed, handles) == 0


def test_marks_are_bounded(model):
    assert model.bounded() == 0


@pytest.mark.parametrize("sizes", [[100], [1000, 10], [10, 1000], [10, 100, 1000], [10, 10000, 100, 1000], [7, 900, 30, 30, 5000, 8]])
def test_changing_sizes_settle(model, sizes):
    a = (ctypes.c_int * len(sizes))(*sizes)
    assert model.allocations(a, len(sizes), 40, 0) == 0
    for busy_every in (2, 3, 5):
        assert model.allocations(a, len(sizes), 40, busy_every) >= 0
