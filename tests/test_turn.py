"""The turn that overlapping calls take on a graph's scratch (csrc/turn.h), with
streams and events that only note what was put on them: the work of all calls is
ordered on the device, whatever the streams, and no call names another's."""
import os
import shutil
import subprocess

import pytest

from paper_2311_12281_amd import build as B

FAKE_HIP = r"""
#pragma once
#include <cstdint>
enum hipError_t { hipSuccess = 0, hipErrorInvalidHandle = 400 };
struct Stream; struct Event;
using hipStream_t = Stream*;
using hipEvent_t = Event*;
#define hipStreamPerThread ((hipStream_t)2)
hipError_t hipEventRecord(hipEvent_t, hipStream_t);
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned);
hipError_t hipStreamSynchronize(hipStream_t);
"""

PROGRAM = r"""
#include "turn.h"
#include <atomic>
#include <chrono>
#include <cstdio>
#include <memory>
#include <thread>
#include <vector>

// An operation comes after the one before it on its stream, and after what it waits for.
struct Op { std::vector<int> after; int work; };
struct Stream { int last = -1; bool alive = true; bool synced = false; };
struct Event { int op = -1; };
static std::vector<Op> ops;
static int thread = 0;         // the thread that calls
static Stream per_thread[4];
static bool broken = false;    // a destroyed stream was named
static Stream* real(hipStream_t s) {
  Stream* r = s == hipStreamPerThread ? &per_thread[thread] : s;
  broken = broken || !r->alive;
  return r;
}
static int put(Stream* r, int work, int also = -1) {
  Op o{{}, work};
  if (r->last >= 0) o.after.push_back(r->last);
  if (also >= 0) o.after.push_back(also);
  ops.push_back(o);
  return r->last = (int)ops.size() - 1;
}
static bool fail_record = false;
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (fail_record) return hipErrorInvalidHandle;
  e->op = put(real(s), -1);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { put(real(s), -1, e->op); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { real(s)->synced = true; return hipSuccess; }

static bool before(int a, int b) {
  if (a == b) return true;
  for (int x : ops[(size_t)b].after)
    if (before(a, x)) return true;
  return false;
}

struct Call {  // one call's turn, on a thread
  int t;
  hipStream_t s;
  std::unique_ptr<scan::Turn> turn;
  int op = -1;
  Call(scan::TurnState& T, int t, hipStream_t s) : t(t), s(s) {
    thread = t;
    turn = std::make_unique<scan::Turn>(T, s, false);
    op = put(real(s), t);
    turn->enqueued();
  }
  void leave() {
    thread = t;
    turn->done();
    turn.reset();
  }
};

static int failures = 0;
static void expect(bool ok, const char* what) {
  if (!ok || broken) { std::printf("FAILED: %s\n", what); ++failures; }
}
static void start() {
  ops.clear();
  broken = false;
  for (auto& s : per_thread) s = Stream();
}

int main() {
  {  // each thread's own hipStreamPerThread
    start();
    Event e; scan::TurnState T; T.ev = &e;
    Call a(T, 0, hipStreamPerThread), b(T, 1, hipStreamPerThread), c(T, 2, hipStreamPerThread);
    expect(before(a.op, b.op) && before(b.op, c.op), "per-thread streams of three threads");
    a.leave(); b.leave(); c.leave();
  }
  {  // mixed with a stream of the caller's
    start();
    Event e; scan::TurnState T; T.ev = &e; Stream x;
    Call a(T, 0, hipStreamPerThread), b(T, 1, &x), c(T, 1, hipStreamPerThread);
    expect(before(a.op, b.op) && before(b.op, c.op), "a per-thread stream, then another");
    c.leave(); b.leave(); a.leave();
  }
  {  // the stream of a call that has left is gone while an earlier call is still counted
    start();
    Event e; scan::TurnState T; T.ev = &e; Stream x, y, z;
    Call a(T, 0, &x), b(T, 1, &y);
    b.leave();
    y.alive = false;
    Call c(T, 2, &z);
    expect(before(a.op, c.op), "after a destroyed stream");
    a.leave(); c.leave();
  }
  {  // calls that do not overlap wait for nothing
    start();
    Event e; scan::TurnState T; T.ev = &e; Stream x, y;
    { Call a(T, 0, &x); a.leave(); }
    Call b(T, 1, &y);
    expect(ops[(size_t)b.op].after.empty() && T.inflight == 1, "alone");
    b.leave();
    expect(T.inflight == 0, "left");
  }
  {  // a call that fails leaves no work behind on its stream
    start();
    Event e; scan::TurnState T; T.ev = &e; Stream x, y;
    fail_record = true;
    { scan::Turn a(T, &x, false); put(&x, 0); expect(a.enqueued() != hipSuccess, "record fails"); }
    fail_record = false;
    expect(x.synced && T.inflight == 0, "a failed record");
    for (bool hold : {false, true}) {
      y.synced = false;
      { scan::Turn a(T, &y, hold); put(&y, 0); a.enqueued(); }
      expect(y.synced && T.inflight == 0, "a call that never got to wait");
    }
  }
  {  // a call that holds its turn: the next one comes when it has left, and queues the third
    start();
    Event e; scan::TurnState T; T.ev = &e; Stream x, y, z;
    auto a = std::make_unique<scan::Turn>(T, &x, true);
    const int wa = put(&x, 0);
    expect(a->enqueued() == hipSuccess && e.op < 0, "no event while alone");
    std::atomic<bool> entered{false};
    std::atomic<int> step{0};
    int wb = -1;
    std::thread other([&] {
      scan::Turn b(T, &y, true);
      entered = true;
      wb = put(&y, 1);
      b.enqueued();
      step = 1;
      while (step != 2) std::this_thread::yield();
      b.done();
    });
    std::this_thread::sleep_for(std::chrono::milliseconds(50));
    expect(!entered, "the second waits for the first");
    x.synced = true;  // (the first call waits for its stream)
    a->done();
    a.reset();
    while (step != 1) std::this_thread::yield();
    expect(e.op >= 0, "the second records");
    { scan::Turn c(T, &z, true); const int wc = put(&z, 2); expect(before(wb, wc), "the third queues"); c.enqueued(); c.done(); }
    step = 2;
    other.join();
    expect(wa >= 0 && T.inflight == 0, "all left");
  }
  return failures ? 1 : 0;
}
"""


def test_turns_are_ordered(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(FAKE_HIP)
    (tmp_path / "turns.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "turns")
    subprocess.run([cxx, "-std=c++17", "-Wall", f"-I{tmp_path}", f"-I{B.CSRC}", str(tmp_path / "turns.cpp"), "-o", exe,
                    "-pthread"], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
