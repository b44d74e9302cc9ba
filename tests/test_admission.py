"""Admission of solver launches to one device (kf_admit.h), without a device: a
host program runs the rule over simulated streams, whose launches wait for the
waits before them and else start and end whenever a seeded draw says so."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <vector>
#include "kf_admit.h"

struct Mark { bool done = false; struct Queue* on = nullptr; };
struct Op { enum { WAIT, SOLVE, RECORD } kind; std::shared_ptr<Mark> mark; int blocks, per_cu; };
struct Queue { std::vector<Op> ops; size_t head = 0; bool running = false, capturing = false, gone = false; };

struct SimOps {
  using Stream = Queue*;
  using Event = std::shared_ptr<Mark>;
  static int events, waits, dangling;
  static Queue own;
  void use(Event& e) { dangling += e->on && e->on->gone; }   // an event of a stream that is gone
  bool create(Event& e) { ++events; e = std::make_shared<Mark>(); e->done = true; return true; }
  void destroy(Event& e) { --events; e.reset(); }
  bool record(Event& e, Queue* q) {
    if (q->capturing) return false;
    e = std::make_shared<Mark>();   // a wait made before keeps the mark that it saw
    e->on = q;
    q->ops.push_back({Op::RECORD, e, 0, 0});
    return true;
  }
  bool done(Event& e) { use(e); return e->done; }
  bool wait(Queue* q, Event& e) { use(e); ++waits; q->ops.push_back({Op::WAIT, e, 0, 0}); return true; }
  bool idle(Queue* q) { return !q->capturing && q->head == q->ops.size(); }
  bool detach(Event& e) { return wait(&own, e) && record(e, &own); }
  bool same(Queue* a, Queue* b) { return a == b; }
  bool capturing(Queue* q) { dangling += q->gone; return q->capturing; }
};
int SimOps::events = 0, SimOps::waits = 0, SimOps::dangling = 0;
Queue SimOps::own;
using Adm = kf::Admission<SimOps>;

int main(int argc, char** argv) {
  const unsigned seed = atoi(argv[1]);
  const bool rule = atoi(argv[2]) != 0;
  std::mt19937 rng(seed);
  auto draw = [&](int n) { return (int)(rng() % n); };
  const int cus = 256, streams = 1 + draw(6);
  Adm adm(cus);
  std::vector<Queue*> q;          // every stream there ever was
  std::vector<Queue*> live(streams);
  for (Queue*& s : live) q.push_back(s = new Queue());
  q.push_back(&SimOps::own);
  std::vector<Adm::Lane*> lane(streams, nullptr);
  int worst = 0, over = 0, solved = 0, stuck = 0;
  long left = 2000;
  auto solves = [&](int& n, int& least) {   // in flight on the device now
    n = 0; least = 1 << 20;
    int teams = 0;
    for (Queue* s : q)
      if (s->running) { ++teams; n += s->ops[s->head].blocks; least = std::min(least, s->ops[s->head].per_cu); }
    return teams;
  };
  while (left > 0 || stuck == 0) {
    if (left > 0 && draw(3) == 0) {   // the program enqueues
      --left;
      const int i = draw(streams);
      Queue& s = *live[i];
      if (draw(40) == 0 && (s.capturing || s.head == s.ops.size())) s.capturing = !s.capturing;
      if (streams > 1 && draw(60) == 0 && lane[i]) {   // its last context goes, and then the stream
        adm.leave(lane[i], draw(2) && s.head == s.ops.size());
        lane[i] = nullptr;
        s.gone = true;
        q.push_back(live[i] = new Queue());
        continue;
      }
      const int blocks = 1 + draw(draw(4) == 0 ? 512 : 256), per_cu = 1 + draw(6);
      auto go = [&] { if (!s.capturing) s.ops.push_back({Op::SOLVE, nullptr, std::min(blocks, per_cu * cus), per_cu}); return 0; };
      if (!lane[i]) lane[i] = adm.join(&s);
      if (rule) { if (adm.launch(lane[i], std::min(blocks, per_cu * cus), per_cu, 0, 1, go)) return 3; }
      else go();
    } else {   // the device goes on at one stream
      bool any = false;
      for (int k = 0, n = (int)q.size(), i = draw(n); k < n; ++k, i = (i + 1) % n) {
        Queue& s = *q[i];
        if (s.head == s.ops.size()) continue;
        Op& op = s.ops[s.head];
        if (op.kind == Op::WAIT && !op.mark->done) continue;
        any = true;
        if (op.kind == Op::RECORD) op.mark->done = true;
        if (op.kind == Op::SOLVE && !s.running) {
          s.running = true;
          ++solved;
          int n, least;
          if (solves(n, least) > 1) { worst = std::max(worst, n); over += n > adm.places(least); }
          break;
        }
        s.running = false;
        ++s.head;
        break;
      }
      if (!any && left <= 0) stuck = 1;
    }
  }
  int unfinished = 0;
  for (Queue* s : q) unfinished += s->head != s->ops.size();
  for (Adm::Lane* l : lane) if (l) adm.leave(l, true);
  printf("streams %d solved %d over %d unfinished %d waits %d worst %d dangling %d\n", streams, solved, over, unfinished,
         SimOps::waits, worst, SimOps::dangling);
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("admission")
    src, exe = d / "sim.cpp", d / "sim"
    src.write_text(PROGRAM)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-pthread", "-I", os.path.join(ROOT, "paper_2207_12244_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    return str(exe)


def _run(program, seed, rule):
    out = subprocess.run([program, str(seed), str(int(rule))], capture_output=True, text=True, check=True, timeout=60)
    w = out.stdout.split()
    return {w[i]: int(w[i + 1]) for i in range(0, len(w), 2)}


def test_solves_on_different_streams_fit_together(program):
    """Whatever the order in which streams make progress, the solves on the device
    at one time have places for all their workgroups, and every launch comes to
    its end; without the rule they do not fit. No event is used after the stream
    that it was recorded on is gone."""
    broken = 0
    for seed in range(200):
        r = _run(program, seed, True)
        assert r["over"] == 0 and r["unfinished"] == 0 and r["dangling"] == 0, (seed, r)
        if r["streams"] == 1:
            assert r["waits"] == 0, (seed, r)
        broken += _run(program, seed, False)["over"] > 0
    assert broken > 100
