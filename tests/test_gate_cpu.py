"""The order among launches whose workgroups wait for each other (csrc/gate.hpp), on a model device: what
runs together fits the device, nothing waits in a circle, and calls enter in the order they came."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), 'paper_2412_16638_amd', 'csrc')

SRC = r'''
#include "gate.hpp"
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <random>
#include <set>
#include <thread>

#define CHECK(x) do { if (!(x)) { std::printf("failed: %s (line %d)\n", #x, __LINE__); std::exit(1); } } while (0)

// A device of streams: an item waits for its stream's last item and for the events its stream was told
// to wait for; every item whose predecessors have ended runs.
struct Item { std::set<int> pred; int wgs; bool ended = false; };
struct Dev {
  std::vector<Item> items;
  std::vector<std::set<int>> stream;  // what the stream's next item waits for
  std::vector<int> event;             // item each event stands behind (-1: recorded on nothing)
  int put(int s, int wgs) {
    const int id = (int)items.size();
    items.push_back(Item{stream[s], wgs});
    stream[s] = {id};
    return id;
  }
} dev;
struct Model {
  using Stream = int;
  using Event = int;
  // (an event stands behind a marker item of no workgroups)
  static int record(Event e, Stream s) { dev.event[e] = dev.put(s, 0); return 0; }
  static int wait(Stream s, Event e) { if (dev.event[e] >= 0) dev.stream[s].insert(dev.event[e]); return 0; }
  static bool done(Event e) { return dev.event[e] < 0 || dev.items[dev.event[e]].ended; }
};
using G = mprk::Gate<Model>;

static std::vector<int> running() {
  std::vector<int> r;
  for (int i = 0; i < (int)dev.items.size(); ++i) {
    if (dev.items[i].ended) continue;
    bool ready = true;
    for (int p : dev.items[i].pred) ready = ready && dev.items[p].ended;
    if (ready) r.push_back(i);
  }
  return r;
}
// what runs now fits the device, or is one launch; then one of it ends
static bool advance(std::mt19937& rng, int room) {
  const std::vector<int> r = running();
  if (r.empty()) return false;
  int sum = 0, waiting = 0;
  for (int i : r) { sum += dev.items[i].wgs; waiting += dev.items[i].wgs > 0; }
  CHECK(sum <= room || waiting <= 1);
  dev.items[r[rng() % r.size()]].ended = true;
  return true;
}

static void model(unsigned seed) {
  std::mt19937 rng(seed);
  const int room = 768, NC = 5, NB = 3;
  dev = Dev{};
  dev.stream.resize(NC + NB);
  dev.event.assign(NB, -1);
  G g(room);
  std::vector<G::Call> calls(NC);
  std::vector<int> in(NC, 0);
  const int sizes[] = {2, 60, 100, 123, 128};
  const int bsizes[] = {40, 200, 512, 700, 768, 1000, 1280};
  int bw[NB];
  for (int& b : bw) b = bsizes[rng() % 7];
  const bool shared = seed % 3 == 0;  // a batch on a call's stream
  for (int op = 0; op < 300; ++op) {
    const int k = rng() % 10;
    if (k < 4) {
      const int c = rng() % NC;
      if (!in[c]) {
        calls[c] = G::Call{c, sizes[rng() % 5]};
        int used = 0;
        for (int i = 0; i < NC; ++i) used += in[i] ? calls[i].wgs : 0;
        if (used + calls[c].wgs > room) continue;
        g.enter(calls[c]);
        in[c] = 1;
      }
      CHECK(g.begin_step(calls[c]) == 0);
      dev.put(c, calls[c].wgs);
      g.end_step();
    } else if (k < 6) {
      const int b = rng() % NB, s = shared && b == 0 ? 0 : NC + b;
      CHECK(g.batch(&bw[b], s, b, bw[b], rng() % 8 == 0, [&] { dev.put(s, bw[b]); return 0; }) == 0);
    } else if (k < 9) {
      advance(rng, room);
    } else {  // a call ends: the device has ended its work first
      const int c = rng() % NC;
      if (!in[c]) continue;
      auto open = [&] { for (int p : dev.stream[c]) if (!dev.items[p].ended) return true; return false; };
      while (open()) CHECK(advance(rng, room));  // (some item can always run)
      g.leave(calls[c]);
      in[c] = 0;
    }
  }
  while (advance(rng, room)) {}
  for (const Item& i : dev.items) CHECK(i.ended);
}

static void threads() {  // calls too many to be inside together all get their turn, in order
  dev = Dev{};
  dev.stream.resize(8);
  dev.event.assign(1, -1);
  G g(300);
  std::atomic<int> inside{0}, most{0}, finished{0};
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&, t] {
      for (int r = 0; r < 50; ++r) {
        G::Call c{t, 100};
        g.enter(c);
        const int now = ++inside;
        int m = most;
        while (now > m && !most.compare_exchange_weak(m, now)) {}
        CHECK(now <= 3);
        std::this_thread::sleep_for(std::chrono::microseconds(20));
        --inside;
        g.leave(c);
      }
      ++finished;
    });
  for (auto& t : ts) t.join();
  CHECK(finished == 8);
  // in order: while the gate is full, callers queue and enter as they came
  G::Call first{0, 300};
  g.enter(first);
  std::vector<int> order;
  std::mutex mu;
  std::vector<std::thread> qs;
  for (int t = 0; t < 4; ++t) {
    qs.emplace_back([&, t] {
      G::Call c{t, 300};
      g.enter(c);
      { std::lock_guard<std::mutex> lk(mu); order.push_back(t); }
      g.leave(c);
    });
    std::this_thread::sleep_for(std::chrono::milliseconds(20));
    CHECK(g.crowded());
  }
  g.leave(first);
  for (auto& t : qs) t.join();
  CHECK((order == std::vector<int>{0, 1, 2, 3}));
  CHECK(!g.crowded());
}

int main() {
  for (unsigned s = 0; s < 400; ++s) model(s);
  threads();
  std::printf("ok\n");
}
'''


@pytest.mark.skipif(shutil.which('g++') is None, reason='needs g++')
def test_gate_on_a_model_device(tmp_path):
    src, exe = tmp_path / 'gate.cpp', tmp_path / 'gate'
    src.write_text(SRC)
    subprocess.run(['g++', '-O1', '-std=c++17', '-pthread', f'-I{CSRC}', str(src), '-o', str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == 'ok', r.stdout + r.stderr
