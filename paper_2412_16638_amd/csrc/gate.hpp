// Order among launches whose workgroups wait for each other, on one device.
//
// A one-launch CG stage and a batched stage need all of their workgroups resident at once.  Such
// launches in flight together on several streams therefore have to fit the device together, or run
// one after the other: partly resident beside each other they would wait for workgroups that
// cannot start.  `room` counts the workgroups the device holds of any of these kernels (each takes
// at most a third of a compute unit), so whatever fits by that count fits wherever the workgroups
// land; kernels that do not wait for each other end by themselves.
//
//   * Calls (mprk_step, mprk_solve with one-launch stages) end before they return.  A call enters
//     when its workgroups fit beside those of the calls inside, in the order the calls came.
//   * Batches (mprk_batch_step) return at once: they never wait on the host for the device.  A
//     batch step that does not fit beside what is in flight is ordered behind it on the device, by
//     events recorded on the calls' streams; and every step of a call asks in turn whether it fits
//     beside the batches in flight and is ordered behind them if not.  So where not all of it
//     fits, calls and batches take turns by steps, and a wait is always for work enqueued before.
//
// Api: Stream, Event, and static int record(Event, Stream), int wait(Stream, Event) (0: done) and
// bool done(Event).
#pragma once

#include <algorithm>
#include <condition_variable>
#include <mutex>
#include <vector>

namespace mprk {

template <class Api>
class Gate {
 public:
  using Stream = typename Api::Stream;
  using Event = typename Api::Event;
  struct Call {
    Stream stream;
    int wgs;
  };

  explicit Gate(int room) : room_(room) {}

  void enter(Call& c) {
    std::unique_lock<std::mutex> lk(mu_);
    const unsigned long long t = calls_in_++;
    cv_.wait(lk, [&] { return calls_admitted_ == t && (calls_.empty() || used_ + c.wgs <= room_); });
    ++calls_admitted_;
    used_ += c.wgs;
    calls_.push_back(&c);
    cv_.notify_all();
  }
  // (the call's launches have ended)
  void leave(Call& c) {
    std::lock_guard<std::mutex> lk(mu_);
    used_ -= c.wgs;
    calls_.erase(std::find(calls_.begin(), calls_.end(), &c));
    cv_.notify_all();
  }
  bool crowded() {  // a call waits to enter
    std::lock_guard<std::mutex> lk(mu_);
    return calls_admitted_ != calls_in_;
  }

  // Around the launches of one step of a call.  Steps of several calls are enqueued side by side;
  // a batch step between them, in the order they came.
  int begin_step(const Call& c) {
    std::unique_lock<std::mutex> lk(mu_);
    const unsigned long long t = turns_in_++;
    cv_.wait(lk, [&] { return turns_done_ == t; });
    ++turns_done_;
    ++enqueuing_;
    cv_.notify_all();
    reap();
    int held = used_, rc = 0;
    for (const Flight& b : batches_) held += b.stream != c.stream ? b.wgs : 0;
    if (held > room_)
      for (const Flight& b : batches_)
        if (b.stream != c.stream && !rc) rc = Api::wait(c.stream, b.ev);
    return rc;
  }
  void end_step() {
    std::lock_guard<std::mutex> lk(mu_);
    --enqueuing_;
    cv_.notify_all();
  }

  // One step of a batch: launch() on stream s.  ev: the batch's own event, recorded behind the step.
  // alone: behind everything in flight, and nothing else is enqueued until launch() returns.
  template <class F>
  int batch(const void* owner, Stream s, Event ev, int wgs, bool alone, F&& launch) {
    std::unique_lock<std::mutex> lk(mu_);
    const unsigned long long t = turns_in_++;
    cv_.wait(lk, [&] { return turns_done_ == t && enqueuing_ == 0; });
    reap();
    int held = wgs, rc = 0;
    for (const Call* c : calls_) held += c->stream != s ? c->wgs : 0;
    for (const Flight& b : batches_) held += b.stream != s ? b.wgs : 0;
    if (alone || held > room_) {
      for (const Flight& b : batches_)
        if (b.stream != s && !rc) rc = Api::wait(s, b.ev);
      drop(owner);  // (its event marks other streams for a moment)
      for (const Call* c : calls_)
        if (c->stream != s && !rc && !(rc = Api::record(ev, c->stream))) rc = Api::wait(s, ev);
    }
    if (!rc) rc = launch();
    drop(owner);
    const int rr = Api::record(ev, s);
    batches_.push_back(Flight{owner, s, ev, wgs});
    ++turns_done_;
    cv_.notify_all();
    return rc ? rc : rr;
  }
  void forget(const void* owner) {
    std::lock_guard<std::mutex> lk(mu_);
    drop(owner);
  }

 private:
  struct Flight {
    const void* owner;
    Stream stream;
    Event ev;
    int wgs;
  };
  void drop(const void* owner) {
    batches_.erase(std::remove_if(batches_.begin(), batches_.end(),
                                  [&](const Flight& b) { return b.owner == owner; }),
                   batches_.end());
  }
  void reap() {
    batches_.erase(std::remove_if(batches_.begin(), batches_.end(), [](const Flight& b) { return Api::done(b.ev); }),
                   batches_.end());
  }

  const int room_;
  std::mutex mu_;
  std::condition_variable cv_;
  unsigned long long calls_in_ = 0, calls_admitted_ = 0;  // order of the calls that enter
  unsigned long long turns_in_ = 0, turns_done_ = 0;      // order of steps
  int used_ = 0;                                          // workgroups of the calls inside
  int enqueuing_ = 0;                                     // calls' steps being enqueued
  std::vector<Call*> calls_;
  std::vector<Flight> batches_;  // at most one step of each owner: its last
};

}  // namespace mprk
