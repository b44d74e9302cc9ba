// Admission of solver launches to one device.
//
// The workgroups of a solver team wait for each other, so a team that is only
// partly resident holds its places until the rest gets some. A team alone always
// fits (checked against the device before its launch), but two launches on
// different streams may each hold a part of the compute units and wait for the
// other's. So launches that could not all be resident together are ordered: the
// later one's stream first waits for the earlier one's event. Plain C++ over
// `Ops` (streams and events), so that the rule is tested without a device.
#pragma once

#include <cstdint>
#include <mutex>
#include <new>

namespace kf {

// Ops: Stream, Event; bool create(Event&), destroy(Event&); bool record(Event&, Stream)
// (false: not possible now, for instance because the stream is being captured);
// bool done(Event&); bool wait(Stream, Event&); bool same(Stream, Stream);
// bool capturing(Stream); bool idle(Stream): nothing is enqueued there any more, as far
// as can be asked; bool detach(Event&): the event, recorded, no longer refers to the
// stream that it was recorded on, which may go (false: waited for instead).
template <class Ops>
class Admission {
 public:
  using Stream = typename Ops::Stream;
  using Event = typename Ops::Event;

  // The solver launches of one stream, of all contexts that use it. They run in
  // order, so at most one is on the device and the last one's end is that of all.
  struct Lane {
    Stream stream{};
    Event event{};
    int refs = 0;          // 0: its contexts are gone, its last launch may be in flight
    enum State { IDLE, UNMARKED, MARKED } state = IDLE;   // UNMARKED: launched, event not recorded yet
    int blocks = 0;        // the largest unfinished launch
    int per_cu = 0;        // and the fewest workgroups of one that a compute unit holds
    Lane* next = nullptr;  // in order of the last launch
    bool waited = false;   // by the launch in hand
  };

  explicit Admission(int cus, Ops ops = Ops()) : cus_(cus), ops_(ops) {}

  // The lane of a stream, or nullptr (out of memory, no event).
  Lane* join(Stream s) {
    std::lock_guard<std::mutex> lock(mu_);
    for (Lane* l = first_; l; l = l->next)
      if (l->refs > 0 && ops_.same(l->stream, s)) {
        ++l->refs;
        return l;
      }
    Lane* l = new (std::nothrow) Lane();
    if (!l) return nullptr;
    if (!ops_.create(l->event)) {
      delete l;
      return nullptr;
    }
    l->stream = s;
    l->refs = 1;
    append(l);
    return l;
  }

  // The stream has to live until its last context has left, with no launch in
  // flight if `ended`.
  void leave(Lane* l, bool ended) {
    std::lock_guard<std::mutex> lock(mu_);
    if (--l->refs > 0) return;
    if (!ended && l->state != Lane::IDLE && !ops_.idle(l->stream) && in_flight(l) && ops_.detach(l->event))
      return;   // kept until a later launch finds it done
    remove(l);
  }

  // Makes one launch of `blocks` workgroups, of which a compute unit holds per_cu,
  // by calling go() (which returns ok on success).
  template <class Err, class F>
  Err launch(Lane* own, int blocks, int per_cu, Err ok, Err wait_failed, F&& go) {
    std::lock_guard<std::mutex> lock(mu_);
    // alone on the device nothing is recorded or asked: one stream pays nothing
    bool others = false;
    for (Lane* l = first_; l; l = l->next) others = others || (l != own && l->state != Lane::IDLE);
    // what a graph replays is not seen here, and other streams are left alone meanwhile
    if ((others || own->state == Lane::MARKED) && ops_.capturing(own->stream)) return go();
    int held = 0, least = per_cu;
    bool shared = false;
    for (Lane *l = first_, *next; l; l = next) {
      next = l->next;
      l->waited = false;
      if (l == own) continue;
      if (in_flight(l)) {
        shared = true;
        held += l->blocks;
        least = l->per_cu < least ? l->per_cu : least;
      } else if (l->refs == 0) {
        remove(l);
      }
    }
    for (Lane* l = first_; l && held > 0 && held + blocks > places(least); l = l->next) {
      if (l == own || l->state != Lane::MARKED) continue;
      if (!ops_.wait(own->stream, l->event)) return wait_failed;
      l->waited = true;
      held -= l->blocks;
      least = per_cu;
      for (Lane* m = first_; m; m = m->next)
        if (m != own && m->state == Lane::MARKED && !m->waited && m->per_cu < least) least = m->per_cu;
    }
    const Err e = go();
    if (e != ok) return e;
    if (own->state == Lane::MARKED && ops_.done(own->event)) own->state = Lane::IDLE;
    const bool more = own->state != Lane::IDLE;
    own->blocks = more && own->blocks > blocks ? own->blocks : blocks;
    own->per_cu = more && own->per_cu < per_cu ? own->per_cu : per_cu;
    own->state = shared && ops_.record(own->event, own->stream) ? Lane::MARKED : Lane::UNMARKED;
    unlink(own);
    append(own);
    return ok;
  }

  // Workgroups that are certain to be resident together if a compute unit with
  // nothing else on it holds at least per_cu of each kind. Registers and LDS are
  // handed out in contiguous pieces, and kernels that have ended in the meantime
  // leave the pieces apart: k workgroups of at most 1 / per_cu of a resource can
  // keep one more of that size out only if their gaps are all smaller,
  // (2 k + 1) / per_cu > 1, so per_cu / 2 of them always find a place.
  int places(int per_cu) const { return cus_ * (per_cu >= 4 ? per_cu / 2 : 1); }

 private:
  bool in_flight(Lane* l) {
    if (l->state == Lane::UNMARKED) {
      // the first launch of another stream since: the event takes in what was
      // enqueued after the solve, too. While that stream is captured it cannot
      // be recorded and its earlier launch counts as ended.
      if (!ops_.record(l->event, l->stream)) return false;
      l->state = Lane::MARKED;
    }
    if (l->state == Lane::MARKED && ops_.done(l->event)) l->state = Lane::IDLE;
    return l->state == Lane::MARKED;
  }

  void append(Lane* l) {
    Lane** p = &first_;
    while (*p) p = &(*p)->next;
    *p = l;
    l->next = nullptr;
  }
  void unlink(Lane* l) {
    Lane** p = &first_;
    while (*p != l) p = &(*p)->next;
    *p = l->next;
  }
  void remove(Lane* l) {
    unlink(l);
    ops_.destroy(l->event);
    delete l;
  }

  std::mutex mu_;
  int cus_;
  Ops ops_;
  Lane* first_ = nullptr;
};

}  // namespace kf
