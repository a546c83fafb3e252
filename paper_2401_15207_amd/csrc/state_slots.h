// Which part of which device slot the parked state of a group occupies (hift_step in model.hip).  Host bookkeeping only, so that
// it can be checked without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace hift {

// Three slots, each as long as the largest group's state, filled one after the other in the order in which groups are fetched;
// a slot holds as many groups as fit.  While the groups of one slot are updated, those of the next arrive and those of the one
// before drain.  A slot is emptied as a whole when it is opened again, so a copy into it waits for the write-backs of what it held
// and for nothing else.
//
// Several groups to a slot let small groups be fetched many steps ahead, so that a large one among them has arrived when its turn
// comes and drains while they are updated: the embeddings of a 12-layer encoder of width 768 are six of its layers.  With one
// group to a slot every sweep waited for them in both directions: sweeps of that model, 8 x 128 tokens, one after the other 28.2 ms
// each, now 25.5 (20.6 with resident state: what is left is the contractions that run beside the copies, nothing waits).
class StateSlots {
 public:
  static constexpr int N = 3;
  static constexpr int64_t ALIGN = 64;  // floats; a group starts aligned as a slot does

  // `groups` groups, `cap` floats to a slot; all slots empty
  void reset(int groups, int64_t cap) {
    cap_ = cap;
    place_.assign(groups, Place());
    for (int q = 0; q < N; ++q) { in_[q].clear(); fill_[q] = 0; }
    open_ = 0;
    last_[0] = last_[1] = -1;
    followed_ = groups;
  }

  bool holds(int g) const { return place_[g].slot >= 0; }   // as the host has it, or newer if its write-back is pending
  bool kept(int g) const { return place_[g].kept; }          // not to be emptied before its update
  int slot(int g) const { return place_[g].slot; }
  int64_t at(int g) const { return place_[g].at; }           // floats from the start of the slot
  int last() const { return last_[0]; }
  bool recent(int g) const { return g == last_[0] || g == last_[1]; }  // one of the last two updated

  void keep(int g) { place_[g].kept = true; }
  void let_go() {
    for (Place& p : place_) p.kept = false;
  }
  void updated(int g) {
    place_[g].kept = false;
    if (g != last_[0]) { last_[1] = last_[0]; last_[0] = g; }
  }

  // What step t has copied in before its own group's update: the group, if no slot holds it, then groups that the schedule visits
  // next, as far ahead as the slots have room but two at most, so that a step of another group, or a wait for all streams, finds
  // little queued before it.  The next one always gets its place; further ones leave the state of the group updated last where it is
  // (a caller may step it again), and never are groups whose own update is so recent that their write-back would hold up the copies
  // behind it.  fetch(g, spare, &done) puts g (see put) and queues its copy; a status other than 0 ends the step.
  // A caller that leaves the schedule has what was fetched ahead still in place when it comes back: as long as the last step off
  // the schedule is less than a cycle ago, nothing is copied again that a slot holds, and directly after it only the next group is
  // fetched.  (Fetched again, 34 groups of which one is large moved 3.3 times the state they updated where every other step was off the
  // schedule, and 1.4 times with one in ten; 1.15 and 1.02 now, 1.3 and 1.08 with one group to a slot.)
  template <class Fetch>
  auto advance(int gid, const std::vector<int32_t>& order, int64_t t, Fetch fetch) -> decltype(fetch(0, 0, (bool*)nullptr)) {
    using Status = decltype(fetch(0, 0, (bool*)nullptr));
    const int k = (int)order.size();
    const bool on_schedule = order[t % k] == gid;
    followed_ = on_schedule ? std::min(followed_ + 1, k) : 0;
    bool done = true;
    Status st{};
    if (!holds(gid)) {
      if ((st = fetch(gid, -1, &done)) != Status{}) return st;
      if (!done) {
        let_go();  // what was fetched ahead gives way
        if ((st = fetch(gid, -1, &done)) != Status{}) return st;
      }
    }
    keep(gid);
    const int ahead = k > N + 1 && followed_ >= 2 ? k - N : 1;
    for (int j = 1, fetched = 0; on_schedule && done && j <= ahead && fetched < 2; ++j) {
      const int next = order[(t + j) % k];
      if (kept(next)) continue;
      if (holds(next) && (followed_ < k || (j == 1 && (k <= N || recent(next))))) {
        keep(next);
        continue;
      }
      if ((st = fetch(next, j == 1 ? -1 : last(), &done)) != Status{}) return st;
      if (!done && j == 1) {
        let_go();
        keep(gid);
        if ((st = fetch(next, -1, &done)) != Status{}) return st;
      }
      ++fetched;
    }
    return st;
  }

  // Group g has no place any more (its copy could not be queued).
  void drop(int g) {
    if (!holds(g)) return;
    std::vector<int>& v = in_[place_[g].slot];
    v.erase(std::find(v.begin(), v.end(), g));
    place_[g] = Place();
  }

  // A place for `floats` values of group g, kept from now on; false if that takes a slot with a kept group, or the one of group
  // `spare` (-1: none).  `emptied` receives the groups whose place is given up for it.
  bool put(int g, int64_t floats, int spare, std::vector<int>& emptied) {
    emptied.clear();
    int q = open_;
    if (fill_[q] + floats > cap_) {
      for (q = (open_ + 1) % N; blocked(q, g, spare); q = (q + 1) % N)
        if (q == open_) return false;
      for (int o : in_[q])
        if (o != g) { emptied.push_back(o); place_[o].slot = -1; }
    }
    drop(g);  // what it had is given up too; the caller orders the copy behind its write-back
    if (q != open_ || fill_[q] + floats > cap_) {
      in_[q].clear();
      fill_[q] = 0;
      open_ = q;
    }
    place_[g].slot = q;
    place_[g].at = fill_[q];
    place_[g].kept = true;
    in_[q].push_back(g);
    fill_[q] = std::min(cap_, fill_[q] + (floats + ALIGN - 1) / ALIGN * ALIGN);
    return true;
  }

 private:
  struct Place {
    int slot = -1;
    int64_t at = 0;
    bool kept = false;
  };
  bool blocked(int q, int g, int spare) const {
    for (int o : in_[q])
      if (o != g && (place_[o].kept || o == spare)) return true;
    return false;
  }
  std::vector<Place> place_;
  std::vector<int> in_[N];
  int64_t fill_[N] = {0, 0, 0}, cap_ = 0;
  int open_ = 0, last_[2] = {-1, -1};
  int followed_ = 0;  // steps in a row in the schedule's order, counted up to a cycle
};

}  // namespace hift
