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
};

}  // namespace hift
