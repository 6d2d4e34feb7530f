// Host check of the multi-view adjoint's slot and pass order: for every
// number of views up to 40, one or two changes of the render time at any
// view, and groups of 1, 2, 3 and 8 views, no pass takes more views than its
// arrays hold, no view takes a slot that a queued view still holds or that a
// launched pass may be reading (no wait in between), and the views are summed
// in the groups of the rule "a pass per group, per render time and per eighth
// slot taken".
#include <cstdio>
#include <vector>

#include "view_queue.hpp"

using Groups = std::vector<std::vector<int>>;

// A pass per group: queued views leave when a group is full, when the last
// slot was taken, and before a view of another time is queued (which has
// taken its slot by then).
static Groups by_groups(const std::vector<int>& time, int group, int slots) {
  Groups out;
  std::vector<int> cur;
  int used = 0;
  auto flush = [&] {
    if (cur.empty()) return;
    out.push_back(cur);
    cur.clear();
    if (used == slots) used = 0;
  };
  for (int k = 0; k < static_cast<int>(time.size()); ++k) {
    ++used;
    if (!cur.empty() && time[k] != time[cur[0]]) flush();
    cur.push_back(k);
    if (static_cast<int>(cur.size()) == group || used == slots) flush();
  }
  flush();
  return out;
}

static bool check(const std::vector<int>& time, int group) {
  constexpr int kSlots = 8;
  pvg::ViewQueue q{kSlots, group};
  Groups got;
  std::vector<int> cur, slot_of(time.size());
  int held[kSlots];        // the view whose gradients a slot holds until its pass, or -1
  bool reading[kSlots];    // a launched pass reads the slot and no wait followed
  for (int s = 0; s < kSlots; ++s) { held[s] = -1; reading[s] = false; }
  auto flush = [&](bool pending) {
    if (cur.empty()) return;
    for (size_t i = 0; i < cur.size(); ++i) {
      if (i % group == 0) got.emplace_back();
      got.back().push_back(cur[i]);
      held[slot_of[cur[i]]] = -1;
      reading[slot_of[cur[i]]] = true;
    }
    cur.clear();
    if (q.passed(pending))
      for (bool& r : reading) r = false;
  };
  for (int k = 0; k < static_cast<int>(time.size()); ++k) {
    const int s = q.take();
    if (s < 0 || s >= kSlots) { std::printf("view %d takes slot %d\n", k, s); return false; }
    if (held[s] >= 0) { std::printf("view %d overwrites slot %d of queued view %d\n", k, s, held[s]); return false; }
    if (reading[s]) { std::printf("view %d writes slot %d beside the pass that reads it\n", k, s); return false; }
    held[s] = k;
    slot_of[k] = s;
    if (!cur.empty() && time[k] != time[cur[0]]) flush(true);
    if (q.queued >= kSlots) { std::printf("view %d is number %d of a pass\n", k, q.queued); return false; }
    ++q.queued;
    cur.push_back(k);
    if (q.full()) flush(false);
  }
  flush(false);
  if (got != by_groups(time, group, kSlots)) { std::printf("other groups\n"); return false; }
  return true;
}

int main() {
  for (int group : {1, 2, 3, 8})
    for (int n = 1; n <= 40; ++n)
      for (int a = 1; a <= n; ++a)
        for (int b = a; b <= n; ++b) {
          std::vector<int> time(n);
          for (int k = 0; k < n; ++k) time[k] = (k >= a) + (k >= b);
          if (!check(time, group)) {
            std::printf("group %d, %d views, time changes at %d and %d\n", group, n, a, b);
            return 1;
          }
        }
  std::printf("view queue ok\n");
  return 0;
}
