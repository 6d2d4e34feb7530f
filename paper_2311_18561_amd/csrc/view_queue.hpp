// The order in which the multi-view adjoint takes its screen-space gradient
// slots and runs its per-Gaussian passes (host bookkeeping only).
#pragma once

#include <cstdint>

namespace pvg {

// A view's compositing adjoint writes the slot it takes(); the view is then
// queued for the next per-Gaussian pass, which reads the slots of all queued
// views (of one render time) and sums them `group` at a time.  Slots are taken
// in turn and start over once a pass has run behind the last one.
//
// A render time that changes at the view of the last slot runs the pass before
// that view is queued.  If the views queued so far are whole groups, the view
// then gets a pass of its own.  Else the slots start over while it still holds
// the last one (`carried`), and its pass comes after one group: with more
// views queued, one of the next would write the slot it has yet to read.
// These are the groups of a pass per group of views, which is what the order
// of each gradient's sum rests on.
struct ViewQueue {
  int32_t slots;   // slots there are, and the most views a pass takes
  int32_t group;
  int32_t used = 0;    // slots taken since they last started over
  int32_t queued = 0;  // views the next pass takes
  bool carried = false;

  int32_t take() { return used++; }
  bool full() const { return carried ? queued == group : used == slots; }
  // A pass over the queued views was launched; `pending`: a view has taken a
  // slot and is not queued yet.  True if slots that the pass reads will be
  // written before another pass does: those writers must wait for it.
  bool passed(bool pending) {
    const bool over = used == slots && !(pending && queued % group == 0);
    const bool reuse = carried || over;
    carried = over && pending;
    if (over) used = 0;
    queued = 0;
    return reuse;
  }
};

}  // namespace pvg
