// The order of a selection launch's workgroups over its camera groups, and the
// identifiers that a stream's groups hand on.
//
// A group waits for the next free identifier of the stream's group before it, so
// that group has to be running by then. Workgroup numbers do not promise this:
// the chip's eight XCDs start their shares of a launch independently of each
// other, each when it has a place free, so a later group may be waiting in one
// while an earlier one has no place yet in another (and with enough launches at a
// time every place could be taken by one that waits). So a workgroup takes its
// group from a ticket: whoever holds an earlier one has started before, the one
// with the lowest ticket waits for nobody, and every wait ends. The ticket's round
// trip does not show: the selection of a four-camera rig
// 22.3 us with numbers and 21.6 with tickets, of four rigs of 640x480 13.3 and 13.0
// (deferred matches: 26.5 and 25.4, 15.9 and 16.3).
//
// Mem: atomic access to memory that the workgroups share, and a pause between
// two looks at it.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define VIO_GROUP_FN __device__ __forceinline__
#else
#define VIO_GROUP_FN inline
#endif

namespace vio {

// The calling workgroup's group of n (called once by each of n workgroups; the
// counter is zero before and after).
template <class Mem>
VIO_GROUP_FN int take_group(int32_t* ticket, int n) {
  const int32_t t = Mem::add(ticket, 1);
  if (t == n - 1) Mem::store(ticket, (int32_t)0);
  return t;
}

// A chain entry is twice the identifier plus one, and zero before it is there and
// after it was taken.
template <class Mem>
VIO_GROUP_FN int64_t take_id(int64_t* chain) {
  int64_t v;
  while ((v = Mem::load(chain)) == 0) Mem::pause();
  Mem::store(chain, (int64_t)0);
  return v >> 1;
}
template <class Mem>
VIO_GROUP_FN void hand_on_id(int64_t* chain, int64_t id) {
  Mem::store(chain, id * 2 + 1);
}

}  // namespace vio
