// How much of a workspace goes to what only gains from room: `fixed` bytes have to be there, and at least `least`,
// at most `most` bytes behind them (most >= least). have: the workspace's size; grow(bytes) puts one of that size in
// its place, or, on a failure, none.
// Where the room is refused once, the call makes do with the least, and later calls, which would be refused
// too, do not ask again: each would give the workspace up for it. stay: graphs hold addresses in the workspace, so it
// is only replaced where not even the least fits.
#pragma once
#include <cstddef>

template <typename Grow>
int fit_room(size_t have, size_t fixed, size_t least, size_t most, bool stay, int refused_status, bool *refused, size_t *room, Grow grow) {
  if (have < fixed + most && have >= fixed + least && (stay || *refused)) {
    *room = (have - fixed) / 256 * 256 > least ? (have - fixed) / 256 * 256 : least;
    return 0;
  }
  *room = most;
  if (have >= fixed + most) return 0;
  if (!*refused) {
    const int rc = grow(fixed + most);
    if (rc != refused_status || most == least) return rc;
    *refused = true;
  }
  *room = least;
  return grow(fixed + least);
}
