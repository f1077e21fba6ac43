// Arithmetic of the tile kernel's list operators that has no need of a GPU: the kernel calls it, and so does a host test.
#pragma once

#include <cstdint>

namespace fbx {

// Which (operator, record) pair each of the 64 signs of a unit belongs to (Pass::pair_at).  64 pairs at a time, one a lane,
// send a number to a lane each, and a running maximum over the lanes fills those that got none.  Lanes that send to the same
// one send the same number, so that it does not matter which of them is heard.
// s: the unit's sign at which the lane's pair starts, at most 63; next: where the next lane's pair does (the last lane: 63);
// number: the lane's pair, plus one; last: the last of the 64 pairs that starts inside the unit, plus one.
// Of pairs that start at the same sign all but the last are without signs: they, and those that start at the unit's last sign
// or beyond it, send what that sign is to know.
struct PairSend { uint32_t lane, number; };
constexpr PairSend pair_send(uint32_t s, uint32_t next, uint32_t number, uint32_t last) {
  return s != next ? PairSend{s, number} : PairSend{63u, last};
}

// Where a pass's lists lie on chip (Pass::keep_lists), in words: `all` is the section of the staged text, of which the pass's
// text takes `text`; `cap` the section for lists of layer 1.  Those go behind the text where there is more room; later layers'
// lists go where the text was, or, if none is staged (a record read in place), to all of its section.
struct ListRoom { bool behind; uint32_t first, later; };
constexpr ListRoom list_room(bool staged, uint32_t all, uint32_t text, uint32_t cap) {
  const bool behind = staged && all - text > cap;
  return ListRoom{behind, behind ? all - text : cap, behind ? text : all};
}

}  // namespace fbx
