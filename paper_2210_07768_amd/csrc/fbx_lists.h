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

}  // namespace fbx
