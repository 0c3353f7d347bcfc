// The record of a sector's rank lookup.
#pragma once

#include <cstdint>

namespace ftlm {
namespace dev {

// One word of the rank lookup: bit k of (hi, lo) is set when rank 64 w + k is
// a representative, base counts the representatives before the word.  One
// record, because a lookup is a random access: bits and base in arrays of
// their own cost two lines each.  Twelve bytes: the records are the largest
// table of a sector without entries, and few of them straddle two lines.
struct RankWord {
  uint32_t lo, hi, base;
};

}  // namespace dev
}  // namespace ftlm
