// Generations of exchange slots (internal; plain C++, also built by a host test).
#pragma once
#include <stdint.h>

namespace hac {

// The words of exchange e carry the 16 bits e & 0xFFFF.  A unit of a slot that an
// exchange does not use keeps the words of an older one, or the zeros before the
// first, and would pass for those of e if that was exactly 65536 exchanges ago (e =
// 65536: never).  So twice in that time, in two exchanges running (one for each of
// the two buffers taken in turn), every unit is written, used or not.
#if defined(__HIP__)
__host__ __device__
#endif
constexpr bool writes_whole_slot(uint32_t e) { return (e & 0x7FFEu) == 0; }

}  // namespace hac
