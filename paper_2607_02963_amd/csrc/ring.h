// Lane masks of the DMA pieces that fill a ring of LDS stages.  (Host and
// device: a test runs the ring's schedule on the CPU.)
#pragma once

#include <stdint.h>

namespace pdec {

// Lanes of a piece of stage st, where stages 0 .. nst - 1 exist.  The waits
// count a wave's pieces from the newest back, the same number at every stage,
// so a stage past the last has pieces too: of one lane, which loads 16 bytes of
// the last unit again, into a slot that nothing reads any more.  (A piece
// without lanes would be cheaper still, but whether such an instruction takes
// part in the count, in order, is the hardware's affair.)
constexpr uint64_t ring_lanes(int st, int nst) { return st < nst ? ~0ull : 1ull; }

}  // namespace pdec
