// Byte offsets of buffer loads that guard themselves: an offset beyond the buffer gives zeros and fetches nothing (k_gemm_norm.hip).  Plain
// C++ with constant evaluation, which refuses any overflow.
#pragma once

namespace sprinter {

// Beyond any buffer, whose size is an int below it, and so is every sum with it: what is added stays below 2^31 - 2^20, and the unsigned sum below 2^32.
constexpr unsigned NOWHERE = 0x7ffffff0u;

// Unit `unit` of `bytes` bytes behind this lane's offset in the first one (which may be NOWHERE), or NOWHERE and more.
constexpr unsigned unit_offset(bool there, unsigned lane, int unit, int bytes) { return (there ? lane : NOWHERE) + (unsigned)unit * (unsigned)bytes; }

}  // namespace sprinter
