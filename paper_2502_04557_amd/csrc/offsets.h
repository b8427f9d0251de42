// Byte offsets of buffer loads that guard themselves: an offset beyond the buffer gives zeros and fetches nothing (k_gemm_norm.hip).  Plain
// C++ with constant evaluation, which refuses any overflow.
#pragma once

namespace sprinter {

// Beyond any buffer of at most FEW_ROWS_MAX_K columns, whose size is an int below it, and so is every sum with it: what is added stays below 2^31, and the unsigned sum below 2^32.
constexpr unsigned NOWHERE = 0x7ffffff0u;
// Longest K whose product of few rows adds itself (64 bytes per k of two float16 operands, or of 16 float32 rows: 2^26); longer ones take the K shares, whose addresses are 64 bits.
constexpr int FEW_ROWS_MAX_K = 1 << 20;

// Unit `unit` of `bytes` bytes behind this lane's offset in the first one (which may be NOWHERE), or NOWHERE and more.
constexpr unsigned unit_offset(bool there, unsigned lane, int unit, int bytes) { return (there ? lane : NOWHERE) + (unsigned)unit * (unsigned)bytes; }

}  // namespace sprinter
