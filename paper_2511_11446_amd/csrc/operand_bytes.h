// Byte sizes and row offsets of the GEMM operands: 32 bits, unsigned.  A layer has up to 2^31 - 1 elements per operand, which in binary16
// are more bytes than a signed int holds.  Plain C++, no HIP.
#pragma once

namespace ql {

constexpr unsigned operand_bytes(int rows, int row_bytes) { return (unsigned)rows * (unsigned)row_bytes; }
constexpr unsigned row_start(int row, int row_bytes) { return (unsigned)row * (unsigned)row_bytes; }

// the largest binary16 operand that the entry points accept
static_assert(operand_bytes(2147483647 / 8, 16) == 4294967280u, "2^31 - 8 values");
static_assert(row_start(1048575, 4094) == 4292866050u, "its rows start behind 2^31");

}  // namespace ql
