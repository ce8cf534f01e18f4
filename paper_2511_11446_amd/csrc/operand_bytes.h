// Byte sizes and row offsets of the GEMM operands: 32 bits, unsigned.  A layer has up to 2^31 - 1 elements per operand, which in binary16
// are more bytes than a signed int holds.  Plain C++, no HIP.
#pragma once

namespace ql {

constexpr unsigned operand_bytes(int rows, int row_bytes) { return (unsigned)rows * (unsigned)row_bytes; }
constexpr unsigned row_start(int row, int row_bytes) { return (unsigned)row * (unsigned)row_bytes; }

// Rows of at least 16 bytes that may be no whole K steps of 128: where 16-byte piece c of a row is read in its first K step, and how far back of
// kt * 128 behind that in step kt of nk.  A piece that crosses the end of its row, or lies behind it, is the row's last one.  Neither may leave
// the row before it comes back: behind the last row of the largest operands 32 bits wrap.
constexpr unsigned first_piece(int row, int row_bytes, int c) { return row_start(row, row_bytes) + (unsigned)(16 * c + 16 < row_bytes ? 16 * c : row_bytes - 16); }
constexpr unsigned piece_back(int kt, int nk, int row_bytes, int c)
{
    const int over = kt * 128 + 16 * c + 16 - row_bytes;
    return kt == 0 || kt + 1 < nk || over < 0 ? 0u : (unsigned)over;
}

// the largest binary16 operand that the entry points accept
static_assert(operand_bytes(2147483647 / 8, 16) == 4294967280u, "2^31 - 8 values");
static_assert(row_start(1048575, 4094) == 4292866050u, "its rows start behind 2^31");

}  // namespace ql
