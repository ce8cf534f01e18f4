// Host check of the addresses of the tiles that take rows of any whole number of words (the header is the kernel's own): every 16-byte piece
// of every K step lies inside its row, where it belongs or at the row's end.
#include <cstdio>
#include <initializer_list>
#include "../paper_2511_11446_amd/csrc/operand_bytes.h"

static long check(long long rows, int row_bytes)
{
    const int nk = (row_bytes + 127) / 128;
    long bad = 0;
    for (long long row : {0ll, rows / 2, rows - 2, rows - 1}) {
        if (row < 0) continue;
        const long long begin = row * row_bytes, last = begin + row_bytes - 16;
        for (int kt = 0; kt < nk; ++kt)
            for (int c = 0; c < 8; ++c) {
                // as the kernel adds them to the operand's 64-bit address
                const long long at = (long long)kt * 128 + ql::first_piece((int)row, row_bytes, c) - ql::piece_back(kt, nk, row_bytes, c);
                const long long want = begin + kt * 128 + 16 * c < last ? begin + kt * 128 + 16 * c : last;
                bad += at != want;
            }
    }
    return bad;
}

int main()
{
    long cases = 0, bad = 0;
    for (int bytes = 1; bytes <= 2; ++bytes)
        for (int row_bytes = 16; row_bytes <= 2600; row_bytes += 4) {
            const long long most = 2147483647ll / (row_bytes / bytes);   // rows of the largest operand that the entry points accept
            for (long long rows : {1ll, 2ll, 65ll, most / 2, most - 1, most}) {
                const long b = check(rows, row_bytes);
                if (b) std::printf("rows %lld of %d bytes: %ld pieces\n", rows, row_bytes, b);
                bad += b;
                ++cases;
            }
        }
    std::printf("cases %ld bad %ld\n", cases, bad);
    return bad != 0;
}
