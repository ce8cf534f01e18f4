// Host check of the walk that qgemm_splitk's wavefronts take over K (the header is the kernel's own): every 32-wide slice of a row is
// taken exactly once and by the wavefront that owns its group, every step begins inside the row, and what is read of the
// resident codes lies inside the LDS that is asked for.
#include <cstdio>
#include <vector>
#include "../paper_2511_11446_amd/csrc/split_walk.h"

template <bool GROUPED>
static long check(int K, int group, int T)
{
    const int G = GROUPED ? K / group : 0, gpr = GROUPED ? ql::split_groups_per_round(G, T) : 0, rounds = GROUPED ? (G + 4 * gpr - 1) / (4 * gpr) : 0;
    std::vector<int> taken((K + 31) / 32, 0);
    long bad = 0;
    for (int wave = 0; wave < 4; ++wave) {
        const ql::SplitWalk<GROUPED> walk(wave, K, group, G, gpr, rounds);
        auto p = walk.first(wave);
        for (int i = 0; i < walk.steps; ++i, walk.next(p)) {
            if (p.kb < 0 || p.kb >= K) ++bad;                                                        // begins inside the row
            if (K <= ql::SPLIT_FUSE_K_MAX && (p.kb + 127) / 128 >= ql::split_resident_steps(K, GROUPED)) ++bad;   // resident codes read
            for (int s = 0; s < 4; ++s) {
                const int k = p.kb + 32 * s;
                if (k >= K) continue;
                // with group scales a round's last step stops at the end of the wavefront's groups
                if (GROUPED && (k / (gpr * group)) % 4 != wave) continue;
                ++taken[k / 32];
            }
        }
    }
    for (int t : taken) bad += t != 1;
    return bad;
}

int main()
{
    long cases = 0, bad = 0;
    for (int K = 16; K <= 5120; K += 16) {
        for (int T = 16; T <= 32; T += 16) {
            bad += check<false>(K, 128, T);
            ++cases;
            for (int group = 32; group <= K; group += 32) {
                if (K % group) continue;
                const long b = check<true>(K, group, T);
                if (b) std::printf("K %d group %d tile %d: %ld\n", K, group, T, b);
                bad += b;
                ++cases;
            }
        }
    }
    std::printf("cases %ld bad %ld\n", cases, bad);
    return bad != 0;
}
