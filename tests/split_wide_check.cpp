// Host check of the walk over K on eight wavefronts and of the LDS slots that the launcher asks for (the header is the kernel's own): every
// 32-wide slice of a row is taken exactly once and by the wavefront that owns its group, and no step uses a slot that is not there.
#include <cstdio>
#include <vector>
#include "../paper_2511_11446_amd/csrc/split_walk.h"

template <bool GROUPED, int W>
static long check(int K, int group, int T)
{
    const int G = GROUPED ? K / group : 0, gpr = GROUPED ? ql::split_groups_per_round(G, T, W) : 0, rounds = GROUPED ? (G + W * gpr - 1) / (W * gpr) : 0;
    std::vector<int> taken((K + 31) / 32, 0);
    long bad = GROUPED && gpr < 1;
    for (int S = 2; S <= 4; ++S) {
        const int slots = ql::split_slots<GROUPED, W>(S, K, group, G, gpr, rounds);
        bad += slots > W * S || (!GROUPED && slots < W);
        for (int wave = 0; wave < W; ++wave) {
            const ql::SplitWalk<GROUPED, W> walk(wave, K, group, G, gpr, rounds);
            auto p = walk.first(wave);
            for (int i = 0; i < walk.steps; ++i, walk.next(p)) {
                bad += wave + W * (i % S) >= slots;
                bad += p.kb < 0 || p.kb >= K || (K <= ql::SPLIT_FUSE_K_MAX && (p.kb + 127) / 128 >= ql::split_resident_steps(K, GROUPED));
                for (int s = 0; s < 4 && S == 2; ++s) {
                    const int k = p.kb + 32 * s;
                    if (k >= K || (GROUPED && (k / (gpr * group)) % W != wave)) continue;
                    ++taken[k / 32];
                }
            }
        }
    }
    for (int t : taken) bad += t != 1;
    return bad;
}

int main()
{
    long cases = 0, bad = 0;
    for (int K = 16; K <= 5120; K += 16)
        for (int T = 16; T <= 32; T += 16) {
            bad += check<false, 8>(K, 128, T) + check<false, 4>(K, 128, T);
            for (int group = 32; group <= K; group += 32)
                if (K % group == 0) bad += check<true, 8>(K, group, T) + check<true, 4>(K, group, T);
            ++cases;
        }
    std::printf("cases %ld bad %ld\n", cases, bad);
    return bad != 0;
}
