// Index arithmetic of qgemm_splitk that the kernel, its launcher and the host check of its bounds share: the K steps of a wavefront, and
// the LDS that a workgroup's own codes take.  Plain C++, no HIP.
#pragma once

namespace ql {

constexpr int SPLIT_FUSE_K_MAX = 1536;   // row length up to which the workgroup quantizes its own rows

// groups of a wavefront's round (T x T tiles, W wavefronts): the partial tiles of all wavefronts' groups are in LDS at once
constexpr int split_groups_per_round(int groups, int T, int W = 4)
{
    const int all = (groups + W - 1) / W, most = (T == 32 ? 12 : 40) / W;
    return all < most ? all : most;
}

// A K step is 128 bytes of an activation row.  Without group scales, wavefront w of W takes steps w, w + W, ...; with group
// scales it takes rounds of `gpr` consecutive groups, and cuts each round into steps from the round's own start: such a step begins
// at a multiple of 32 (of the group size), not of 128, and the last one of a round may be cut short.
template <bool GROUPED, int W = 4>
struct SplitWalk {
    int steps, round_k, round_steps;
    constexpr SplitWalk(int wave, int row_bytes, int group, int groups, int gpr, int rounds)
        : steps(0), round_k(GROUPED ? gpr * group : 0), round_steps(GROUPED ? (gpr * group + 127) / 128 : 0)
    {
        if (GROUPED) {
            const int last = groups - ((rounds - 1) * W + wave) * gpr;   // groups of the last round
            const int mine = (rounds - 1) * gpr + (last < 0 ? 0 : last < gpr ? last : gpr);
            const int full = mine / gpr, rest = mine - full * gpr;       // every round but the last is full
            steps = full * round_steps + (rest * group + 127) / 128;
        } else {
            const int nk = (row_bytes + 127) / 128;
            steps = nk > wave ? (nk - wave + W - 1) / W : 0;
        }
    }
    // first byte of a step inside its row; one of these for the step to be requested next, one for the step to be read next
    struct Position {
        int kb, in_round;
    };
    constexpr Position first(int wave) const { return {GROUPED ? wave * round_k : wave * 128, 0}; }
    constexpr void next(Position &p) const
    {
        if (!GROUPED) {
            p.kb += W * 128;
        } else if (++p.in_round == round_steps) {
            p.in_round = 0;
            p.kb += W * round_k - (round_steps - 1) * 128;
        } else {
            p.kb += 128;
        }
    }
};

// LDS slots of the rings, S per wavefront: slot i of wavefront w is number w + W i.  As many as the steps reach, and without group scales one for each
// wavefront's sums.
template <bool GROUPED, int W>
constexpr int split_slots(int S, int row_bytes, int group, int groups, int gpr, int rounds)
{
    int slots = GROUPED ? 1 : W;
    for (int wave = 0; wave < W; ++wave) {
        const int steps = SplitWalk<GROUPED, W>(wave, row_bytes, group, groups, gpr, rounds).steps, used = steps < S ? steps : S;
        if (used > 0 && wave + W * (used - 1) + 1 > slots) slots = wave + W * (used - 1) + 1;
    }
    return slots;
}

// K steps of codes that a workgroup which quantizes its own rows keeps in LDS: a wavefront reads whole steps, and with group scales its
// last one can begin up to 96 bytes behind a multiple of 128 and then ends in the step behind the row's last (K = 1152, groups of
// 288: bytes 1120 to 1247 of 1152).  What lies there is read and not used.
constexpr int split_resident_steps(int K, bool grouped) { return (K + 127) / 128 + (grouped ? 1 : 0); }

}  // namespace ql
