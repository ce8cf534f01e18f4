// Several layers of a plan in one launch, for gfx950: the GEMMs of layers that do not wait for each other (their activations are
// quantized already, none writes what another one reads or writes).
//
// What bounds a layer of a few hundred tiles is how they divide by the CUs: 128x128 tiles at two workgroups per CU come in rounds of 512,
// and M = 4096, N = 1152 has 288 of them, M = 2048 144; every launch fills and drains the chip for itself.  Here every workgroup takes one
// tile of one layer, and the hardware hands out the next one where one ends, whatever layer it is from, so that only the end of
// the launch leaves CUs idle.  The tiles are those of qgemm_dma and qgemm_w4, not persistent, all kinds in one kernel: the
// kind is uniform over a workgroup.  The layers come in descending order of a tile's time, so that no long tile starts last.
#include "qgemm_dma.h"
#include "qgemm_w4.h"

namespace ql {

using ManyW8 = TileD<2, 2, 2, 2, 3, 2, true, 1, 2>;
using ManyF16 = TileD<2, 2, 2, 2, 3, 2, true, 1, 2, false, true>;
using ManyW4 = TileW4<2, 3, 2>;
constexpr int MANY_LDS = ManyW8::LDS_BYTES > ManyW4::LDS_BYTES ? ManyW8::LDS_BYTES : ManyW4::LDS_BYTES;
static_assert(ManyF16::LDS_BYTES <= MANY_LDS && 2 * MANY_LDS <= 160 * 1024, "two workgroups per CU");

// the kinds of tiles; 4-bit ones by the K slices of 32 per weight group that the loop is unrolled for
enum ManyKind : int { MANY_W8, MANY_F16, MANY_W4_1, MANY_W4_2, MANY_W4_4, MANY_W4_6, MANY_W4_9, MANY_NONE };

struct ManyLayer {
    const int8_t *q;
    const float *s_a;
    const void *w, *s_w, *bias;
    void *y;
    int N, K, group, kind;
    int tiles_n, padded;   // tile columns; workgroups of the layer: its tiles, rounded up to a multiple of XCDS
};
struct ManyArgs {
    ManyLayer l[PLAN_WINDOW];
    int M, R, tiles_m, group_m;
};

__global__ __launch_bounds__(256, 2) void qgemm_many(ManyArgs b)
{
    int i = 0, block = blockIdx.x;
    while (block >= b.l[i].padded) block -= b.l[i++].padded;   // the grid is the sum of all
    const ManyLayer &l = b.l[i];
    GemmArgs a{};
    a.q = l.q;
    a.s_a = l.s_a;
    a.w = l.w;
    a.s_w = l.s_w;
    a.bias = l.bias;
    a.y = l.y;
    a.M = b.M;
    a.N = l.N;
    a.K = l.K;
    a.R = b.R;
    a.group = l.group;
    const int tiles_n = l.tiles_n, padded = l.padded;
    switch (l.kind) {
    case MANY_W8: qgemm_dma_tiles<ManyW8, false>(a, block, padded, b.tiles_m, tiles_n, padded, b.group_m); break;
    case MANY_F16: qgemm_dma_tiles<ManyF16, false>(a, block, padded, b.tiles_m, tiles_n, padded, b.group_m); break;
    case MANY_W4_1: qgemm_w4_tiles<ManyW4, 1, false, false, Channel::no, true>(a, block, padded, b.tiles_m, tiles_n, padded, b.group_m); break;
    case MANY_W4_2: qgemm_w4_tiles<ManyW4, 2, false, false, Channel::no, true>(a, block, padded, b.tiles_m, tiles_n, padded, b.group_m); break;
    case MANY_W4_4: qgemm_w4_tiles<ManyW4, 4, false, false, Channel::no, true>(a, block, padded, b.tiles_m, tiles_n, padded, b.group_m); break;
    case MANY_W4_6: qgemm_w4_tiles<ManyW4, 6, false, false, Channel::no, true>(a, block, padded, b.tiles_m, tiles_n, padded, b.group_m); break;
    default: qgemm_w4_tiles<ManyW4, 9, false, false, Channel::no, true>(a, block, padded, b.tiles_m, tiles_n, padded, b.group_m); break;
    }
}

static int many_kind(const GemmArgs &a)
{
    if (a.w_bits != 4) return a.w_bits == 8 ? MANY_W8 : MANY_F16;
    const int nk = a.K / 128;   // a period of the unrolled loop is 3 or 9 K steps for groups of 192 and 288
    switch (a.group) {
    case 32: return MANY_W4_1;
    case 64: return MANY_W4_2;
    case 128: return MANY_W4_4;
    case 192: return nk % 3 == 0 ? MANY_W4_6 : MANY_NONE;
    case 288: return nk % 9 == 0 ? MANY_W4_9 : MANY_NONE;
    default: return MANY_NONE;
    }
}

bool qgemm_many_takes(const GemmArgs &a)
{
    if (a.w_grouped || a.s_ag || a.acc_out || a.act != 0 || a.residual || a.gate || a.row_absmax) return false;
    if (a.w_bits == 4) return qgemm_w4_takes(a) && a.K / a.group <= ManyW4::MAX_GROUPS && many_kind(a) != MANY_NONE;
    return (a.w_bits == 8 || a.w_bits == 16) && a.K * (a.w_bits == 16 ? 2 : 1) % 128 == 0 && ((uintptr_t)a.q | (uintptr_t)a.w) % 16 == 0;
}

// What a tile takes of its CU, in microseconds, K steps of 128 bytes.  From plans of 1 to 4 blocks of widths 384, 768 and 1152 at M = 512 to 16384,
// with this launch and without.  (8-bit: 3, 6 and 9 steps 3.2, 4.2 to 4.6 and 6.3 us.)
static float tile_us(const GemmArgs &a)
{
    const float steps = (float)(a.K * (a.w_bits == 16 ? 2 : 1) / 128);
    if (a.w_bits == 8) return 1.2f + 0.56f * steps;
    if (a.w_bits == 16) return 1.9f + 0.44f * steps;
    return 2.0f + 0.347f * steps + 0.18f * (float)(a.K / a.group);
}

// all tiles spread evenly over 256 CUs, and half a tile of idling at the end
static float many_us(const GemmArgs *const *layers, int count)
{
    float work = 0.0f, longest = 0.0f;
    for (int i = 0; i < count; ++i) {
        const GemmArgs &a = *layers[i];
        const float us = tile_us(a);
        work += us * (float)((a.M + ManyW8::BM - 1) / ManyW8::BM) * (float)((a.N + ManyW8::BN - 1) / ManyW8::BN);
        longest = us > longest ? us : longest;
    }
    return 3.2f + work / 256.0f + 0.5f * longest;
}

// The same layers on 256x288 tiles, where these are one round (one tile of qgemm_big as choose_tile prices it; the longest K decides).  Three 8-bit layers of
// a block of width 1152 at M = 2048, 256 tiles: 28.1 us, 32.9 on the 1152 tiles of 128x128.  With DAQ and fc2, 128x128 -> here: width 768, M = 2560 48.7 ->
// 47.0, 2816 56.4 -> 49.9; 1024, M = 1792 53.7 -> 50.4; 1152, M = 1664 58.0 -> 55.0, 2048 70.4 -> 64.5; 1536, M = 1280 70.2 -> 66.2; 2048, M = 1024 96.0 -> 88.8.
static float big_many_us(const GemmArgs *const *layers, int count)
{
    if (!qgemm_big_many_takes(layers, count)) return 1e9f;
    int longest = 0;
    for (int i = 0; i < count; ++i) longest = layers[i]->K > longest ? layers[i]->K : longest;
    return 11.7f + 1.773f * (float)(longest / 128);
}

// A layer that splits K by itself stays out, but for 4-bit ones of more 32x32 tiles than CUs whose groups are more than four wavefronts take in one go: two workgroups of them
// fit a CU, and yet the launch costs a plan more than these tiles do (four blocks of width 768 with 4-bit projections, us, own launches -> shared: M = 325 175 -> 157, M =
// 602 165 -> 153).
static bool stays_out(const GemmArgs &a)
{
    const int split = qgemm_split_choice(a);
    return split && !(split == 32 && a.w_bits == 4 && a.K / a.group > 4 && (long long)((a.M + 31) / 32) * ((a.N + 31) / 32) > 256);
}

// One launch for all that it takes, where that is estimated to be the faster: filling the chip once, the tiles spread evenly
// over 256 CUs and half a tile of idling at the end, against the layers' own best tiles and 1.5 us for each launch more.  Two 8-bit blocks of width
// 1152, us with the layers' own launches -> in one: M = 512 91 -> 72, 2048 155 -> 143, 4096 250 -> 213, 6144 317 -> 309; not taken: 8192 403 -> 421,
// 16384 695 -> 753, where the large tiles come in whole rounds.
int qgemm_many_choice(const GemmArgs *layers, int n, const GemmArgs **chosen)
{
    int count = 0;
    float alone = -1.5f;
    for (int i = 0; i < n; ++i) {
        const GemmArgs &a = layers[i];
        if (!qgemm_many_takes(a) || stays_out(a)) continue;
        chosen[count++] = &a;
        alone += qgemm_alone_us(a) + 1.5f;
    }
    if (count < 2) return 0;
    return (qgemm_many_one_round(chosen, count) ? big_many_us(chosen, count) : many_us(chosen, count)) < alone ? count : 0;
}

bool qgemm_many_one_round(const GemmArgs *const *layers, int count) { return big_many_us(layers, count) < many_us(layers, count); }

hipError_t launch_qgemm_many(const GemmArgs *const *layers, int count, hipStream_t stream)
{
    if (qgemm_many_one_round(layers, count)) return launch_qgemm_big_many(layers, count, stream);
    static const hipError_t opt_in = hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_many), hipFuncAttributeMaxDynamicSharedMemorySize, MANY_LDS);
    if (opt_in != hipSuccess) return opt_in;
    ManyArgs b{};
    b.M = layers[0]->M;
    b.R = 1;
    b.tiles_m = (b.M + ManyW8::BM - 1) / ManyW8::BM;
    b.group_m = pick_group_m(ManyW8::BM);
    int order[PLAN_WINDOW];
    for (int i = 0; i < count; ++i) {
        if (layers[i]->w_bits != 16) b.R = layers[i]->R;   // one for all quantized layers
        int at = i;
        for (; at > 0 && tile_us(*layers[order[at - 1]]) < tile_us(*layers[i]); --at) order[at] = order[at - 1];
        order[at] = i;
    }
    unsigned grid = 0;
    for (int i = 0; i < count; ++i) {
        const GemmArgs &a = *layers[order[i]];
        const int tiles_n = (a.N + ManyW8::BN - 1) / ManyW8::BN;
        b.l[i] = {a.q, a.s_a, a.w, a.s_w, a.bias, a.y, a.N, a.K, a.group, many_kind(a), tiles_n, (b.tiles_m * tiles_n + XCDS - 1) / XCDS * XCDS};
        grid += (unsigned)b.l[i].padded;
    }
    hipLaunchKernelGGL(qgemm_many, dim3(grid), dim3(256), MANY_LDS, stream, b);
    return hipGetLastError();
}

}  // namespace ql
