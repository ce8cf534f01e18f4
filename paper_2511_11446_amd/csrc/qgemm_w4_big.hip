// INT8 x INT4 -> INT32 GEMM with one weight scale per 128 inputs on large tiles, for gfx950: the 4-bit layers with groups of 128
// (Step 2; Algorithm 2 Phase B) where M and N fill the chip with such tiles.
//
//   P[m,g,n] = sum_{k in group g} q[m,k] * w4[n,k]              v_mfma_i32_16x16x64_i8, nibbles fed as value * 16
//   f        = fma(float(P[m,g,n]), s_w[n,g], f)                 g ascending, fp32
//   y[m,n]   = fp16(fma(f, alpha[m/R], bias[n]))
//
// What bounds such a layer is the vector ALU: a conversion and a multiply-add per result and group, and the unpacking of the
// nibbles.  A K step of 128 bytes is one group, and a wavefront finishes it block by block: the two MFMAs of a 16x16
// block follow each other, so the int32 sums live for a few MFMAs only (two sets of two blocks) and the fp32 sums alone fill the
// register file.  That allows a tile twice as large as qgemm_w4's (the unpacking is shared by twice as many MFMAs), and the fold of
// one pair of blocks is issued between the MFMAs of the next.
//   - Eight wavefronts own a tile of 256 x 288, 256 x 256 or 128 x 288; the columns, the ring that does not drain between tiles, the
//     scales by DMA and the stores straight from registers are those of qgemm_big.
//   - Within a K step, which k an MFMA multiplies is free as long as both operands agree: lane quarter c holds k = 32 c .. 32 c + 31,
//     so that a lane reads the packed weights of both MFMAs at once (16 bytes).
// At M = 16384 the vector ALU is busy 69 % of the kernel, the matrix cores 34 %, and LDS bank conflicts take 15 % of the CU cycles
// (profiles/qgemm_big_qgemm_w4_big_c5_stack_m16384_sq_counters.txt).  The 16 lanes of a group-scale read hold columns 8 apart, hence lie 16 G bytes
// apart: on 16 different banks where G is odd (K = 1152), on 4 of the 64 where G = 36 (K = 4608).
// Same bits as qgemm_w4.  M = 16384, random operands, us against its 128x128 tiles: K = 1152: N = 1152 36 -> 32, N = 3456 94 -> 87,
// N = 4608 126 -> 115; K = 4608, N = 1152 111 -> 100.
#include "qgemm_common.h"

namespace ql {

template <int MT_, int NT_>
struct TileW4Big {
    static constexpr int MT = MT_, WM = 4, WN = 2, NW = 8, NTHR = 512;
    static constexpr bool TAIL = NT_ == 9;
    static constexpr int NM = 8;                                             // main blocks of a wavefront: 128 columns
    static constexpr int TI = TAIL ? MT / 2 : 0;                             // row blocks of the tail, two column blocks each
    static constexpr int BM = 16 * MT * WM, BN = 16 * NT_ * WN;
    static constexpr int A_GROUPS = BM / 8, B_GROUPS = BN / 16;              // 1024-byte DMA instructions per K step
    static constexpr int NA = A_GROUPS / NW, NB = (B_GROUPS + NW - 1) / NW;  // per wavefront
    static constexpr int LEAST = NA + B_GROUPS / NW;                         // the fewest a wavefront issues
    static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 64, STAGE = A_BYTES + B_BYTES;
    static constexpr int FR = NM + (TAIL ? 2 : 0);                           // weight fragments per K step
    static constexpr int NBUF = FR / 2, DIST = NBUF - 1, GAP = 1;            // a fragment is read DIST ahead; the stages change hands
    static constexpr int HAND = FR - DIST + GAP, SPAN = FR - HAND;           // GAP fragments behind the last read of a step
    static constexpr int LOADS = (NA + NB + SPAN - 1) / SPAN;
    static constexpr int STORES = 4 * MT + 4 * TI;                           // per wavefront and full tile
    // fragments of the next step requested by the end of fragment HAND + k
    static constexpr int ahead(int k) { return 2 * (k + 1) < k + GAP + 1 ? 2 * (k + 1) : k < 0 ? 0 : k + GAP + 1; }
    static constexpr bool is_tail(int f) { return TAIL && f >= NM / 2 && f < NM / 2 + 2; }
    // column block of fragment f: the two of the tail in the middle
    static constexpr int block_of(int f) { return !TAIL || f < NM / 2 ? f : is_tail(f) ? f - NM / 2 : f - 2; }
    // a fragment's row blocks are multiplied two at a time
    static constexpr int rows(int f) { return is_tail(f) ? TI : MT; }
    static constexpr int units(int f) { return (rows(f) + 1) / 2; }
    static constexpr int unit_rows(int f, int u) { return rows(f) - 2 * u < 2 ? rows(f) - 2 * u : 2; }
    static constexpr int units_before(int f)
    {
        int n = 0;
        for (int i = 0; i < f; ++i) n += units(i);
        return n;
    }
    // behind the stages: twice (this tile, next tile) the group scales of the tile's columns, the row scales and the binary16 biases,
    // each rounded up to whole DMA instructions
    static constexpr int MAX_GROUPS = 40, SG_Q = (BN * MAX_GROUPS * 2 + 1023) / 1024;
    static constexpr int SA_Q = (BM + 63) / 64, SB_Q = (BN + 127) / 128;
    static constexpr int ROWS0 = SG_Q * 1024, SCALES = ROWS0 + (SA_Q + SB_Q) * 256, S0 = 2 * STAGE, LDS_BYTES = S0 + 2 * SCALES;
    static_assert(FR % NBUF == 0 && NBUF > DIST && A_GROUPS % NW == 0 && units_before(FR) % 2 == 0, "shape");
    static_assert(LDS_BYTES <= 160 * 1024 && STORES < 64 && SPAN > 0 && ahead(SPAN - 1) == DIST, "LDS, outstanding operations, ring");
};

template <class T, bool GLUE>
__global__ __launch_bounds__(T::NTHR, 2) void qgemm_w4_big(GemmArgs a, int tiles_m, int tiles_n, int nblk_padded, int group_m)
{
    constexpr int MT = T::MT, NM = T::NM, TI = T::TI, NA = T::NA, NB = T::NB, FR = T::FR;
    extern __shared__ __align__(1024) unsigned char smem[];

    const int per_xcd = nblk_padded / XCDS, slots_per_xcd = gridDim.x / XCDS;
    const int xcd_first = (blockIdx.x % XCDS) * per_xcd;
    int in_xcd = blockIdx.x / XCDS;
    if (in_xcd >= per_xcd || xcd_first + in_xcd >= tiles_m * tiles_n) return;
    int m0, n0;
    auto set_tile = [&](int logical) {
        const int group_sz = group_m * tiles_n;
        const int first_m = (logical / group_sz) * group_m;
        const int gm = min(tiles_m - first_m, group_m);
        m0 = (first_m + (logical % group_sz) % gm) * T::BM;
        n0 = ((logical % group_sz) / gm) * T::BN;
    };
    set_tile(xcd_first + in_xcd);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::WN, wn = wave % T::WN;
    const int M = a.M, N = a.N, K = a.K;
    const int nk = K / 128, G = nk;   // at least 2

    // ---- DMA: of a 1024-byte group lane l fills bytes [16 l, 16 l + 16): activations: row l/8, slot l%8, chunk c of row r at slot
    // c ^ ((r >> 1) & 7); packed weights: row l/4, slot l%4, chunk c at slot c ^ ((r >> 2) & 3).
    // LDS row 16 j + p of a wavefront's 128 columns is column 8 p + j of them, and row 16 b + p of the tail its column 2 p + b.
    unsigned offA[NA], offB[NB];
    auto set_off = [&]() {
        int lane = tid & 63;   // opaque: what is computed from it is not kept in registers through the K loop
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int row = 8 * (wave + i * T::NW) + (lane >> 3);
            offA[i] = (unsigned)(min(m0 + row, M - 1) * K + 16 * ((lane & 7) ^ ((row >> 1) & 7)));
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int g = wave + i * T::NW, p = lane >> 2;
            const int col = g < NM * T::WN ? (g / NM) * 16 * NM + 8 * p + g % NM : 16 * NM * T::WN + 2 * p + (g - NM * T::WN);
            offB[i] = (unsigned)(min(n0 + col, N - 1) * (K / 2) + 16 * ((lane & 3) ^ ((p >> 2) & 3)));
        }
    };
    auto issue = [&](int kt, int stage, int li) {
        unsigned char *st = smem + stage * T::STAGE;
        if (li < NA) dma16_buf(a.q, M * K, st + (wave + li * T::NW) * 1024, offA[li < NA ? li : 0], kt * 128);
        else if (T::B_GROUPS % T::NW == 0 || wave + (li - NA) * T::NW < T::B_GROUPS)
            dma16_buf(a.w, N * (K / 2), st + T::A_BYTES + (wave + (li - NA) * T::NW) * 1024, offB[li < NA ? 0 : li - NA], kt * 64);
    };
    // the tile's scales, straight to LDS; the group scales of its columns are one run of BN * G values, and what lies behind the end of
    // the tensor reads as zero
    auto fetch_scales = [&](int par) {
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        unsigned char *s = smem + T::S0 + par * T::SCALES;
        for (int c = wave; c * 1024 < T::BN * G * 2; c += T::NW)
            dma16_buf(a.s_w, N * G * 2, s + c * 1024, (unsigned)(n0 * G * 2 + c * 1024 + lane * 16), 0);
#pragma unroll
        for (int c = 0; c < T::SA_Q + T::SB_Q; ++c) {
            if (wave != c % T::NW) continue;
            if (c < T::SA_Q) dma4_buf(a.s_a, ((M - 1) / a.R + 1) * 4, s + T::ROWS0 + c * 256, (unsigned)(min(m0 + 64 * c + lane, M - 1) / a.R * 4));
            else if (a.bias) dma4_buf(a.bias, N * 2, s + T::ROWS0 + c * 256, (unsigned)(n0 + 128 * (c - T::SA_Q) + 2 * lane) * 2u);
        }
    };

    // ---- fragments: lane = row (lane & 15) of a 16-row block; quarter c = lane >> 4: of the activations chunks 2 c and 2 c + 1 (one per
    // MFMA), of the packed weights chunk c
    v4f acc[MT][NM], tail[TI > 0 ? TI : 1][2];
    v4i part[2][2], af[2][MT], bf[T::NBUF];
    unsigned short sraw[T::NBUF];
    // LDS addresses of the fragments in this step's stage.  A wavefront with wn = 1 starts with the upper half of its row
    // blocks, so that the tail's blocks are the first ones of both.
    int pa[2], pb;
    const int hi_step = T::TAIL ? wn * TI * 4096 : 0;   // from the lower to the upper half of the row blocks, and back
    {
        const int lane = tid & 63;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            pa[h] = (lane & 15) * 128 + ((2 * (lane >> 4) + h) ^ ((lane >> 1) & 7)) * 16 + (wm * MT + (T::TAIL ? wn * TI : 0)) * 2048;
        pb = T::A_BYTES + (lane & 15) * 64 + ((lane >> 4) ^ ((lane >> 2) & 3)) * 16;
    }
    const int p_lane = tid & 15;
    auto turn = [&](int &p, int stage) { p += stage ? -T::STAGE : T::STAGE; };
    auto row_block = [&](int i) { return T::TAIL ? (wn ? (i < TI ? i + TI : i - TI) : i) : i; };
    auto read_a = [&](int h, int i) {
        af[h][i] = *reinterpret_cast<const v4i *>(smem + (i < TI || !T::TAIL ? pa[h] : pa[h] - hi_step) + i * 2048);
    };
    auto read_b = [&](int f, int step, int par) {   // fragment f of K step `step` and the group scale of this lane's column
        const int b = T::block_of(f);
        bf[f % T::NBUF] = *reinterpret_cast<const v4i *>(smem + pb + (T::is_tail(f) ? T::WN * NM + b : wn * NM + b) * 1024);
        const int col = T::is_tail(f) ? T::WN * 16 * NM + 2 * p_lane + b : wn * 16 * NM + 8 * p_lane + b;
        sraw[f % T::NBUF] = *reinterpret_cast<const unsigned short *>(smem + T::S0 + par * T::SCALES + (col * G + step) * 2);
    };

    set_off();
    fetch_scales(0);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int li = 0; li < NA + NB; ++li) issue(kt, kt, li);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(T::LEAST) : "memory");   // step 0 and the scales
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        read_a(0, i);
        read_a(1, i);
    }
#pragma unroll
    for (int f = 0; f < T::DIST; ++f) read_b(f, 0, 0);

    bool stores_behind = false;   // this wavefront's youngest vector memory operations are STORES stores
    for (int cur = 0, par = 0;; par ^= 1) {   // one pass per tile
        const int em0 = m0, en0 = n0;
        in_xcd += slots_per_xcd;
        const bool has_next = in_xcd < per_xcd && xcd_first + in_xcd < tiles_m * tiles_n;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NM; ++j) acc[i][j][r] = 0.0f;
#pragma unroll
            for (int i = 0; i < TI; ++i) tail[i][0][r] = tail[i][1][r] = 0.0f;
            part[1][0][r] = part[1][1][r] = 0;
        }
        float sc_prev = 0.0f;   // scale of the last fragment of the step before

        // the int32 sums of unit u of fragment f -> fp32 sums
        auto fold = [&](int f, int u, float s) {
            const int b = T::block_of(f), set = (T::units_before(f) + u) & 1;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (i >= T::unit_rows(f, u)) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = (float)part[set][i][r];
                    if (T::is_tail(f)) tail[T::is_tail(f) ? 2 * u + i : 0][b & 1][r] = __builtin_fmaf(v, s, tail[T::is_tail(f) ? 2 * u + i : 0][b & 1][r]);
                    else acc[2 * u + i][b][r] = __builtin_fmaf(v, s, acc[2 * u + i][b][r]);
                }
            }
        };

        // the folded sums are needed here: left alone, the compiler moves all folds behind the K step, out of the MFMAs' shadow
        auto keep = [&](int f, int u) {
            const int b = T::block_of(f);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (i >= T::unit_rows(f, u)) continue;
                if (T::is_tail(f)) asm volatile("" : "+v"(tail[T::is_tail(f) ? 2 * u + i : 0][b & 1]));
                else asm volatile("" : "+v"(acc[2 * u + i][b]));
            }
        };

        // One K step per pass.  Fragment f: its MFMAs, two row blocks at a time, with the folds of the two before between them; then
        // fragment f + DIST is requested.  Before fragment HAND every fragment of this stage has been requested, and the activations of
        // the whole step are in registers: once they have arrived and the next step is in LDS, the stages change hands; from
        // there on the fragments of the next step are read, and this stage is refilled with the step after it.  Behind the very last
        // step the reads find stale bytes, which nothing uses.
        for (int kt = 0; kt < nk; ++kt, cur ^= 1) {
            const bool refill = kt + 2 < nk || has_next;
            const int step = kt + 2 < nk ? kt + 2 : kt + 2 - nk;
            const int next = kt + 1 < nk ? kt + 1 : 0, next_par = kt + 1 < nk ? par : par ^ 1;
#pragma unroll
            for (int f = 0; f < FR; ++f) {
                if (f == T::HAND) {
                    // behind a tile's stores, step 1 is older than they are
                    if (stores_behind) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(T::STORES) : "memory");
                    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                    stores_behind = false;
                    __builtin_amdgcn_s_barrier();
                }
                __builtin_amdgcn_sched_barrier(0);
                const v4i p = bf[f % T::NBUF];
                float sc = half_to_float_dev(sraw[f % T::NBUF]);
                asm volatile("" : "+v"(sc));   // converted once, not in every multiply-add
                const v4i w0 = {(int)(((unsigned)p[0] << 4) & 0xf0f0f0f0u), (int)((unsigned)p[0] & 0xf0f0f0f0u),
                                (int)(((unsigned)p[1] << 4) & 0xf0f0f0f0u), (int)((unsigned)p[1] & 0xf0f0f0f0u)};
                const v4i w1 = {(int)(((unsigned)p[2] << 4) & 0xf0f0f0f0u), (int)((unsigned)p[2] & 0xf0f0f0f0u),
                                (int)(((unsigned)p[3] << 4) & 0xf0f0f0f0u), (int)((unsigned)p[3] & 0xf0f0f0f0u)};
#pragma unroll
                for (int u = 0; u < T::units(f); ++u) {
                    const int set = (T::units_before(f) + u) & 1;
                    const v4i zero = {0, 0, 0, 0};
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (i < T::unit_rows(f, u)) part[set][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[0][2 * u + i], w0, zero, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (i < T::unit_rows(f, u)) part[set][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[1][2 * u + i], w1, part[set][i], 0, 0, 0);
                    if (u > 0) fold(f, u - 1, sc);
                    else if (f > 0) fold(f - 1, T::units(f - 1) - 1, sc_prev);
                    else fold(FR - 1, T::units(FR - 1) - 1, sc_prev);
                    // vector ALU work between the MFMAs; the first unit waits for its weights
                    if (u == 0) __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
#pragma unroll
                    for (int i = 0; i < 2 * T::unit_rows(f, u); ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                    }
                    if (u > 0) keep(f, u - 1);
                    else if (f > 0) keep(f - 1, T::units(f - 1) - 1);
                    else keep(FR - 1, T::units(FR - 1) - 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (f == FR - 1) {   // these row blocks' activations are done with: the next step's
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            read_a(0, 2 * u + i);
                            read_a(1, 2 * u + i);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                sc_prev = sc;
                if (f == T::HAND) {
                    turn(pa[0], cur);
                    turn(pa[1], cur);
                    turn(pb, cur);
                    if (kt == nk - 2 && has_next) {
                        set_tile(xcd_first + in_xcd);
                        set_off();
                        fetch_scales(par ^ 1);
                    }
                }
                if (f >= T::HAND) {
#pragma unroll
                    for (int n = T::ahead(f - T::HAND - 1); n < T::ahead(f - T::HAND); ++n) read_b(n, next, next_par);
                    if (refill) {
#pragma unroll
                        for (int li = (f - T::HAND) * T::LOADS; li < (f - T::HAND + 1) * T::LOADS; ++li)
                            if (li < NA + NB) issue(step, cur, li);
                    }
                } else if (f + T::DIST < FR) {
                    read_b(f + T::DIST, kt, par);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        fold(FR - 1, T::units(FR - 1) - 1, sc_prev);

        // ---- epilogue
        int lane = tid & 63;   // opaque, as in set_off
        asm volatile("" : "+v"(lane));
        const int p = lane & 15, kq = lane >> 4;
        _Float16 *y = static_cast<_Float16 *>(a.y);
        const float *s_row = reinterpret_cast<const float *>(smem + T::S0 + par * T::SCALES + T::ROWS0) + wm * 16 * MT + 4 * kq;
        const _Float16 *b_col = reinterpret_cast<const _Float16 *>(smem + T::S0 + par * T::SCALES + T::ROWS0 + T::SA_Q * 256);
        const int m_base = em0 + wm * 16 * MT + 4 * kq;
        const int c_main = wn * 16 * NM + 8 * p, c_tail = T::WN * 16 * NM + 2 * p;
        const bool full = em0 + T::BM <= M && en0 + T::BN <= N;
        const GateRows gate_rows(GLUE ? a.gate : nullptr, a.gate_rows, em0, T::BM);
        // C neighbouring columns from column c of the tile; v(i, e): fp32 sum of row block i and column e
        auto columns = [&](auto count_tag, int c, int blocks, auto v) {
            constexpr int C = decltype(count_tag)::value;
            typedef _Float16 hC __attribute__((ext_vector_type(C)));
            float b[C];
#pragma unroll
            for (int e = 0; e < C; ++e) b[e] = a.bias ? (float)b_col[c + e] : -0.0f;   // x + -0.0 is x, signed zeros included
            const int n = en0 + c;
#pragma unroll
            for (int i = 0; i < blocks; ++i) {
                const int blk = row_block(i);
                const v4f sa = *reinterpret_cast<const v4f *>(s_row + 16 * blk) * 0.0625f;   // the nibbles were used as value * 16
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int m = m_base + 16 * blk + r;
                    const bool mine = full || (m < M && n < N);
                    const unsigned off = (unsigned)(m * N + n);
                    hC g, res, out;
                    if (GLUE && mine && a.gate) g = *reinterpret_cast<const hC *>(static_cast<const _Float16 *>(a.gate) + (unsigned)(gate_rows.of(m - em0) * N + n));
                    if (GLUE && mine && a.residual) res = *reinterpret_cast<const hC *>(static_cast<const _Float16 *>(a.residual) + off);
#pragma unroll
                    for (int e = 0; e < C; ++e) {
                        float u = __builtin_fmaf(v(i, e)[r], sa[r], b[e]);
                        if (GLUE && a.act == 1) u = gelu_tanh_dev(u);
                        asm volatile("" : "+v"(u));   // keep the fp32 rounding before the fp16 one
                        out[e] = (_Float16)u;
                        if (GLUE && (a.gate || a.residual)) {
                            u = __builtin_fmaf(a.gate ? (float)g[e] : 1.0f, (float)out[e], a.residual ? (float)res[e] : 0.0f);
                            asm volatile("" : "+v"(u));
                            out[e] = (_Float16)u;
                        }
                    }
                    // streamed out from the last tile, through the L2 before another one (as in qgemm_big)
                    typedef hC hC_alias __attribute__((may_alias));
                    if (mine) {
                        if (has_next) *reinterpret_cast<hC_alias *>(y + off) = out;
                        else __builtin_nontemporal_store(out, reinterpret_cast<hC_alias *>(y + off));
                    }
                    if (GLUE && a.row_absmax) {
                        // the row's largest over the 16 lanes that hold it, then one atomic
                        typedef unsigned short usC __attribute__((ext_vector_type(C)));
                        const usC mag = __builtin_bit_cast(usC, out) & (unsigned short)0x7fff;
                        unsigned top = mine ? __builtin_reduce_max(mag) : 0;
                        top = max(top, (unsigned)__builtin_amdgcn_mov_dpp((int)top, 0x128 /* row_ror:8 */, 0xF, 0xF, true));
                        top = max(top, (unsigned)__builtin_amdgcn_mov_dpp((int)top, 0x124, 0xF, 0xF, true));
                        top = max(top, (unsigned)__builtin_amdgcn_mov_dpp((int)top, 0x122, 0xF, 0xF, true));
                        top = max(top, (unsigned)__builtin_amdgcn_mov_dpp((int)top, 0x121, 0xF, 0xF, true));
                        if (p == 0 && m < M && top) atomicMax(a.row_absmax + m, top);
                    }
                }
            }
        };
        columns(std::integral_constant<int, 8>{}, c_main, MT, [&](int i, int e) { return acc[i][e]; });
        if constexpr (T::TAIL) columns(std::integral_constant<int, 2>{}, c_tail, TI, [&](int i, int e) { return tail[i][e]; });
        stores_behind = full && !GLUE;
        if (!has_next) break;
    }
}

template <class T, bool GLUE>
static hipError_t run_w4_big(const GemmArgs &a, hipStream_t s)
{
    static const hipError_t opt_in = hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_w4_big<T, GLUE>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    if (opt_in != hipSuccess) return opt_in;
    const int tiles_m = (a.M + T::BM - 1) / T::BM, tiles_n = (a.N + T::BN - 1) / T::BN;
    const int padded = (tiles_m * tiles_n + XCDS - 1) / XCDS * XCDS;
    static const int resident = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < XCDS)
            return 0;
        return cus / XCDS * XCDS;
    }();
    if (resident <= 0) return hipErrorInvalidDevice;
    hipLaunchKernelGGL((qgemm_w4_big<T, GLUE>), dim3(padded < resident ? padded : resident), dim3(T::NTHR), T::LDS_BYTES, s, a, tiles_m, tiles_n,
                       padded, pick_group_m(T::BM));
    return hipGetLastError();
}

// what these kernels take of a layer: groups of one K step, at least two of them, 16-byte rows everywhere
bool qgemm_w4_big_takes(const GemmArgs &a)
{
    return a.w_bits == 4 && a.group == 128 && !a.w_grouped && !a.s_ag && !a.acc_out && a.K % 128 == 0 && a.K >= 256 && a.K / 128 <= 40 &&
           a.N % 8 == 0 && (uintptr_t)a.q % 16 == 0 && (uintptr_t)a.w % 16 == 0 && (uintptr_t)a.s_w % 4 == 0 && (uintptr_t)a.y % 16 == 0 &&
           (uintptr_t)a.bias % 4 == 0 && (uintptr_t)a.gate % 16 == 0 && (uintptr_t)a.residual % 16 == 0;
}

#define BIG(name, ...)                                                                                           \
    hipError_t launch_big_##name(const GemmArgs &a, hipStream_t s) { return run_w4_big<TileW4Big<__VA_ARGS__>, false>(a, s); }  \
    hipError_t launch_big_##name##_glue(const GemmArgs &a, hipStream_t s) { return run_w4_big<TileW4Big<__VA_ARGS__>, true>(a, s); }
BIG(w4_256x288, 4, 9)
BIG(w4_256x256, 4, 8)
BIG(w4_128x288, 2, 9)

}  // namespace ql
