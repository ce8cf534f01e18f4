// GEMM + dequantization for the shapes the pipelined kernels do not serve well, for gfx950:
//
//   qgemm_splitk   few rows: 32x32 or 16x16 output tiles, K split over the four or eight wavefronts of a workgroup
//   qgemm_edge     an inner size or an alignment that the DMA kernels do not take, and rows of a few K steps that are no whole ones:
//                workgroup tiles staged through registers, the last K step padded with zeros.  Its 16-byte loads may be misaligned (the hardware splits them), and a
//                piece that crosses the end of a row is read byte by byte, so that no access leaves the operand.
//
// Both take 8-bit weights, packed 4-bit weights, int8 codes with group scales and binary16 operands.
#include "daq_device.h"
#include "qgemm_common.h"
#include "split_walk.h"

namespace ql {

constexpr size_t SPLIT_LDS_MAX = 160 * 1024;

enum OperandKind : int { OP_I8 = 0, OP_W4 = 1, OP_I8G = 2, OP_F16 = 3 };

struct __attribute__((packed, aligned(1))) v4i_unaligned {
    v4i v;
};
struct __attribute__((packed, aligned(1))) v2i_unaligned {
    v2i v;
};

__device__ __forceinline__ v4i load16(const unsigned char *p) { return reinterpret_cast<const v4i_unaligned *>(p)->v; }

// bytes [kb, kb + 16) of a row of row_bytes bytes, zeros past its end (only the last K step of a row needs this form)
__device__ __forceinline__ v4i load_piece(const unsigned char *row, int kb, int row_bytes)
{
    if (kb + 16 <= row_bytes) return load16(row + kb);
    if ((row_bytes & 7) == 0) {
        // rows of whole 8-byte words: at most the first half is there
        v2i h = {0, 0};
        if (kb < row_bytes) h = reinterpret_cast<const v2i_unaligned *>(row + kb)->v;
        return v4i{h[0], h[1], 0, 0};
    }
    unsigned w[4] = {0, 0, 0, 0};
    // static indexes: a run-time one would put the piece into scratch memory
#pragma unroll
    for (int b = 0; b < 15; ++b)
        if (kb + b < row_bytes) w[b / 4] |= (unsigned)row[kb + b] << (8 * (b % 4));
    return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
}

// the int8 MFMA operand of 8 packed bytes (16 nibbles): nibble values times 16
__device__ __forceinline__ v4i nibbles_x16(int p0, int p1)
{
    return v4i{(int)(((unsigned)p0 << 4) & 0xf0f0f0f0u), (int)((unsigned)p0 & 0xf0f0f0f0u), (int)(((unsigned)p1 << 4) & 0xf0f0f0f0u),
               (int)((unsigned)p1 & 0xf0f0f0f0u)};
}

// Which tile a workgroup takes: ids go round-robin over the XCDs, each XCD owns consecutive logical tiles, and group_m
// tile rows are walked together so that one L2 sees few distinct panels of both operands.
__device__ __forceinline__ bool pick_tile(int tiles_m, int tiles_n, int nblk_padded, int group_m, int &tm, int &tn)
{
    const int logical = (blockIdx.x % XCDS) * (nblk_padded / XCDS) + blockIdx.x / XCDS;
    if (logical >= tiles_m * tiles_n) return false;
    const int group_sz = group_m * tiles_n;
    const int first_m = (logical / group_sz) * group_m;
    const int gm = min(tiles_m - first_m, group_m);
    tm = first_m + (logical % group_sz) % gm;
    tn = (logical % group_sz) / gm;
    return true;
}

// the layer's fp32 value of one element from its integer or fp32 sum (formulas in the public header)
template <int KIND>
__device__ __forceinline__ float dequant_one(const GemmArgs &a, int acc, float f, float sa, float sw, float b)
{
    if (KIND == OP_F16) return f + b;
    if (KIND == OP_I8) {
        const float t = (float)acc * sa;
        return a.bias ? __builtin_fmaf(t, sw, b) : t * sw;
    }
    if (a.s_ag) return a.bias ? f + b : f;
    return a.bias ? __builtin_fmaf(f, sa, b) : f * sa;
}

// ---- few rows ------------------------------------------------------------------------------------------------------
// A workgroup of W = 4 or 8 wavefronts owns NB neighbouring T x T output tiles (T = 32 or 16, one MFMA each) and SPLITS K: every wavefront walks
// its own K steps, whose operand pieces go global -> LDS by DMA through a ring of its own, and waits for nobody until the
// partial results meet in LDS.
//
// What bounds it: at these sizes neither bytes nor MFMAs but the chain launch -> first bytes -> serial walk over K ->
// store.  The 64x64 workgroup tiles of the other kernels leave most CUs empty (M = 64, N = 1152: 18 workgroups) and pay
// a workgroup hand-over for every K step of 128.  A wavefront's K step still costs some 400 cycles of latency (LDS
// read, MFMA, fold), so the walk is cut into four or eight.
//
// Group scales (4-bit weights, int8 codes with group scales): a wavefront takes whole groups and leaves every group's sum
// in LDS; the fp32 sum over the groups, whose ascending order is part of the definition, is then taken by the thread that
// owns the element.  Where the sums of all groups do not fit, this happens in rounds.
//
// FUSE: the activations arrive as fp16 and are quantized by the workgroup itself (Step 3, eq. (4) with tau = the absolute
// maximum), its T rows of codes resident in LDS while only the weights pass through the rings.  The codes are
// recomputed by every workgroup of the row - 36 elements per thread for 16 rows of 1152 - but a kernel launch
// less is worth more: some 3.6 us of host time and 2.6-3.5 us of GPU time at these sizes.
// W wavefronts; NB tiles side by side; S: ring depth per wavefront
template <int KIND, int T, bool FUSE, int W_ = 4, int NB_ = 1>
struct SplitTile {
    static constexpr int W = W_, NB = NB_, NTHR = 64 * W;
    static constexpr bool GROUPED = KIND == OP_W4 || KIND == OP_I8G;
    static constexpr int A_GROUPS = FUSE ? 0 : T / 8, B_GROUPS = NB * (KIND == OP_W4 ? T / 16 : T / 8);   // 1024-byte DMA instructions per K step
    static constexpr int LOADS = A_GROUPS + B_GROUPS;
    static constexpr int STAGE = LOADS * 1024;
    // ring depth per wavefront; how many workgroups a CU holds is counted from all that they keep in LDS (split_rounds)
    static constexpr int S = T == 32 || W == 8 ? 2 : GROUPED ? 3 : 4;
    static constexpr int TILE = NB * T * T * 4;                 // partial tiles of a wavefront or group, bytes
};

// EXPORT: the integer sums are also written to a.acc_out (verification)
template <int KIND, int T, bool GLUE, bool EXPORT, bool FUSE, int W, int NB>
__global__ __launch_bounds__(64 * W, W == 8 && NB <= 2 ? 4 : 2) void qgemm_splitk(GemmArgs a, int tiles_m, int tiles_n, int nblk_padded, int gpr, int rounds, int slots)
{
    using C = SplitTile<KIND, T, FUSE, W, NB>;
    constexpr bool GROUPED = C::GROUPED;
    constexpr int EB = KIND == OP_F16 ? 2 : 1;
    constexpr int S = C::S, RG = T * T / 64;        // accumulator registers per lane and tile: 16 or 4
    constexpr int EPT = (NB * RG + W - 1) / W;      // elements a thread finishes
    constexpr int BSTEP = KIND == OP_W4 ? 64 : 128; // bytes of a weight row per K step
    typedef typename std::conditional<KIND == OP_F16, float, int>::type elem_t;
    typedef elem_t acc_t __attribute__((ext_vector_type(RG)));
    extern __shared__ __align__(1024) unsigned char smem[];
    int tm, tn;
    if (!pick_tile(tiles_m, tiles_n, nblk_padded, tiles_m, tm, tn)) return;
    const int m0 = tm * T, n0 = tn * T * NB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & (T - 1), kq = lane / T;   // fragment row, and the lane's part of a slice
    const int M = a.M, N = a.N, K = a.K;
    const int KB = K * EB, WB = KIND == OP_W4 ? K / 2 : KB;
    const int group = GROUPED ? a.group : 128, G = GROUPED ? K / group : 0;

    // ---- the K steps of this wavefront; the next one to be requested, and the next one to be read
    const SplitWalk<GROUPED, W> walk(wave, KB, group, G, gpr, rounds);
    const int steps = walk.steps;
    typename SplitWalk<GROUPED, W>::Position ask = walk.first(wave), use = ask;

    // ---- DMA: lane l fills bytes [16 l, 16 l + 16) of a 1024-byte group.  128-byte rows: row l/8, chunk c of row r at slot
    // c ^ ((r >> 1) & 7); packed 4-bit rows (64 bytes): row l/4, chunk c at slot c ^ ((r >> 2) & 3).
    // slot i of a wavefront lies behind slot i of the others, so that a short row leaves nothing unused between them
    auto slot_at = [&](int slot) { return smem + (wave + slot * W) * C::STAGE; };
    const int rings = slots * C::STAGE;
    // The buffer form: descriptor and step offset in scalar registers, the lane's fixed offset in one vector register.
    constexpr int NA = FUSE ? 1 : C::A_GROUPS;
    int offA[NA], offB[C::B_GROUPS], ca[NA], cb[C::B_GROUPS];   // c*: the lane's byte inside a row's K step
#pragma unroll
    for (int i = 0; i < C::A_GROUPS; ++i) {
        const int row = 8 * i + (lane >> 3);
        ca[i] = 16 * ((lane & 7) ^ ((row >> 1) & 7));
        offA[i] = min(m0 + row, M - 1) * KB + ca[i];
    }
#pragma unroll
    for (int i = 0; i < C::B_GROUPS; ++i) {
        const int row = KIND == OP_W4 ? 16 * i + (lane >> 2) : 8 * i + (lane >> 3);
        cb[i] = KIND == OP_W4 ? 16 * ((lane & 3) ^ ((row >> 2) & 3)) : 16 * ((lane & 7) ^ ((row >> 1) & 7));
        offB[i] = min(n0 + row, N - 1) * WB + cb[i];
    }
    auto issue = [&](int slot) {
        const int kb = ask.kb, wb = KIND == OP_W4 ? kb / 2 : kb;
        walk.next(ask);
        unsigned char *dst = slot_at(slot);
        if (kb + 128 <= KB) {
#pragma unroll
            for (int j = 0; j < C::A_GROUPS; ++j) dma16_buf(a.q, M * KB, dst + j * 1024, offA[j], kb);
#pragma unroll
            for (int j = 0; j < C::B_GROUPS; ++j)
                dma16_buf(a.w, N * WB, dst + (C::A_GROUPS + j) * 1024, offB[j], wb);
        } else {
            // a chunk past the end of its row reads the row's last one instead (such slices are skipped, or zeroed in registers)
#pragma unroll
            for (int j = 0; j < C::A_GROUPS; ++j)
                dma16_buf(a.q, M * KB, dst + j * 1024, offA[j] - max(kb + ca[j] - (KB - 16), 0), kb);
#pragma unroll
            for (int j = 0; j < C::B_GROUPS; ++j)
                dma16_buf(a.w, N * WB, dst + (C::A_GROUPS + j) * 1024, offB[j] - max(wb + cb[j] - (WB - 16), 0), wb);
        }
    };
    // FUSE: the rows first, since loads return in order
    constexpr int CH = SPLIT_FUSE_K_MAX / 512, RB = FUSE ? T / W : 1;    // 8-value pieces per lane and row; rows of this wavefront
    uint4 v[RB][CH];
    if constexpr (FUSE) {
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const unsigned short *xr = static_cast<const unsigned short *>(a.x) + (size_t)min(m0 + wave * RB + r, M - 1) * K;
#pragma unroll
            for (int i = 0; i < CH; ++i) v[r][i] = load_row_piece(xr, K * 2, lane * 16, i * 1024);
        }
    }
#pragma unroll
    for (int st = 0; st < S; ++st)
        if (st < steps) issue(st);
    // ---- what the folds and the epilogue need: requested behind the first K steps (the waits for these, which count loads
    // issued later, then at most wait longer than they must)
    // the elements a thread finishes: registers EPT * wave + e, of all NB tiles one after the other
    auto reg_of = [&](int e) { return EPT * wave + e; };
    auto row_of = [&](int e) { return T == 32 ? 8 * (reg_of(e) % RG / 4) + 4 * kq + reg_of(e) % 4 : 4 * kq + reg_of(e) % RG; };
    auto tile_of = [&](int e) { return NB == 1 ? 0 : reg_of(e) / RG; };
    auto col_of = [&](int e) { return n0 + tile_of(e) * T + fr; };
    auto owns = [&](int e) { return NB * RG % W == 0 || reg_of(e) < NB * RG; };
    // partial tiles: of every group of a round, or one per wavefront in its own ring, which by then is idle
    unsigned char *part = smem + (GROUPED ? rings : 0);
    constexpr int PART = GROUPED ? C::TILE : C::STAGE;
    static_assert(GROUPED || C::STAGE >= C::TILE, "a partial tile fits its wavefront's first slot");
    float *ctab = reinterpret_cast<float *>(smem + rings + (GROUPED ? min(W * gpr, G) * C::TILE : 0));   // [G][T * NB] group scales of the tile's columns
    if constexpr (GROUPED) {
        // a thread looks after every NTHR-th entry; nibbles enter the products as value * 16, the scale carries the 1/16 (exact)
        const unsigned short *src = static_cast<const unsigned short *>(a.s_w);
        const float *sag = a.s_ag ? a.s_ag + (size_t)(min(m0, M - 1) / a.R) * G : nullptr;   // one scale block per tile
        constexpr int COLS = T * NB;
        for (int at = threadIdx.x; at < G * COLS; at += 4 * C::NTHR) {
            unsigned short h[4];
            float al[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int g = min((at + u * C::NTHR) / COLS, G - 1);
                h[u] = src[(size_t)min(n0 + (at + u * C::NTHR) % COLS, N - 1) * G + g];
                al[u] = sag ? sag[g] : 1.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (at + u * C::NTHR < G * COLS) ctab[at + u * C::NTHR] = half_to_float_dev(h[u]) * (KIND == OP_W4 ? 0.0625f : 1.0f) * al[u];
        }
    }
    constexpr int COLUMNS = NB == 1 ? 1 : EPT;      // one tile: a thread's elements are of one column
    unsigned short bias_h[COLUMNS];
    float sw[COLUMNS];
#pragma unroll
    for (int e = 0; e < COLUMNS; ++e) {
        const int n_in = min(col_of(e), N - 1);
        bias_h[e] = a.bias ? static_cast<const unsigned short *>(a.bias)[n_in] : (unsigned short)0;
        sw[e] = KIND == OP_I8 ? static_cast<const float *>(a.s_w)[n_in] : 1.0f;
    }
    GlueTerms terms[EPT];
    if constexpr (GLUE && NB == 1) {
        request_glue<EPT>(a, terms, min(col_of(0), N - 1), EPT, [&](int e) { return min(m0 + row_of(e), M - 1); }, [&](int m) { return m / a.gate_rows; });
    } else if constexpr (GLUE) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int m = min(m0 + row_of(e), M - 1);
            terms[e] = glue_terms(a, m, min(col_of(e), N - 1), a.gate ? m / a.gate_rows : 0);
        }
    }
    // FUSE: the codes of the tile's rows, [K step][row][128 bytes] with the chunks of a row swizzled as in the rings, and the
    // rows' scales
    unsigned char *resident = reinterpret_cast<unsigned char *>(ctab + (GROUPED ? T * NB * G : 0));
    float *srow = reinterpret_cast<float *>(resident + T * split_resident_steps(K, GROUPED) * 128);
    if constexpr (FUSE) {
        const int npad = (K + 127) / 128 * 16;                    // pieces of a row of codes, whole K steps
        // all rows' maxima first, then all codes: the chains of one row are short on instructions and long on latency
        unsigned mx[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            mx[r] = 0;
            if (a.parts == 0) {
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    mx[r] = absmax_word(absmax_word(absmax_word(absmax_word(mx[r], v[r][i].x), v[r][i].y), v[r][i].z), v[r][i].w);
                mx[r] = (mx[r] & 0xffffu) > (mx[r] >> 16) ? (mx[r] & 0xffffu) : (mx[r] >> 16);
            } else {
                const unsigned *pm = a.partmax + (size_t)(min(m0 + wave * RB + r, M - 1) / a.R) * a.parts;
                for (int i = lane; i < a.parts; i += 64) mx[r] = mx[r] > pm[i] ? mx[r] : pm[i];
            }
        }
        const int rows_here = M - m0 - wave * RB;   // rows past the last one: their codes are never stored
        float alpha[RB], rcp[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            alpha[r] = alpha_from_bits(wave_max_u32(mx[r]));
            rcp[r] = 1.0f / alpha[r];
        }
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            if (r >= rows_here) continue;
            const int row = wave * RB + r;
            if (lane == 0) srow[row] = alpha[r];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int c = lane + 64 * i;        // past the end of the row: zeros
                if (c < npad)
                    *reinterpret_cast<uint2 __attribute__((may_alias)) *>(resident + ((c >> 4) * T + row) * 128 + ((((c >> 1) & 7) ^ ((row >> 1) & 7)) * 16) + (c & 1) * 8) =
                        daq_piece(v[r][i], alpha[r], rcp[r]);
            }
        }
        __syncthreads();
    }
    float sa[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int m = min(m0 + row_of(e), M - 1);
        if (FUSE) sa[e] = srow[row_of(e)];
        else sa[e] = (KIND != OP_F16 && !a.s_ag) ? a.s_a[a.R == 1 ? m : m / a.R] : 1.0f;
    }

    constexpr int NF = (T == 32 || GROUPED) ? 4 : 2;  // MFMAs per K step
    // fragments of a lane: T = 32: 16 bytes of every 32-byte slice; T = 16: 16 bytes of every 64-byte pair of slices, or with
    // group scales 8 bytes of every slice (a group may end after any slice)
    constexpr bool HALF = T == 16 && GROUPED;
    typedef typename std::conditional<HALF, v2i, v4i>::type frag_a;
    typedef typename std::conditional<KIND == OP_W4, typename std::conditional<HALF, int, v2i>::type, frag_a>::type frag_b;
    typedef frag_a frag_a_alias __attribute__((may_alias));
    typedef frag_b frag_b_alias __attribute__((may_alias));
    const int keyA = (fr >> 1) & 7, key4 = (fr >> 2) & 3;
    auto read_frags = [&](int slot, frag_a(&af)[NF], frag_b(&bf)[NF][NB]) {
        const unsigned char *st = slot_at(slot), *stb = st + C::A_GROUPS * 1024;
        const int c0 = use.kb >> 4;   // first chunk of the step inside its row
        walk.next(use);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            // first byte of the lane's part: 16-byte chunk and offset inside it
            const int chunk = HALF ? 2 * f + (kq >> 1) : f * (8 / NF) + kq, off = HALF ? 8 * (kq & 1) : 0;
            if constexpr (FUSE) {
                const int c = c0 + chunk;
                af[f] = *reinterpret_cast<const frag_a_alias *>(resident + ((c >> 3) * T + fr) * 128 + (((c & 7) ^ keyA) * 16) + off);
            } else {
                af[f] = *reinterpret_cast<const frag_a_alias *>(st + fr * 128 + ((chunk ^ keyA) * 16) + off);
            }
            // the swizzle's key repeats every 16 rows
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if constexpr (KIND == OP_W4)
                    bf[f][b] = *reinterpret_cast<const frag_b_alias *>(stb + (b * T + fr) * 64 + (((chunk >> 1) ^ key4) * 16) + (chunk & 1) * 8 + off / 2);
                else
                    bf[f][b] = *reinterpret_cast<const frag_b_alias *>(stb + (b * T + fr) * 128 + ((chunk ^ keyA) * 16) + off);
            }
        }
    };
    acc_t acc[NB];
    auto clear = [&]() {
#pragma unroll
        for (int r = 0; r < NB * RG; ++r) acc[r / RG][r % RG] = 0;
    };
    auto mma_one = [&](const frag_a &af, const frag_b &bf, acc_t c) -> acc_t {
        if constexpr (HALF) {
            long b;
            if constexpr (KIND == OP_W4)
                b = __builtin_bit_cast(long, v2i{(int)(((unsigned)bf << 4) & 0xf0f0f0f0u), (int)((unsigned)bf & 0xf0f0f0f0u)});
            else
                b = __builtin_bit_cast(long, bf);
            return __builtin_amdgcn_mfma_i32_16x16x32_i8(__builtin_bit_cast(long, af), b, c, 0, 0, 0);
        } else if constexpr (T == 32) {
            if constexpr (KIND == OP_W4) return mfma_step<false>(af, nibbles_x16(bf[0], bf[1]), c);
            else return mfma_step<KIND == OP_F16>(af, bf, c);
        } else if constexpr (KIND == OP_F16) {
            return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, af), __builtin_bit_cast(v8h, bf), c, 0, 0, 0);
        } else {
            return __builtin_amdgcn_mfma_i32_16x16x64_i8(af, bf, c, 0, 0, 0);
        }
    };
    auto mma = [&](const frag_a &af, const frag_b(&bf)[NB]) {
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b] = mma_one(af, bf[b], acc[b]);
    };
    // partial tile layout: register r of a lane at [r][lane], so that thread (wavefront w, lane) finds its elements at
    // registers EPT * w + e of the same lane
    auto park = [&](int slot) {
        elem_t *p = reinterpret_cast<elem_t *>(part + slot * PART);
#pragma unroll
        for (int r = 0; r < NB * RG; ++r) p[r * 64 + lane] = acc[r / RG][r % RG];
    };
    auto wait_for = [&](int later) {   // steps issued after the one that is needed
        if (later >= S - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * C::LOADS) : "memory");
        else if (S > 3 && later == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * C::LOADS) : "memory");
        else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(C::LOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    float f[EPT];
    elem_t sum[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        f[e] = 0.0f;
        sum[e] = 0;
    }
    frag_a af0[NF], af1[NF];
    frag_b bf0[NF][NB], bf1[NF][NB];
    int slot = 0;
    // Step i: its fragments are in (afc, bfc).  Their LDS slot is free once they have arrived: it is refilled with step i + S;
    // then the fragments of step i + 1 are requested, and step i is multiplied while they travel.
    auto advance = [&](int i, frag_a(&afn)[NF], frag_b(&bfn)[NF][NB]) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + S < steps) issue(slot);
        slot = slot + 1 == S ? 0 : slot + 1;
        if (i + 1 < steps) {
            wait_for(min(S - 1, steps - 2 - i));
            read_frags(slot, afn, bfn);
        }
    };
    if (steps > 0) {
        wait_for(min(S - 1, steps - 1));
        read_frags(0, af0, bf0);
    }
    clear();
    if constexpr (!GROUPED) {
        auto one = [&](int i, frag_a(&afc)[NF], frag_b(&bfc)[NF][NB], frag_a(&afn)[NF], frag_b(&bfn)[NF][NB]) {
            advance(i, afn, bfn);
            const int kb = (wave + W * i) * 128;
            if (!FUSE && kb + 128 > KB) {
#pragma unroll
                for (int q = 0; q < NF; ++q)
                    if (kb + (q * (8 / NF) + kq) * 16 >= KB) {
                        afc[q] = frag_a{0, 0, 0, 0};
                        if constexpr (KIND == OP_F16) bfc[q][0] = frag_b{0, 0, 0, 0};   // 0 * Inf is not 0
                    }
            }
#pragma unroll
            for (int q = 0; q < NF; ++q) mma(afc[q], bfc[q]);
        };
        for (int i = 0; i < steps; i += 2) {
            one(i, af0, bf0, af1, bf1);
            if (i + 1 < steps) one(i + 1, af1, bf1, af0, bf0);
        }
        park(wave);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w)
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (owns(e)) sum[e] += reinterpret_cast<const elem_t *>(part + w * PART)[reg_of(e) * 64 + lane];
    } else {
        const int QG = group / 32;
        int i = 0;
        for (int r = 0; r < rounds; ++r) {
            const int g_first = r * W * gpr;                                     // of the round, over all wavefronts
            const int mine = max(0, min(gpr, G - g_first - wave * gpr));
            const int i_end = i + (mine * group + 127) / 128;
            int qs = 0, done = 0;
            auto one = [&](frag_a(&afc)[NF], frag_b(&bfc)[NF][NB], frag_a(&afn)[NF], frag_b(&bfn)[NF][NB]) {
                advance(i, afn, bfn);
#pragma unroll
                for (int q = 0; q < NF; ++q) {
                    if (done < mine) {      // a round's last step may be cut short
                        mma(afc[q], bfc[q]);
                        if (++qs == QG) {
                            park(wave * gpr + done);
                            clear();
                            qs = 0;
                            ++done;
                        }
                    }
                }
                ++i;
            };
            // the fragments alternate between the two sets by the parity of i
            if ((i & 1) && i < i_end) one(af1, bf1, af0, bf0);
            while (i < i_end) {
                one(af0, bf0, af1, bf1);
                if (i < i_end) one(af1, bf1, af0, bf0);
            }
            __syncthreads();
            const int have = min(W * gpr, G - g_first);
            // U groups at a time: their sums and scales are requested together, the fp32 sum takes them in ascending order
            constexpr int U = EPT == 4 ? 4 : 8;
            auto take = [&](int g, auto count_tag) {
                constexpr int CNT = decltype(count_tag)::value;
                int p[CNT][EPT];
                float c[CNT][EPT];
#pragma unroll
                for (int u = 0; u < CNT; ++u) {
#pragma unroll
                    for (int e = 0; e < EPT; ++e) {
                        const int reg = owns(e) ? reg_of(e) : 0;
                        c[u][e] = ctab[(g_first + g + u) * T * NB + (NB == 1 ? 0 : reg / RG * T) + fr];
                        p[u][e] = reinterpret_cast<const int *>(part + (g + u) * PART)[reg * 64 + lane];
                    }
                }
#pragma unroll
                for (int u = 0; u < CNT; ++u)
#pragma unroll
                    for (int e = 0; e < EPT; ++e) {
                        if (EXPORT) {
                            const int m = m0 + row_of(e), n = col_of(e);
                            if (m < M && n < N) a.acc_out[((size_t)m * G + g_first + g + u) * N + n] = KIND == OP_W4 ? p[u][e] >> 4 : p[u][e];
                        }
                        f[e] = __builtin_fmaf((float)p[u][e], c[u][e], f[e]);
                    }
            };
            int g = 0;
            for (; g + U <= have; g += U) take(g, std::integral_constant<int, U>{});
            for (; g < have; ++g) take(g, std::integral_constant<int, 1>{});
            if (r + 1 < rounds) __syncthreads();
        }
    }

#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int m = m0 + row_of(e), n = col_of(e);
        if (m >= M || n >= N || !owns(e)) continue;
        const float b = half_to_float_dev(bias_h[e % COLUMNS]);
        float u;
        if constexpr (GROUPED) u = dequant_one<KIND>(a, 0, f[e], sa[e], 1.0f, b);
        else if constexpr (KIND == OP_F16) u = dequant_one<KIND>(a, 0, sum[e], 1.0f, 1.0f, b);
        else u = dequant_one<KIND>(a, sum[e], 0.0f, sa[e], sw[e % COLUMNS], b);
        if constexpr (KIND == OP_I8 && EXPORT) a.acc_out[(size_t)m * N + n] = sum[e];
        asm volatile("" : "+v"(u));   // keep the fp32 rounding before the fp16 one
        static_cast<_Float16 *>(a.y)[(size_t)m * N + n] = GLUE ? glue_one(a, u, m, terms[e]) : (_Float16)u;
    }
}

// ---- more rows, any inner size -------------------------------------------------------------------------------------
// 2 x 2 wavefronts of TM x TN MFMA tiles; a K step is 128 bytes of an activation row, two LDS buffers, the next step's
// global loads in flight while this one is multiplied.
// table != 0: the group scales of the tile's columns sit in LDS behind the stages (a load per group, issued among the next
// step's operand loads, would make every group wait for those); 0: more groups than the table holds, loaded as they open.
constexpr int EDGE_TABLE_GROUPS = 144;
template <int KIND, int TM, int TN, bool GLUE>
__global__ __launch_bounds__(256, TM * TN == 1 ? 4 : 2) void qgemm_edge(GemmArgs a, int tiles_m, int tiles_n, int nblk_padded, int group_m, int table)
{
    constexpr bool GROUPED = KIND == OP_W4 || KIND == OP_I8G;
    constexpr int EB = KIND == OP_F16 ? 2 : 1;
    constexpr int BM = 64 * TM, BN = 64 * TN;
    constexpr int BSTEP = KIND == OP_W4 ? 64 : 128;          // bytes of a weight row per K step
    constexpr int LDA = 128 + 16, LDB = BSTEP + 16;           // padded against bank conflicts
    constexpr int NA = BM * 8 / 256, NB = BN * (BSTEP / 16) / 256;
    constexpr int A_BYTES = BM * LDA, B_BYTES = BN * LDB;
    constexpr int STRIP = 32 * (TN * 64 + 16);
    static_assert(BM * 4 + 4 * STRIP <= 2 * A_BYTES + 2 * B_BYTES, "the epilogue's scratch reuses the stages");
    typedef typename std::conditional<KIND == OP_F16, v16f, v16i>::type acc_t;
    extern __shared__ __align__(16) unsigned char smem[];
    float *ctab = reinterpret_cast<float *>(smem + 2 * A_BYTES + 2 * B_BYTES);   // [G][BN]
    int tm, tn;
    if (!pick_tile(tiles_m, tiles_n, nblk_padded, group_m, tm, tn)) return;
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int fr = lane & 31, half = lane >> 5;
    const int M = a.M, N = a.N, K = a.K;
    const int KB = K * EB, WB = KIND == OP_W4 ? K / 2 : KB;
    const int nk = (KB + 127) / 128;
    const int G = GROUPED ? K / a.group : 0, QG = GROUPED ? a.group / 32 : 0;
    const unsigned char *qa = reinterpret_cast<const unsigned char *>(a.q), *wb = static_cast<const unsigned char *>(a.w);

    v4i ga[NA], gb[NB];
    auto load_step = [&](int kt) {
        const bool whole = (kt + 1) * 128 <= KB;   // uniform: only a row's last step can be cut short
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int c = tid + i * 256, kb = kt * 128 + (c % 8) * 16;
            const unsigned char *row = qa + (size_t)min(m0 + c / 8, M - 1) * KB;
            ga[i] = whole ? load16(row + kb) : load_piece(row, kb, KB);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int c = tid + i * 256, kb = kt * BSTEP + (c % (BSTEP / 16)) * 16;
            const unsigned char *row = wb + (size_t)min(n0 + c / (BSTEP / 16), N - 1) * WB;
            gb[i] = whole ? load16(row + kb) : load_piece(row, kb, WB);
        }
    };
    auto store_step = [&](int kt) {
        unsigned char *dA = smem + (kt & 1) * A_BYTES, *dB = smem + 2 * A_BYTES + (kt & 1) * B_BYTES;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int c = tid + i * 256;
            *reinterpret_cast<v4i *>(dA + (c / 8) * LDA + (c % 8) * 16) = ga[i];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int c = tid + i * 256;
            *reinterpret_cast<v4i *>(dB + (c / (BSTEP / 16)) * LDB + (c % (BSTEP / 16)) * 16) = gb[i];
        }
    };
    acc_t acc[TM][TN];
    float fsum[GROUPED ? TM : 1][GROUPED ? TN : 1][16];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] = 0;
                if (GROUPED) fsum[GROUPED ? i : 0][GROUPED ? j : 0][r] = 0.0f;
            }
    int qs = 0, grp = 0;             // slice inside the current weight group, and the group's number
    unsigned short sgrp[TN] = {};
    float agrp[TM] = {};
    load_step(0);
    // What the epilogue needs from memory, behind the first step: two trips to memory less at the end of the kernel (8-bit, M = 1021, K = 1160,
    // N = 1000: 10.35 -> 9.4 us).  Binary16 layers, which have no scales, were not faster for it.
    static_assert(BM <= 256, "one row scale per thread");
    float row_scale, swt[TN];
    unsigned short bias_h[TN];
    auto load_scalars = [&]() {
        row_scale = (KIND != OP_F16 && !a.s_ag && tid < BM) ? a.s_a[min(m0 + tid, M - 1) / a.R] : 1.0f;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = min(n0 + wn * TN * 32 + j * 32 + fr, N - 1);
            swt[j] = KIND == OP_I8 ? static_cast<const float *>(a.s_w)[n] : 1.0f;
            bias_h[j] = a.bias ? static_cast<const unsigned short *>(a.bias)[n] : (unsigned short)0;
        }
    };
    if (KIND != OP_F16) load_scalars();
    if (GROUPED && table) {
        const unsigned short *src = static_cast<const unsigned short *>(a.s_w) + (size_t)min(n0 + tid % BN, N - 1) * G;
        for (int g = tid / BN; g < G; g += 256 / BN) ctab[g * BN + tid % BN] = half_to_float_dev(src[g]) * (KIND == OP_W4 ? 0.0625f : 1.0f);
    }
    store_step(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) load_step(kt + 1);
        const unsigned char *pa = smem + (kt & 1) * A_BYTES + (wm * TM * 32 + fr) * LDA + half * 16;
        const unsigned char *pb = smem + 2 * A_BYTES + (kt & 1) * B_BYTES + (wn * TN * 32 + fr) * LDB + half * (KIND == OP_W4 ? 8 : 16);
        auto slice = [&](int ks) {
            v4i af[TM], bf[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const v4i *>(pa + i * 32 * LDA + ks * 32);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (KIND == OP_W4) {
                    const v2i p = *reinterpret_cast<const v2i *>(pb + j * 32 * LDB + ks * 16);
                    bf[j] = nibbles_x16(p[0], p[1]);
                } else {
                    bf[j] = *reinterpret_cast<const v4i *>(pb + j * 32 * LDB + ks * 32);
                }
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = mfma_step<KIND == OP_F16>(af[i], bf[j], acc[i][j]);
        };
        if constexpr (!GROUPED) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) slice(ks);   // slices past the end of the row hold zeros
        } else {
            const int ns = min(4, K / 32 - 4 * kt);     // whole slices only: groups are multiples of 32 that divide K
            for (int ks = 0; ks < ns; ++ks) {
                if (qs == 0) {
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        if (!table) sgrp[j] = static_cast<const unsigned short *>(a.s_w)[(size_t)min(n0 + wn * TN * 32 + j * 32 + fr, N - 1) * G + grp];
                    // channel-group activation scales: a 32-row block lies inside one scale block (the dispatcher sees to it)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        agrp[i] = a.s_ag ? a.s_ag[(size_t)(min(m0 + wm * TM * 32 + i * 32, M - 1) / a.R) * G + grp] : 1.0f;
                }
                slice(ks);
                if (++qs == QG) {
                    qs = 0;
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int n = n0 + wn * TN * 32 + j * 32 + fr;
                        const float s = table ? ctab[grp * BN + wn * TN * 32 + j * 32 + fr] : half_to_float_dev(sgrp[j]) * (KIND == OP_W4 ? 0.0625f : 1.0f);
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            const float c = s * agrp[i];
#pragma unroll
                            for (int r = 0; r < 16; ++r) {
                                const int p = (int)acc[i][j][r];
                                if (a.acc_out) {
                                    const int m = m0 + wm * TM * 32 + i * 32 + 8 * (r / 4) + 4 * half + (r % 4);
                                    if (m < M && n < N) a.acc_out[(unsigned)((m * G + grp) * N + n)] = KIND == OP_W4 ? p >> 4 : p;
                                }
                                float &fs = fsum[GROUPED ? i : 0][GROUPED ? j : 0][r];
                                fs = __builtin_fmaf((float)p, c, fs);
                                acc[i][j][r] = 0;
                            }
                        }
                    }
                    ++grp;
                }
            }
        }
        if (kt + 1 < nk) store_step(kt + 1);
        __syncthreads();
    }

    float *sRow = reinterpret_cast<float *>(smem);
    if (KIND == OP_F16) load_scalars();
    if (tid < BM) sRow[tid] = row_scale;
    __syncthreads();
    _Float16 *y = static_cast<_Float16 *>(a.y);
    float bj[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bj[j] = half_to_float_dev(bias_h[j]);
    auto value = [&](int i, int j, int r) {
        const float sa = sRow[wm * TM * 32 + i * 32 + 8 * (r / 4) + 4 * half + (r % 4)];
        if constexpr (GROUPED) return dequant_one<KIND>(a, 0, fsum[i][j][r], sa, 1.0f, bj[j]);
        else if constexpr (KIND == OP_F16) return dequant_one<KIND>(a, 0, acc[i][j][r], sa, 1.0f, bj[j]);
        else return dequant_one<KIND>(a, acc[i][j][r], 0.0f, sa, swt[j], bj[j]);
    };
    const bool pieces = GLUE && (a.residual || a.gate);
    const bool aligned = ((reinterpret_cast<uintptr_t>(a.y) | (pieces ? reinterpret_cast<uintptr_t>(a.residual) | reinterpret_cast<uintptr_t>(a.gate) : 0)) & 15) == 0;
    if (m0 + BM <= M && n0 + BN <= N && (N % 8) == 0 && aligned && (GROUPED || !a.acc_out)) {
        GluePieces gl;
        if (pieces) {
            gl.gate = static_cast<const _Float16 *>(a.gate);
            gl.residual = static_cast<const _Float16 *>(a.residual);
            gl.gate_rows = a.gate_rows;
            gl.on = true;
        }
        if (GLUE) gl.rowmax = a.row_absmax;
        unsigned char *strip = smem + BM * 4 + wave * STRIP;
        if (GLUE && a.act == 1)
            store_tile_staged<TM, TN, true, 32>(strip, lane, y, N, m0 + wm * TM * 32, n0 + wn * TN * 32,
                                                [&](int i, int j, int r) { return gelu_tanh_dev(value(i, j, r)); }, gl);
        else
            store_tile_staged<TM, TN, true, 32>(strip, lane, y, N, m0 + wm * TM * 32, n0 + wn * TN * 32, value, gl);
        return;
    }
    const GateRows gate_rows(GLUE ? a.gate : nullptr, a.gate_rows, m0, BM);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i)
            store_column<GLUE, true, GLUE ? Behind::PASSED : Behind::ASKED>(a, gate_rows, m0, wm * TM * 32 + i * 32 + 4 * half, n0 + wn * TN * 32 + j * 32 + fr, [&](int r, unsigned off) {
                const float u = value(i, j, r);   // ahead of the question, which the read of the row's scale would wait behind
                if constexpr (KIND == OP_I8) {
                    if (a.acc_out) a.acc_out[off] = acc[i][j][r];
                }
                return u;
            });
}

// ---- launches ------------------------------------------------------------------------------------------------------
static OperandKind kind_of(const GemmArgs &a)
{
    return a.w_bits == 16 ? OP_F16 : a.w_bits == 4 ? OP_W4 : a.w_grouped ? OP_I8G : OP_I8;
}

static bool glue_of(const GemmArgs &a) { return a.act != 0 || a.residual != nullptr || a.gate != nullptr || a.row_absmax != nullptr; }

template <int KIND, int T, int W>
static int split_gpr(const GemmArgs &a)
{
    return SplitTile<KIND, T, false>::GROUPED ? split_groups_per_round(a.K / a.group, T, W) : 0;
}

// how a layer is laid out: groups per round, rounds, LDS slots, LDS bytes
struct SplitLayout {
    int gpr, rounds, slots;
    size_t lds;
};
template <int KIND, int T, bool FUSE, int W, int NB>
static SplitLayout split_layout(const GemmArgs &a)
{
    using C = SplitTile<KIND, T, FUSE, W, NB>;
    const int G = C::GROUPED ? a.K / a.group : 0, gpr = split_gpr<KIND, T, W>(a), rounds = gpr ? (G + W * gpr - 1) / (W * gpr) : 0;
    const int slots = split_slots<C::GROUPED, W>(C::S, a.K * (KIND == OP_F16 ? 2 : 1), C::GROUPED ? a.group : 128, G, gpr, rounds);
    return {gpr, rounds, slots,
            (size_t)slots * C::STAGE + (size_t)(W * gpr < G ? W * gpr : G) * C::TILE + (size_t)T * NB * G * 4 +
                (FUSE ? (size_t)T * (split_resident_steps(a.K, C::GROUPED) * 128 + 4) : 0)};
}

template <int KIND, int T, bool GLUE, bool EXPORT, bool FUSE, int W, int NB>
static hipError_t run_split_as(const GemmArgs &a, hipStream_t s)
{
    static const hipError_t opt_in = hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_splitk<KIND, T, GLUE, EXPORT, FUSE, W, NB>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, SPLIT_LDS_MAX);
    if (opt_in != hipSuccess) return opt_in;
    const int tiles_m = (a.M + T - 1) / T, tiles_n = (a.N + T * NB - 1) / (T * NB);
    const int padded = (tiles_m * tiles_n + XCDS - 1) / XCDS * XCDS;
    const SplitLayout l = split_layout<KIND, T, FUSE, W, NB>(a);
    if (l.lds > SPLIT_LDS_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((qgemm_splitk<KIND, T, GLUE, EXPORT, FUSE, W, NB>), dim3(padded), dim3(64 * W), l.lds, s, a, tiles_m, tiles_n, padded, l.gpr, l.rounds, l.slots);
    return hipGetLastError();
}

// rounds of workgroups that a layer takes in this form; 0: it does not fit
template <int KIND, int T, bool FUSE, int W, int NB>
static long long split_rounds(const GemmArgs &a)
{
    const size_t lds = split_layout<KIND, T, FUSE, W, NB>(a).lds;
    if (lds > SPLIT_LDS_MAX) return 0;
    const long long tiles = (long long)((a.M + T - 1) / T) * ((a.N + T * NB - 1) / (T * NB)), resident = 256 * (long long)min((size_t)2, SPLIT_LDS_MAX / lds);
    return (tiles + resident - 1) / resident;
}

// What a wavefront does one after the other: its K steps, and a hand-over for every round of groups
template <int KIND, int T, int W>
static int split_serial(const GemmArgs &a, int rounds)
{
    return rounds * ((split_gpr<KIND, T, W>(a) * a.group + 127) / 128 + 1);
}

// Eight wavefronts share K where their workgroups, which take more LDS with group scales, are all resident at once; 16x16 tiles of integer codes come
// two to a workgroup where there are more of them than CUs.  us, DAQ and GEMM, four wavefronts -> chosen: 8-bit, K = 4608, N = 1152: M = 16 7.5 -> 7.0,
// 64 8.7 -> 8.2; 4-bit M = 16 9.9 -> 9.1, 64 11.2 -> 10.4, 128 14.3 -> 13.0; K = 1152, M = 256 11.3 -> 9.0.  32x32 tiles without group scales, whose steps go round
// the wavefronts, were up to 7 % slower with eight, and binary16 ones of short rows up to 16 %.
//
// 32x32 tiles with group scales: the sums of 12 groups fit LDS at once, which are three for each of four wavefronts and only one for each of eight.  Short groups
// then take more rounds on eight and no fewer steps (groups of 32, K = 4608, M = 133, N = 1152: 18 rounds of a step against 12, 33.0 against 27.6 us; groups of 128
// 5 against 3 rounds of three steps, 0.90 to 0.93 of the time).  int8 codes gain on eight in a single round only (0.94 to 1.04 of the time over 17 layers, mostly 0.98;
// in several rounds 0.99 to 1.06).
template <int KIND, int T>
static hipError_t run_split(const GemmArgs &a, hipStream_t s)
{
    if (a.acc_out) return glue_of(a) ? hipErrorInvalidValue : run_split_as<KIND, T, false, true, false, 4, 1>(a, s);   // no call exports and glues
    auto run = [&](auto w, auto nb) {
        constexpr int W = decltype(w)::value, NB = decltype(nb)::value;
        return glue_of(a) ? run_split_as<KIND, T, true, false, false, W, NB>(a, s) : run_split_as<KIND, T, false, false, false, W, NB>(a, s);
    };
    typedef std::integral_constant<int, 8> eight;
    if constexpr (T == 16 && KIND != OP_F16) {
        if ((long long)((a.M + 15) / 16) * ((a.N + 15) / 16) > 256 && split_rounds<KIND, T, false, 8, 2>(a) == 1) return run(eight{}, std::integral_constant<int, 2>{});
    }
    constexpr bool GROUPED = KIND == OP_W4 || KIND == OP_I8G;
    if constexpr (T == 16 || GROUPED) {
        bool worth = KIND != OP_F16 || (a.K >= 1152 && (long long)((a.M + 15) / 16) * ((a.N + 15) / 16) <= 256);
        if constexpr (T == 32) {
            const int r4 = split_layout<KIND, T, false, 4, 1>(a).rounds, r8 = split_layout<KIND, T, false, 8, 1>(a).rounds;
            const int s4 = split_serial<KIND, T, 4>(a, r4), s8 = split_serial<KIND, T, 8>(a, r8);
            worth = KIND == OP_I8G ? r8 == 1 : s8 < s4 || (s8 == s4 && r8 == r4);
        }
        if (worth && split_rounds<KIND, T, false, 8, 1>(a) == 1) return run(eight{}, std::integral_constant<int, 1>{});
    }
    return run(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{});
}

template <int KIND, int NB>
static hipError_t run_split_fused(const GemmArgs &a, hipStream_t s)
{
    return glue_of(a) ? run_split_as<KIND, 16, true, false, true, 8, NB>(a, s) : run_split_as<KIND, 16, false, false, true, 8, NB>(a, s);
}

template <int T>
static size_t split_lds_of(const GemmArgs &a)
{
    switch (kind_of(a)) {
    case OP_I8: return split_layout<OP_I8, T, false, 4, 1>(a).lds;
    case OP_W4: return split_layout<OP_W4, T, false, 4, 1>(a).lds;
    case OP_I8G: return split_layout<OP_I8G, T, false, 4, 1>(a).lds;
    default: return split_layout<OP_F16, T, false, 4, 1>(a).lds;
    }
}

// DMA needs 16-byte pieces; the scale table of a tile has to fit beside the rings
bool qgemm_split_takes(const GemmArgs &a, int T)
{
    if (((uintptr_t)a.q | (uintptr_t)a.w) % 16 != 0 || (a.w_bits == 16 ? a.K % 8 : a.K % 16) != 0) return false;
    if (a.w_bits == 16 && (long long)(a.M > a.N ? a.M : a.N) * a.K >= 1ll << 30) return false;   // 32-bit byte offsets
    if (a.s_ag && a.R % T != 0 && a.R < a.M) return false;   // a tile inside one scale block
    return (T == 32 ? split_lds_of<32>(a) : split_lds_of<16>(a)) <= SPLIT_LDS_MAX;
}

// Which tile, if any, splits K to advantage.  The kernel's time is nearly flat as long as all its workgroups are resident
// at once and then goes up by a whole walk over K per further round (M = 64..192, N = 1152, K = 4608, 8-bit: 5.4-5.7 us, M =
// 256: 8.3; the 64x64 workgroup tiles take 12.2 there).  16x16 tiles have the shortest walk, 32x32 tiles move half the
// operand bytes.  A second round does not pay where 64x64 workgroup tiles can run instead (16.8 against 11.8 us at M = N = 1024,
// K = 4096, 37.6 against 21.5 in binary16; from 576 tiles on they are level at best), only for inner sizes that those do not
// take, and there where the walk is long (K >= 2304).
int qgemm_split_choice(const GemmArgs &a)
{
    auto rounds = [&](int T, size_t lds) {
        const long long tiles = (long long)((a.M + T - 1) / T) * ((a.N + T - 1) / T);
        const long long resident = 256 * (long long)min((size_t)2, SPLIT_LDS_MAX / lds);
        return (tiles + resident - 1) / resident;
    };
    if (qgemm_split_takes(a, 16) && rounds(16, split_lds_of<16>(a)) == 1) return 16;
    const long long kb = (long long)a.K * (a.w_bits == 16 ? 2 : 1);
    const bool two = kb >= 2304 && kb % 128 != 0 && a.w_bits != 4 && !a.w_grouped;
    if (qgemm_split_takes(a, 32) && rounds(32, split_lds_of<32>(a)) <= (two ? 2 : 1)) return 32;
    return 0;
}

// Whether the layer runs in one launch, codes made by the GEMM's own workgroups (a.x is the fp16 input), and how many column tiles each of them
// covers: the fewest that leave no CU a second workgroup, which has to fit its LDS.  Every workgroup makes the codes of its 16 rows, so that more columns are
// fewer repetitions, but fewer CUs too.  The launch that it saves also costs the host 3.6 us, which is what bounds a sequence of such small calls.
//
// us, M x K x N, two launches or (up to 256 tiles) four wavefronts -> now: 8-bit 16 x 384 x 384 4.9 -> 4.2, 16 x 1152 x 1152 6.4 -> 5.4, 16 x 1152 x 4608 6.9 -> 5.5 (NB
// = 2), 64 x 1152 x 1152 7.2 -> 5.6 (2), 128 7.9 -> 6.6 (3), 256 8.6 -> 8.1 (5), 64 x 1152 x 4096 7.9 -> 6.7 (4), 64 x 1152 x 4608 8.2 -> 7.6 (5), 128 9.2 -> 9.2 (none);
// 4-bit 16 x 1152 x 1152 7.6 -> 5.9, 128 9.5 -> 7.3; one scale for all rows, 8-bit, 256 x 1152 x 1152 11.7 -> 10.7.  Without NB = 4, rows of 1536 were slower than
// in two launches (8-bit, 24 x 1536 x 6448: two launches 7.9, NB = 5 8.2, NB = 4 6.7; 256 x 1536 x 1024 8.3, 8.5, 7.3).  With four wavefronts NB = 2 to 5 were no
// faster than the two launches, and up to 1.2 times as long.  Short 4-bit groups whose scales and sums do not fit beside the codes take the two launches.
static int fuse_tiles(const GemmArgs &a)   // NB; 0: DAQ runs by itself
{
    if ((a.w_bits != 8 && a.w_bits != 4) || a.w_grouped || a.s_ag || a.acc_out || (uintptr_t)a.x % 16 != 0 || a.K > SPLIT_FUSE_K_MAX) return 0;
    if (!qgemm_split_takes(a, 16)) return 0;
    auto takes = [&](auto nb) {
        constexpr int NB = decltype(nb)::value;
        if ((long long)((a.M + 15) / 16) * ((a.N + 16 * NB - 1) / (16 * NB)) > 256) return 0;
        return (a.w_bits == 8 ? split_rounds<OP_I8, 16, true, 8, NB>(a) : split_rounds<OP_W4, 16, true, 8, NB>(a)) == 1 ? NB : 0;
    };
    int nb = takes(std::integral_constant<int, 1>{});
    if (!nb) nb = takes(std::integral_constant<int, 2>{});
    if (!nb) nb = takes(std::integral_constant<int, 3>{});
    if (!nb) nb = takes(std::integral_constant<int, 4>{});
    return nb ? nb : takes(std::integral_constant<int, 5>{});
}
bool qgemm_fuse_takes(const GemmArgs &a) { return fuse_tiles(a) != 0; }
bool qgemm_fuse_one_tile(const GemmArgs &a) { return fuse_tiles(a) == 1; }
hipError_t launch_qgemm_fused(const GemmArgs &a, hipStream_t stream)
{
    switch (fuse_tiles(a)) {
    case 1: return a.w_bits == 8 ? run_split_fused<OP_I8, 1>(a, stream) : run_split_fused<OP_W4, 1>(a, stream);
    case 2: return a.w_bits == 8 ? run_split_fused<OP_I8, 2>(a, stream) : run_split_fused<OP_W4, 2>(a, stream);
    case 3: return a.w_bits == 8 ? run_split_fused<OP_I8, 3>(a, stream) : run_split_fused<OP_W4, 3>(a, stream);
    case 4: return a.w_bits == 8 ? run_split_fused<OP_I8, 4>(a, stream) : run_split_fused<OP_W4, 4>(a, stream);
    case 5: return a.w_bits == 8 ? run_split_fused<OP_I8, 5>(a, stream) : run_split_fused<OP_W4, 5>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

template <int T>
static hipError_t launch_split(const GemmArgs &a, hipStream_t stream)
{
    switch (kind_of(a)) {
    case OP_I8: return run_split<OP_I8, T>(a, stream);
    case OP_W4: return run_split<OP_W4, T>(a, stream);
    case OP_I8G: return run_split<OP_I8G, T>(a, stream);
    default: return run_split<OP_F16, T>(a, stream);
    }
}
hipError_t launch_qgemm_split32(const GemmArgs &a, hipStream_t stream) { return launch_split<32>(a, stream); }
hipError_t launch_qgemm_split16(const GemmArgs &a, hipStream_t stream) { return launch_split<16>(a, stream); }

template <int KIND, int T, bool GLUE>
static hipError_t run_edge_as(const GemmArgs &a, hipStream_t s)
{
    constexpr int B = 64 * T, STAGES = 2 * B * 144 + 2 * B * (KIND == OP_W4 ? 80 : 144);
    constexpr bool GROUPED = KIND == OP_W4 || KIND == OP_I8G;
    static const hipError_t opt_in = hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_edge<KIND, T, T, GLUE>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, STAGES + (GROUPED ? B * EDGE_TABLE_GROUPS * 4 : 0));
    if (opt_in != hipSuccess) return opt_in;
    const int tiles_m = (a.M + B - 1) / B, tiles_n = (a.N + B - 1) / B;
    const int padded = (tiles_m * tiles_n + XCDS - 1) / XCDS * XCDS;
    const int G = GROUPED ? a.K / a.group : 0, table = G <= EDGE_TABLE_GROUPS ? 1 : 0;
    hipLaunchKernelGGL((qgemm_edge<KIND, T, T, GLUE>), dim3(padded), dim3(256), STAGES + (GROUPED && table ? B * G * 4 : 0), s, a, tiles_m, tiles_n,
                       padded, pick_group_m(B), table);
    return hipGetLastError();
}

template <int KIND, int T>
static hipError_t run_edge(const GemmArgs &a, hipStream_t s)
{
    return glue_of(a) ? run_edge_as<KIND, T, true>(a, s) : run_edge_as<KIND, T, false>(a, s);
}

bool qgemm_edge_takes(const GemmArgs &a) { return !a.s_ag || a.R % 32 == 0 || a.R >= a.M; }

hipError_t launch_qgemm_edge(const GemmArgs &a, hipStream_t stream)
{
    // 128x128 tiles move half the operand bytes of 64x64 ones but need 512 of them for two workgroups per CU
    const bool big = (long long)((a.M + 127) / 128) * ((a.N + 127) / 128) >= 512;
    switch (kind_of(a)) {
    case OP_I8: return big ? run_edge<OP_I8, 2>(a, stream) : run_edge<OP_I8, 1>(a, stream);
    case OP_W4: return run_edge<OP_W4, 1>(a, stream);
    case OP_I8G: return run_edge<OP_I8G, 1>(a, stream);
    default: return big ? run_edge<OP_F16, 2>(a, stream) : run_edge<OP_F16, 1>(a, stream);
    }
}

}  // namespace ql
