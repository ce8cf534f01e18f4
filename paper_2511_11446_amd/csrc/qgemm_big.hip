// INT8 x INT8 -> INT32 (and binary16 x binary16 -> fp32) GEMM + dequantization on large tiles, for gfx950: the layers with
// 8-bit weights (one scale per output channel; Step 3, Step 5, Section 6) and the FP16 layers, where M and N fill the chip with
// such tiles.
//
// Eight wavefronts own a tile of 256 x 288, 256 x 256 or 128 x 288; a wavefront holds MT x NT blocks of 16x16 of it.
//   - With random operands (no clock or power reading is kept that would say why) v_mfma_i32_16x16x64_i8 from registers reaches 4.0 POPS where
//     v_mfma_i32_32x32x32_i8 reaches 3.36 (4.7 and 4.8 on zeros), and a large tile moves fewer bytes through the L2 and the LDS
//     per operation.  256 x 288: a K step of 128 bytes is 2304 MFMA clocks of a SIMD, 1660 clocks of LDS reads and 540 of
//     LDS writes; it measured 3100.  Over a whole kernel at M = 16384 the matrix cores are busy 43
//     to 46 % of the time (profiles/qgemm_big_qgemm_w4_big_c5_stack_m16384_sq_counters.txt).
//   - 288 divides 1152, 3456 and 4608, so that 256-row tiles at M = 16384 fill 256 CUs in whole rounds.  The 32 columns behind
//     2 x 128 are shared by the two wavefronts of a row, each taking half of the row blocks.
//   - A lane's columns of the result are 8 neighbouring ones (the rows of W enter LDS in that order), so that 16 lanes
//     store 256 bytes of a row straight from registers.  Segments of 288 bytes, which do not end on a 128-byte line, took
//     20 us longer at M = 16384, K = 1152, N = 4608.
//   - Two LDS stages of one K step.  The stages change hands two groups of MFMAs behind the last fragment read, so that no wavefront
//     waits for LDS there (at once: 9 % slower), and a stage has a whole step to be filled again.
//   - The launch is persistent and the ring does not drain between tiles: the last two steps of a tile request the first two of the
//     next one, the scales come by DMA as well, and the epilogue touches LDS only to read them; its stores are still on
//     their way while the next tile starts.  What is left of the epilogue is 2 us of vector ALU work and up to 4 us of stores per
//     tile, since all CUs store at about the same time.
// M = 16384, random operands, us before -> after: K = 1152: N = 3456 81 -> 70, N = 4608 108 -> 94; K = 4608, N = 1152 88 -> 75
// (2.3 POPS); in binary16 146 -> 119, 183 -> 157, 171 -> 144.
#include "qgemm_common.h"

namespace ql {

template <int MT_, int NT_, int WM_, int WN_, bool F16_>
struct TileBig {
    static constexpr int MT = MT_, WM = WM_, WN = WN_;
    static constexpr bool F16 = F16_;
    static constexpr bool TAIL = NT_ == 9;
    static constexpr int NM = 8;                                             // main blocks of a wavefront: 128 columns
    static constexpr int TI = TAIL ? MT / 2 : 0;                             // row blocks of the tail, two column blocks each
    static constexpr int NW = WM * WN, NTHR = 64 * NW;
    static constexpr int BM = 16 * MT * WM, BN = 16 * NT_ * WN;
    static constexpr int A_GROUPS = BM / 8, B_GROUPS = BN / 8;               // 1024-byte DMA instructions per K step
    static constexpr int NA = A_GROUPS / NW, NB = (B_GROUPS + NW - 1) / NW;  // per wavefront
    static constexpr int LEAST = NA + B_GROUPS / NW;                         // the fewest a wavefront issues
    static constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, STAGE = A_BYTES + B_BYTES;
    static constexpr int FR = NM + (TAIL ? 2 : 0), GROUPS = 2 * FR;          // weight fragments per half step of 64 bytes, and per step
    static constexpr int DIST = 6, GAP = 2;                       // a weight fragment is read DIST groups ahead; the stages change hands
    static constexpr int HAND = GROUPS - DIST + GAP;                         // GAP groups behind the last read of a step
    static constexpr int NBUF = GROUPS / 2;                                  // fragment buffers: divides GROUPS, > DIST
    static constexpr int SPAN = GROUPS - HAND;                               // groups left to read the next step's first fragments
    static constexpr int LOADS = (NA + NB + SPAN - 1) / SPAN, READS = (MT + SPAN - 1) / SPAN;   // per group from HAND on
    static constexpr int STORES = 4 * MT + 4 * TI;                           // per wavefront and full tile
    // fragments of the next step requested by the end of group HAND + k
    static constexpr int ahead(int k) { return 2 * (k + 1) < k + GAP + 1 ? 2 * (k + 1) : k < 0 ? 0 : k + GAP + 1; }
    // behind the stages: twice (this tile, next tile) row scales, weight scales and binary16 biases of the tile's columns, each rounded up
    // to whole DMA instructions of 64 words
    static constexpr int SA_Q = (BM + 63) / 64, SW_Q = (BN + 63) / 64, SB_Q = (BN + 127) / 128;
    static constexpr int SCALES = (SA_Q + SW_Q + SB_Q) * 256, S0 = 2 * STAGE, LDS_BYTES = S0 + 2 * SCALES;
    static_assert(GROUPS % NBUF == 0 && NBUF > DIST && A_GROUPS % NW == 0 && BM % 64 == 0 && (!TAIL || WN == 2), "shape");
    static_assert(LDS_BYTES <= 160 * 1024 && STORES < 64 && SPAN > 0, "LDS, outstanding operations");
};

// workgroup `block` of `blocks` (a multiple of XCDS) that share the layer
template <class T, bool GLUE>
__device__ __forceinline__ void qgemm_big_tiles(const GemmArgs &a, int block, int blocks, int tiles_m, int tiles_n, int nblk_padded, int group_m)
{
    constexpr int MT = T::MT, NM = T::NM, TI = T::TI, NA = T::NA, NB = T::NB, FR = T::FR;
    constexpr bool F16 = T::F16;
    constexpr int EB = F16 ? 2 : 1;
    typedef typename std::conditional<F16, float, int>::type elem_t;
    typedef elem_t acc_t __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(1024) unsigned char smem[];

    const int per_xcd = nblk_padded / XCDS, slots_per_xcd = blocks / XCDS;
    const int xcd_first = (block % XCDS) * per_xcd;
    int in_xcd = block / XCDS;
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
    const int M = a.M, N = a.N, KB = a.K * EB;
    const int nk = KB / 128;   // whole steps, at least 2

    // ---- DMA: lane l fills bytes [16 l, 16 l + 16) of a 1024-byte group = row l/8, slot l%8; chunk c of row r at slot c ^ ((r >> 1) & 7).
    // LDS row 16 j + p of a wavefront's 128 columns is column 8 p + j of them, and row 16 b + p of the tail its column 2 p + b.
    unsigned offA[NA], offB[NB];
    auto set_off = [&]() {
        int lane = tid & 63;   // opaque: what is computed from it is not kept in registers through the K loop
        asm volatile("" : "+v"(lane));
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int row = 8 * (wave + i * T::NW) + (lane >> 3);
            offA[i] = row_start(min(m0 + row, M - 1), KB) + 16 * ((lane & 7) ^ ((row >> 1) & 7));
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int row = 8 * (wave + i * T::NW) + (lane >> 3);
            const int g = (wave + i * T::NW) >> 1, p = 8 * ((wave + i * T::NW) & 1) + (lane >> 3);
            const int col = g < NM * T::WN ? (g / NM) * 16 * NM + 8 * p + g % NM : 16 * NM * T::WN + 2 * p + (g - NM * T::WN);
            offB[i] = row_start(min(n0 + col, N - 1), KB) + 16 * ((lane & 7) ^ ((row >> 1) & 7));
        }
    };
    auto issue = [&](int kt, int stage, int li) {
        unsigned char *st = smem + stage * T::STAGE;
        if (li < NA) dma16_buf(a.q, operand_bytes(M, KB), st + (wave + li * T::NW) * 1024, offA[li < NA ? li : 0], kt * 128);
        else if (T::B_GROUPS % T::NW == 0 || wave + (li - NA) * T::NW < T::B_GROUPS)
            dma16_buf(a.w, operand_bytes(N, KB), st + T::A_BYTES + (wave + (li - NA) * T::NW) * 1024, offB[li < NA ? 0 : li - NA], kt * 128);
    };
    // the epilogue's scales, straight to LDS
    auto fetch_scales = [&](int par) {
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        unsigned char *s = smem + T::S0 + par * T::SCALES;
#pragma unroll
        for (int c = 0; c < T::SA_Q + T::SW_Q + T::SB_Q; ++c) {
            if (wave != c % T::NW) continue;
            if (c < T::SA_Q) {
                if (!F16) dma4_buf(a.s_a, ((M - 1) / a.R + 1) * 4, s + c * 256, (unsigned)(min(m0 + 64 * c + lane, M - 1) / a.R * 4));
            } else if (c < T::SA_Q + T::SW_Q) {
                if (!F16) dma4_buf(a.s_w, N * 4, s + c * 256, (unsigned)(n0 + 64 * (c - T::SA_Q) + lane) * 4u);
            } else if (a.bias) {
                dma4_buf(a.bias, N * 2, s + c * 256, (unsigned)(n0 + 128 * (c - T::SA_Q - T::SW_Q) + 2 * lane) * 2u);
            }
        }
    };

    // ---- fragments: lane = row (lane & 15) of a 16-row block, 16 bytes at chunk 4 * half + (lane >> 4) of the step
    acc_t acc[MT][NM], tail[TI > 0 ? TI : 1][2];
    v4i af[2][MT], bf[T::NBUF];
    // LDS addresses of the fragments in this step's stage, by half.  A wavefront with wn = 1 starts with the upper half of its row
    // blocks, so that the tail's blocks are the first ones of both.
    int pa_lo[2], pa_hi[2], pb[2], pt[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int lane = tid & 63, at = (lane & 15) * 128 + ((4 * h + (lane >> 4)) ^ ((lane >> 1) & 7)) * 16;
        pa_lo[h] = at + (wm * MT + (T::TAIL ? wn * TI : 0)) * 2048;
        pa_hi[h] = at + (wm * MT - (T::TAIL ? wn * TI : 0)) * 2048;
        pb[h] = at + T::A_BYTES + wn * NM * 2048;
        pt[h] = at + T::A_BYTES + T::WN * NM * 2048;
    }
    auto turn = [&](int &p, int stage) { p += stage ? -T::STAGE : T::STAGE; };
    auto row_block = [&](int i) { return T::TAIL ? (wn ? (i < TI ? i + TI : i - TI) : i) : i; };
    auto read_a = [&](int h, int i) { af[h][i] = *reinterpret_cast<const v4i *>(smem + (i < TI || !T::TAIL ? pa_lo[h] : pa_hi[h]) + i * 2048); };
    // the column blocks of a half step in the order they are multiplied: the two of the tail (-1, -2) in the middle
    auto block_of = [](int f) constexpr { return !T::TAIL || f < NM / 2 ? f : f < NM / 2 + 2 ? NM / 2 - 1 - f : f - 2; };
    auto read_b = [&](int s) {   // fragment s of the step's GROUPS
        const int h = (s / FR) & 1, b = block_of(s % FR);
        bf[s % T::NBUF] = *reinterpret_cast<const v4i *>(smem + (b >= 0 ? pb[h] + b * 2048 : pt[h] + (-1 - b) * 2048));
    };
    auto mfma = [&](v4i x, v4i w, acc_t c) {
        if constexpr (F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, x), __builtin_bit_cast(v8h, w), c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_i32_16x16x64_i8(x, w, c, 0, 0, 0);
    };

    set_off();
    fetch_scales(0);
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int li = 0; li < NA + NB; ++li) issue(kt, kt, li);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(T::LEAST) : "memory");   // step 0
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < MT; ++i) read_a(0, i);
#pragma unroll
    for (int s = 0; s < T::DIST; ++s) read_b(s);

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
                for (int j = 0; j < NM; ++j) acc[i][j][r] = 0;
#pragma unroll
            for (int i = 0; i < TI; ++i) tail[i][0][r] = tail[i][1][r] = 0;
        }

        // One K step per pass.  Group s: MFMAs of a fragment, then the fragment of group s + DIST is requested.  Before group HAND every
        // fragment of this stage has been requested, GAP groups ago: once they have arrived and the next step is in LDS, the
        // stages change hands; from there on the fragments of the next step are read, two per group until they are DIST
        // groups ahead again, and this stage is refilled with the step after it.  Behind the very last step the reads find
        // stale bytes, which nothing uses.
        for (int kt = 0; kt < nk; ++kt, cur ^= 1) {
            const bool refill = kt + 2 < nk || has_next;
            const int step = kt + 2 < nk ? kt + 2 : kt + 2 - nk;
#pragma unroll
            for (int s = 0; s < T::GROUPS; ++s) {
                if (s == T::HAND) {
                    // behind a tile's stores, step 1 is older than they are
                    if (stores_behind) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(T::STORES) : "memory");
                    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                    stores_behind = false;
                    __builtin_amdgcn_s_barrier();
                }
                __builtin_amdgcn_sched_barrier(0);
                const int h = s / FR, b = block_of(s % FR);
                const v4i w = bf[s % T::NBUF];
                if (b >= 0) {
#pragma unroll
                    for (int i = 0; i < MT; ++i) acc[i][b >= 0 ? b : 0] = mfma(af[h][i], w, acc[i][b >= 0 ? b : 0]);
                } else {
#pragma unroll
                    for (int i = 0; i < TI; ++i) tail[i][b >= 0 ? 0 : -1 - b] = mfma(af[h][i], w, tail[i][b >= 0 ? 0 : -1 - b]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (s == T::HAND) {
#pragma unroll
                    for (int hh = 0; hh < 2; ++hh) {
                        turn(pa_lo[hh], cur);
                        turn(pa_hi[hh], cur);
                        turn(pb[hh], cur);
                        turn(pt[hh], cur);
                    }
                    if (kt == nk - 2 && has_next) {
                        set_tile(xcd_first + in_xcd);
                        set_off();
                        fetch_scales(par ^ 1);
                    }
                }
                if (s < MT) read_a(1, s);
                if (s >= T::HAND) {
#pragma unroll
                    for (int i = (s - T::HAND) * T::READS; i < (s - T::HAND + 1) * T::READS; ++i)
                        if (i < MT) read_a(0, i);
#pragma unroll
                    for (int n = T::ahead(s - T::HAND - 1); n < T::ahead(s - T::HAND); ++n) read_b(T::GROUPS + n);
                } else if (s + T::DIST < T::GROUPS) {
                    read_b(s + T::DIST);
                }
                if (s >= T::HAND && refill) {
#pragma unroll
                    for (int li = (s - T::HAND) * T::LOADS; li < (s - T::HAND + 1) * T::LOADS; ++li)
                        if (li < NA + NB) issue(step, cur, li);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        // ---- epilogue
        int lane = tid & 63;   // opaque, as in set_off
        asm volatile("" : "+v"(lane));
        const int p = lane & 15, kq = lane >> 4;
        _Float16 *y = static_cast<_Float16 *>(a.y);
        const float *s_row = reinterpret_cast<const float *>(smem + T::S0 + par * T::SCALES) + wm * 16 * MT + 4 * kq;
        const float *s_col = reinterpret_cast<const float *>(smem + T::S0 + par * T::SCALES) + 64 * T::SA_Q;
        const _Float16 *b_col = reinterpret_cast<const _Float16 *>(s_col + 64 * T::SW_Q);
        const int m_base = em0 + wm * 16 * MT + 4 * kq;
        const int c_main = wn * 16 * NM + 8 * p, c_tail = T::WN * 16 * NM + 2 * p;
        const bool full = em0 + T::BM <= M && en0 + T::BN <= N;
        const GateRows gate_rows(GLUE ? a.gate : nullptr, a.gate_rows, em0, T::BM);
        // C neighbouring columns from column c of the tile; v(i, e): accumulator of row block i and column e
        auto columns = [&](auto count_tag, int c, int blocks, auto v) {
            constexpr int C = decltype(count_tag)::value;
            typedef _Float16 hC __attribute__((ext_vector_type(C)));
            float sw[C], b[C];
#pragma unroll
            for (int e = 0; e < C; ++e) {
                sw[e] = F16 ? 1.0f : s_col[c + e];
                b[e] = a.bias ? (float)b_col[c + e] : -0.0f;   // x + -0.0 is x, signed zeros included
            }
            const int n = en0 + c;
#pragma unroll
            for (int i = 0; i < blocks; ++i) {
                const int blk = row_block(i);
                v4f sa = {1.0f, 1.0f, 1.0f, 1.0f};
                if (!F16) sa = *reinterpret_cast<const v4f *>(s_row + 16 * blk);
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
                        float u;
                        if constexpr (F16) u = v(i, e)[r] + b[e];
                        else u = __builtin_fmaf((float)v(i, e)[r] * sa[r], sw[e], b[e]);
                        if (GLUE && a.act == 1) u = gelu_tanh_dev(u);
                        asm volatile("" : "+v"(u));   // keep the fp32 rounding before the fp16 one
                        out[e] = (_Float16)u;
                        if (GLUE && (a.gate || a.residual)) {
                            u = __builtin_fmaf(a.gate ? (float)g[e] : 1.0f, (float)out[e], a.residual ? (float)res[e] : 0.0f);
                            asm volatile("" : "+v"(u));
                            out[e] = (_Float16)u;
                        }
                    }
                    // The workgroup's last tile is streamed out; before another one the L2 takes the burst of stores that all
                    // CUs send at about the same time, and passes it on during the next tile (M = 16384, K = 1152, N = 4608: 103 -> 98 us)
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
__global__ __launch_bounds__(T::NTHR, 2) void qgemm_big(GemmArgs a, int tiles_m, int tiles_n, int nblk_padded, int group_m)
{
    qgemm_big_tiles<T, GLUE>(a, blockIdx.x, gridDim.x, tiles_m, tiles_n, nblk_padded, group_m);
}

template <class T, bool GLUE>
static hipError_t run_big(const GemmArgs &a, hipStream_t s)
{
    static const hipError_t opt_in = hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_big<T, GLUE>),
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
    hipLaunchKernelGGL((qgemm_big<T, GLUE>), dim3(padded < resident ? padded : resident), dim3(T::NTHR), T::LDS_BYTES, s, a, tiles_m, tiles_n,
                       padded, pick_group_m(T::BM));
    return hipGetLastError();
}

// what these kernels take of a layer: whole K steps of 128 bytes, at least two, 16-byte rows everywhere
bool qgemm_big_takes(const GemmArgs &a)
{
    const long kb = (long)a.K * (a.w_bits == 16 ? 2 : 1);
    return (a.w_bits == 8 || a.w_bits == 16) && !a.w_grouped && !a.s_ag && !a.acc_out && kb % 128 == 0 && kb >= 256 && a.N % 8 == 0 &&
           (uintptr_t)a.q % 16 == 0 && (uintptr_t)a.w % 16 == 0 && (uintptr_t)a.y % 16 == 0 && (uintptr_t)a.bias % 4 == 0 &&
           (uintptr_t)a.gate % 16 == 0 && (uintptr_t)a.residual % 16 == 0;
}

// ---- several 8-bit layers of a plan in one launch (qgemm_many.hip), where all their tiles are one round: a workgroup, a tile
using BigMany = TileBig<4, 9, 4, 2, false>;
struct BigManyLayer {
    const int8_t *q, *w;
    const float *s_a, *s_w;
    const void *bias;
    void *y;
    int N, K, tiles_n, padded;
};
struct BigManyArgs {
    BigManyLayer l[PLAN_WINDOW];
    int M, R, tiles_m, group_m;
};
__global__ __launch_bounds__(BigMany::NTHR, 2) void qgemm_big_many(BigManyArgs b)
{
    int i = 0, block = blockIdx.x;
    while (block >= b.l[i].padded) block -= b.l[i++].padded;   // the grid is the sum of all
    const BigManyLayer &l = b.l[i];
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
    qgemm_big_tiles<BigMany, false>(a, block, l.padded, b.tiles_m, l.tiles_n, l.padded, b.group_m);
}

static int big_many_padded(const GemmArgs &a)
{
    const int tiles = ((a.M + BigMany::BM - 1) / BigMany::BM) * ((a.N + BigMany::BN - 1) / BigMany::BN);
    return (tiles + XCDS - 1) / XCDS * XCDS;
}

bool qgemm_big_many_takes(const GemmArgs *const *layers, int count)
{
    int blocks = 0;
    for (int i = 0; i < count; ++i) {
        if (layers[i]->w_bits != 8 || !qgemm_big_takes(*layers[i])) return false;
        blocks += big_many_padded(*layers[i]);
    }
    return blocks <= 256;
}

hipError_t launch_qgemm_big_many(const GemmArgs *const *layers, int count, hipStream_t stream)
{
    static const hipError_t opt_in = hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_big_many), hipFuncAttributeMaxDynamicSharedMemorySize, BigMany::LDS_BYTES);
    if (opt_in != hipSuccess) return opt_in;
    BigManyArgs b{};
    b.M = layers[0]->M;
    b.R = layers[0]->R;
    b.tiles_m = (b.M + BigMany::BM - 1) / BigMany::BM;
    b.group_m = pick_group_m(BigMany::BM);
    unsigned grid = 0;
    for (int i = 0; i < count; ++i) {
        const GemmArgs &a = *layers[i];
        b.l[i] = {a.q, static_cast<const int8_t *>(a.w), a.s_a, static_cast<const float *>(a.s_w), a.bias, a.y, a.N, a.K, (a.N + BigMany::BN - 1) / BigMany::BN, big_many_padded(a)};
        grid += (unsigned)b.l[i].padded;
    }
    hipLaunchKernelGGL(qgemm_big_many, dim3(grid), dim3(BigMany::NTHR), BigMany::LDS_BYTES, stream, b);
    return hipGetLastError();
}

#define BIG(name, ...)                                                                                           \
    hipError_t launch_big_##name(const GemmArgs &a, hipStream_t s) { return run_big<TileBig<__VA_ARGS__>, false>(a, s); }  \
    hipError_t launch_big_##name##_glue(const GemmArgs &a, hipStream_t s) { return run_big<TileBig<__VA_ARGS__>, true>(a, s); }
BIG(w8_256x288, 4, 9, 4, 2, false)
BIG(w8_256x256, 4, 8, 4, 2, false)
BIG(w8_128x288, 2, 9, 4, 2, false)
BIG(f16_256x288, 4, 9, 4, 2, true)
BIG(f16_256x256, 4, 8, 4, 2, true)

}  // namespace ql
