// The pipelined tile of 8-bit and binary16 layers (qgemm.hip launches it layer by layer, qgemm_many.hip for several layers at once).
// Not part of the public ABI.
#pragma once
#include "qgemm_common.h"

namespace ql {

// ---------------------------------------------------------------------------------------------
// Pipelined variant: tiles go from global memory straight into LDS (global_load_lds_dwordx4, no
// register staging) through a ring of S stages.  One K step is 128 int8 = one 128-byte LDS row, so
// every DMA instruction moves 8 rows x 128 contiguous bytes (whole cache lines; 64-byte pieces were
// measured at little more than half the L1 fill rate).  The 16-byte chunk c of row r is kept at slot
// c ^ ((r >> 1) & 7) of its row: rows are unpadded (a wavefront's DMA writes 1024 contiguous bytes),
// and the XOR spreads the 16 lanes that read one chunk index of 16 consecutive rows over all banks.
// The K step is multiplied in four 32-wide quarters with double-buffered fragments: the reads of
// the next quarter, the hand-over barrier and the next DMA issue all sit behind an MFMA that is
// already executing.
// ---------------------------------------------------------------------------------------------
template <int TM_, int TN_, int WGM_, int WGN_, int S_, int WPS_, bool STG_ = true, int EV_ = 0, int SB_ = S_, bool PERSIST_ = false, bool F16_ = false, bool ANYK_ = false>
struct TileD {
    static constexpr int TM = TM_, TN = TN_, WGM = WGM_, WGN = WGN_, WPS = WPS_;
    // ring depth of the activation tile and of the weight tile (K steps resident or in flight); they may differ by one
    static constexpr int SA = S_, SB = SB_;
    // both operands binary16 (a layer the plan leaves unquantized): one K step is 64 values = the same 128 bytes per row
    static constexpr bool F16 = F16_;
    // rows of any whole number of words, at least 16 bytes: their last K step may be cut short
    static constexpr bool ANYK = ANYK_;
    static constexpr int NW = WGM * WGN, NT = NW * 64;
    static constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32, BK = 128;
    // 1024-byte DMA groups per K step: 8 rows x 128 B
    static constexpr int A_GROUPS = BM / 8, B_GROUPS = BN / 8;
    static constexpr int NA = A_GROUPS / NW, NB = B_GROUPS / NW;   // DMA instructions per wavefront per K step
    static constexpr int A_BYTES = A_GROUPS * 1024, B_BYTES = B_GROUPS * 1024;
    static constexpr int B_RING = SA * A_BYTES;           // the weight ring follows the activation ring
    static constexpr bool STAGED_STORE = STG_;
    static constexpr int DMA_EVERY = EV_;                 // one DMA instruction behind every EV_-th MFMA; 0: all at the hand-over
    static constexpr int STRIP_OFF = (BM * 4 + 255) / 256 * 256;   // epilogue: row scales first, then one strip per wavefront
    // a persistent workgroup parks its epilogue beside stage 0; where a 32-row strip per wavefront does not fit there,
    // the strip holds 16 rows
    static constexpr int STRIP_ROWS = (PERSIST_ && (SA - 1) * A_BYTES < STRIP_OFF + NW * 32 * (TN * 64 + 16)) ? 16 : 32;
    static constexpr int STRIP_BYTES = STRIP_ROWS * (TN * 64 + 16);
    static constexpr int RINGS = SA * A_BYTES + SB * B_BYTES;
    static constexpr int LDS_BYTES = RINGS > STRIP_OFF + NW * STRIP_BYTES ? RINGS : STRIP_OFF + NW * STRIP_BYTES;
    static constexpr int SMAX = SA > SB ? SA : SB;
    // Persistent launch: a workgroup walks several tiles and requests the first K step of the next tile before it
    // starts the epilogue of the current one, into stage 0 of both rings; the epilogue's scratch then lives in the
    // later stages of the activation ring.
    static constexpr bool PERSIST = PERSIST_;
    static constexpr int EPI_OFF = PERSIST ? A_BYTES : 0;
    static_assert(!PERSIST || (SA - 1) * A_BYTES >= STRIP_OFF + NW * STRIP_BYTES, "epilogue scratch beside stage 0");
    // loads that may still be in flight when K step 0 is first read, and at the hand-over from step kt to kt+1
    static constexpr int WAIT_START = (SA - 1) * NA + (SB - 1) * NB;
    static constexpr int WAIT_HAND = SA > SB ? NA + (SB - 2) * (NA + NB) : SA < SB ? NB + (SA - 2) * (NA + NB) : (SA - 2) * (NA + NB);
    static_assert(A_GROUPS % NW == 0 && B_GROUPS % NW == 0, "every wavefront issues the same number of DMA instructions");
    static_assert(SA >= 2 && SB >= 2 && (SA - SB) * (SA - SB) <= 1, "ring depths differ by at most one");
    static_assert(WAIT_START <= 63, "vmcnt is a 6-bit counter");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of one CU");
};

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;

// one workgroup's part: workgroup `block` of `blocks` (a multiple of XCDS) that share the layer
template <class T, bool GLUE>
__device__ __forceinline__ void qgemm_dma_tiles(const GemmArgs &a, int block, int blocks, int tiles_m, int tiles_n, int nblk_padded, int group_m)
{
    constexpr int TM = T::TM, TN = T::TN, BM = T::BM, BN = T::BN, NT = T::NT, NW = T::NW;
    constexpr bool F16 = T::F16;
    constexpr int EB = F16 ? 2 : 1;   // bytes per element of both operands
    extern __shared__ __align__(1024) unsigned char smem[];

    // Workgroup ids go round-robin over the XCDs; each XCD owns per_xcd consecutive logical tiles and its resident
    // workgroups take them in order, blocks / XCDS at a time (all of them at once unless the launch is persistent).
    const int per_xcd = nblk_padded / XCDS;
    const int slots_per_xcd = blocks / XCDS;
    const int xcd_first = (block % XCDS) * per_xcd;
    int in_xcd = block / XCDS;
    if (in_xcd >= per_xcd || xcd_first + in_xcd >= tiles_m * tiles_n) return;
    int m0, n0;
    auto set_tile = [&](int logical) {
        const int group_sz = group_m * tiles_n;
        const int first_m = (logical / group_sz) * group_m;
        const int gm = min(tiles_m - first_m, group_m);
        m0 = (first_m + (logical % group_sz) % gm) * BM;
        n0 = ((logical % group_sz) / gm) * BN;
    };
    set_tile(xcd_first + in_xcd);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keep it in a scalar register
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    const int M = a.M, N = a.N, K = a.K;
    const int nk = T::ANYK ? (K * EB + 127) / 128 : K * EB / 128;   // K steps (128 bytes per row)
    QL_PHASE(0)

    // Everything the epilogue needs from global memory is requested now, ahead of the first DMA (the oldest loads
    // return first, so the vmcnt bookkeeping of the ring is unaffected): the activation scale of one tile row per
    // thread, and the weight scale and bias of this lane's columns.
    static_assert(BM <= NT, "one row scale per thread");
    float sa_pre, swt[TN], bj[TN];
    auto load_scales = [&]() {
        sa_pre = (!F16 && tid < BM) ? a.s_a[min(m0 + tid, M - 1) / a.R] : 1.0f;
        const unsigned short *bias_h = static_cast<const unsigned short *>(a.bias);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = min(n0 + wn * TN * 32 + j * 32 + (lane & 31), N - 1);
            swt[j] = F16 ? 1.0f : static_cast<const float *>(a.s_w)[n];
            bj[j] = bias_h ? half_to_float_dev(bias_h[n]) : 0.0f;
        }
    };
    if (!T::PERSIST) load_scales();

    // DMA addressing: lane l of a wavefront fills bytes [16 l, 16 l + 16) of a 1024-byte group = row l/8, slot l%8.
    // Group g covers tile rows [8 g, 8 g + 8) of its operand.  Wavefront w takes groups w, w+NW, ... of both operands.
    constexpr int SA = T::SA, SB = T::SB, NA = T::NA, NB = T::NB;
    unsigned goffA[NA], goffB[NB];
    auto set_goff = [&]() {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int row = 8 * (wave + i * NW) + (lane >> 3);
            const int c = (lane & 7) ^ ((row >> 1) & 7);
            goffA[i] = T::ANYK ? first_piece(min(m0 + row, M - 1), K * EB, c) : row_start(min(m0 + row, M - 1), K * EB) + 16 * c;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int row = 8 * (wave + i * NW) + (lane >> 3);
            const int c = (lane & 7) ^ ((row >> 1) & 7);
            goffB[i] = T::ANYK ? first_piece(min(n0 + row, N - 1), K * EB, c) : row_start(min(n0 + row, N - 1), K * EB) + 16 * c;
        }
    };
    set_goff();
    // ANYK: a piece of the last K step that crosses or lies behind the end of its row reads the row's last 16 bytes instead
    auto back = [&](int kt, int i) { return T::ANYK ? piece_back(kt, nk, K * EB, (lane & 7) ^ ((4 * (wave + i * NW) + (lane >> 4)) & 7)) : 0u; };
    auto issue_a = [&](int kt, int slot, int i) {
        __builtin_amdgcn_global_load_lds((global_void *)(a.q + (size_t)kt * 128 + goffA[i] - back(kt, i)),
                                         (lds_void *)(smem + slot * T::A_BYTES + (wave + i * NW) * 1024), 16, 0, 0);
    };
    auto issue_b = [&](int kt, int slot, int i) {
        __builtin_amdgcn_global_load_lds((global_void *)(static_cast<const int8_t *>(a.w) + (size_t)kt * 128 + goffB[i] - back(kt, i)),
                                         (lds_void *)(smem + T::B_RING + slot * T::B_BYTES + (wave + i * NW) * 1024), 16, 0, 0);
    };
    // Refill window j = the loads issued after the hand-over barrier of K step j, into the slots that step used:
    // weight tile of step j+SB and activation tile of step j+SA.  The operand with the shallower ring is needed sooner
    // and goes first.  li numbers the NA+NB instructions of the window.
    constexpr bool B_FIRST = SB <= SA;
    auto issue_win = [&](int j, int slot_a, int slot_b, int li) {
        const bool is_b = B_FIRST ? li < NB : li >= NA;
        if (is_b) {
            if (j + SB < nk) issue_b(j + SB, slot_b, B_FIRST ? li : li - NA);
        } else {
            if (j + SA < nk) issue_a(j + SA, slot_a, B_FIRST ? li - NB : li);
        }
    };
    // ANYK, once the last K step is in LDS (slots sl_a and sl_b) and before it is read: what its pieces hold twice, or from behind the end of
    // the row, becomes zero; in one operand for integers, in both for binary16, where 0 * Inf is not 0
    auto clear_behind = [&](int sl_a, int sl_b) {
        const int left = K * EB - (nk - 1) * 128, first = left / 16, again = 16 - left % 16;   // again: bytes of piece `first` that are there twice
        auto clear = [&](unsigned char *st, int rows) {
            for (int e = tid; e < rows * 8; e += NT) {
                const int row = e >> 3, c = e & 7;
                if (c < first) continue;
                int *p = reinterpret_cast<int *>(st + row * 128 + ((c ^ ((row >> 1) & 7)) * 16));
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    if (c > first || 4 * w < again) p[w] = 0;
            }
        };
        if (left == 128) return;
        clear(smem + sl_a * T::A_BYTES, BM);
        if (F16) clear(smem + T::B_RING + sl_b * T::B_BYTES, BN);
        __syncthreads();
    };
    auto wait_vm = [&](auto n_tag) {
        constexpr int n = decltype(n_tag)::value;
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory");
    };

    typedef typename std::conditional<F16, v16f, v16i>::type acc_t;   // fp32 accumulators for FP16 operands
    acc_t acc[TM][TN];
    auto clear_sums = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    };

    // fragment of a lane: row (lane & 31) of a 32-row tile, 16 k starting at 32 * quarter + 16 * (lane >> 5)
    const int frag_row = lane & 31, frag_half = lane >> 5;
    const int key = (lane >> 1) & 7;  // swizzle key of this lane's row (tile rows start at multiples of 32)
    const int a_off = (wm * TM * 32 + frag_row) * 128;
    const int b_off = T::B_RING + (wn * TN * 32 + frag_row) * 128;
    auto read_frags = [&](int sl_a, int sl_b, int quarter, v4i(&af)[TM], v4i(&bf)[TN]) {
        const unsigned char *st = smem + sl_a * T::A_BYTES;
        const unsigned char *stb = smem + sl_b * T::B_BYTES;
        const int so = ((2 * quarter + frag_half) ^ key) * 16;
#pragma unroll
        for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const v4i *>(st + a_off + i * 32 * 128 + so);
#pragma unroll
        for (int j = 0; j < TN; ++j) bf[j] = *reinterpret_cast<const v4i *>(stb + b_off + j * 32 * 128 + so);
    };
    // MFMAs number [first, last) of one quarter, in (i, j) order
    auto mma = [&](const v4i(&af)[TM], const v4i(&bf)[TN], int first, int last) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (i * TN + j >= first && i * TN + j < last) acc[i][j] = mfma_step<F16>(af[i], bf[j], acc[i][j]);
    };
    constexpr int NMMA = TM * TN;
    // The same, with one DMA instruction of K step kt_i slipped in after every EVERY-th MFMA, starting with load i0:
    // 64 loads issued back to back fill the texture-address queue and stall the MFMA issue of every wavefront.
    constexpr int EVERY = T::DMA_EVERY > 0 ? T::DMA_EVERY : 1;
    constexpr bool SPREAD = T::DMA_EVERY > 0;
    auto mma_dma = [&](const v4i(&af)[TM], const v4i(&bf)[TN], int first, int last, bool on, int win, int slot_a, int slot_b, int i0) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int idx = i * TN + j;
                if (idx >= first && idx < last) {
                    acc[i][j] = mfma_step<F16>(af[i], bf[j], acc[i][j]);
                    const int li = i0 + (idx - first) / EVERY;
                    if (SPREAD && (idx - first) % EVERY == EVERY - 1 && li < NA + NB) {
                        if (on) issue_win(win, slot_a, slot_b, li);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
    };
    constexpr int N_Q = (NMMA - 1) / EVERY;    // loads that fit behind the MFMAs of one quarter
    static_assert(!SPREAD || 3 * N_Q >= NA + NB, "the loads of a refill window must be issued within three quarters");

    // prologue: the first SA activation tiles and SB weight tiles, in K-step order.  A persistent workgroup requests
    // step 0 ahead of everything else (for its first tile here, for later tiles before the previous epilogue).
    auto issue_step0 = [&]() {
        if (0 < nk) {
#pragma unroll
            for (int i = 0; i < NA; ++i) issue_a(0, 0, i);
#pragma unroll
            for (int i = 0; i < NB; ++i) issue_b(0, 0, i);
        }
    };
    if (T::PERSIST) issue_step0();
    for (;;) {   // one pass per tile; a single pass unless the launch is persistent
    if (T::PERSIST) load_scales();
    clear_sums();
    if (!T::PERSIST) issue_step0();
#pragma unroll
    for (int st = 1; st < T::SMAX; ++st) {
        if (st < SA && st < nk) {
#pragma unroll
            for (int i = 0; i < NA; ++i) issue_a(st, st, i);
        }
        if (st < SB && st < nk) {
#pragma unroll
            for (int i = 0; i < NB; ++i) issue_b(st, st, i);
        }
    }
    QL_PHASE(1)
    v4i af0[TM], bf0[TN], af1[TM], bf1[TN];
    // K step 0 has landed once only the later steps of the prologue are outstanding
    if (nk >= T::SMAX) wait_vm(std::integral_constant<int, T::WAIT_START>{});
    else wait_vm(std::integral_constant<int, 0>{});
    __builtin_amdgcn_s_barrier();
    if (T::ANYK && nk == 1) clear_behind(0, 0);
    read_frags(0, 0, 0, af0, bf0);
    int sa = 0, sb = 0, pa = SA - 1, pb = SB - 1;   // ring slots of K step kt and of step kt-1
    for (int kt = 0; kt < nk; ++kt) {
        const int na = sa + 1 == SA ? 0 : sa + 1, nb = sb + 1 == SB ? 0 : sb + 1;
        const bool refill = kt > 0;   // refill window kt-1 is still being issued during quarters 0 and 1
        // quarter 0 (fragments 0) while reading quarter 1 (fragments 1)
        mma(af0, bf0, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(sa, sb, 1, af1, bf1);
        __builtin_amdgcn_sched_barrier(0);
        mma_dma(af0, bf0, 1, NMMA, refill, kt - 1, pa, pb, N_Q);
        __builtin_amdgcn_sched_barrier(0);
        // quarter 1 while reading quarter 2
        mma(af1, bf1, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(sa, sb, 2, af0, bf0);
        __builtin_amdgcn_sched_barrier(0);
        mma_dma(af1, bf1, 1, NMMA, refill, kt - 1, pa, pb, 2 * N_Q);
        __builtin_amdgcn_sched_barrier(0);
        // quarter 2 while reading quarter 3
        mma(af0, bf0, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(sa, sb, 3, af1, bf1);
        __builtin_amdgcn_sched_barrier(0);
        mma(af0, bf0, 1, NMMA);
        __builtin_amdgcn_sched_barrier(0);
        // quarter 3: its first MFMA needs the last fragments of this K step, so once it has issued every read of
        // this step's slots by this wavefront is complete.  Then hand over: step kt+1 must be in LDS (only loads
        // issued after its last one may still be in flight), and after the barrier this step's slots can be refilled.
        mma(af1, bf1, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        if (kt + T::SMAX <= nk) wait_vm(std::integral_constant<int, T::WAIT_HAND>{});
        else wait_vm(std::integral_constant<int, 0>{});
        __builtin_amdgcn_s_barrier();
        if (T::ANYK && kt + 2 == nk) clear_behind(na, nb);
        if (!SPREAD) {
#pragma unroll
            for (int li = 0; li < NA + NB; ++li) issue_win(kt, sa, sb, li);
        }
        if (kt + 1 < nk) read_frags(na, nb, 0, af0, bf0);
        __builtin_amdgcn_sched_barrier(0);
        mma_dma(af1, bf1, 1, NMMA, true, kt, sa, sb, 0);
        __builtin_amdgcn_sched_barrier(0);
        pa = sa;
        pb = sb;
        sa = na;
        sb = nb;
    }
    QL_PHASE(2)
    __syncthreads();

    // the tile being written out; a persistent workgroup moves on to its next tile first and requests that tile's
    // first K step, so that it travels while the epilogue runs
    const int em0 = m0, en0 = n0;
    bool has_next = false;
    if (T::PERSIST) {
        in_xcd += slots_per_xcd;
        has_next = in_xcd < per_xcd && xcd_first + in_xcd < tiles_m * tiles_n;
        if (has_next) {
            set_tile(xcd_first + in_xcd);
            set_goff();
            issue_step0();
        }
    }
    float *sRow = reinterpret_cast<float *>(smem + T::EPI_OFF);
    if (tid < BM) sRow[tid] = sa_pre;
    __syncthreads();
    QL_PHASE(3)
    _Float16 *y = static_cast<_Float16 *>(a.y);
    const unsigned short *bias = static_cast<const unsigned short *>(a.bias);
    const bool full = (em0 + BM <= M) && (en0 + BN <= N);
    const bool glue_pieces = GLUE && (a.residual || a.gate);
    const bool glue_aligned = !glue_pieces || (((reinterpret_cast<uintptr_t>(a.residual) | reinterpret_cast<uintptr_t>(a.gate)) & 15) == 0);
    if (full && (N % 8) == 0 && (reinterpret_cast<uintptr_t>(a.y) & 15) == 0 && !a.acc_out && glue_aligned) {
        GluePieces gl;
        if (glue_pieces) {
            gl.gate = static_cast<const _Float16 *>(a.gate);
            gl.residual = static_cast<const _Float16 *>(a.residual);
            gl.gate_rows = a.gate_rows;
            gl.on = true;
        }
        if (GLUE) gl.rowmax = a.row_absmax;
        unsigned char *strip = smem + T::EPI_OFF + T::STRIP_OFF + wave * T::STRIP_BYTES;
        // the 16 row scales of each 32-row block of this lane (rows 8g + 4*frag_half + 0..3), read once as 4 x 16 bytes
        float sr[TM * 16];
        {
            const float *srow = sRow + wm * TM * 32 + 4 * frag_half;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4f t = *reinterpret_cast<const v4f *>(srow + i * 32 + 8 * g);
                    sr[i * 16 + 4 * g + 0] = t[0];
                    sr[i * 16 + 4 * g + 1] = t[1];
                    sr[i * 16 + 4 * g + 2] = t[2];
                    sr[i * 16 + 4 * g + 3] = t[3];
                }
        }
        // the activation is chosen once per kernel, not per element
        auto emit_fast = [&](auto act_tag) {
            constexpr bool ACT = decltype(act_tag)::value;
            auto act_of = [&](float u) { return ACT ? gelu_tanh_dev(u) : u; };
            if (F16)
                store_tile_staged<TM, TN, T::STAGED_STORE, T::STRIP_ROWS>(strip, lane, y, N, em0 + wm * TM * 32, en0 + wn * TN * 32, [&](int i, int j, int r) {
                    return act_of((float)acc[i][j][r] + bj[j]);
                }, gl);
            else if (bias)
                store_tile_staged<TM, TN, T::STAGED_STORE, T::STRIP_ROWS>(strip, lane, y, N, em0 + wm * TM * 32, en0 + wn * TN * 32, [&](int i, int j, int r) {
                    return act_of(__builtin_fmaf((float)acc[i][j][r] * sr[i * 16 + r], swt[j], bj[j]));
                }, gl);
            else
                store_tile_staged<TM, TN, T::STAGED_STORE, T::STRIP_ROWS>(strip, lane, y, N, em0 + wm * TM * 32, en0 + wn * TN * 32, [&](int i, int j, int r) {
                    return act_of((float)acc[i][j][r] * sr[i * 16 + r] * swt[j]);
                }, gl);
        };
        if (GLUE && a.act == 1) emit_fast(std::true_type{});
        else emit_fast(std::false_type{});
    } else {
        const GateRows gate_rows(GLUE ? a.gate : nullptr, a.gate_rows, em0, BM);
        auto emit = [&](auto edge) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int row = wm * TM * 32 + i * 32 + 4 * frag_half;
                    const int n = en0 + wn * TN * 32 + j * 32 + frag_row;
                    store_column<GLUE, decltype(edge)::value, GLUE ? Behind::PASSED : F16 ? Behind::ASKED : Behind::LEFT>(a, gate_rows, em0, row, n, [&](int r, unsigned off) {
                        if (F16) return (float)acc[i][j][r] + bj[j];
                        const float t = (float)acc[i][j][r] * sRow[row + 8 * (r / 4) + r % 4];
                        if (a.acc_out) a.acc_out[off] = (int)acc[i][j][r];
                        return bias ? __builtin_fmaf(t, swt[j], bj[j]) : t * swt[j];
                    });
                }
        };
        // glue keeps one form: a second one is a quarter more code in this library's largest object (with six blocks per wavefront it also spills), and a plan that
        // uses one plain kernel of it was 1 % slower (32 images of 256 rows, percentile scales, 313 against 317 us)
        if (!GLUE && full) emit(std::false_type{});
        else emit(std::true_type{});
    }
    QL_PHASE(4)
    if (!has_next) break;
    __syncthreads();   // the epilogue's scratch is free again: the rest of the next prologue may overwrite it
    }
}

}  // namespace ql
