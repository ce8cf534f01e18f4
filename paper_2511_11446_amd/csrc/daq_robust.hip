// Percentile-clipped dynamic activation quantization (Step 3, eq. (4) as printed; activation width b from the
// time-bin policy of Step 6 / Algorithm 2 Phase B) for gfx950.
//
//   tau   = the c-th largest magnitude of the scale block (nearest-rank percentile: c = n - ceil(n p) + 1)
//   alpha = tau / qmax, qmax = 2^(b-1) - 1   (1 if tau = 0)
//   code  = clamp(round_half_even(clip(x, -tau, tau) / alpha), -qmax, qmax)
//
// The selection is exact and works on the 15-bit magnitude patterns of binary16 (their integer order is the numeric
// order).  One row per scale: the row sits in registers and tau is found by a bitwise binary search (15 counting
// rounds over the registers).  Several rows per scale: two histogram passes (upper 8 bits, then the lower 7 bits of
// the values that share the selected upper bits) and the quantize pass; whoever needs a selection scans the bins from the top
// itself.
#include "daq_device.h"

namespace ql {

__device__ __forceinline__ unsigned wave_sum_u32(unsigned m)
{
#define QL_ROR_ADD(ctrl) m += (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, ctrl, 0xF, 0xF, false);
    QL_ROR_ADD(0x128)  // row_ror:8
    QL_ROR_ADD(0x124)  // row_ror:4
    QL_ROR_ADD(0x122)  // row_ror:2
    QL_ROR_ADD(0x121)  // row_ror:1
#undef QL_ROR_ADD
    return (unsigned)__builtin_amdgcn_readlane((int)m, 0) + (unsigned)__builtin_amdgcn_readlane((int)m, 16) +
           (unsigned)__builtin_amdgcn_readlane((int)m, 32) + (unsigned)__builtin_amdgcn_readlane((int)m, 48);
}

// clip to [-tau, tau], then the code with the given full scale (same arithmetic as the oracle's: IEEE division)
__device__ __forceinline__ int robust_code(float v, float tau, float alpha, float qmax)
{
    v = fminf(fmaxf(v, -tau), tau);
    float r = __builtin_rintf(v / alpha);
    r = fminf(fmaxf(r, -qmax), qmax);
    return (int)r;
}

__device__ __forceinline__ unsigned robust_pack4(unsigned w0, unsigned w1, float tau, float alpha, float qmax)
{
    const int c0 = robust_code(half_bits_to_float(w0 & 0xffffu), tau, alpha, qmax);
    const int c1 = robust_code(half_bits_to_float(w0 >> 16), tau, alpha, qmax);
    const int c2 = robust_code(half_bits_to_float(w1 & 0xffffu), tau, alpha, qmax);
    const int c3 = robust_code(half_bits_to_float(w1 >> 16), tau, alpha, qmax);
    return (unsigned)(c0 & 0xff) | ((unsigned)(c1 & 0xff) << 8) | ((unsigned)(c2 & 0xff) << 16) | ((unsigned)c3 << 24);
}

// division-free form, as in daq_piece(): |clip(x)/alpha| <= qmax <= 127, so the same error bound holds
__device__ __forceinline__ unsigned robust_fast_code(unsigned hbits, float tau, float rcp, float &dmax)
{
    float x = half_bits_to_float(hbits);
    x = fminf(fmaxf(x, -tau), tau);
    const float y = __builtin_fmaf(x, rcp, DAQ_MAGIC);
    const float r = y - DAQ_MAGIC;
    const float d = __builtin_fmaf(x, rcp, -r);
    dmax = fmaxf(dmax, fabsf(d));
    return __builtin_bit_cast(unsigned, y);
}

__device__ __forceinline__ uint2 robust_piece(const uint4 &v, float tau, float alpha, float rcp, float qmax)
{
    float dmax = 0.0f;
    unsigned y[8];
    const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        y[2 * i] = robust_fast_code(w[i] & 0xffffu, tau, rcp, dmax);
        y[2 * i + 1] = robust_fast_code(w[i] >> 16, tau, rcp, dmax);
    }
    uint2 out;
    out.x = __builtin_amdgcn_perm(__builtin_amdgcn_perm(y[3], y[2], 0x0c0c0400u), __builtin_amdgcn_perm(y[1], y[0], 0x0c0c0400u), 0x05040100u);
    out.y = __builtin_amdgcn_perm(__builtin_amdgcn_perm(y[7], y[6], 0x0c0c0400u), __builtin_amdgcn_perm(y[5], y[4], 0x0c0c0400u), 0x05040100u);
    if (__builtin_expect(!(dmax < DAQ_NEAR_TIE), 0))
        out = make_uint2(robust_pack4(v.x, v.y, tau, alpha, qmax), robust_pack4(v.z, v.w, tau, alpha, qmax));
    return out;
}

struct RobustScale {
    float tau, alpha, rcp;
};
__device__ __forceinline__ RobustScale robust_scale(unsigned tau_bits, float qmax)
{
    RobustScale s;
    s.tau = half_bits_to_float(tau_bits);
    s.alpha = s.tau == 0.0f ? 1.0f : s.tau / qmax;
    s.rcp = 1.0f / s.alpha;
    return s;
}

// ---- selection from histograms -------------------------------------------------------------------------------------
// A magnitude has 15 bits: level 0 counts by the upper 8, level 1 by the lower 7 of the magnitudes whose upper bits level 0
// selected.  Where a scale block has few parts (HIST_FEW), every part leaves its own 16-bit histogram with plain stores and
// the next pass adds them up: no clearing pass, no global atomics, no launch that only selects.  Scratch (a.hist):
// [block][part][256] level 0, then [block][part][128] level 1, 16 bits each; blockmax[b] = selected upper bits | rank left
// inside that bin << 8.  With more parts: 32-bit counts collected with atomics, [block][DAQ_ROBUST_WORDS].
constexpr int HIST_PART = DAQ_HIST_PART;
constexpr int HIST_BINS = 256;

// The bin, counted from the top, in which the `left`-th largest value falls, and the rank left inside it.  One wavefront; bins
// 0 .. 64 * PER - 1 at `count`.
template <int PER>
__device__ __forceinline__ void select_bin(const unsigned *count, unsigned &left, unsigned &bin)
{
    const int lane = threadIdx.x & 63;
    unsigned c[PER], sum = 0;       // lane 0 has the highest bins
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = count[64 * PER - 1 - (lane * PER + i)];
        sum += c[i];
    }
    unsigned upto = sum;            // inclusive sum over the lanes
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const unsigned o = __shfl_up(upto, d);
        if (lane >= d) upto += o;
    }
    unsigned before = upto - sum;
    const unsigned long long hit = __ballot(upto >= left);
    const int owner = hit ? __ffsll((long long)hit) - 1 : 63;
    unsigned b = 0, l = 0;
    bool found = false;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (!found && (before + c[i] >= left || i == PER - 1)) {
            found = true;
            b = 64 * PER - 1 - (lane * PER + i);
            l = left - before;
        }
        before += c[i];
    }
    bin = __shfl(b, owner);
    left = __shfl(l, owner);
}

// level 0: sums of the parts' histograms into LDS, then the selection, by the whole workgroup
__device__ __forceinline__ void first_selection(const DaqArgs &a, unsigned b, int parts, unsigned *bins, unsigned &prefix, unsigned &left)
{
    __shared__ unsigned found[2];
    const unsigned short *h0 = reinterpret_cast<const unsigned short *>(a.hist) + (size_t)b * parts * 256;
    unsigned n = 0;
#pragma unroll 8
    for (int p = 0; p < parts; ++p) n += h0[p * 256 + threadIdx.x];
    bins[threadIdx.x] = n;
    __syncthreads();
    if (threadIdx.x < 64) {
        unsigned l = a.top_rank, bin;
        select_bin<4>(bins, l, bin);
        if (threadIdx.x == 0) {
            found[0] = bin;
            found[1] = l;
        }
    }
    __syncthreads();
    prefix = found[0];
    left = found[1];
}

// level 1: the magnitude pattern of tau
__device__ __forceinline__ unsigned second_selection(const DaqArgs &a, int b, unsigned *bins)
{
    __shared__ unsigned tau;
    const int parts = a.quant_parts;
    const unsigned short *h1 = reinterpret_cast<const unsigned short *>(a.hist) + (size_t)(a.M / a.R) * parts * 256 + (size_t)b * parts * 128;
    if (threadIdx.x < 128) {
        unsigned n = 0;
#pragma unroll 8
        for (int p = 0; p < parts; ++p) n += h1[p * 128 + threadIdx.x];
        bins[threadIdx.x] = n;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const unsigned first = a.blockmax[b];
        unsigned l = first >> 8, bin;
        select_bin<2>(bins, l, bin);
        if (threadIdx.x == 0) tau = (first & 0xffu) << 7 | bin;
    }
    __syncthreads();
    return tau;
}

// ---- one row per scale, row in registers ------------------------------------------------------------------------
// mode DAQ_FUSED: select tau, then quantize; mode DAQ_QUANT: tau of the row's block comes from blockmax, or with HIST from the second
// histogram pass (quant_parts partial histograms, R % 4 == 0: the workgroup's rows share a block).  HIST is a kernel of its own: its LDS
// and barriers inside the others cost one row per scale 8 % (M = 16384, K = 1152: 18.0 -> 19.6 us)
template <int CH, bool HIST>
__device__ __forceinline__ void robust_rows(const DaqArgs &a, int mode, int wg)
{
    const int lane = threadIdx.x & 63;
    const int row = wg * 4 + (threadIdx.x >> 6);
    if (row >= a.M) return;   // whole workgroups at a time where the rows share a block
    const int nch = a.K >> 3;
    const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(a.x) + (size_t)row * a.K);
    uint4 v[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int c = lane + 64 * i;
        v[i] = c < nch ? xr[c] : make_uint4(0, 0, 0, 0);
    }
    unsigned tau_bits;
    if constexpr (HIST) {
        __shared__ unsigned bins[HIST_BINS];
        tau_bits = second_selection(a, row / a.R, bins);
        // the row has arrived by now: said once, here, or every piece below waits for all of memory, its predecessor's store included (K =
        // 4608, 64 rows: 7.0 us against 5.8)
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    } else if (mode == DAQ_QUANT) {
        tau_bits = a.blockmax[row / a.R];
    } else {
        // Each half word is 0x8000 | magnitude (OR-ing 0x8000 in overwrites the sign bit); subtracting T from both
        // halves at once leaves bit 15 of a half set iff its magnitude >= T (no half can borrow from its neighbour:
        // every half result is >= 1).  Lanes past the end of the row hold zeros, which no T >= 1 counts.
        auto count_ge = [&](unsigned t) {
            const unsigned t2 = t * 0x00010001u;
            unsigned cnt = 0;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                cnt += (((v[i].x | 0x80008000u) - t2) >> 15) & 0x00010001u;
                cnt += (((v[i].y | 0x80008000u) - t2) >> 15) & 0x00010001u;
                cnt += (((v[i].z | 0x80008000u) - t2) >> 15) & 0x00010001u;
                cnt += (((v[i].w | 0x80008000u) - t2) >> 15) & 0x00010001u;
            }
            return wave_sum_u32((cnt & 0xffffu) + (cnt >> 16));
        };
        unsigned mx = 0;   // the row maximum
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            mx = absmax_word(mx, v[i].x);
            mx = absmax_word(mx, v[i].y);
            mx = absmax_word(mx, v[i].z);
            mx = absmax_word(mx, v[i].w);
        }
        mx = wave_max_u32((mx & 0xffffu) > (mx >> 16) ? (mx & 0xffffu) : (mx >> 16));
        unsigned T = 0;
        if (a.top_rank <= 8) {
            // tau is among the few largest values (the paper's p = 99.9 %: the 2nd largest of 1152, the 5th of 4608):
            // walk down the distinct magnitudes from the top.  One sweep over the registers finds the next magnitude
            // below `prev` and, with the same comparison, counts the values at or above `prev`; the walk ends at the
            // first magnitude with top_rank values at or above it (after at most top_rank sweeps), or where everything left is zero (tau = 0).
            // That the walk begins below the maximum is written out: left to itself the compiler sometimes sweeps with the comparison for
            // the maximum too (M = 16384, K = 1152: 18.3 us against 19.6)
            unsigned prev = mx;
            for (unsigned pass = 1; pass <= a.top_rank && prev != 0; ++pass) {
                const unsigned p2 = prev * 0x00010001u;
                unsigned m2 = 0, cnt = 0;
                auto sweep = [&](unsigned w) {
                    const unsigned mag = w & 0x7fff7fffu;
                    const unsigned ge = (((mag | 0x80008000u) - p2) >> 15) & 0x00010001u;   // bit 0 / 16: magnitude >= prev
                    cnt += ge;
                    m2 = absmax_word(m2, mag & ((ge ^ 0x00010001u) * 0xffffu));              // the halves below prev
                };
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    sweep(v[i].x);
                    sweep(v[i].y);
                    sweep(v[i].z);
                    sweep(v[i].w);
                }
                if (wave_sum_u32((cnt & 0xffffu) + (cnt >> 16)) >= a.top_rank) {
                    T = prev;
                    break;
                }
                prev = wave_max_u32((m2 & 0xffffu) > (m2 >> 16) ? (m2 & 0xffffu) : (m2 >> 16));
            }
        } else {
            // largest T with count(magnitude >= T) >= top_rank, built bit by bit from the top; a candidate above the
            // row maximum cannot succeed and costs no counting round
            for (int bit = 14; bit >= 0; --bit) {
                const unsigned cand = T | (1u << bit);
                if (cand <= mx && count_ge(cand) >= a.top_rank) T = cand;
            }
        }
        tau_bits = T;
    }
    const float qmax = (float)a.qmax;
    const RobustScale s = robust_scale(tau_bits, qmax);
    if (lane == 0 && (row % a.R) == 0) a.scales[row / a.R] = s.alpha;
    uint2 *qr = reinterpret_cast<uint2 *>(a.q + (size_t)row * a.K);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) qr[c] = robust_piece(v[i], s.tau, s.alpha, s.rcp, qmax);
    }
}

template <int CH, bool HIST>
__global__ __launch_bounds__(256) void daq_rows_robust(DaqArgs a, int mode)
{
    robust_rows<CH, HIST>(a, mode, mode == DAQ_QUANT ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x);
}

// The rows of several layers.  LONG: some of more than 1536 values; their registers (127 against 55) would halve the wavefronts that the shorter
// rows' selections keep in flight (99.9th percentile of each row, M = 16384, us a plan: eight layers of K = 384 102 -> 80, four of K = 1152 172 -> 161; a
// launch per layer 131 and 170)
template <bool LONG, bool HIST>
__global__ __launch_bounds__(256) void daq_rows_robust_many(DaqMany b, int mode)
{
    const int block = mode == DAQ_QUANT ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x;
    const int layer = block / b.row_blocks, wg = block - layer * b.row_blocks;
    const DaqArgs &l = b.l[layer];
    if (l.K <= 512) robust_rows<1, HIST>(l, mode, wg);
    else if (l.K <= 1024) robust_rows<2, HIST>(l, mode, wg);
    else if (!LONG || l.K <= 1536) robust_rows<3, HIST>(l, mode, wg);
    else if (l.K <= 2048) robust_rows<LONG ? 4 : 3, HIST>(l, mode, wg);
    else if (l.K <= 3072) robust_rows<LONG ? 6 : 3, HIST>(l, mode, wg);
    else robust_rows<LONG ? 9 : 3, HIST>(l, mode, wg);
}

template <bool HIST>
static void run_robust_rows_many(const DaqMany &b, int mode, hipStream_t s)
{
    bool long_rows = false;
    for (int i = 0; i < b.count; ++i) long_rows = long_rows || b.l[i].K > 1536;
    const dim3 grid((unsigned)b.row_blocks * (unsigned)b.count);
    if (long_rows) hipLaunchKernelGGL((daq_rows_robust_many<true, HIST>), grid, dim3(256), 0, s, b, mode);
    else hipLaunchKernelGGL((daq_rows_robust_many<false, HIST>), grid, dim3(256), 0, s, b, mode);
}

// any row length and alignment: the row is re-read from memory (cache) in every counting round
__global__ __launch_bounds__(256) void daq_rows_robust_loop(DaqArgs a, int mode)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= a.M) return;
    const unsigned short *xs = static_cast<const unsigned short *>(a.x) + (size_t)row * a.K;
    unsigned tau_bits;
    if (mode == DAQ_QUANT) {
        tau_bits = a.blockmax[row / a.R];
    } else {
        unsigned T = 0;
        for (int bit = 14; bit >= 0; --bit) {
            const unsigned cand = T | (1u << bit);
            unsigned cnt = 0;
            for (int k = lane; k < a.K; k += 64) cnt += ((unsigned)(xs[k] & 0x7fffu) >= cand) ? 1u : 0u;
            cnt = wave_sum_u32(cnt);
            if (cnt >= a.top_rank) T = cand;
        }
        tau_bits = T;
    }
    const float qmax = (float)a.qmax;
    const RobustScale s = robust_scale(tau_bits, qmax);
    if (lane == 0 && (row % a.R) == 0) a.scales[row / a.R] = s.alpha;
    int8_t *qs = a.q + (size_t)row * a.K;
    for (int k = lane; k < a.K; k += 64) qs[k] = (int8_t)robust_code(half_bits_to_float(xs[k]), s.tau, s.alpha, qmax);
}

// ---- several rows per scale: histogram passes ------------------------------------------------------------------------
// FEW: partial histograms (see above); otherwise atomics into hist[b*DAQ_ROBUST_WORDS ...]: 0..255 level 0, [256] selected
// upper bits, [257] rank left, [258..385] level 1.
// The magnitudes of a real activation tensor fall into some thirty of the 256 bins: sixteen copies of the LDS histogram, one
// per quarter wavefront, keep the lanes of an LDS atomic from queueing for one word.
// What bounds a pass over a large tensor is the arithmetic per value, since all parts are resident at once: the level is a template argument,
// a whole part (all but the last of a block) loads and counts without a condition per piece, and level 1 looks at two
// values with one branch.  M = 8192, R = 256, us with a branch per load and the level as an argument -> now: three layers of K = 1152 18.7 and 19.1 ->
// 15.7 and 14.1, K = 4608 23.3 and 17.6 -> 20.1 and 13.3 (level 0 is left with its LDS atomics).
template <bool FEW, int LEVEL>
__device__ __forceinline__ void hist_part(const DaqArgs &a, unsigned block, unsigned parts_per_block, bool self)
{
    constexpr int COPIES = 16;
    __shared__ unsigned h[COPIES * (HIST_BINS + 1)];
    __shared__ unsigned bins[HIST_BINS];
    const unsigned b = block / parts_per_block, part = block - b * parts_per_block;
    const size_t n_per_block = (size_t)a.R * a.K;
    const unsigned short *xb = static_cast<const unsigned short *>(a.x) + (size_t)b * n_per_block;
    const size_t i0 = (size_t)part * HIST_PART;
    const size_t i1 = i0 + HIST_PART < n_per_block ? i0 + HIST_PART : n_per_block;
    const bool vec = ((uintptr_t)(xb + i0) % 16 == 0);
    const size_t pieces = vec ? (i1 - i0) / 8 : 0;
    constexpr int U = HIST_PART / 8 / 256;   // 16-byte pieces per thread
    const bool whole = pieces == HIST_PART / 8;
    uint4 v[U];
    // zeros past the part's end, without a branch between the loads
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = load_row_piece(xb + i0, (int)pieces * 16, threadIdx.x * 16, u * 4096);
    for (int i = threadIdx.x; i < COPIES * (HIST_BINS + 1); i += 256) h[i] = 0;
    unsigned prefix = 0;
    if (LEVEL) {
        if (FEW && self) {
            unsigned left;
            first_selection(a, b, (int)parts_per_block, bins, prefix, left);
            if (part == 0 && threadIdx.x == 0) a.blockmax[b] = prefix | left << 8;
        } else if (FEW) {
            prefix = a.blockmax[b] & 0xffu;
        } else {
            prefix = a.hist[(size_t)b * DAQ_ROBUST_WORDS + 256];
        }
    }
    __syncthreads();
    unsigned *mine = h + (threadIdx.x >> 4) * (HIST_BINS + 1);
    auto tally = [&](unsigned m) {
        if (LEVEL == 0) atomicAdd(&mine[m >> 7], 1u);
        else if ((m >> 7) == prefix) atomicAdd(&mine[m & 127u], 1u);
    };
    const unsigned prefix2 = prefix * (128u * 0x00010001u);
    auto tally2 = [&](unsigned w) {
        // a half of z is zero where its upper bits are the selected ones; 0x8000 minus it then keeps bit 15
        const unsigned z = (w ^ prefix2) & 0x7f807f80u;
        if (LEVEL == 0 || ((0x80008000u - z) & 0x80008000u)) {
            tally(w & 0x7fffu);
            tally((w >> 16) & 0x7fffu);
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (whole || threadIdx.x + 256 * (size_t)u < pieces) {
            tally2(v[u].x);
            tally2(v[u].y);
            tally2(v[u].z);
            tally2(v[u].w);
        }
    }
    for (size_t i = i0 + pieces * 8 + threadIdx.x; i < i1; i += 256) tally(xb[i] & 0x7fffu);
    __syncthreads();
    unsigned cnt = 0;
#pragma unroll
    for (int c = 0; c < COPIES; ++c) cnt += h[c * (HIST_BINS + 1) + threadIdx.x];
    if (FEW) {
        unsigned short *h16 = reinterpret_cast<unsigned short *>(a.hist);
        if (LEVEL == 0) h16[(size_t)block * 256 + threadIdx.x] = (unsigned short)cnt;
        else if (threadIdx.x < 128) h16[(size_t)(a.M / a.R) * parts_per_block * 256 + (size_t)block * 128 + threadIdx.x] = (unsigned short)cnt;
    } else if (cnt && (LEVEL == 0 || threadIdx.x < 128)) {
        atomicAdd(a.hist + (size_t)b * DAQ_ROBUST_WORDS + (LEVEL ? 258 : 0) + threadIdx.x, cnt);
    }
}

template <bool FEW, int LEVEL>
__global__ __launch_bounds__(256) void daq_hist(DaqArgs a, unsigned parts_per_block)
{
    hist_part<FEW, LEVEL>(a, blockIdx.x, parts_per_block, parts_per_block <= DAQ_HIST_SELF);
}

// the parts of several layers, few per scale block
template <bool SELF, int LEVEL>
__global__ __launch_bounds__(256) void daq_hist_many(DaqMany b)
{
    const int i = many_layer(b, blockIdx.x);
    hist_part<true, LEVEL>(b.l[i], blockIdx.x - b.first[i], (unsigned)b.l[i].quant_parts, SELF);
}

template <bool FEW>
static void run_hist(const DaqArgs &a, unsigned parts, int level, hipStream_t s)
{
    const dim3 grid(parts * (unsigned)(a.M / a.R));
    if (level == 0) hipLaunchKernelGGL((daq_hist<FEW, 0>), grid, dim3(256), 0, s, a, parts);
    else hipLaunchKernelGGL((daq_hist<FEW, 1>), grid, dim3(256), 0, s, a, parts);
}

template <bool SELF>
static void run_hist_many(const DaqMany &b, unsigned grid, int level, hipStream_t s)
{
    if (level == 0) hipLaunchKernelGGL((daq_hist_many<SELF, 0>), dim3(grid), dim3(256), 0, s, b);
    else hipLaunchKernelGGL((daq_hist_many<SELF, 1>), dim3(grid), dim3(256), 0, s, b);
}

// many parts: one wavefront per scale block
__global__ __launch_bounds__(64) void daq_hist_select(DaqArgs a, int level)
{
    unsigned *hb = a.hist + (size_t)blockIdx.x * DAQ_ROBUST_WORDS;
    unsigned left = level ? hb[257] : a.top_rank, bin;
    if (level == 0) select_bin<4>(hb, left, bin);
    else select_bin<2>(hb + 258, left, bin);
    if (threadIdx.x != 0) return;
    if (level == 0) {
        hb[256] = bin;
        hb[257] = left;
    } else {
        a.blockmax[blockIdx.x] = (hb[256] << 7) | bin;
    }
}

// partial histograms whose consumers do not select for themselves: one workgroup per scale block adds them up, four threads
// per bin, and selects; level 0 leaves blockmax = upper bits | rank left << 8, level 1 the pattern of tau
__device__ __forceinline__ void part_select(const DaqArgs &a, int b, int parts, int level)
{
    __shared__ unsigned bins[4][HIST_BINS];
    const int width = level ? 128 : 256, bin_of = threadIdx.x & 255, q = threadIdx.x >> 8;
    const unsigned short *h = reinterpret_cast<const unsigned short *>(a.hist) + (level ? (size_t)(a.M / a.R) * parts * 256 : 0) + (size_t)b * parts * width;
    unsigned n = 0;
    if (bin_of < width) {
#pragma unroll 8
        for (int p = q; p < parts; p += 4) n += h[p * width + bin_of];
    }
    bins[q][bin_of] = n;
    __syncthreads();
    if (threadIdx.x < 256) bins[0][threadIdx.x] += bins[1][threadIdx.x] + bins[2][threadIdx.x] + bins[3][threadIdx.x];
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const unsigned first = level ? a.blockmax[b] : 0;
    unsigned left = level ? first >> 8 : a.top_rank, bin;
    if (level == 0) select_bin<4>(bins[0], left, bin);
    else select_bin<2>(bins[0], left, bin);
    if (threadIdx.x == 0) a.blockmax[b] = level == 0 ? bin | left << 8 : (first & 0xffu) << 7 | bin;
}

__global__ __launch_bounds__(1024) void daq_part_select(DaqArgs a, int parts, int level) { part_select(a, blockIdx.x, parts, level); }

__global__ __launch_bounds__(1024) void daq_part_select_many(DaqMany b, int level)
{
    const int nblk = b.l[0].M / b.l[0].R, layer = blockIdx.x / nblk;
    part_select(b.l[layer], blockIdx.x - layer * nblk, b.l[layer].quant_parts, level);
}

__global__ void fill_zero_u32(unsigned *p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

template <int CH>
static void run_robust_cached(const DaqArgs &a, int mode, hipStream_t s)
{
    if (mode == DAQ_QUANT && a.quant_parts > 0) hipLaunchKernelGGL((daq_rows_robust<CH, true>), dim3((a.M + 3) / 4), dim3(256), 0, s, a, mode);
    else hipLaunchKernelGGL((daq_rows_robust<CH, false>), dim3((a.M + 3) / 4), dim3(256), 0, s, a, mode);
}

static void run_robust_rows(const DaqArgs &a, int mode, hipStream_t s)
{
    const bool vec = (a.K % 8 == 0) && ((uintptr_t)a.x % 16 == 0) && ((uintptr_t)a.q % 8 == 0);
    const int per_lane = (a.K / 8 + 63) / 64;
    if (!vec || per_lane > 16) {
        hipLaunchKernelGGL(daq_rows_robust_loop, dim3((a.M + 3) / 4), dim3(256), 0, s, a, mode);
        return;
    }
    if (per_lane <= 1) run_robust_cached<1>(a, mode, s);
    else if (per_lane <= 2) run_robust_cached<2>(a, mode, s);
    else if (per_lane <= 3) run_robust_cached<3>(a, mode, s);
    else if (per_lane <= 4) run_robust_cached<4>(a, mode, s);
    else if (per_lane <= 6) run_robust_cached<6>(a, mode, s);
    else if (per_lane <= 9) run_robust_cached<9>(a, mode, s);
    else if (per_lane <= 12) run_robust_cached<12>(a, mode, s);
    else run_robust_cached<16>(a, mode, s);
}

hipError_t launch_daq_robust(const DaqArgs &a, hipStream_t stream)
{
    if (a.R == 1) {
        run_robust_rows(a, DAQ_FUSED, stream);
        return hipGetLastError();
    }
    const int nblk = a.M / a.R;
    const unsigned parts = (unsigned)daq_hist_parts(a.K, a.R);
    if (parts <= DAQ_HIST_FEW && a.scratch_bytes >= daq_hist_bytes(a.M, a.K, a.R)) {
        // few parts: every consumer adds them up and selects for itself; more: a selection launch in between (M = 8192, R = 256, K =
        // 4608, 72 parts: 57 us against 77 with twice the part size and no selection launches)
        const bool self = parts <= DAQ_HIST_SELF;
        // rows of one workgroup in one block, and a row kernel that holds the row in registers
        const bool self_rows = self && a.R % 4 == 0 && a.K % 8 == 0 && a.K <= 8192 && (uintptr_t)a.x % 16 == 0 && (uintptr_t)a.q % 8 == 0;
        DaqArgs q = a;
        q.quant_parts = self_rows ? (int)parts : 0;
        for (int level = 0; level < 2; ++level) {
            run_hist<true>(a, parts, level, stream);
            if (level == 0 ? !self : !self_rows) hipLaunchKernelGGL(daq_part_select, dim3(nblk), dim3(1024), 0, stream, a, (int)parts, level);
        }
        run_robust_rows(q, DAQ_QUANT, stream);
        return hipGetLastError();
    }
    const size_t words = (size_t)nblk * DAQ_ROBUST_WORDS;
    hipLaunchKernelGGL(fill_zero_u32, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, a.hist, words);
    for (int level = 0; level < 2; ++level) {
        run_hist<false>(a, parts, level, stream);
        hipLaunchKernelGGL(daq_hist_select, dim3(nblk), dim3(64), 0, stream, a, level);
    }
    run_robust_rows(a, DAQ_QUANT, stream);
    return hipGetLastError();
}

// The same passes over several layers (daq_many_takes): a pass selects for itself where every layer's would.  us against a launch per layer and pass, block
// of four layers of width 1152 with its GEMMs, M = 8192, R = 256: 348 -> 330.
hipError_t launch_daq_robust_many(DaqMany &b, hipStream_t stream)
{
    const int M = b.l[0].M, R = b.l[0].R, nblk = M / R;
    b.row_blocks = (M + 3) / 4;
    if (R == 1) {
        run_robust_rows_many<false>(b, DAQ_FUSED, stream);
        return hipGetLastError();
    }
    bool self = true;
    unsigned grid = 0;
    for (int i = 0; i < b.count; ++i) {
        b.l[i].quant_parts = (int)daq_hist_parts(b.l[i].K, R);
        self = self && b.l[i].quant_parts <= (int)DAQ_HIST_SELF;
        b.first[i] = grid;
        grid += (unsigned)b.l[i].quant_parts * (unsigned)nblk;
    }
    for (int i = b.count; i < PLAN_WINDOW; ++i) b.first[i] = ~0u;
    const bool self_rows = self && R % 4 == 0;
    for (int level = 0; level < 2; ++level) {
        if (self) run_hist_many<true>(b, grid, level, stream);
        else run_hist_many<false>(b, grid, level, stream);
        if (level == 0 ? !self : !self_rows) hipLaunchKernelGGL(daq_part_select_many, dim3((unsigned)(nblk * b.count)), dim3(1024), 0, stream, b, level);
    }
    if (self_rows) run_robust_rows_many<true>(b, DAQ_QUANT, stream);
    else run_robust_rows_many<false>(b, DAQ_QUANT, stream);
    return hipGetLastError();
}

}  // namespace ql
