// Dynamic activation quantization kernels for gfx950 (wave64).
//
// Step 3, eq. (4) of the paper with tau = the absolute maximum of the scale
// block: alpha = amax / 127 (1 for an all-zero block),
// code = clamp(round_half_even(x / alpha), -127, 127).
//
// One wavefront owns one or a few rows.  A row is read once with 16-byte loads and
// kept in registers (2 bytes in, 1 byte out per element is all the HBM traffic
// of the per-token mode).  The absolute maximum is taken on the fp16 bit
// patterns: for non-negative binary16 numbers the integer order of the
// patterns is the numeric order, so a packed 16-bit integer max is exact.
#include "daq_device.h"

namespace ql {

__device__ __forceinline__ void publish_block_max(unsigned *slot, unsigned bits)
{
    // most rows lose against an earlier, larger maximum: look before the atomic
    if (__hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < bits) atomicMax(slot, bits);
}

// Second pass of the modes with several rows per scale: the maximum of scale block b, either reduced already
// (blockmax) or, when the block has few parts, taken here from its partial maxima (saves a launch)
__device__ __forceinline__ unsigned block_max_bits(const DaqArgs &a, int b, int lane)
{
    if (a.quant_parts <= 0) return a.blockmax[b];
    const unsigned *pm = a.partmax + (size_t)b * a.quant_parts;
    unsigned m = 0;
    for (int i = lane; i < a.quant_parts; i += 64) {
        const unsigned o = pm[i];
        m = m > o ? m : o;
    }
    return wave_max_u32(m);
}

constexpr int ROWS_PER_BLOCK = 4;  // 4 wavefronts, one row each (loop kernels)

// Rows held in registers: CH 16-byte chunks per lane and row (K/8 <= 64*CH), RW rows per wavefront (all loads of the
// RW rows are issued before the first reduction).  The dispatcher uses RW = 1: see run_rows().
template <int CH, int RW>
__global__ __launch_bounds__(256) void daq_rows_cached(DaqArgs a, int mode)
{
    const int lane = threadIdx.x & 63;
    // the second pass of the two-pass modes walks the rows backwards: the rows read last by the first pass are
    // the ones most likely still in cache
    const int wg = mode == DAQ_QUANT ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x;
    const int row0 = (wg * 4 + (threadIdx.x >> 6)) * RW;
    if (row0 >= a.M) return;
    const int nch = a.K >> 3;
    uint4 v[RW][CH];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int row = min(row0 + r, a.M - 1);
        const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(a.x) + (size_t)row * a.K);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = lane + 64 * i;
            v[r][i] = c < nch ? xr[c] : make_uint4(0, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int row = row0 + r;
        if (row >= a.M) break;
        unsigned bits;
        if (mode != DAQ_QUANT) {
            unsigned m = 0;
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                m = absmax_word(m, v[r][i].x);
                m = absmax_word(m, v[r][i].y);
                m = absmax_word(m, v[r][i].z);
                m = absmax_word(m, v[r][i].w);
            }
            m = (m & 0xffffu) > (m >> 16) ? (m & 0xffffu) : (m >> 16);
            bits = wave_max_u32(m);
            if (mode == DAQ_ABSMAX) {
                if (lane == 0) publish_block_max(a.blockmax + row / a.R, bits);
                continue;
            }
        } else {
            bits = block_max_bits(a, row / a.R, lane);
        }
        const float alpha = alpha_from_bits(bits);
        const float rcp = 1.0f / alpha;
        if (lane == 0 && (row % a.R) == 0) a.scales[row / a.R] = alpha;
        uint2 *qr = reinterpret_cast<uint2 *>(a.q + (size_t)row * a.K);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int c = lane + 64 * i;
            if (c < nch) qr[c] = daq_piece(v[r][i], alpha, rcp);
        }
    }
}

// DAQ of several layers with as many rows each in one launch (a plan whose next inputs are there already): workgroup ids run
// through the layers, a wavefront takes one row as above.  At M = 2048 a launch of K = 1152 is mostly fill and drain: one
// HBM round trip, one reduction, one store.  Three layers of K = 1152 in one launch instead of three, us per block of four layers: M =
// 2048 80.6 -> 73.3, M = 8192 (4-bit MLP) 242 -> 231, M = 16384 357 -> 350.
template <int CH, bool QUANT>
__device__ __forceinline__ void daq_one_row(const DaqArgs &l, int row, int lane)
{
    const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(l.x) + (size_t)row * l.K);
    const int nch = l.K >> 3;
    uint4 v[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) v[i] = lane + 64 * i < nch ? xr[lane + 64 * i] : make_uint4(0, 0, 0, 0);
    unsigned bits;
    if (QUANT) {
        bits = block_max_bits(l, row / l.R, lane);
    } else {
        unsigned m = 0;
#pragma unroll
        for (int i = 0; i < CH; ++i) m = absmax_word(absmax_word(absmax_word(absmax_word(m, v[i].x), v[i].y), v[i].z), v[i].w);
        bits = wave_max_u32((m & 0xffffu) > (m >> 16) ? (m & 0xffffu) : (m >> 16));
    }
    const float alpha = alpha_from_bits(bits);
    const float rcp = 1.0f / alpha;
    if (!QUANT && lane == 0) l.scales[row] = alpha;
    if (QUANT && lane == 0 && row % l.R == 0) l.scales[row / l.R] = alpha;
    uint2 *qr = reinterpret_cast<uint2 *>(l.q + (size_t)row * l.K);
#pragma unroll
    for (int i = 0; i < CH; ++i)
        if (lane + 64 * i < nch) qr[lane + 64 * i] = daq_piece(v[i], alpha, rcp);
}

// QUANT: several rows per scale, second pass, from the end as above
template <bool QUANT>
__global__ __launch_bounds__(256) void daq_rows_many(DaqMany b)
{
    const int wg = QUANT ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x;
    const int layer = wg / b.row_blocks, lane = threadIdx.x & 63;
    const DaqArgs &l = b.l[layer];
    const int row = (wg - layer * b.row_blocks) * 4 + (threadIdx.x >> 6);
    if (row >= l.M) return;
    if (l.K <= 1024) daq_one_row<2, QUANT>(l, row, lane);
    else if (l.K <= 1536) daq_one_row<3, QUANT>(l, row, lane);
    else if (l.K <= 3072) daq_one_row<6, QUANT>(l, row, lane);
    else daq_one_row<9, QUANT>(l, row, lane);
}

// Long rows, few of them: the four wavefronts of a workgroup share one, CH pieces per thread, so that four times as many loads are in
// flight (a row of 4608 per wavefront leaves two wavefronts per SIMD at M = 2048).
template <int CH>
__global__ __launch_bounds__(256) void daq_rows_wide(DaqArgs a)
{
    __shared__ unsigned wave_max[4];
    const int nch = a.K >> 3;
    const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(a.x) + (size_t)blockIdx.x * a.K);
    uint4 v[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int c = threadIdx.x + 256 * i;
        v[i] = c < nch ? xr[c] : make_uint4(0, 0, 0, 0);
    }
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < CH; ++i) m = absmax_word(absmax_word(absmax_word(absmax_word(m, v[i].x), v[i].y), v[i].z), v[i].w);
    m = wave_max_u32((m & 0xffffu) > (m >> 16) ? (m & 0xffffu) : (m >> 16));
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    const unsigned m01 = wave_max[0] > wave_max[1] ? wave_max[0] : wave_max[1];
    const unsigned m23 = wave_max[2] > wave_max[3] ? wave_max[2] : wave_max[3];
    const float alpha = alpha_from_bits(m01 > m23 ? m01 : m23);
    const float rcp = 1.0f / alpha;
    if (threadIdx.x == 0) a.scales[blockIdx.x] = alpha;
    uint2 *qr = reinterpret_cast<uint2 *>(a.q + (size_t)blockIdx.x * a.K);
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int c = threadIdx.x + 256 * i;
        if (c < nch) qr[c] = daq_piece(v[i], alpha, rcp);
    }
}

// Any row length: the row is read twice (the second read normally hits L2).
// VEC = 8: 16-byte loads (K % 8 == 0, aligned); VEC = 1: element-wise, no alignment needs.
template <int VEC>
__global__ __launch_bounds__(256) void daq_rows_loop(DaqArgs a, int mode)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * ROWS_PER_BLOCK + (threadIdx.x >> 6);
    if (row >= a.M) return;
    const unsigned short *xs = static_cast<const unsigned short *>(a.x) + (size_t)row * a.K;
    const int nch = a.K / VEC;
    unsigned bits;
    if (mode != DAQ_QUANT) {
        unsigned m = 0;
        for (int c = lane; c < nch; c += 64) {
            if (VEC == 8) {
                uint4 v = reinterpret_cast<const uint4 *>(xs)[c];
                m = absmax_word(m, v.x);
                m = absmax_word(m, v.y);
                m = absmax_word(m, v.z);
                m = absmax_word(m, v.w);
            } else {
                m = absmax_word(m, xs[c]);
            }
        }
        m = (m & 0xffffu) > (m >> 16) ? (m & 0xffffu) : (m >> 16);
        bits = wave_max_u32(m);
        if (mode == DAQ_ABSMAX) {
            if (lane == 0) publish_block_max(a.blockmax + row / a.R, bits);
            return;
        }
    } else {
        bits = block_max_bits(a, row / a.R, lane);
    }
    const float alpha = alpha_from_bits(bits);
    const float rcp = 1.0f / alpha;
    if (lane == 0 && (row % a.R) == 0) a.scales[row / a.R] = alpha;
    int8_t *qs = a.q + (size_t)row * a.K;
    for (int c = lane; c < nch; c += 64) {
        if (VEC == 8) {
            uint4 v = reinterpret_cast<const uint4 *>(xs)[c];
            reinterpret_cast<uint2 *>(qs)[c] = daq_piece(v, alpha, rcp);
        } else {
            qs[c] = (int8_t)daq_code(half_bits_to_float(xs[c]), alpha);
        }
    }
}

// First pass of the modes with several rows per scale: a scale block is one contiguous run of R*K values, cut into
// parts of DAQ_PART_PIECES 16-byte pieces; one workgroup per part leaves the part's maximum in partmax (plain stores:
// thousands of atomics on a few neighbouring words cost more than the whole pass).
constexpr int ABSMAX_U = DAQ_PART_PIECES / 256;
__device__ __forceinline__ void part_absmax(unsigned block, const uint4 *x, unsigned pieces_per_block, unsigned parts_per_block,
                                            unsigned *partmax)
{
    __shared__ unsigned wave_max[4];
    const unsigned b = block / parts_per_block, part = block - b * parts_per_block;
    const uint4 *xb = x + (size_t)b * pieces_per_block;
    const unsigned c0 = part * DAQ_PART_PIECES + threadIdx.x;
    uint4 v[ABSMAX_U];
#pragma unroll
    for (int i = 0; i < ABSMAX_U; ++i) {
        const unsigned c = c0 + 256 * i;
        v[i] = c < pieces_per_block ? xb[c] : make_uint4(0, 0, 0, 0);
    }
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < ABSMAX_U; ++i) {
        m = absmax_word(m, v[i].x);
        m = absmax_word(m, v[i].y);
        m = absmax_word(m, v[i].z);
        m = absmax_word(m, v[i].w);
    }
    m = (m & 0xffffu) > (m >> 16) ? (m & 0xffffu) : (m >> 16);
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned m01 = wave_max[0] > wave_max[1] ? wave_max[0] : wave_max[1];
        const unsigned m23 = wave_max[2] > wave_max[3] ? wave_max[2] : wave_max[3];
        partmax[block] = m01 > m23 ? m01 : m23;
    }
}

__global__ __launch_bounds__(256) void daq_part_absmax(const uint4 *x, unsigned pieces_per_block, unsigned parts_per_block, unsigned *partmax)
{
    part_absmax(blockIdx.x, x, pieces_per_block, parts_per_block, partmax);
}

__global__ __launch_bounds__(256) void daq_part_absmax_many(DaqMany b)
{
    const int i = many_layer(b, blockIdx.x);
    const DaqArgs &l = b.l[i];
    part_absmax(blockIdx.x - b.first[i], static_cast<const uint4 *>(l.x), (unsigned)l.R * (unsigned)(l.K >> 3), (unsigned)l.quant_parts, l.partmax);
}

// one workgroup per scale block: maximum of its partial maxima
__global__ __launch_bounds__(256) void daq_reduce_parts(const unsigned *partmax, unsigned parts_per_block, unsigned *blockmax)
{
    __shared__ unsigned wave_max[4];
    const unsigned *pm = partmax + (size_t)blockIdx.x * parts_per_block;
    unsigned m = 0;
    for (unsigned i = threadIdx.x; i < parts_per_block; i += 256) {
        const unsigned o = pm[i];
        m = m > o ? m : o;
    }
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned m01 = wave_max[0] > wave_max[1] ? wave_max[0] : wave_max[1];
        const unsigned m23 = wave_max[2] > wave_max[3] ? wave_max[2] : wave_max[3];
        blockmax[blockIdx.x] = m01 > m23 ? m01 : m23;
    }
}

__global__ void fill_u32(unsigned *p, int n, unsigned v)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

template <int CH, int RW>
static void run_cached(const DaqArgs &a, int mode, hipStream_t s)
{
    dim3 grid((a.M + 4 * RW - 1) / (4 * RW));
    hipLaunchKernelGGL((daq_rows_cached<CH, RW>), grid, dim3(256), 0, s, a, mode);
}

static void run_rows(const DaqArgs &a, int mode, hipStream_t s)
{
    dim3 grid((a.M + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK);
    const bool vec = (a.K % 8 == 0) && ((uintptr_t)a.x % 16 == 0) && ((uintptr_t)a.q % 8 == 0);
    if (!vec) {
        hipLaunchKernelGGL(daq_rows_loop<1>, grid, dim3(256), 0, s, a, mode);
        return;
    }
    // one row per wavefront at every size: with the division-free codes the kernel is no longer VALU-bound, and more,
    // shorter wavefronts beat several rows per wavefront (measured 4.5 against 3.4 TB/s at M = 16384, K = 1152)
    const int per_lane = (a.K / 8 + 63) / 64;
    // us, a wavefront per row -> a workgroup per row: K = 4608: M = 64 4.7 -> 3.2, 1024 7.8 -> 5.6, 4096 14.0 -> 11.2, 16384 39.0 -> 35.9;
    // K = 2304: 64 3.8 -> 2.8, 8192 13.4 -> 11.6, but 16384 21.0 -> 21.5
    if (mode == DAQ_FUSED && per_lane > 4 && per_lane <= 16 && (a.M <= 8192 || per_lane > 5)) {
        if (per_lane <= 8) hipLaunchKernelGGL(daq_rows_wide<2>, dim3(a.M), dim3(256), 0, s, a);
        else if (per_lane <= 12) hipLaunchKernelGGL(daq_rows_wide<3>, dim3(a.M), dim3(256), 0, s, a);
        else hipLaunchKernelGGL(daq_rows_wide<4>, dim3(a.M), dim3(256), 0, s, a);
        return;
    }
    if (per_lane <= 1) run_cached<1, 1>(a, mode, s);
    else if (per_lane <= 2) run_cached<2, 1>(a, mode, s);
    else if (per_lane <= 3) run_cached<3, 1>(a, mode, s);
    else if (per_lane <= 4) run_cached<4, 1>(a, mode, s);
    else if (per_lane <= 6) run_cached<6, 1>(a, mode, s);
    else if (per_lane <= 9) run_cached<9, 1>(a, mode, s);
    else if (per_lane <= 12) run_cached<12, 1>(a, mode, s);
    else if (per_lane <= 16) run_cached<16, 1>(a, mode, s);
    else hipLaunchKernelGGL(daq_rows_loop<8>, grid, dim3(256), 0, s, a, mode);
}

// ---- eq. (4) with its channel groups: one scale per block of R rows AND group of `cg` consecutive channels ------------
// pass 1: every wavefront takes one row; a lane's 16-byte piece lies inside one channel group (cg % 8 == 0), its maximum
// goes to the wavefront's LDS table and from there, once per row and group, to blockmax[block][group]
constexpr int DAQ_CG_MAX_GROUPS = 1024;
__global__ __launch_bounds__(256) void daq_cg_absmax(DaqArgs a, int cg)
{
    __shared__ unsigned gmax[4][DAQ_CG_MAX_GROUPS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = blockIdx.x * 4 + wave;
    const int G = a.K / cg, nch = a.K >> 3;
    for (int g = lane; g < G; g += 64) gmax[wave][g] = 0;
    __builtin_amdgcn_wave_barrier();
    if (row < a.M) {
        const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(a.x) + (size_t)row * a.K);
        for (int c = lane; c < nch; c += 64) {
            const uint4 v = xr[c];
            unsigned m = absmax_word(absmax_word(absmax_word(absmax_word(0, v.x), v.y), v.z), v.w);
            m = (m & 0xffffu) > (m >> 16) ? (m & 0xffffu) : (m >> 16);
            atomicMax(&gmax[wave][(c * 8) / cg], m);
        }
    }
    __syncthreads();
    if (row < a.M)
        for (int g = lane; g < G; g += 64) publish_block_max(a.blockmax + (size_t)(row / a.R) * G + g, gmax[wave][g]);
}

// pass 2: codes from the block maxima; the row is read again (the first read normally left it in L2)
__global__ __launch_bounds__(256) void daq_cg_quant(DaqArgs a, int cg)
{
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= a.M) return;
    const int G = a.K / cg, nch = a.K >> 3;
    const unsigned *bm = a.blockmax + (size_t)(row / a.R) * G;
    const uint4 *xr = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(a.x) + (size_t)row * a.K);
    uint2 *qr = reinterpret_cast<uint2 *>(a.q + (size_t)row * a.K);
    for (int c = lane; c < nch; c += 64) {
        const float alpha = alpha_from_bits(bm[(c * 8) / cg]);
        qr[c] = daq_piece(xr[c], alpha, 1.0f / alpha);
    }
    if (row % a.R == 0)
        for (int g = lane; g < G; g += 64) a.scales[(size_t)(row / a.R) * G + g] = alpha_from_bits(bm[g]);
}

// The same for blocks of rows that 8 divides (daq_cg_slab_rows).  A workgroup takes a slab of rows; a thread keeps one 16-byte piece of
// columns (hence one channel group) and walks down every rpw-th of the slab's rows, so that the group arithmetic - a division
// by cg, the scale and its reciprocal - is paid once per thread and not per piece.  Pass 1 leaves the slab's maximum per
// group with plain stores, no clearing pass and no atomics; pass 2 takes the maximum over its block's slabs.
// M = 4096, K = 1152, R = 256, cg = 128: 32.7 -> 13 us.
// rows in flight per thread (six, a whole slab of 16 for three rows side by side, were not faster, and 3 % slower at K = 3072 from 64 slabs on)
constexpr int DAQ_CG_ROWS = 4;
// Slabs per scale block up to which every thread takes the maximum of its group over them by itself; beyond that the workgroup does it
// together (both passes, cg = 128, M = R = 16384, 1024 slabs: K = 1152 131 -> 22 us, K = 4608 404 -> 91, where the atomic kernels take
// 79 and 185; M = 4096, R = 1024, K = 1152: 15.5 -> 8.4)
constexpr int DAQ_CG_OWN = 16;
template <bool QUANT>
__global__ __launch_bounds__(1024) void daq_cg_slab(DaqArgs a, int cg, int slab, int slabs, int rpw)
{
    extern __shared__ unsigned gmax_lds[];
    const int P = a.K >> 3, G = a.K / cg;
    const int p = threadIdx.x % P, r0 = threadIdx.x / P, g = p * 8 / cg;
    const bool on = r0 < rpw;
    const int row0 = blockIdx.x * slab;
    unsigned *part = a.blockmax;          // [M / slab][G]
    float alpha = 1.0f, rcp = 1.0f;
    if (!QUANT || slabs > DAQ_CG_OWN) {
        for (int i = threadIdx.x; i < G; i += blockDim.x) gmax_lds[i] = 0;
        __syncthreads();
    }
    const uint4 *x = reinterpret_cast<const uint4 *>(a.x) + (size_t)row0 * P + p;
    uint4 v[DAQ_CG_ROWS];
    auto load = [&](int r) {
#pragma unroll
        for (int u = 0; u < DAQ_CG_ROWS; ++u) v[u] = on && r + u * rpw < slab ? x[(size_t)(r + u * rpw) * P] : make_uint4(0, 0, 0, 0);
    };
    if (!QUANT || slabs <= DAQ_CG_OWN) load(r0);
    if (QUANT) {
        const unsigned *pm = part + (size_t)(row0 / a.R) * slabs * G;
        unsigned m = 0;
        if (slabs > DAQ_CG_OWN) {
            for (int i = threadIdx.x; i < slabs * G; i += blockDim.x) atomicMax(&gmax_lds[i % G], pm[i]);
            __syncthreads();
            if (on) m = gmax_lds[g];
        } else if (on && slabs == 1) {
            m = pm[g];
        } else if (on) {
            // all requested at once: in a loop each one waited for the one before (M = 1024, R = 256, K = 1152: 9.3 -> 6.9 us)
            unsigned o[DAQ_CG_OWN];
#pragma unroll
            for (int s = 0; s < DAQ_CG_OWN; ++s) o[s] = pm[(s < slabs ? s : 0) * G + g];
#pragma unroll
            for (int s = 0; s < DAQ_CG_OWN; ++s) m = m > o[s] ? m : o[s];
        }
        if (on) {
            alpha = alpha_from_bits(m);
            rcp = 1.0f / alpha;
            if (row0 % a.R == 0 && r0 == 0 && p * 8 % cg == 0) a.scales[(size_t)(row0 / a.R) * G + g] = alpha;
        }
    }
    if (on) {
        uint2 *q = reinterpret_cast<uint2 *>(a.q) + (size_t)row0 * P + p;
        unsigned m = 0;
        for (int r = r0; r < slab; r += rpw * DAQ_CG_ROWS) {
            if (r != r0 || (QUANT && slabs > DAQ_CG_OWN)) load(r);
#pragma unroll
            for (int u = 0; u < DAQ_CG_ROWS; ++u) {
                if (QUANT) {
                    if (r + u * rpw < slab) q[(size_t)(r + u * rpw) * P] = daq_piece(v[u], alpha, rcp);
                } else {
                    m = absmax_word(absmax_word(absmax_word(absmax_word(m, v[u].x), v[u].y), v[u].z), v[u].w);
                }
            }
        }
        if (!QUANT) atomicMax(&gmax_lds[g], (m & 0xffffu) > (m >> 16) ? (m & 0xffffu) : (m >> 16));
    }
    if (!QUANT) {
        __syncthreads();
        for (int i = threadIdx.x; i < G; i += blockDim.x) part[(size_t)blockIdx.x * G + i] = gmax_lds[i];
    }
}

hipError_t launch_daq_cg(const DaqArgs &a, int cg, bool slabs, hipStream_t stream)
{
    const int slab = slabs ? daq_cg_slab_rows(a.R) : 0, P = a.K / 8, G = a.K / cg;
    // few wide rows in short blocks make a few large workgroups and nothing to merge: the kernels with a wavefront per row
    // (K = 4608, R = 16, 512 rows: 12 against 15.5 us; from 4096 rows on they are level)
    const bool few = P > 512 && a.R <= 64 && a.M <= 2048;
    if (slab > 0 && P <= 1024 && !few) {
        // rows walked side by side: half a workgroup's threads where rows are short, all of them where one row at a time would leave a
        // chain of four trips to memory (M = 512, R = 64, K = 3072: 14.5 -> 11.3 us; all threads at M = 16384, R = 64, K = 384: 10.0 -> 12.6)
        const int rpw = P > 512 ? 1 : P > 256 ? 1024 / P : 512 / P;
        const dim3 grid(a.M / slab), block((P * rpw + 63) / 64 * 64);
        hipLaunchKernelGGL(daq_cg_slab<false>, grid, block, G * 4, stream, a, cg, slab, a.R / slab, rpw);
        // The codes are written by workgroups of 8 rows where those of 16 make at most 8 wavefronts per CU, or walk row by row.  They merge few
        // slabs and have at most 4 rows side by side.  Both passes, us, workgroups of 16 -> 8: M = 2048, R = 64, K = 1152 9.0 -> 7.5, K = 3072 11.6 -> 11.1,
        // M = 4096, R = 256, K = 1152 9.3 -> 9.05, K = 4608 21.4 -> 18.9, M = 16384 72.6 -> 70.7; but M = 4096, K = 3072, R = 64 14.8 -> 15.7, M = 8192,
        // R = 256 22.6 -> 24.3, M = 16384, K = 1152 19.1 -> 20.0
        const bool few_waves = (int64_t)grid.x * (block.x / 64) <= 8 * 256;
        const int rows = a.R / slab <= DAQ_CG_OWN && rpw <= 4 && (rpw == 1 || few_waves) ? 8 : slab;
        hipLaunchKernelGGL(daq_cg_slab<true>, dim3(a.M / rows), block, G * 4, stream, a, cg, rows, a.R / slab, rpw);
        return hipGetLastError();
    }
    const int n = (a.M / a.R) * G;
    hipLaunchKernelGGL(fill_u32, dim3((n + 255) / 256), dim3(256), 0, stream, a.blockmax, n, 0u);
    hipLaunchKernelGGL(daq_cg_absmax, dim3((a.M + 3) / 4), dim3(256), 0, stream, a, cg);
    hipLaunchKernelGGL(daq_cg_quant, dim3((a.M + 3) / 4), dim3(256), 0, stream, a, cg);
    return hipGetLastError();
}

hipError_t launch_daq_part_absmax(const DaqArgs &a, hipStream_t stream)
{
    const unsigned parts = (unsigned)daq_parts_per_block(a.K, a.R);
    hipLaunchKernelGGL(daq_part_absmax, dim3(parts * (unsigned)(a.M / a.R)), dim3(256), 0, stream, static_cast<const uint4 *>(a.x),
                       (unsigned)((size_t)a.R * a.K / 8), parts, a.partmax);
    return hipGetLastError();
}

bool daq_many_takes(const DaqArgs &a, bool robust)
{
    if (a.K % 8 != 0 || a.K > 4608 || (uintptr_t)a.x % 16 != 0 || (uintptr_t)a.q % 8 != 0) return false;
    if (a.R == 1) return true;
    // Percentiles of very many blocks gain nothing: a workgroup per block, with histograms larger than its values, is what takes the time (two rows per
    // scale, us, a launch per layer and pass -> shared: M = 4096, eight layers of K = 384 129 -> 86; but 65536 rows 1742 -> 1942, M = 16384, two of K =
    // 1152 298 -> 311)
    if (robust) return a.M / a.R <= 4096 && daq_hist_parts(a.K, a.R) <= DAQ_HIST_FEW && a.scratch_bytes >= daq_hist_bytes(a.M, a.K, a.R);
    // every wavefront of the quantize pass reduces the partial maxima itself
    const size_t parts = daq_parts_per_block(a.K, a.R);
    return parts > 0 && parts <= 256 && parts * (size_t)(a.M / a.R) * 4 <= a.scratch_bytes;
}

// Several rows per scale: both passes take all layers, the maxima first.  us against a launch per layer and pass, 8-bit blocks of four layers with their
// GEMMs, R = 256: width 1152, M = 2048 94.8 -> 74.8, M = 8192 241 -> 228; width 384, M = 1024 49 -> 34.
hipError_t launch_daq_many(DaqMany &b, hipStream_t stream)
{
    const int M = b.l[0].M, R = b.l[0].R;
    b.row_blocks = (M + 3) / 4;
    const dim3 rows((unsigned)b.row_blocks * (unsigned)b.count);
    if (R == 1) {
        hipLaunchKernelGGL(daq_rows_many<false>, rows, dim3(256), 0, stream, b);
        return hipGetLastError();
    }
    unsigned grid = 0;
    for (int i = 0; i < b.count; ++i) {
        b.l[i].quant_parts = (int)daq_parts_per_block(b.l[i].K, R);
        b.first[i] = grid;
        grid += (unsigned)b.l[i].quant_parts * (unsigned)(M / R);
    }
    for (int i = b.count; i < PLAN_WINDOW; ++i) b.first[i] = ~0u;
    hipLaunchKernelGGL(daq_part_absmax_many, dim3(grid), dim3(256), 0, stream, b);
    hipLaunchKernelGGL(daq_rows_many<true>, rows, dim3(256), 0, stream, b);
    return hipGetLastError();
}

hipError_t launch_daq(const DaqArgs &a, hipStream_t stream)
{
    if (a.R == 1) {
        run_rows(a, DAQ_FUSED, stream);
    } else {
        const int nblk = a.M / a.R;
        const size_t parts = daq_parts_per_block(a.K, a.R);
        if (parts > 0 && (uintptr_t)a.x % 16 == 0 && parts * nblk < (1ull << 31) && parts * nblk * 4 <= a.scratch_bytes) {
            const hipError_t e = launch_daq_part_absmax(a, stream);
            if (e != hipSuccess) return e;
            if (parts <= 256) {
                // few parts per block: every wavefront of the quantize pass reduces them itself
                DaqArgs q = a;
                q.quant_parts = (int)parts;
                run_rows(q, DAQ_QUANT, stream);
                return hipGetLastError();
            }
            hipLaunchKernelGGL(daq_reduce_parts, dim3(nblk), dim3(256), 0, stream, a.partmax, (unsigned)parts, a.blockmax);
        } else {
            hipLaunchKernelGGL(fill_u32, dim3((nblk + 255) / 256), dim3(256), 0, stream, a.blockmax, nblk, 0u);
            run_rows(a, DAQ_ABSMAX, stream);
        }
        run_rows(a, DAQ_QUANT, stream);
    }
    return hipGetLastError();
}

hipError_t launch_fill_u32(unsigned *p, int n, unsigned v, hipStream_t stream)
{
    hipLaunchKernelGGL(fill_u32, dim3((n + 255) / 256), dim3(256), 0, stream, p, n, v);
    return hipGetLastError();
}

// The first pass is already done: the producing layer's epilogue left every row's maximum.  A block's R row maxima are
// laid out like the partial maxima of the two-pass modes, so the quantize pass reduces them itself (R <= 256) or after
// one reduction launch.
hipError_t launch_daq_from_rowmax(const DaqArgs &a, const unsigned *row_absmax, hipStream_t stream)
{
    DaqArgs q = a;
    q.partmax = const_cast<unsigned *>(row_absmax);
    if (a.R <= 256) {
        q.quant_parts = a.R;
    } else {
        hipLaunchKernelGGL(daq_reduce_parts, dim3(a.M / a.R), dim3(256), 0, stream, row_absmax, (unsigned)a.R, a.blockmax);
        q.quant_parts = 0;
    }
    run_rows(q, DAQ_QUANT, stream);
    return hipGetLastError();
}

}  // namespace ql
