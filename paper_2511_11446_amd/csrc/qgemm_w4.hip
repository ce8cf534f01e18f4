// INT8 x INT4 -> INT32 GEMM with group-wise weight scales for gfx950 (CDNA4): the 4-bit layers of the bit plan
// (Step 2: integer weights with one scale per group of input channels; Algorithm 2 Phase B runs them with 8-bit
// dynamic activations).
//
//   P[m,g,n] = sum_{k in group g} q[m,k] * w4[n,k]              v_mfma_i32_32x32x32_i8, nibbles fed as value * 16
//   f        = fma(float(P[m,g,n]), s_w[n,g], f)                 g ascending, fp32
//   y[m,n]   = fp16(fma(f, alpha[m/R], bias[n]))
//
// A workgroup owns a 128x128 (4 wavefronts) or 256x128 (8 wavefronts) tile; every wavefront a 64x64 block of it as
// 2x2 MFMA tiles.  Both operands go global -> LDS by DMA (global_load_lds_dwordx4) through rings of their own: one
// K step is 128 k = 128 bytes per activation row and 64 bytes per packed weight row.  The launch is persistent: as
// many workgroups as the chip holds walk their XCD's tiles, and the first K step of the next tile is requested before
// the epilogue of the current one.
//
// The per-group work is what bounds this kernel: 16 conversions and 16 multiply-adds per 32x32 tile and group on the
// vector ALU against group/32 MFMAs on the matrix cores.  It is placed where the matrix cores stay busy: the partial
// sums of tile (i,j) are folded right before that tile's first MFMA of the next group, which then starts from a zero
// C operand (no clearing pass), while the MFMAs of the other tiles and of the SIMD's second wavefront execute.  The
// nibble unpacking (6 ALU operations per 16-byte operand) is done once per pair of MFMAs, directly before them, on
// words that were read from LDS one quarter of a K step earlier.
#include "qgemm_w4.h"

namespace ql {

template <class T, int QGF, bool EXPORT, bool GLUE, Channel CHANNEL>
__global__ __launch_bounds__(T::NT, T::WPS) void qgemm_w4(GemmArgs a, int tiles_m, int tiles_n, int nblk_padded, int group_m)
{
    qgemm_w4_tiles<T, QGF, EXPORT, GLUE, CHANNEL>(a, blockIdx.x, gridDim.x, tiles_m, tiles_n, nblk_padded, group_m);
}

template <class T, int QGF, bool EXPORT, bool GLUE, Channel CHANNEL>
static hipError_t run_w4(const GemmArgs &a, hipStream_t s)
{
    static const hipError_t lds_opt_in = hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_w4<T, QGF, EXPORT, GLUE, CHANNEL>),
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    if (lds_opt_in != hipSuccess) return lds_opt_in;
    const int tiles_m = (a.M + T::BM - 1) / T::BM, tiles_n = (a.N + T::BN - 1) / T::BN;
    const int nblk = tiles_m * tiles_n;
    const int padded = (nblk + XCDS - 1) / XCDS * XCDS;
    // as many workgroups as the chip holds at once (LDS decides), a multiple of the XCD count
    static const int resident = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < XCDS)
            return 0;
        const int per_cu = 160 * 1024 / T::LDS_BYTES > 0 ? 160 * 1024 / T::LDS_BYTES : 1;
        return cus / XCDS * XCDS * per_cu;
    }();
    if (resident <= 0) return hipErrorInvalidDevice;
    const int grid = padded < resident ? padded : resident;
    hipLaunchKernelGGL((qgemm_w4<T, QGF, EXPORT, GLUE, CHANNEL>), dim3(grid), dim3(T::NT), T::LDS_BYTES, s, a, tiles_m, tiles_n, padded,
                       pick_group_m(T::BM));
    return hipGetLastError();
}

// more than 40 groups (K = 4608 with groups of 32 or 64): a table of up to 144 groups
constexpr int W4_MANY_GROUPS = 144;

bool qgemm_w4_takes(const GemmArgs &a)
{
    if (a.K % 128 != 0 || a.group % 32 != 0 || a.K % a.group != 0 || (uintptr_t)a.q % 16 != 0 || (uintptr_t)a.w % 16 != 0) return false;
    if (a.s_ag && (a.R % 64 != 0 || a.M % a.R != 0)) return false;   // channel-group activation scales: tiles inside one scale block
    return a.w_grouped ? a.w_bits == 8 && a.K / a.group <= W4_MANY_GROUPS : a.w_bits == 4 && a.K / a.group <= W4_MANY_GROUPS;
}

// the group set of Algorithm 1 (32, 64, 128, 192, 288) with the restart pattern unrolled, when K holds whole periods of it
template <class T, bool MANY, Channel CHANNEL>
static hipError_t run_w4_group(const GemmArgs &a, hipStream_t stream)
{
    const int nk = a.K / 128;
    if (a.group == 32) return run_w4<T, 1, false, false, CHANNEL>(a, stream);
    if (a.group == 64) return run_w4<T, 2, false, false, CHANNEL>(a, stream);
    if constexpr (!MANY) {                                       // larger groups number more than 40 only beyond K = 5120
        if (a.group == 128) return run_w4<T, 4, false, false, CHANNEL>(a, stream);
        if (a.group == 192 && nk % 3 == 0) return run_w4<T, 6, false, false, CHANNEL>(a, stream);
        if (a.group == 288 && nk % 9 == 0) return run_w4<T, 9, false, false, CHANNEL>(a, stream);
    }
    return run_w4<T, 0, false, false, CHANNEL>(a, stream);
}

template <int T, bool B8, bool MANY>
static hipError_t run_w4_tile(const GemmArgs &a, hipStream_t stream)
{
    // int8 codes on 128x128 tiles: a third activation stage would leave one workgroup per CU
    using TT = TileW4<2, B8 && T == 2 ? 2 : 3, 2, B8, MANY ? W4_MANY_GROUPS : 40, T>;
    const bool glue = a.act != 0 || a.residual != nullptr || a.gate != nullptr || a.row_absmax != nullptr;
    if (a.acc_out) return run_w4<TT, 0, true, !B8, Channel::ask>(a, stream);   // verification: group partial sums exported
    if constexpr (B8) {
        if (glue) return hipErrorInvalidValue;                                 // no call asks for glue on int8-held codes
    } else {
        if (glue) return a.group == 128 ? run_w4<TT, 4, false, true, Channel::no>(a, stream) : run_w4<TT, 0, false, true, Channel::no>(a, stream);
    }
    if (a.s_ag) return run_w4_group<TT, MANY, Channel::yes>(a, stream);
    // int8 codes without them on 128x128 tiles keep the question: where it is left out the compiler spills 18 registers instead of 8 with groups of 32
    // (7 % slower in the mean of 18 shapes) and 8 instead of 2 with groups of 64 (1.5 %); on 64x64 tiles leaving it out gains 1 to 3 %
    return run_w4_group<TT, MANY, B8 && T == 2 ? Channel::ask : Channel::no>(a, stream);
}

template <int T>
static hipError_t launch_w4_tile(const GemmArgs &a, hipStream_t stream)
{
    const bool many = a.K / a.group > 40;
    if (a.w_grouped) return many ? run_w4_tile<T, true, true>(a, stream) : run_w4_tile<T, true, false>(a, stream);
    return many ? run_w4_tile<T, false, true>(a, stream) : run_w4_tile<T, false, false>(a, stream);
}

hipError_t launch_qgemm_w4_64(const GemmArgs &a, hipStream_t stream) { return launch_w4_tile<1>(a, stream); }
hipError_t launch_qgemm_w4_128(const GemmArgs &a, hipStream_t stream)
{
    return a.s_ag && a.R % 128 != 0 ? launch_w4_tile<1>(a, stream) : launch_w4_tile<2>(a, stream);
}

// Group-scaled codes and channel-group activation scales (packed 4-bit layers without those choose by cost, in launch_qgemm): 64x64 tiles
// (32x32 per wavefront; four workgroups per CU, three with int8 codes or more than 40 groups) or 128x128 (64x64 per wavefront; two, one
// with more than 40 groups).  The small tiles hide the folds and the hand-overs behind more wavefronts but move twice the operand
// bytes.  The line was drawn on packed 4-bit layers: 64x64 up to 1024 tiles, up to about twice as many where K is short, and wherever more
// than 40 groups leave the large tiles one workgroup per CU.  M = 2048, K = 4608, N = 1152, group 128: 28 against 34 us; M = 8192: 80
// against 74; group 32: 134 against 198.
// Int8 codes leave three small workgroups per CU instead of four: where those take more than two rounds (of 768) and the large tiles one (of
// 512), the large ones.  Over the 13 such (M, N) of 1280 to 8192 rows and 640 to 4608 columns, eight K from 256 to 1536 and groups of 32 and 128, layers without
// channel scales take 0.82 to 0.93 of their time on 64x64 tiles in the mean, at most 0.98 (K = 1152, M = 2048, N = 3456 29.0 -> 24.1 us).  Two rounds against
// one and three against two are level: K = 1152, M = 4096, N = 1152 26.6 -> 25.7, but groups of 32 33.5 -> 37.0; M = 2048, N = 4608 34.0 -> 34.5.
hipError_t launch_qgemm_w4(const GemmArgs &a, hipStream_t stream)
{
    const long long tiles = (long long)((a.M + 63) / 64) * ((a.N + 63) / 64);
    const long long large_tiles = (long long)((a.M + 127) / 128) * ((a.N + 127) / 128);
    const bool one_round = a.w_grouped && tiles > 2 * 768 && large_tiles <= 512;
    const bool small = a.K / a.group > 40 || tiles <= 1024 || (a.K <= 1536 && tiles <= 2304 && !one_round);
    return small ? launch_qgemm_w4_64(a, stream) : launch_qgemm_w4_128(a, stream);
}

// Pair order (byte i of a row: k = 2i low nibble, k = 2i+1 high nibble) -> the storage order unpack_w4 reads (byte j of a
// 4-byte block: k = 8b+j low, k = 8b+4+j high).  One thread per 4-byte block; `blocks` = N*K/8.
__global__ __launch_bounds__(256) void prepack_w4_pairs(const unsigned *__restrict__ pairs, unsigned *__restrict__ packed, long long blocks)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= blocks) return;
    const unsigned s = pairs[i];                       // nibble t (bits 4t..4t+3) holds k = 8b+t
    unsigned d = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) d |= (((s >> (4 * j)) & 0xfu) | (((s >> (4 * (4 + j))) & 0xfu) << 4)) << (8 * j);
    packed[i] = d;
}

hipError_t launch_prepack_w4(const void *pairs, void *packed, long long blocks, hipStream_t stream)
{
    hipLaunchKernelGGL(prepack_w4_pairs, dim3((unsigned)((blocks + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const unsigned *>(pairs), static_cast<unsigned *>(packed), blocks);
    return hipGetLastError();
}

}  // namespace ql
