// INT8 x INT8 -> INT32 GEMM with fused dequantization for gfx950 (CDNA4).
//
// The paper's linears multiply int8 codes into int32 sums, with one weight scale per
// output channel (Step 3, Step 5, Section 6) or per weight group (Step 2).
// Here: acc[m,n] = sum_k q[m,k] * w[n,k] on v_mfma_i32_32x32x32_i8, both
// operands K-contiguous, and the dequantization + bias + fp16 conversion applied
// to the accumulators in registers.  The kernel families:
//   qgemm_big, qgemm_w4_big (qgemm_big.hip, qgemm_w4_big.hip) tiles of up to 256x288: 8-bit weights and binary16 operands,
//               and packed 4-bit weights with groups of 128
//   qgemm_dma   (launched here, the tile in qgemm_dma.h) tiles of 64x64 to 256x192 go global -> LDS by DMA through rings of 2-3 stages,
//               optional persistent walk over tiles; 8-bit weights, and binary16 operands for the layers a plan leaves in FP16; two of
//               the tiles take rows of any whole number of words
//   qgemm_w4    (qgemm_w4.hip, the tile in qgemm_w4.h) group scales: packed 4-bit weights and int8 codes with group scales
//   qgemm_many  (qgemm_many.hip) 128x128 tiles of these two for several layers of a plan in one launch
//   qgemm_k64   (here) 8-bit layers of many tiles whose inner size is an odd multiple of 64
//   qgemm_splitk, qgemm_edge (qgemm_small.hip) few rows; any inner size and alignment
// plus a one-thread-per-element kernel: the tuning hooks' reference, and the last resort for channel-group activation
// scales over blocks of rows that no tile boundary meets.
// Activation, gate and residual can be folded into the epilogue (GLUE instantiations).
#include "qgemm_dma.h"

namespace ql {

template <class T, bool GLUE = false>
__global__ __launch_bounds__(T::NT, T::WPS) void qgemm_dma(GemmArgs a, int tiles_m, int tiles_n, int nblk_padded, int group_m)
{
    qgemm_dma_tiles<T, GLUE>(a, blockIdx.x, gridDim.x, tiles_m, tiles_n, nblk_padded, group_m);
}

template <class T, bool GLUE = false>
static hipError_t run_dma(const GemmArgs &a, hipStream_t s)
{
    // LDS above 64 KB needs an opt-in, once per kernel (initialised thread-safely on first use)
    static const hipError_t lds_opt_in = [] {
        if (T::LDS_BYTES <= 64 * 1024) return hipSuccess;
        return hipFuncSetAttribute(reinterpret_cast<const void *>(&qgemm_dma<T, GLUE>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    }();
    if (lds_opt_in != hipSuccess) return lds_opt_in;
    const int tiles_m = (a.M + T::BM - 1) / T::BM, tiles_n = (a.N + T::BN - 1) / T::BN;
    const int nblk = tiles_m * tiles_n;
    const int padded = (nblk + XCDS - 1) / XCDS * XCDS;
    int grid = padded;
    if (T::PERSIST) {
        // as many workgroups as the chip holds at once (LDS decides), a multiple of the XCD count
        static const int resident = [] {
            int dev = 0, cus = 0;
            if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
                cus < XCDS)
                return 0;   // no guess: the launch fails instead
            const int per_cu = 160 * 1024 / T::LDS_BYTES > 0 ? 160 * 1024 / T::LDS_BYTES : 1;
            return cus / XCDS * XCDS * per_cu;
        }();
        if (resident <= 0) return hipErrorInvalidDevice;
        if (grid > resident) grid = resident;
    }
    hipLaunchKernelGGL((qgemm_dma<T, GLUE>), dim3(grid), dim3(T::NT), T::LDS_BYTES, s, a, tiles_m, tiles_n, padded, pick_group_m(T::BM));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// 8-bit layers whose inner size is a multiple of 64 but not of 128 (the DMA kernels walk K in steps of 128 bytes): 128x128 tiles of
// 2 x 2 wavefronts, K steps of 64 staged through registers into two LDS buffers.  qgemm_edge takes any K but pads the last step of 128
// and has two workgroups per CU on such tiles; three here (M = 4096, N = 2560: K = 320 14.6 against 20.3 us, K = 2240 48 against 66).
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 3) void qgemm_k64(GemmArgs a, int tiles_m, int tiles_n, int nblk_padded, int group_m)
{
    constexpr int T = 2, B = 128, BK = 64, LD = BK + 16, BYTES = B * LD, PIECES = B * BK / 16 / 256;
    __shared__ __align__(16) unsigned char smem[4 * BYTES];
    unsigned char *sA = smem, *sB = smem + 2 * BYTES;
    const int logical = (blockIdx.x % XCDS) * (nblk_padded / XCDS) + blockIdx.x / XCDS;
    if (logical >= tiles_m * tiles_n) return;
    const int group_sz = group_m * tiles_n, first_m = (logical / group_sz) * group_m, gm = min(tiles_m - first_m, group_m);
    const int m0 = (first_m + (logical % group_sz) % gm) * B, n0 = ((logical % group_sz) / gm) * B;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int M = a.M, N = a.N, K = a.K, nk = K / BK;
    v4i ga[PIECES], gb[PIECES];
    auto load_tile = [&](int kt) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int row = (tid + i * 256) / (BK / 16), k = kt * BK + (tid + i * 256) % (BK / 16) * 16;
            ga[i] = *reinterpret_cast<const v4i *>(a.q + (size_t)min(m0 + row, M - 1) * K + k);
            gb[i] = *reinterpret_cast<const v4i *>(static_cast<const int8_t *>(a.w) + (size_t)min(n0 + row, N - 1) * K + k);
        }
    };
    auto store_tile = [&](int kt) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int at = (kt & 1) * BYTES + (tid + i * 256) / (BK / 16) * LD + (tid + i * 256) % (BK / 16) * 16;
            *reinterpret_cast<v4i *>(sA + at) = ga[i];
            *reinterpret_cast<v4i *>(sB + at) = gb[i];
        }
    };
    v16i acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;
    // fragment of a lane: row (lane & 31) of a 32-row block, 16 k starting at 16 * (lane >> 5) of a 32-wide slice
    const int fr = lane & 31, half = lane >> 5;
    load_tile(0);
    store_tile(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) load_tile(kt + 1);
        const unsigned char *pa = sA + (kt & 1) * BYTES + (wm * T * 32 + fr) * LD + half * 16;
        const unsigned char *pb = sB + (kt & 1) * BYTES + (wn * T * 32 + fr) * LD + half * 16;
#pragma unroll
        for (int ks = 0; ks < BK / 32; ++ks) {
            v4i af[T], bf[T];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                af[i] = *reinterpret_cast<const v4i *>(pa + i * 32 * LD + ks * 32);
                bf[i] = *reinterpret_cast<const v4i *>(pb + i * 32 * LD + ks * 32);
            }
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int j = 0; j < T; ++j) acc[i][j] = mfma_step<false>(af[i], bf[j], acc[i][j]);
        }
        if (kt + 1 < nk) store_tile(kt + 1);
        __syncthreads();
    }

    // ---- epilogue: activation scale per row (staged in LDS), weight scale and bias per column
    float *s_row = reinterpret_cast<float *>(smem);
    for (int t = tid; t < B; t += 256) s_row[t] = a.s_a[min(m0 + t, M - 1) / a.R];
    __syncthreads();
    _Float16 *y = static_cast<_Float16 *>(a.y);
    auto emit = [&](auto edge) {
        constexpr bool EDGE = decltype(edge)::value;
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const int n = n0 + wn * T * 32 + j * 32 + fr;
            const bool n_ok = !EDGE || n < N;
            const float sw = n_ok ? static_cast<const float *>(a.s_w)[n] : 1.0f;
            const float b = (a.bias && n_ok) ? half_to_float_dev(static_cast<const unsigned short *>(a.bias)[n]) : 0.0f;
#pragma unroll
            for (int i = 0; i < T; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = wm * T * 32 + i * 32 + 8 * (r / 4) + 4 * half + (r % 4), m = m0 + row;
                    if (!EDGE || (m < M && n_ok)) {
                        const float t = (float)acc[i][j][r] * s_row[row];
                        float u = a.bias ? __builtin_fmaf(t, sw, b) : t * sw;
                        const unsigned off = (unsigned)(m * N + n);
                        if (a.acc_out) a.acc_out[off] = acc[i][j][r];
                        asm volatile("" : "+v"(u));   // keep the fp32 rounding before the fp16 one
                        __builtin_nontemporal_store((_Float16)u, &y[off]);
                    }
                }
        }
    };
    if (m0 + B <= M && n0 + B <= N) emit(std::false_type{});
    else emit(std::true_type{});
}

static bool k64_takes(const GemmArgs &a)
{
    const bool glue = a.act != 0 || a.residual != nullptr || a.gate != nullptr || a.row_absmax != nullptr;
    return a.w_bits == 8 && !a.w_grouped && !a.s_ag && !glue && a.K % 64 == 0 && ((uintptr_t)a.q | (uintptr_t)a.w) % 16 == 0;
}

// Where it is the faster one: more tiles than CUs (320 tiles: 10 to 25 % faster than qgemm_edge, 240: 15 to 45 % slower) and whole tile columns; others are written element by
// element, which only a long K and more than two tiles per CU outweigh (N = 1000: M = 8192, K = 192 22.5 against 19.5 us, K = 2240 53 against 51).  Of very many tiles only with
// rows that are mostly padding on the DMA tiles for any K, which take steps of 128 (from 1152 tiles on, DMA tiles over this kernel: K = 64 0.94 to 1.07 of the time,
// mostly 1.04 and more; 192 0.97 to 1.06; 320 0.95 to 1.05, mostly 0.98; 576 0.95 to 1.01; 2240 0.91 to 0.94).
static bool k64_wins(const GemmArgs &a)
{
    const long tiles = (long)((a.M + 127) / 128) * ((a.N + 127) / 128);
    return k64_takes(a) && tiles > 256 && (tiles <= 1024 || a.K <= 192) && (a.N % 128 == 0 || (a.K >= 2048 && tiles > 512));
}

static hipError_t run_k64(const GemmArgs &a, hipStream_t s)
{
    const int tiles_m = (a.M + 127) / 128, tiles_n = (a.N + 127) / 128, padded = (tiles_m * tiles_n + XCDS - 1) / XCDS * XCDS;
    hipLaunchKernelGGL(qgemm_k64, dim3(padded), dim3(256), 0, s, a, tiles_m, tiles_n, padded, pick_group_m(128));
    return hipGetLastError();
}

// Any shape, no alignment needs: one thread per output element.
__global__ __launch_bounds__(256) void qgemm_naive(GemmArgs a)
{
    const int n = blockIdx.y * 64 + (threadIdx.x & 63);
    const int m = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (m >= a.M || n >= a.N) return;
    const int K = a.K;
    const unsigned short *bias = static_cast<const unsigned short *>(a.bias);
    const float b = bias ? half_to_float_dev(bias[n]) : 0.0f;
    if (a.w_bits == 16) {
        // a layer left in FP16: a.q holds the binary16 activations, a.w the binary16 weights; fp32 running sum
        const unsigned short *xr = reinterpret_cast<const unsigned short *>(a.q) + (size_t)m * K;
        const unsigned short *wr = static_cast<const unsigned short *>(a.w) + (size_t)n * K;
        float s = 0.0f;
        for (int k = 0; k < K; ++k) s = __builtin_fmaf(half_to_float_dev(xr[k]), half_to_float_dev(wr[k]), s);
        const float u16 = s + b;
        static_cast<_Float16 *>(a.y)[(size_t)m * a.N + n] = has_glue(a) ? glue_one(a, u16, m, glue_terms(a, m, n, a.gate ? m / a.gate_rows : 0)) : (_Float16)u16;
        return;
    }
    const float sa = a.s_ag ? 1.0f : a.s_a[m / a.R];
    const int8_t *q = a.q + (size_t)m * K;
    float u;
    if (a.w_bits == 8 && !a.w_grouped) {
        const int8_t *w = static_cast<const int8_t *>(a.w) + (size_t)n * K;
        int s = 0;
        for (int k = 0; k < K; ++k) s += (int)q[k] * (int)w[k];
        if (a.acc_out) a.acc_out[(size_t)m * a.N + n] = s;
        const float t = (float)s * sa;
        const float sw = static_cast<const float *>(a.s_w)[n];
        u = bias ? __builtin_fmaf(t, sw, b) : t * sw;
    } else {
        // group-wise weight scales: packed nibbles, or int8 codes of any width up to 8 bits
        const unsigned char *w = static_cast<const unsigned char *>(a.w) + (size_t)n * (a.w_grouped ? K : K / 2);
        const int gsz = a.group;
        const int G = K / gsz;
        float f = 0.0f;
        for (int g = 0; g < G; ++g) {
            int s = 0;
            for (int k = gsz * g; k < gsz * g + gsz; ++k) {
                int v;
                if (a.w_grouped) {
                    v = (int)(int8_t)w[k];
                } else {
                    const unsigned byte = w[4 * (k / 8) + (k % 4)];
                    v = (k % 8) >= 4 ? (int)(byte >> 4) : (int)(byte & 0xf);
                    v = v >= 8 ? v - 16 : v;
                }
                s += (int)q[k] * v;
            }
            if (a.acc_out) a.acc_out[((size_t)m * G + g) * a.N + n] = s;
            float c = half_to_float_dev(static_cast<const unsigned short *>(a.s_w)[(size_t)n * G + g]);
            if (a.s_ag) c = c * a.s_ag[(size_t)(m / a.R) * G + g];
            f = __builtin_fmaf((float)s, c, f);
        }
        u = bias ? __builtin_fmaf(f, sa, b) : f * sa;
    }
    static_cast<_Float16 *>(a.y)[(size_t)m * a.N + n] = has_glue(a) ? glue_one(a, u, m, glue_terms(a, m, n, a.gate ? m / a.gate_rows : 0)) : (_Float16)u;
}

// ---- variants -----------------------------------------------------------------
struct Variant {
    const char *name;
    int w_bits;
    bool (*takes)(const GemmArgs &);
    hipError_t (*run)(const GemmArgs &, hipStream_t);
    hipError_t (*run_glue)(const GemmArgs &, hipStream_t) = nullptr;   // the same tile with block glue in the epilogue
};

// the DMA kernels need 16-byte loads along K and whole K steps of 128 bytes
static bool dma_takes(const GemmArgs &a)
{
    return (a.K * (a.w_bits == 16 ? 2 : 1)) % 128 == 0 && ((uintptr_t)a.q | (uintptr_t)a.w) % 16 == 0;
}

template <int T>
static bool split_takes(const GemmArgs &a) { return qgemm_split_takes(a, T); }

//                          TM TN WGM WGN S WPS
using D8_128x128_s3 = TileD<2, 2, 2, 2, 3, 2>;
using D8_128x128_s2 = TileD<2, 2, 2, 2, 2, 2>;
using D8_128x192_s3 = TileD<2, 3, 2, 2, 3, 2>;
using D8_128x192_s2 = TileD<2, 3, 2, 2, 2, 2>;
using D8_256x128_s3 = TileD<4, 2, 2, 2, 3, 1>;
using D8_256x192_s2 = TileD<4, 3, 2, 2, 2, 1>;
using D8_256x256_8w = TileD<4, 2, 2, 4, 2, 2>;
using D8_256x192_8w = TileD<2, 3, 4, 2, 2, 2>;
using D8_256x192_8w_e1 = TileD<2, 3, 4, 2, 2, 2, true, 1>;
using D8_256x256_8w_e1 = TileD<4, 2, 2, 4, 2, 2, true, 1>;
using D8_256x256_8w_e2 = TileD<4, 2, 2, 4, 2, 2, true, 2>;
using D8_256x192_4w_e2 = TileD<4, 3, 2, 2, 2, 1, true, 2>;
using D8_64x64_s3 = TileD<1, 1, 2, 2, 3, 4>;
//                                                       SA                  SB
using D8_256x192_8w_a3b2 = TileD<2, 3, 4, 2, 3, 2, true, 1, 2>;
using D8_256x192_8w_a2b3 = TileD<2, 3, 4, 2, 2, 2, true, 1, 3>;
using D8_256x256_8w_a3b2 = TileD<4, 2, 2, 4, 3, 2, true, 1, 2>;
using D8_128x128_a3b2 = TileD<2, 2, 2, 2, 3, 2, true, 0, 2>;
using D8_128x128_a3b2_e1 = TileD<2, 2, 2, 2, 3, 2, true, 1, 2>;
using D8_128x128_s2_e1 = TileD<2, 2, 2, 2, 2, 2, true, 1>;
//                                                                               persistent
using P8_128x128_a3b2 = TileD<2, 2, 2, 2, 3, 2, true, 1, 2, true>;
using P8_128x192_s2 = TileD<2, 3, 2, 2, 2, 2, true, 1, 2, true>;
//                                                                                      FP16 operands
using H_256x192_8w = TileD<2, 3, 4, 2, 3, 2, true, 1, 2, false, true>;
using H_128x128_4w = TileD<2, 2, 2, 2, 3, 2, true, 1, 2, false, true>;
using H_64x64_4w = TileD<1, 1, 2, 2, 3, 4, true, 0, 3, false, true>;
using H_p192 = TileD<2, 3, 2, 2, 2, 2, true, 1, 2, true, true>;
using H_p128 = TileD<2, 2, 2, 2, 3, 2, true, 1, 2, true, true>;

//                                                                                            rows of any whole number of words
using K8_64x64 = TileD<1, 1, 2, 2, 3, 4, true, 0, 3, false, false, true>;
using K8_128x128 = TileD<2, 2, 2, 2, 3, 2, true, 1, 2, false, false, true>;
using KH_64x64 = TileD<1, 1, 2, 2, 3, 4, true, 0, 3, false, true, true>;
using KH_128x128 = TileD<2, 2, 2, 2, 3, 2, true, 1, 2, false, true, true>;

static bool any_k_takes(const GemmArgs &a)
{
    const long kb = (long)a.K * (a.w_bits == 16 ? 2 : 1);
    return (a.w_bits == 8 || a.w_bits == 16) && !a.w_grouped && !a.s_ag && kb % 4 == 0 && kb >= 16 && ((uintptr_t)a.q | (uintptr_t)a.w) % 4 == 0;
}

static const Variant VARIANTS[] = {
    {"w8 dma 64x64 s3 4w", 8, dma_takes, run_dma<D8_64x64_s3>, run_dma<D8_64x64_s3, true>},
    {"w8 dma 256x192 a3b2 8w spread1", 8, dma_takes, run_dma<D8_256x192_8w_a3b2>, run_dma<D8_256x192_8w_a3b2, true>},
    {"w8 dma 128x128 a3b2 4w", 8, dma_takes, run_dma<D8_128x128_a3b2>, run_dma<D8_128x128_a3b2, true>},
    {"w8 dma 128x128 a3b2 4w spread1", 8, dma_takes, run_dma<D8_128x128_a3b2_e1>, run_dma<D8_128x128_a3b2_e1, true>},
    {"w8 dma 128x128 a3b2 4w spread1 persistent", 8, dma_takes, run_dma<P8_128x128_a3b2>},
    {"w8 dma 128x192 s2 4w spread1 persistent", 8, dma_takes, run_dma<P8_128x192_s2>},
    {"f16 dma 256x192 a3b2 8w spread1", 16, dma_takes, run_dma<H_256x192_8w>, run_dma<H_256x192_8w, true>},
    {"f16 dma 128x128 a3b2 4w spread1", 16, dma_takes, run_dma<H_128x128_4w>, run_dma<H_128x128_4w, true>},
    {"f16 dma 64x64 s3 4w", 16, dma_takes, run_dma<H_64x64_4w>, run_dma<H_64x64_4w, true>},
    {"f16 dma 128x192 s2 4w spread1 persistent", 16, dma_takes, run_dma<H_p192>},
    {"w4 pipelined 128x128 a3b2 4w any-group", 4, qgemm_w4_takes, launch_qgemm_w4_128, launch_qgemm_w4_128},
    {"w4 pipelined 64x64 a3b2 4w any-group", 4, qgemm_w4_takes, launch_qgemm_w4_64, launch_qgemm_w4_64},
    {"w8 big 256x288", 8, qgemm_big_takes, launch_big_w8_256x288, launch_big_w8_256x288_glue},
    {"w8 big 256x256", 8, qgemm_big_takes, launch_big_w8_256x256, launch_big_w8_256x256_glue},
    {"w8 big 128x288", 8, qgemm_big_takes, launch_big_w8_128x288, launch_big_w8_128x288_glue},
    {"f16 big 256x288", 16, qgemm_big_takes, launch_big_f16_256x288, launch_big_f16_256x288_glue},
    {"f16 big 256x256", 16, qgemm_big_takes, launch_big_f16_256x256, launch_big_f16_256x256_glue},
    {"w4 big 256x288", 4, qgemm_w4_big_takes, launch_big_w4_256x288, launch_big_w4_256x288_glue},
    {"w4 big 256x256", 4, qgemm_w4_big_takes, launch_big_w4_256x256, launch_big_w4_256x256_glue},
    {"w4 big 128x288", 4, qgemm_w4_big_takes, launch_big_w4_128x288, launch_big_w4_128x288_glue},
    {"w8 split-K 32x32", 8, split_takes<32>, launch_qgemm_split32, launch_qgemm_split32},
    {"w4 any-group split-K 32x32", 4, split_takes<32>, launch_qgemm_split32, launch_qgemm_split32},
    {"f16 split-K 32x32", 16, split_takes<32>, launch_qgemm_split32, launch_qgemm_split32},
    {"w8 split-K 16x16", 8, split_takes<16>, launch_qgemm_split16, launch_qgemm_split16},
    {"w4 any-group split-K 16x16", 4, split_takes<16>, launch_qgemm_split16, launch_qgemm_split16},
    {"f16 split-K 16x16", 16, split_takes<16>, launch_qgemm_split16, launch_qgemm_split16},
    {"w8 edge any-K", 8, qgemm_edge_takes, launch_qgemm_edge, launch_qgemm_edge},
    {"w4 any-group edge any-K", 4, qgemm_edge_takes, launch_qgemm_edge, launch_qgemm_edge},
    {"f16 edge any-K", 16, qgemm_edge_takes, launch_qgemm_edge, launch_qgemm_edge},
    {"w8 staged 128x128 k64", 8, k64_takes, run_k64},
    {"w8 dma any-K 64x64 s3 4w", 8, any_k_takes, run_dma<K8_64x64>, run_dma<K8_64x64, true>},
    {"w8 dma any-K 128x128 a3b2 4w spread1", 8, any_k_takes, run_dma<K8_128x128>, run_dma<K8_128x128, true>},
    {"f16 dma any-K 64x64 s3 4w", 16, any_k_takes, run_dma<KH_64x64>, run_dma<KH_64x64, true>},
    {"f16 dma any-K 128x128 a3b2 4w spread1", 16, any_k_takes, run_dma<KH_128x128>, run_dma<KH_128x128, true>},
#ifdef QL_SWEEP_VARIANTS   // the other tile shapes of the sweeps that chose the ones above
    {"w8 dma 128x128 s3 4w", 8, dma_takes, run_dma<D8_128x128_s3>},
    {"w8 dma 128x128 s2 4w", 8, dma_takes, run_dma<D8_128x128_s2>},
    {"w8 dma 128x192 s3 4w", 8, dma_takes, run_dma<D8_128x192_s3>},
    {"w8 dma 128x192 s2 4w", 8, dma_takes, run_dma<D8_128x192_s2>},
    {"w8 dma 256x128 s3 4w", 8, dma_takes, run_dma<D8_256x128_s3>},
    {"w8 dma 256x192 s2 4w", 8, dma_takes, run_dma<D8_256x192_s2>},
    {"w8 dma 256x256 s2 8w", 8, dma_takes, run_dma<D8_256x256_8w>},
    {"w8 dma 256x192 s2 8w", 8, dma_takes, run_dma<D8_256x192_8w>},
    {"w8 dma 256x192 s2 8w spread1", 8, dma_takes, run_dma<D8_256x192_8w_e1>},
    {"w8 dma 256x256 s2 8w spread1", 8, dma_takes, run_dma<D8_256x256_8w_e1>},
    {"w8 dma 256x256 s2 8w spread2", 8, dma_takes, run_dma<D8_256x256_8w_e2>},
    {"w8 dma 256x192 s2 4w spread2", 8, dma_takes, run_dma<D8_256x192_4w_e2>},
    {"w8 dma 256x192 a2b3 8w spread1", 8, dma_takes, run_dma<D8_256x192_8w_a2b3>},
    {"w8 dma 256x256 a3b2 8w spread1", 8, dma_takes, run_dma<D8_256x256_8w_a3b2>},
    {"w8 dma 128x128 s2 4w spread1", 8, dma_takes, run_dma<D8_128x128_s2_e1>},
    {"f16 dma 128x128 a3b2 4w spread1 persistent", 16, dma_takes, run_dma<H_p128>},
#endif
};
constexpr int NUM_VARIANTS = sizeof(VARIANTS) / sizeof(VARIANTS[0]);

int num_gemm_variants() { return NUM_VARIANTS; }
const char *gemm_variant_name(int v) { return (v >= 0 && v < NUM_VARIANTS) ? VARIANTS[v].name : "naive (any shape)"; }

static int find_variant(const char *name)
{
    for (int v = 0; v < NUM_VARIANTS; ++v)
        if (__builtin_strcmp(VARIANTS[v].name, name) == 0) return v;
    return 0;
}

// ---- tile choice --------------------------------------------------------------------------------------------------------
// What a layer takes on each tile, in microseconds: the tiles of the busiest CU one after the other, `resident` of them sharing it.
//
//   base + n * (tile + step * K steps + fold * groups) + rounds * (round_step * K steps + round_fold * groups) + more * (n - resident)
//   n = tiles of the busiest CU, rounds = ceil(n / resident), K steps of 128 bytes, groups of 4-bit weights along K
//   + per 10^4 outputs of the busiest CU: act (GELU), gated (gate or residual)
//   + for the part of a partial tile that is written, per value of a lane: edge, edge_act, edge_gated (the large tiles write theirs in
//     pieces like whole ones)
//
// Fitted to sweeps on MI355X over M = 640..16384 and 27 (K, N) from 256 to 5120, plain, with GELU and with gate and residual; DAQ in front of
// the layer, other weights and outputs in every call, as in a stack; 4-bit weights also with groups of 32, 64, 192 and 288: 0.3 % in the mean over the fastest tile, 2 %
// of 6300 cases more than 5 % over it.  profiles/tile_choice_sweep.txt holds the part of the data with the common widths.  Rules that charged the large tiles per round and the
// others by their rate, without the glue, lost 2 % (4 bits) to 6 % (FP16) in the mean of the plain layers and 5 to 17 % with gate and residual (8-bit, M = 8192, K = 256, N =
// 1024: 40.7 us against 14.3).  The edge terms of 8-bit and FP16 layers were set again when gate and residual of such values came to be requested together; since those kernels
// changed, 1850 layers of M = 512..16384 and widths of any kind, two thirds of them with glue, stay over the fastest tile by 2.0 % (8-bit), 2.2 % (FP16) and 0.7 % (4-bit) in the mean,
// 10, 11 and 3 % of them by more than 5 %, at worst 54 % (odd widths with gate and residual, whose every tile pays what is charged once).
struct GlueCost {
    float act, gated, big_act, big_gated, edge, edge_act, edge_gated;
};
static const GlueCost GLUE_W8 = {0.537f, 0.838f, 1.316f, 2.061f, 0.069f, 0.05f, 0.5f};
static const GlueCost GLUE_F16 = {0.671f, 1.080f, 1.425f, 3.027f, 0.007f, 0.05f, 0.63f};
static const GlueCost GLUE_W4 = {0.834f, 1.750f, 1.002f, 3.037f, 0.045f, 0.193f, 0.835f};
struct TileCost {
    const char *name;
    int bits, BM, BN, resident;
    float base, tile, step, fold, round_step, round_fold, more;
    int most_tiles = 0;   // not beyond this many (0: any)
};
static const TileCost TILE_COSTS[] = {
    {"w8 dma 64x64 s3 4w", 8, 64, 64, 3, 4.685f, 0, 0.133f, 0, 0.154f, 0, 0.890f},
    {"w8 dma 128x128 a3b2 4w", 8, 128, 128, 2, 0.065f, 4.717f, 0.531f, 0, 0, 0, 1.019f, 256},   // the deeper issue of one tile per CU at most
    {"w8 dma 128x128 a3b2 4w spread1", 8, 128, 128, 2, 3.178f, 1.466f, 0.183f, 0, 0.399f, 0, 1.163f},
    {"w8 dma 128x128 a3b2 4w spread1 persistent", 8, 128, 128, 2, 4.291f, 1.123f, 0.245f, 0, 0.276f, 0, 1.187f},
    {"w8 dma 128x192 s2 4w spread1 persistent", 8, 128, 192, 2, 3.888f, 1.543f, 0.250f, 0, 0.752f, 0, 1.600f},
    {"w8 dma 256x192 a3b2 8w spread1", 8, 256, 192, 1, 0, 7.622f, 1.173f, 0, 0, 0, 1.376f},
    {"w8 big 128x288", 8, 128, 288, 1, 3.469f, 5.451f, 1.251f, 0, 0, 0, 1.285f},
    {"w8 big 256x256", 8, 256, 256, 1, 3.808f, 5.434f, 1.422f, 0, 0, 0, 0.176f},
    {"w8 big 256x288", 8, 256, 288, 1, 2.983f, 8.716f, 1.773f, 0, 0, 0, 0.128f},
    {"f16 dma 64x64 s3 4w", 16, 64, 64, 3, 3.401f, 0.047f, 0.163f, 0, 0.095f, 0, 0.784f},
    {"f16 dma 128x128 a3b2 4w spread1", 16, 128, 128, 2, 2.892f, 0.472f, 0.293f, 0, 0.293f, 0, 1.441f},
    {"f16 dma 128x192 s2 4w spread1 persistent", 16, 128, 192, 2, 1.821f, 1.541f, 0.336f, 0, 0.573f, 0, 2.070f},
    {"f16 dma 256x192 a3b2 8w spread1", 16, 256, 192, 1, 0.275f, 5.430f, 1.129f, 0, 0, 0, 4.768f},
    {"f16 big 256x256", 16, 256, 256, 1, 1.395f, 4.703f, 1.423f, 0, 0, 0, 0.007f},
    {"f16 big 256x288", 16, 256, 288, 1, 0, 6.117f, 1.753f, 0, 0, 0, 0.331f},
    // rows that are no whole K steps: the 8-bit DMA tiles as above, those of FP16 and qgemm_edge fitted; qgemm_edge where the rows are a few steps only (its 128x128 tiles, from
    // 512 of them on, were 1.07 to 1.9 times as slow with 8 bits, and with FP16 rows of one step 0.92 to 1.27 times).  us, DAQ and GEMM, qgemm_edge -> chosen, M x K x N: 8-bit
    // 1021 x 1160 x 1000 16.0 -> 12.1, 1021 x 2244 x 1000 42 -> 32, 8192 x 1160 x 2560 59 -> 50, 64 x 1000 x 77 12.9 -> 9.5; FP16 2047 x 2244 x 1000 36 -> 25, 4096 x 1160 x 2560 55 ->
    // 42; 8-bit 4096 x 200 x 1200 13.5 -> 13.1.  Over the fastest kernel 1.4 % (8-bit) and 2.9 % (FP16) in the mean of 570 layers whose rows are whole 16 bytes, 6 and 16 % of
    // 550 others, where qgemm_edge reads the ends of rows byte by byte and is still taken for short ones.
    {"w8 dma any-K 64x64 s3 4w", 8, 64, 64, 3, 4.685f, 0, 0.133f, 0, 0.154f, 0, 0.890f},
    {"w8 dma any-K 128x128 a3b2 4w spread1", 8, 128, 128, 2, 3.178f, 1.466f, 0.183f, 0, 0.399f, 0, 1.163f},
    {"w8 edge any-K", 8, 64, 64, 4, 3.985f, 0.173f, 0.024f, 0, 0.748f, 0, 0},
    {"f16 dma any-K 64x64 s3 4w", 16, 64, 64, 3, 3.430f, 0.196f, 0.215f, 0, 0.120f, 0, 0.303f},
    {"f16 dma any-K 128x128 a3b2 4w spread1", 16, 128, 128, 2, 4.531f, 0.388f, 0.458f, 0, 0.173f, 0, 2.030f},
    {"f16 edge any-K", 16, 64, 64, 4, 1.656f, 0.341f, 0.082f, 0, 0.702f, 0, 0},
    {"w4 pipelined 64x64 a3b2 4w any-group", 4, 64, 64, 4, 4.803f, 0.011f, 0.058f, 0.043f, 0.336f, 0.013f, 0.407f},
    {"w4 pipelined 128x128 a3b2 4w any-group", 4, 128, 128, 2, 4.365f, 1.245f, 0.079f, 0.095f, 0.536f, 0.170f, 0.245f},
    {"w4 big 128x288", 4, 128, 288, 1, 5.977f, 5.191f, 1.495f, 0, 0, 0, 0.347f},
    {"w4 big 256x256", 4, 256, 256, 1, 6.465f, 3.934f, 2.029f, 0, 0, 0, 0.024f},
    {"w4 big 256x288", 4, 256, 288, 1, 12.968f, 0.069f, 2.318f, 0, 0, 0, 4.782f},
};
static int choose_tile(const GemmArgs &a, bool glue, float *us = nullptr)
{
    constexpr int COUNT = sizeof(TILE_COSTS) / sizeof(TILE_COSTS[0]), CUS_PER_XCD = 32;
    static const int *const variants = [] {
        static int v[COUNT];
        for (int i = 0; i < COUNT; ++i) v[i] = find_variant(TILE_COSTS[i].name);
        return (const int *)v;
    }();
    const bool big_takes = a.w_bits == 4 ? qgemm_w4_big_takes(a) : qgemm_big_takes(a);
    const GlueCost &g = a.w_bits == 8 ? GLUE_W8 : a.w_bits == 4 ? GLUE_W4 : GLUE_F16;
    const float act = a.act != 0 || (glue && !a.gate && !a.residual) ? 1.0f : 0.0f, gated = a.gate || a.residual ? 1.0f : 0.0f;
    const int groups = a.w_bits == 4 ? a.K / a.group : 0;
    const float steps = (float)((a.K * (a.w_bits == 16 ? 2 : 1) + 127) / 128), folds = (float)groups;
    const bool any_k = a.w_bits != 4 && !dma_takes(a);
    // outputs that no 16-byte piece reaches are written value by value everywhere
    const bool pieces = a.N % 8 == 0 && ((uintptr_t)a.y | (uintptr_t)a.gate | (uintptr_t)a.residual) % 16 == 0;
    int best = -1;
    float least = 0.0f;
    for (int i = 0; i < COUNT; ++i) {
        const TileCost &t = TILE_COSTS[i];
        const Variant &v = VARIANTS[variants[i]];
        if (t.bits != a.w_bits || (glue && !v.run_glue)) continue;
        const bool edge = v.takes == qgemm_edge_takes;
        if ((edge || v.takes == any_k_takes) != any_k) continue;
        if (edge && (long)((a.M + 127) / 128) * ((a.N + 127) / 128) >= 512) continue;
        const bool big = !any_k && v.takes != dma_takes && v.takes != qgemm_w4_takes;
        if (big && !big_takes) continue;
        if (groups > 40 && t.BM == 128) continue;   // the large scale table leaves such a tile one workgroup per CU (134 against 198 us at 144 groups)
        const long tiles = (long)((a.M + t.BM - 1) / t.BM) * ((a.N + t.BN - 1) / t.BN);
        if (t.most_tiles && tiles > t.most_tiles) continue;
        const float n = (float)(((tiles + XCDS - 1) / XCDS + CUS_PER_XCD - 1) / CUS_PER_XCD), resident = (float)t.resident;
        const float rounds = __builtin_ceilf(n / resident);
        float cost = t.base + n * (t.tile + t.step * steps + t.fold * folds) + rounds * (t.round_step * steps + t.round_fold * folds) +
                     t.more * (n > resident ? n - resident : 0.0f);
        cost += n * (float)(t.BM * t.BN) * 1e-4f * (act * (big ? g.big_act : g.act) + gated * (big ? g.big_gated : g.gated));
        if (!big) {
            const float in_m = (float)(a.M % t.BM) / t.BM, in_n = (float)(a.N % t.BN) / t.BN, part = !pieces ? 1.0f : in_m > in_n ? in_m : in_n;
            cost += part * (float)(t.BM * t.BN / (t.BM == 256 ? 512 : 256)) * (g.edge + act * g.edge_act + gated * g.edge_gated);
        }
        if (best < 0 || cost < least) {
            best = variants[i];
            least = cost;
        }
    }
    if (us) *us = least;
    return best;
}

float qgemm_alone_us(const GemmArgs &a)
{
    float us;
    choose_tile(a, false, &us);
    return us;
}

hipError_t launch_qgemm(const GemmArgs &a, int variant, hipStream_t stream)
{
    const bool glue = a.act != 0 || a.residual != nullptr || a.gate != nullptr || a.row_absmax != nullptr;
    auto naive = [&]() {
        hipLaunchKernelGGL(qgemm_naive, dim3((a.M + 3) / 4, (a.N + 63) / 64), dim3(256), 0, stream, a);
        return hipGetLastError();
    };
    if (variant >= NUM_VARIANTS) return naive();
    const int split = qgemm_split_choice(a);
    auto small = [&]() {
        if (split) return split == 16 ? launch_qgemm_split16(a, stream) : launch_qgemm_split32(a, stream);
        if (k64_wins(a)) return run_k64(a, stream);
        return qgemm_edge_takes(a) ? launch_qgemm_edge(a, stream) : naive();
    };
    if (a.w_grouped || a.s_ag) {
        // plan-space generality: the pipelined grouped kernel where it takes the shape
        if (!split && qgemm_w4_takes(a) && !glue) return launch_qgemm_w4(a, stream);
        return small();
    }
    auto usable = [&](const Variant &v) { return v.w_bits == a.w_bits && v.takes(a) && (!glue || v.run_glue); };
    int v = variant;
    if (v < 0 || !usable(VARIANTS[v])) {
        if (split || !(a.w_bits == 4 ? qgemm_w4_takes(a) : dma_takes(a) || (any_k_takes(a) && !k64_wins(a)))) return small();
        v = choose_tile(a, glue);
    }
    return glue ? VARIANTS[v].run_glue(a, stream) : VARIANTS[v].run(a, stream);
}

}  // namespace ql
