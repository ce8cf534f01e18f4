// Internal launch interface between the host API (api.hip) and the kernels.
// Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ql {

// ---- DAQ (Step 3, eq. (4), tau = block absmax) ---------------------------
// mode of the row kernels
enum DaqMode : int {
    DAQ_FUSED = 0,   // per-token: absmax, scale, codes in one pass over a row held in registers
    DAQ_ABSMAX = 1,  // R > 1, phase 1 (fallback): row absmax -> atomic max into blockmax[row / R]
    DAQ_QUANT = 2    // R > 1, phase 2: codes from blockmax[row / R]
};

struct DaqArgs {
    const void *x;       // [M,K] fp16
    int8_t *q;           // [M,K]
    float *scales;       // [M/R]
    unsigned *blockmax;  // [M/R] fp16 bit patterns of block maxima (workspace), R > 1 only
    unsigned *partmax;   // [M/R][daq_parts_per_block] partial maxima (workspace), R > 1 only
    int M, K, R;
    int quant_parts;     // > 0: the quantize pass takes each block's maximum from this many partial maxima itself
    // percentile-clipped variant only (launch_daq_robust)
    int qmax;            // 2^(b-1) - 1 for b-bit activation codes
    unsigned top_rank;   // tau = the top_rank-th largest magnitude of a scale block (1 = the maximum)
    unsigned *hist;      // selection scratch (workspace, where partmax is), R > 1 only: daq_hist_bytes() for the partial histograms, and
                         //    from DAQ_ROBUST_WORDS words per scale block on the selection with atomics
    // both variants: bytes at partmax and hist; where the partial maxima or histograms need more, the kernels with atomics run
    size_t scratch_bytes;
};
constexpr int DAQ_ROBUST_WORDS = 256 + 2 + 128;
// Partial histograms of the percentile selection: elements per part (at most 65535, so that a 16-bit count holds); parts per
// scale block up to which the next pass adds them up itself, and up to which a selection launch does (beyond: atomics)
constexpr unsigned DAQ_HIST_SELF = 20, DAQ_HIST_FEW = 256;
constexpr unsigned DAQ_HIST_PART = 16384;
inline size_t daq_hist_parts(int64_t K, int64_t R) { return ((size_t)R * (size_t)K + DAQ_HIST_PART - 1) / DAQ_HIST_PART; }
inline size_t daq_hist_bytes(int64_t M, int64_t K, int64_t R)
{
    const size_t nblk = (size_t)(M / R), parts = daq_hist_parts(K, R);
    return parts <= DAQ_HIST_FEW ? nblk * parts * (256 + 128) * 2 : nblk * DAQ_ROBUST_WORDS * 4;
}

// R > 1: the first pass cuts every scale block (R*K contiguous values) into this many parts and leaves one partial
// maximum per part; 0 when the shape takes the row kernels instead (no partials needed).
constexpr int DAQ_PART_PIECES = 2048;  // 16-byte pieces per part: 256 threads x 8 loads
inline size_t daq_parts_per_block(int64_t K, int64_t R)
{
    if (R <= 1 || K % 8 != 0) return 0;
    const size_t pieces = (size_t)R * (size_t)K / 8;
    if (pieces < (size_t)DAQ_PART_PIECES || pieces >= (1ull << 31)) return 0;
    return (pieces + DAQ_PART_PIECES - 1) / DAQ_PART_PIECES;
}

hipError_t launch_daq(const DaqArgs &a, hipStream_t stream);
// DAQ of up to PLAN_WINDOW layers of the same M and R in the launches that one layer takes; every layer has to pass daq_many_takes
constexpr int PLAN_WINDOW = 8;
struct DaqMany {
    DaqArgs l[PLAN_WINDOW];
    int count;
    // set by the launches: workgroups per layer of the row kernels, and where a layer's workgroups begin in the kernels that cut scale blocks into parts
    int row_blocks;
    unsigned first[PLAN_WINDOW];   // (of those that are not there: behind all workgroups)
};
// A layer's codes are read by its GEMM after the codes of the layers with it and the outputs of those before it have been written; layers go together as far
// as Infinity Cache (256 MB) holds these.  us a plan, a launch per layer -> as many together as there are -> within this bound: four layers of K = N = 1152,
// M = 16384 163 -> 159 -> 160, M = 65536 520 -> 564 -> 518; eight of 384 x 384, M = 65536 316 -> 325 -> 297; four of 1160 x 1000, M = 65536 832 -> 925 -> 805.
// It also keeps their launches below 2^32 threads: 64 threads per row of at least 8 codes.
constexpr int64_t PLAN_WINDOW_BYTES = (int64_t)256 << 20;
static_assert(PLAN_WINDOW_BYTES / 8 * 64 < (int64_t)1 << 32, "threads of a launch");
bool daq_many_takes(const DaqArgs &a, bool robust);
hipError_t launch_daq_many(DaqMany &b, hipStream_t stream);
hipError_t launch_daq_robust_many(DaqMany &b, hipStream_t stream);
// the first pass alone: partial maxima of every scale block (daq_parts_per_block of them) into a.partmax
hipError_t launch_daq_part_absmax(const DaqArgs &a, hipStream_t stream);
// eq. (4) with channel groups: scales [M/R, K/cg]; workspace in blockmax: one maximum per group and slab of
// daq_cg_slab_rows(R) rows with `slabs` (per scale block without, or where that is 0); K % 8 == 0, cg % 8 == 0, K/cg <= 1024
inline int daq_cg_slab_rows(int64_t R) { return R % 16 == 0 ? 16 : R % 8 == 0 ? 8 : 0; }
hipError_t launch_daq_cg(const DaqArgs &a, int cg, bool slabs, hipStream_t stream);
// DAQ whose row maxima are already known (row_absmax [M], binary16 bit patterns): scales and the quantize pass only
hipError_t launch_daq_from_rowmax(const DaqArgs &a, const unsigned *row_absmax, hipStream_t stream);
hipError_t launch_fill_u32(unsigned *p, int n, unsigned v, hipStream_t stream);
// eq. (4) with tau = a percentile of the magnitudes and a selectable code width
hipError_t launch_daq_robust(const DaqArgs &a, hipStream_t stream);

// LayerNorm + modulation + per-token DAQ in one pass (daq_ln.hip); K % 8 == 0, K <= 4608, 16-byte aligned rows
struct LnDaqArgs {
    const void *x;       // [M,K] fp16
    const void *shift;   // [M/rows_per_mod, K] fp16 or null (0)
    const void *scale;   // [M/rows_per_mod, K] fp16 or null (0): h = n * (1 + scale) + shift
    void *h;             // [M,K] fp16 out, or null
    int8_t *q;           // [M,K] out, or null (then only h is produced)
    float *scales;       // [M] out
    int M, K, rows_per_mod;
    float eps;
};
hipError_t launch_daq_ln(const LnDaqArgs &a, hipStream_t stream);

// ---- GEMM + dequantization -------------------------------------------------
struct GemmArgs {
    const int8_t *q;      // [M,K] activation codes
    const float *s_a;     // [M/R]
    const void *w;        // int8 [N,K] or packed 4-bit [N,K/2]
    const void *s_w;      // fp32 [N] (W8) or fp16 [N,K/group] (W4)
    const void *bias;     // fp16 [N] or null
    void *y;              // fp16 [M,N]
    int32_t *acc_out;     // optional export: [M,N] (W8) or [M,K/group,N] (W4)
    int M, N, K, R;
    int w_bits;           // 8 or 4
    int group;            // 4-bit weights: k per weight scale (a multiple of 32 dividing K); 128 unless stated
    // block glue folded into the epilogue (all zero = none):  h = f16(act(u));  y = f16(fma(g, h, r))
    int act;              // 0 identity, 1 GELU (tanh form) on the fp32 value u
    const void *residual; // fp16 [M,N] r, or null (0)
    const void *gate;     // fp16 [M/gate_rows, N] g, or null (1)
    int gate_rows;        // rows sharing one gate row
    // plan-space generality (Step 2, Algorithm 1, eq. (4)'s channel groups); all zero = none
    int w_grouped;        // 1: w holds int8 codes [N,K] (W3, W6, W8 or asymmetric codes stored as code - zero) with fp16 scales
                          //    [N,K/group] like the 4-bit layers (w_bits stays 8)
    const float *s_ag;    // activation scales per (scale block, channel group) [M/R, K/group] instead of s_a; the channel
                          //    groups are the weight groups
    unsigned *row_absmax; // optional side output [M] (cleared by the caller of the launch): the largest |y[m,:]| as a binary16
                          //    bit pattern, taken on the fp16 values the layer writes (what the next layer's DAQ would find)
    // quantization inside the GEMM (qgemm_fuse_takes): the fp16 input instead of q and s_a, and where several rows share a
    // scale the partial maxima of their scale block
    const void *x;            // [M,K] fp16, or null
    const unsigned *partmax;  // [M/R][parts]
    int parts;                // 0: every row its own maximum
};

int num_gemm_variants();
const char *gemm_variant_name(int v);
// variant < 0: choose by shape
hipError_t launch_qgemm(const GemmArgs &a, int variant, hipStream_t stream);
// estimated time of a layer without glue on the tile that launch_qgemm would choose for it (layers that its DMA kernels take)
float qgemm_alone_us(const GemmArgs &a);

// the pipelined 4-bit kernel (qgemm_w4.hip): shapes it takes, and its launch (group 128 or any 32 j, exports, glue)
bool qgemm_w4_takes(const GemmArgs &a);
hipError_t launch_qgemm_w4(const GemmArgs &a, hipStream_t stream);
hipError_t launch_qgemm_w4_64(const GemmArgs &a, hipStream_t stream);    // the same with the tile given
hipError_t launch_qgemm_w4_128(const GemmArgs &a, hipStream_t stream);
// any K, N and alignment (qgemm_small.hip): few rows with K split over a workgroup's wavefronts, and register-staged tiles
bool qgemm_split_takes(const GemmArgs &a, int tile);
int qgemm_split_choice(const GemmArgs &a);   // tile (16 or 32) where splitting K is the fastest, else 0
bool qgemm_fuse_takes(const GemmArgs &a);    // one launch that quantizes its own input (a.x) instead of DAQ and GEMM
bool qgemm_fuse_one_tile(const GemmArgs &a); // ... and a CU for every 16x16 tile
hipError_t launch_qgemm_fused(const GemmArgs &a, hipStream_t stream);
hipError_t launch_qgemm_split32(const GemmArgs &a, hipStream_t stream);
hipError_t launch_qgemm_split16(const GemmArgs &a, hipStream_t stream);
bool qgemm_edge_takes(const GemmArgs &a);
hipError_t launch_qgemm_edge(const GemmArgs &a, hipStream_t stream);
bool qgemm_big_takes(const GemmArgs &a);
// 8-bit layers of a plan whose 256x288 tiles are one round of workgroups, in one launch
bool qgemm_big_many_takes(const GemmArgs *const *layers, int count);
hipError_t launch_qgemm_big_many(const GemmArgs *const *layers, int count, hipStream_t stream);
hipError_t launch_big_w8_256x288(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w8_256x288_glue(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w8_256x256(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w8_256x256_glue(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w8_128x288(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w8_128x288_glue(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_f16_256x288(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_f16_256x288_glue(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_f16_256x256(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_f16_256x256_glue(const GemmArgs &a, hipStream_t s);
bool qgemm_w4_big_takes(const GemmArgs &a);
hipError_t launch_big_w4_256x288(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w4_256x288_glue(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w4_256x256(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w4_256x256_glue(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w4_128x288(const GemmArgs &a, hipStream_t s);
hipError_t launch_big_w4_128x288_glue(const GemmArgs &a, hipStream_t s);
// the GEMMs of several layers with as many rows each in one launch; every one has to pass qgemm_many_takes
bool qgemm_many_takes(const GemmArgs &a);
// which of them are better in one launch than one after the other (their number; fewer than two: none)
int qgemm_many_choice(const GemmArgs *layers, int n, const GemmArgs **chosen);
// the launch takes 256x288 tiles (qgemm_big_many_takes) in place of 128x128
bool qgemm_many_one_round(const GemmArgs *const *layers, int count);
hipError_t launch_qgemm_many(const GemmArgs *const *layers, int count, hipStream_t stream);
// pair-order nibbles (device) -> the 4-bit storage order (device); blocks = N*K/8 four-byte blocks
hipError_t launch_prepack_w4(const void *pairs, void *packed, long long blocks, hipStream_t stream);

}  // namespace ql
