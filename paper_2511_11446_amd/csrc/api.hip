// Host side of the C ABI declared in include/diffpro_qlinear.h: argument
// validation (always before the first HIP call), workspace carving, kernel
// dispatch, and the plan runner (Algorithm 2, Phase B restricted to the
// quantized linears).
#include "plan_window.h"

#include <algorithm>
#include <atomic>
#include <new>
#include <vector>

// Scratch of the allocation-free entry point (qlinear_w8a8_noalloc): one array per GPU the library runs on, held until
// the process ends.  In host code this name is only a handle for hipGetSymbolAddress; the device address it yields is
// what kernels and launches receive.
#define QL_NOALLOC_SCRATCH_BYTES (24u << 20)
static __device__ __align__(256) unsigned char scratch[QL_NOALLOC_SCRATCH_BYTES];

namespace {

thread_local int g_last_device_error = 0;
std::atomic<int> g_gemm_variant{-1};

constexpr int64_t K_MAX = 133143;          // 133143 * 127 * 127 < 2^31
constexpr int64_t ELEMS_MAX = 2147483647;  // int32 indexing inside the kernels
constexpr int64_t W4_GROUP_MAX = 132096;   // largest multiple of 32 with 127 * 8 * 16 * group < 2^31

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

int device_status(hipError_t e)
{
    if (e == hipSuccess) return QL_OK;
    g_last_device_error = (int)e;
    return QL_ERR_DEVICE;
}

int check_shape(int64_t M, int64_t K, int64_t R, int64_t N)
{
    if (M < 1 || K < 1 || N < 1 || R < 1) return QL_ERR_SHAPE;
    if (K > K_MAX || M % R != 0) return QL_ERR_SHAPE;
    if (M > ELEMS_MAX / K || M > ELEMS_MAX / N || N > ELEMS_MAX / K) return QL_ERR_SHAPE;
    return QL_OK;
}

inline bool misaligned(const void *p, size_t a) { return p && ((uintptr_t)p % a) != 0; }

// DAQ scratch for R > 1.  Absmax: [block maxima M/R][partial maxima (M/R) * parts]; percentile: [tau patterns M/R]
// [selection histograms].  One size covers both, so a workspace serves either mode.  Its histograms are either the partial ones
// (what the sizing functions return) or, from DAQ_ROBUST_WORDS words per scale block on, those of the atomic selection.
enum class Scratch { full, atomic, least };
size_t daq_scratch_bytes(int64_t M, int64_t K, int64_t R, Scratch kind = Scratch::full)
{
    if (M < 1 || R <= 1 || M % R != 0) return 0;
    const size_t nblk = (size_t)(M / R);
    const size_t plain = align_up(nblk * ql::daq_parts_per_block(K, R) * 4, 256);
    const size_t parts = align_up(ql::daq_hist_bytes(M, K, R), 256), atomics = align_up(nblk * ql::DAQ_ROBUST_WORDS * 4, 256);
    const size_t robust = kind == Scratch::full ? parts : kind == Scratch::atomic || atomics < parts ? atomics : parts;
    return align_up(nblk * 4, 256) + (plain > robust ? plain : robust);
}

// eq. (4): rank from the top of the nearest-rank percentile, c = n - ceil(n p) + 1 with n = R*K values per scale block
int robust_args(const ql_daq_params *dp, int64_t K, int64_t R, ql::DaqArgs &d)
{
    if (dp->p_ppm < 1 || dp->p_ppm > 1000000 || dp->a_bits < 2 || dp->a_bits > 8) return QL_ERR_UNSUPPORTED;
    const int64_t n = R * K;
    if (n > (int64_t)1 << 31) return QL_ERR_SHAPE;
    int64_t k = (n * (int64_t)dp->p_ppm + 999999) / 1000000;
    if (k < 1) k = 1;
    if (k > n) k = n;
    d.top_rank = (unsigned)(n - k + 1);
    d.qmax = (1 << (dp->a_bits - 1)) - 1;
    return QL_OK;
}

// workspace layout of one layer: [codes M*K][scales M/R][DAQ scratch (R > 1)]
struct LayerWs {
    size_t q_off, s_off, bm_off, total;
};

LayerWs layer_ws(int64_t M, int64_t K, int64_t R, Scratch kind = Scratch::full)
{
    LayerWs w;
    w.q_off = 0;
    w.s_off = align_up((size_t)(M * K), 256);
    w.bm_off = w.s_off + align_up((size_t)(M / R) * 4, 256);
    w.total = w.bm_off + daq_scratch_bytes(M, K, R, kind);
    return w;
}

int check_workspace(void *ws, size_t have, size_t need)
{
    if (need == 0) return QL_OK;
    if (!ws || have < need) return QL_ERR_WORKSPACE;
    if ((uintptr_t)ws % 256 != 0) return QL_ERR_ALIGN;
    return QL_OK;
}

// 4-bit weight groups: a multiple of 32 that divides K (Step 2 / Algorithm 1 choose the size per layer)
int check_group(int64_t K, int64_t group)
{
    if (group < 32 || group % 32 != 0) return QL_ERR_UNSUPPORTED;
    if (K % group != 0 || K % 8 != 0) return QL_ERR_SHAPE;
    // the kernels multiply nibbles as value * 16: a group's sum of 127 * 128 * group must stay below 2^31
    if (group > W4_GROUP_MAX) return QL_ERR_SHAPE;
    return QL_OK;
}

inline bool overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes)
{
    return (uintptr_t)a < (uintptr_t)b + b_bytes && (uintptr_t)b < (uintptr_t)a + a_bytes;
}

// a layer's codes, scales and DAQ scratch in `bytes` of workspace
ql::DaqArgs daq_args(const void *x, int64_t M, int64_t K, int64_t R, unsigned char *base, size_t bytes)
{
    const LayerWs lw = layer_ws(M, K, R);
    const size_t blocks = align_up((size_t)(M / R) * 4, 256);
    ql::DaqArgs d{};
    d.x = x;
    d.q = reinterpret_cast<int8_t *>(base + lw.q_off);
    d.scales = reinterpret_cast<float *>(base + lw.s_off);
    if (R > 1) {
        d.blockmax = reinterpret_cast<unsigned *>(base + lw.bm_off);
        d.partmax = reinterpret_cast<unsigned *>(base + lw.bm_off + blocks);
        d.hist = d.partmax;
        d.scratch_bytes = bytes - lw.bm_off - blocks;
    }
    d.M = (int)M;
    d.K = (int)K;
    d.R = (int)R;
    return d;
}

// DAQ then GEMM for one layer; all arguments already validated
int run_layer(const void *x, int64_t M, int64_t K, int64_t R, int w_bits, const void *w, const void *w_scale,
              const void *bias, int64_t N, void *y, const ql_debug *dbg, void *workspace, size_t workspace_bytes, hipStream_t stream,
              const ql_daq_params *dp = nullptr, int64_t group = 128, const ql_fusion *fu = nullptr)
{
    if (w_bits == 16) {
        // a layer the plan leaves in FP16: no quantization, both operands binary16
        ql::GemmArgs g{};
        g.q = static_cast<const int8_t *>(x);
        g.w = w;
        g.bias = bias;
        g.y = y;
        g.M = (int)M;
        g.N = (int)N;
        g.K = (int)K;
        g.R = 1;
        g.w_bits = 16;
        g.group = 128;
        if (fu) {
            g.act = fu->act;
            g.residual = fu->residual;
            g.gate = fu->gate;
            g.gate_rows = (int)fu->gate_rows;
            g.row_absmax = static_cast<unsigned *>(fu->row_absmax);
        }
        if (g.row_absmax) {
            const int rc = device_status(ql::launch_fill_u32(g.row_absmax, (int)M, 0u, stream));
            if (rc) return rc;
        }
        return device_status(ql::launch_qgemm(g, g_gemm_variant.load(), stream));
    }
    ql::DaqArgs d = daq_args(x, M, K, R, static_cast<unsigned char *>(workspace), workspace_bytes);
    if (dbg && dbg->q) d.q = static_cast<int8_t *>(dbg->q);
    if (dbg && dbg->a_scales) d.scales = static_cast<float *>(dbg->a_scales);
    int rc;
    ql::GemmArgs g{};
    g.q = d.q;
    g.s_a = d.scales;
    g.w = w;
    g.s_w = w_scale;
    g.bias = bias;
    g.y = y;
    g.acc_out = dbg ? static_cast<int32_t *>(dbg->acc) : nullptr;
    g.M = (int)M;
    g.N = (int)N;
    g.K = (int)K;
    g.R = (int)R;
    g.w_bits = w_bits;
    g.group = (int)group;
    if (fu) {
        g.act = fu->act;
        g.residual = fu->residual;
        g.gate = fu->gate;
        g.gate_rows = (int)fu->gate_rows;
        g.row_absmax = static_cast<unsigned *>(fu->row_absmax);
    }
    if (g.row_absmax) {
        rc = device_status(ql::launch_fill_u32(g.row_absmax, (int)M, 0u, stream));
        if (rc) return rc;
    }
    const int variant = g_gemm_variant.load();
    const size_t parts = ql::daq_parts_per_block(K, R);
    if (!dp && !dbg && variant < 0 && (R == 1 || (parts > 0 && parts <= 256 && parts * (size_t)(M / R) * 4 <= d.scratch_bytes))) {
        // few rows: the GEMM's workgroups quantize their own rows (one launch; two where rows share a scale), unless the outputs
        // lie over the inputs that other workgroups still read
        ql::GemmArgs f = g;
        f.x = x;
        f.partmax = d.partmax;
        f.parts = R == 1 ? 0 : (int)parts;
        if (ql::qgemm_fuse_takes(f) && !overlap(x, (size_t)(M * K) * 2, y, (size_t)(M * N) * 2)) {
            if (R > 1) {
                rc = device_status(ql::launch_daq_part_absmax(d, stream));
                if (rc) return rc;
            }
            return device_status(ql::launch_qgemm_fused(f, stream));
        }
    }
    if (dp) {
        rc = robust_args(dp, K, R, d);
        if (rc) return rc;
        rc = device_status(ql::launch_daq_robust(d, stream));
    } else {
        rc = device_status(ql::launch_daq(d, stream));
    }
    if (rc) return rc;
    return device_status(ql::launch_qgemm(g, variant, stream));
}

// device address of `scratch` on the current device, looked up once per device
constexpr int NOALLOC_MAX_DEVICES = 64;
std::atomic<void *> g_scratch_ptr[NOALLOC_MAX_DEVICES];

int noalloc_scratch(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return device_status(e);
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return QL_ERR_UNSUPPORTED;
    void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return device_status(e);
        if (!p) return QL_ERR_DEVICE;
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return QL_OK;
}

int check_fusion(const ql_fusion *fu, int64_t M)
{
    if (!fu) return QL_OK;
    if (fu->act != QL_ACT_NONE && fu->act != QL_ACT_GELU_TANH) return QL_ERR_UNSUPPORTED;
    if (misaligned(fu->residual, 2) || misaligned(fu->gate, 2) || misaligned(fu->row_absmax, 4)) return QL_ERR_ALIGN;
    if (fu->gate && (fu->gate_rows < 1 || M % fu->gate_rows != 0)) return QL_ERR_SHAPE;
    return QL_OK;
}

int check_layer_ptrs(const void *x, const void *w, const void *w_scale, const void *bias, const void *y,
                     const ql_debug *dbg, int w_bits)
{
    if (!x || !w || !w_scale || !y) return QL_ERR_NULL;
    if (misaligned(x, 2) || misaligned(y, 2) || misaligned(bias, 2)) return QL_ERR_ALIGN;
    if (misaligned(w_scale, w_bits == 8 ? 4 : 2)) return QL_ERR_ALIGN;
    if (dbg && (misaligned(dbg->a_scales, 4) || misaligned(dbg->acc, 4))) return QL_ERR_ALIGN;
    return QL_OK;
}

int qlinear_any(int w_bits, const void *x, int64_t M, int64_t K, int64_t R, const void *w, const void *w_scale,
                const void *bias, int64_t N, void *y, const ql_debug *dbg, void *workspace, size_t workspace_bytes,
                void *stream, int64_t group = 128, const ql_fusion *fu = nullptr)
{
    int rc = check_layer_ptrs(x, w, w_scale, bias, y, dbg, w_bits);
    if (rc) return rc;
    rc = check_shape(M, K, R, N);
    if (rc) return rc;
    rc = check_fusion(fu, M);
    if (rc) return rc;
    if (w_bits == 4) {
        rc = check_group(K, group);
        if (rc) return rc;
        if (M > ELEMS_MAX / N / (K / group) && dbg && dbg->acc) return QL_ERR_SHAPE;
    }
    rc = check_workspace(workspace, workspace_bytes, layer_ws(M, K, R, Scratch::least).total);
    if (rc) return rc;
    return run_layer(x, M, K, R, w_bits, w, w_scale, bias, N, y, dbg, workspace, workspace_bytes, static_cast<hipStream_t>(stream),
                     nullptr, group, fu);
}

int qgemm_any(int w_bits, const void *q, const void *a_scales, int64_t M, int64_t K, int64_t R, const void *w,
              const void *w_scale, const void *bias, int64_t N, void *y, void *acc, void *stream, int64_t group = 128)
{
    if (!q || !a_scales || !w || !w_scale || !y) return QL_ERR_NULL;
    if (misaligned(a_scales, 4) || misaligned(y, 2) || misaligned(bias, 2) || misaligned(acc, 4) ||
        misaligned(w_scale, w_bits == 8 ? 4 : 2))
        return QL_ERR_ALIGN;
    int rc = check_shape(M, K, R, N);
    if (rc) return rc;
    if (w_bits == 4) {
        rc = check_group(K, group);
        if (rc) return rc;
        if (acc && M > ELEMS_MAX / N / (K / group)) return QL_ERR_SHAPE;
    }
    ql::GemmArgs g{};
    g.q = static_cast<const int8_t *>(q);
    g.s_a = static_cast<const float *>(a_scales);
    g.w = w;
    g.s_w = w_scale;
    g.bias = bias;
    g.y = y;
    g.acc_out = static_cast<int32_t *>(acc);
    g.M = (int)M;
    g.N = (int)N;
    g.K = (int)K;
    g.R = (int)R;
    g.w_bits = w_bits;
    g.group = (int)group;
    return device_status(ql::launch_qgemm(g, g_gemm_variant.load(), static_cast<hipStream_t>(stream)));
}

}  // namespace

namespace ql {

// Do the GEMMs of these layers give the same in any order?  No output overlaps another one's, or what another layer reads (codes and
// scales lie in the workspace).
bool any_order(const GemmArgs *g, size_t n)
{
    for (size_t i = 0; i < n; ++i) {
        const size_t y_bytes = (size_t)g[i].M * g[i].N * 2;
        for (size_t j = 0; j < n; ++j) {
            if (i == j) continue;
            const GemmArgs &o = g[j];
            const size_t w_elems = (size_t)o.N * o.K, scales = o.w_bits == 8 ? (size_t)o.N * 4 : o.w_bits == 4 ? (size_t)o.N * (o.K / o.group) * 2 : 0;
            if (overlap(g[i].y, y_bytes, o.y, (size_t)o.M * o.N * 2) || overlap(g[i].y, y_bytes, o.w, o.w_bits == 16 ? w_elems * 2 : o.w_bits == 8 ? w_elems : w_elems / 2) ||
                (scales && overlap(g[i].y, y_bytes, o.s_w, scales)) || (o.bias && overlap(g[i].y, y_bytes, o.bias, (size_t)o.N * 2)) ||
                (o.w_bits == 16 && overlap(g[i].y, y_bytes, o.q, (size_t)o.M * o.K * 2)))
                return false;
        }
    }
    return true;
}

void plan_window(const ql_layer_desc *layers, size_t n_layers, size_t first, const void *const *x_in, void *const *y_out, int64_t M, int64_t R,
                 const ql_daq_params *dp, void *workspace, size_t workspace_bytes, PlanWindow &w)
{
    unsigned char *base = static_cast<unsigned char *>(workspace);
    w.n = w.count = w.daq.count = 0;
    size_t used = 0, n = 0;
    int64_t codes = 0, outputs = 0;   // bytes; outputs: of the layers before this one
    for (; n < PLAN_WINDOW && first + n < n_layers; ++n) {
        const size_t l = first + n;
        const ql_layer_desc &d = layers[l];
        bool ready = true;
        for (size_t j = first; j < l; ++j)
            ready = ready && !overlap(x_in[l], (size_t)(M * d.K) * 2, y_out[j], (size_t)(M * layers[j].N) * 2);
        if (!ready) break;
        if (n > 0) outputs += M * layers[l - 1].N * 2;
        GemmArgs &a = w.g[n];
        a = GemmArgs{};
        a.w = d.w;
        a.s_w = d.w_scale;
        a.bias = d.bias;
        a.y = y_out[l];
        a.M = (int)M;
        a.N = (int)d.N;
        a.K = (int)d.K;
        a.R = d.w_bits == 16 ? 1 : (int)R;
        a.w_bits = d.w_bits;
        a.group = d.w_bits == 4 ? (int)d.group : 128;
        if (d.w_bits == 16) {
            a.q = static_cast<const int8_t *>(x_in[l]);
            continue;
        }
        const LayerWs lw = layer_ws(M, d.K, R);
        if (used + lw.total > workspace_bytes) break;
        codes += M * d.K;
        if (codes + outputs > PLAN_WINDOW_BYTES) break;
        DaqArgs it = daq_args(x_in[l], M, d.K, R, base + used, lw.total);
        if ((dp && robust_args(dp, d.K, R, it) != QL_OK) || !daq_many_takes(it, dp != nullptr)) break;
        a.q = it.q;
        a.s_a = it.scales;
        if (!dp) {
            GemmArgs f = a;
            f.x = x_in[l];
            f.partmax = it.partmax;
            f.parts = R == 1 ? 0 : (int)daq_parts_per_block(d.K, R);
            if (qgemm_fuse_one_tile(f)) break;
        }
        w.daq.l[w.daq.count++] = it;
        used += lw.total;
    }
    if (w.daq.count < 2) return;
    w.n = (int)n;
    // GEMMs that share a launch: none of the window's layers may read or write what another one writes
    if (any_order(w.g, n)) w.count = qgemm_many_choice(w.g, w.n, w.together);
}

}  // namespace ql

struct ql_plan {
    std::vector<ql_layer_desc> layers;
    int64_t M_max;
    int64_t K_widest;
};

extern "C" {

const char *ql_status_string(int status)
{
    switch (status) {
        case QL_OK: return "QL_OK";
        case QL_ERR_NULL: return "QL_ERR_NULL";
        case QL_ERR_SHAPE: return "QL_ERR_SHAPE";
        case QL_ERR_ALIGN: return "QL_ERR_ALIGN";
        case QL_ERR_UNSUPPORTED: return "QL_ERR_UNSUPPORTED";
        case QL_ERR_WORKSPACE: return "QL_ERR_WORKSPACE";
        case QL_ERR_DEVICE: return "QL_ERR_DEVICE";
        default: return "QL_ERR_?";
    }
}

int ql_last_device_error(void) { return g_last_device_error; }

int ql_version(void) { return 1000; }

size_t daq_workspace_bytes(int64_t M, int64_t K, int64_t R)
{
    return daq_scratch_bytes(M, K, R);
}

static int daq_any(const void *x, int64_t M, int64_t K, int64_t R, const ql_daq_params *dp, void *q, void *scales,
                   void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x || !q || !scales) return QL_ERR_NULL;
    if (misaligned(x, 2) || misaligned(scales, 4)) return QL_ERR_ALIGN;
    int rc = check_shape(M, K, R, 1);
    if (rc) return rc;
    ql::DaqArgs d{};
    if (dp) {
        rc = robust_args(dp, K, R, d);
        if (rc) return rc;
    }
    rc = check_workspace(workspace, workspace_bytes, daq_scratch_bytes(M, K, R, Scratch::least));
    if (rc) return rc;
    d.x = x;
    d.q = static_cast<int8_t *>(q);
    d.scales = static_cast<float *>(scales);
    d.blockmax = R > 1 ? static_cast<unsigned *>(workspace) : nullptr;
    d.partmax = R > 1 ? reinterpret_cast<unsigned *>(static_cast<unsigned char *>(workspace) + align_up((size_t)(M / R) * 4, 256))
                      : nullptr;
    d.hist = d.partmax;
    d.scratch_bytes = R > 1 ? workspace_bytes - align_up((size_t)(M / R) * 4, 256) : 0;
    d.M = (int)M;
    d.K = (int)K;
    d.R = (int)R;
    return device_status(dp ? ql::launch_daq_robust(d, static_cast<hipStream_t>(stream))
                            : ql::launch_daq(d, static_cast<hipStream_t>(stream)));
}

int daq_quantize(const void *x, int64_t M, int64_t K, int64_t R, void *q, void *scales, void *workspace,
                 size_t workspace_bytes, void *stream)
{
    return daq_any(x, M, K, R, nullptr, q, scales, workspace, workspace_bytes, stream);
}

int daq_quantize_robust(const void *x, int64_t M, int64_t K, int64_t R, const ql_daq_params *params, void *q, void *scales,
                        void *workspace, size_t workspace_bytes, void *stream)
{
    if (!params) return QL_ERR_NULL;
    return daq_any(x, M, K, R, params, q, scales, workspace, workspace_bytes, stream);
}

int daq_quantize_rowmax(const void *x, int64_t M, int64_t K, int64_t R, const void *row_absmax, void *q, void *scales,
                        void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x || !q || !scales || !row_absmax) return QL_ERR_NULL;
    if (misaligned(x, 2) || misaligned(scales, 4) || misaligned(row_absmax, 4)) return QL_ERR_ALIGN;
    int rc = check_shape(M, K, R, 1);
    if (rc) return rc;
    rc = check_workspace(workspace, workspace_bytes, daq_scratch_bytes(M, K, R, Scratch::least));
    if (rc) return rc;
    ql::DaqArgs d{};
    d.x = x;
    d.q = static_cast<int8_t *>(q);
    d.scales = static_cast<float *>(scales);
    d.blockmax = R > 1 ? static_cast<unsigned *>(workspace) : nullptr;
    d.M = (int)M;
    d.K = (int)K;
    d.R = (int)R;
    return device_status(ql::launch_daq_from_rowmax(d, static_cast<const unsigned *>(row_absmax), static_cast<hipStream_t>(stream)));
}

// ---- plan-space generality: channel-group activation scales, int8-held codes of any width with group scales ----------
static int check_act_group(int64_t K, int64_t ag)
{
    if (ag < 8 || ag % 8 != 0) return QL_ERR_UNSUPPORTED;
    if (K % 8 != 0 || K % ag != 0 || K / ag > 1024) return QL_ERR_SHAPE;
    return QL_OK;
}

// one word per scale: the scales themselves, and the scratch from which on the atomic kernels run
static size_t cg_scales_bytes(int64_t M, int64_t K, int64_t R, int64_t act_group)
{
    return align_up((size_t)(M / R) * (size_t)(K / act_group) * 4, 256);
}

size_t daq_cg_workspace_bytes(int64_t M, int64_t K, int64_t R, int64_t act_group)
{
    if (M < 1 || K < 1 || R < 1 || M % R != 0 || act_group < 1 || K % act_group != 0) return 0;
    const int64_t slab = ql::daq_cg_slab_rows(R);
    return align_up((size_t)(M / (slab ? slab : R)) * (size_t)(K / act_group) * 4, 256);
}

int daq_quantize_cg(const void *x, int64_t M, int64_t K, int64_t R, int64_t act_group, void *q, void *scales, void *workspace,
                    size_t workspace_bytes, void *stream)
{
    if (!x || !q || !scales) return QL_ERR_NULL;
    if (misaligned(x, 16) || misaligned(q, 8) || misaligned(scales, 4)) return QL_ERR_ALIGN;
    int rc = check_shape(M, K, R, 1);
    if (rc) return rc;
    rc = check_act_group(K, act_group);
    if (rc) return rc;
    rc = check_workspace(workspace, workspace_bytes, cg_scales_bytes(M, K, R, act_group));
    if (rc) return rc;
    ql::DaqArgs d{};
    d.x = x;
    d.q = static_cast<int8_t *>(q);
    d.scales = static_cast<float *>(scales);
    d.blockmax = static_cast<unsigned *>(workspace);
    d.M = (int)M;
    d.K = (int)K;
    d.R = (int)R;
    const bool slabs = workspace_bytes >= daq_cg_workspace_bytes(M, K, R, act_group);
    return device_status(ql::launch_daq_cg(d, (int)act_group, slabs, static_cast<hipStream_t>(stream)));
}

size_t qlinear_grouped_workspace_bytes(int64_t M, int64_t K, int64_t R, int64_t act_group)
{
    if (M < 1 || K < 1 || R < 1 || M % R != 0) return 0;
    if (act_group <= 0) return layer_ws(M, K, R).total;
    if (K % act_group != 0) return 0;
    return align_up((size_t)(M * K), 256) + cg_scales_bytes(M, K, R, act_group) + daq_cg_workspace_bytes(M, K, R, act_group);
}

int qlinear_grouped(const void *x, int64_t M, int64_t K, int64_t R, int64_t act_group, const void *w, int32_t w_storage,
                    const void *w_scale, int64_t group, const void *bias, int64_t N, void *y, const ql_debug *dbg,
                    void *workspace, size_t workspace_bytes, void *stream)
{
    if (w_storage != 4 && w_storage != 8) return QL_ERR_UNSUPPORTED;
    int rc = check_layer_ptrs(x, w, w_scale, bias, y, dbg, 4);
    if (rc) return rc;
    rc = check_shape(M, K, R, N);
    if (rc) return rc;
    rc = check_group(K, group);
    if (rc) return rc;
    if (act_group != 0 && act_group != group) return QL_ERR_UNSUPPORTED;   // the channel groups are the weight groups
    if (act_group != 0) {
        rc = check_act_group(K, act_group);
        if (rc) return rc;
        if (misaligned(x, 16)) return QL_ERR_ALIGN;
    }
    if (dbg && dbg->acc && M > ELEMS_MAX / N / (K / group)) return QL_ERR_SHAPE;
    const size_t full = qlinear_grouped_workspace_bytes(M, K, R, act_group);
    rc = check_workspace(workspace, workspace_bytes, act_group == 0 ? layer_ws(M, K, R, Scratch::least).total
                                                                   : align_up((size_t)(M * K), 256) + 2 * cg_scales_bytes(M, K, R, act_group));
    if (rc) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    unsigned char *base = static_cast<unsigned char *>(workspace);
    ql::GemmArgs g{};
    if (act_group == 0) {
        const LayerWs lw = layer_ws(M, K, R);
        ql::DaqArgs d{};
        d.x = x;
        d.q = (dbg && dbg->q) ? static_cast<int8_t *>(dbg->q) : reinterpret_cast<int8_t *>(base + lw.q_off);
        d.scales = (dbg && dbg->a_scales) ? static_cast<float *>(dbg->a_scales) : reinterpret_cast<float *>(base + lw.s_off);
        d.blockmax = R > 1 ? reinterpret_cast<unsigned *>(base + lw.bm_off) : nullptr;
        d.partmax = R > 1 ? reinterpret_cast<unsigned *>(base + lw.bm_off + align_up((size_t)(M / R) * 4, 256)) : nullptr;
        d.scratch_bytes = R > 1 ? workspace_bytes - lw.bm_off - align_up((size_t)(M / R) * 4, 256) : 0;
        d.M = (int)M;
        d.K = (int)K;
        d.R = (int)R;
        rc = device_status(ql::launch_daq(d, s));
        if (rc) return rc;
        g.q = d.q;
        g.s_a = d.scales;
    } else {
        const size_t cgb = cg_scales_bytes(M, K, R, act_group);
        ql::DaqArgs d{};
        d.x = x;
        d.q = (dbg && dbg->q) ? static_cast<int8_t *>(dbg->q) : reinterpret_cast<int8_t *>(base);
        d.scales = (dbg && dbg->a_scales) ? static_cast<float *>(dbg->a_scales) : reinterpret_cast<float *>(base + align_up((size_t)(M * K), 256));
        d.blockmax = reinterpret_cast<unsigned *>(base + align_up((size_t)(M * K), 256) + cgb);
        d.M = (int)M;
        d.K = (int)K;
        d.R = (int)R;
        rc = device_status(ql::launch_daq_cg(d, (int)act_group, workspace_bytes >= full, s));
        if (rc) return rc;
        g.q = d.q;
        g.s_ag = d.scales;
    }
    g.w = w;
    g.s_w = w_scale;
    g.bias = bias;
    g.y = y;
    g.acc_out = dbg ? static_cast<int32_t *>(dbg->acc) : nullptr;
    g.M = (int)M;
    g.N = (int)N;
    g.K = (int)K;
    g.R = (int)R;
    g.w_bits = w_storage;
    g.w_grouped = w_storage == 8 ? 1 : 0;
    g.group = (int)group;
    return device_status(ql::launch_qgemm(g, g_gemm_variant.load(), s));
}

int ql_pack_bits_host(const int8_t *codes, int64_t N, int64_t K, int32_t bits, uint8_t *packed)
{
    if (!codes || !packed) return QL_ERR_NULL;
    if (bits < 2 || bits > 7) return QL_ERR_UNSUPPORTED;
    if (N < 1 || K < 1 || (K * bits) % 8 != 0) return QL_ERR_SHAPE;
    const int64_t row_bytes = K * bits / 8;
    const int lo = -(1 << (bits - 1)), hi = (1 << (bits - 1)) - 1;
    for (int64_t n = 0; n < N; ++n) {
        uint8_t *dst = packed + n * row_bytes;
        for (int64_t i = 0; i < row_bytes; ++i) dst[i] = 0;
        for (int64_t k = 0; k < K; ++k) {
            const int c = codes[n * K + k];
            if (c < lo || c > hi) return QL_ERR_SHAPE;
            const unsigned u = (unsigned)c & ((1u << bits) - 1);
            for (int b = 0; b < bits; ++b)
                if (u >> b & 1) dst[(k * bits + b) / 8] |= (uint8_t)(1u << ((k * bits + b) % 8));
        }
    }
    return QL_OK;
}

int ql_unpack_bits_host(const uint8_t *packed, int64_t N, int64_t K, int32_t bits, int8_t *codes)
{
    if (!codes || !packed) return QL_ERR_NULL;
    if (bits < 2 || bits > 7) return QL_ERR_UNSUPPORTED;
    if (N < 1 || K < 1 || (K * bits) % 8 != 0) return QL_ERR_SHAPE;
    const int64_t row_bytes = K * bits / 8;
    for (int64_t n = 0; n < N; ++n) {
        const uint8_t *src = packed + n * row_bytes;
        for (int64_t k = 0; k < K; ++k) {
            int u = 0;
            for (int b = 0; b < bits; ++b) u |= ((src[(k * bits + b) / 8] >> ((k * bits + b) % 8)) & 1) << b;
            codes[n * K + k] = (int8_t)(u >= (1 << (bits - 1)) ? u - (1 << bits) : u);
        }
    }
    return QL_OK;
}

int ql_zero_point_fold_host(const int8_t *codes, const int32_t *zeros, int64_t N, int64_t K, int64_t group, int8_t *out)
{
    if (!codes || !zeros || !out) return QL_ERR_NULL;
    if (N < 1 || K < 1 || group < 1 || K % group != 0) return QL_ERR_SHAPE;
    const int64_t G = K / group;
    for (int64_t n = 0; n < N; ++n)
        for (int64_t k = 0; k < K; ++k) {
            const int d = (int)codes[n * K + k] - zeros[n * G + k / group];
            if (d < -127 || d > 127) return QL_ERR_UNSUPPORTED;   // 8-bit codes with a zero point do not fit
            out[n * K + k] = (int8_t)d;
        }
    return QL_OK;
}

int daq_quantize_ln(const void *x, int64_t M, int64_t K, int64_t R, const void *shift, const void *scale, int64_t rows_per_mod,
                    float eps, void *h, void *q, void *scales, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x || (!q && !h) || (q && !scales)) return QL_ERR_NULL;
    if (misaligned(x, 16) || misaligned(shift, 16) || misaligned(scale, 16) || misaligned(h, 16) || misaligned(q, 8) ||
        misaligned(scales, 4))
        return QL_ERR_ALIGN;
    int rc = check_shape(M, K, R, 1);
    if (rc) return rc;
    if (K % 8 != 0 || K > 4608 || !(eps >= 0.0f)) return QL_ERR_SHAPE;
    if ((shift || scale) && (rows_per_mod < 1 || M % rows_per_mod != 0)) return QL_ERR_SHAPE;
    if (R > 1 && q && !h) return QL_ERR_NULL;    // several rows per scale: the normalised rows are staged in h
    if (R > 1 && q) {
        rc = check_workspace(workspace, workspace_bytes, daq_scratch_bytes(M, K, R, Scratch::least));
        if (rc) return rc;
    }
    ql::LnDaqArgs a{};
    a.x = x;
    a.shift = shift;
    a.scale = scale;
    a.h = h;
    a.q = R == 1 ? static_cast<int8_t *>(q) : nullptr;
    a.scales = static_cast<float *>(scales);
    a.M = (int)M;
    a.K = (int)K;
    a.rows_per_mod = (shift || scale) ? (int)rows_per_mod : 1;
    a.eps = eps;
    rc = device_status(ql::launch_daq_ln(a, static_cast<hipStream_t>(stream)));
    if (rc || R == 1 || !q) return rc;
    return daq_any(h, M, K, R, nullptr, q, scales, workspace, workspace_bytes, stream);
}

int ql_time_bin(int64_t step, int64_t num_steps)
{
    if (num_steps < 1 || step < 0 || step >= num_steps) return -1;
    return (int)(step * 3 / num_steps);
}

size_t qlinear_workspace_bytes(int64_t M, int64_t K, int64_t R)
{
    if (M < 1 || K < 1 || R < 1 || M % R != 0) return 0;
    return layer_ws(M, K, R).total;
}

int qlinear_w8a8(const void *x, int64_t M, int64_t K, int64_t R, const void *w, const void *w_scale,
                 const void *bias, int64_t N, void *y, const ql_debug *dbg, void *workspace, size_t workspace_bytes,
                 void *stream)
{
    return qlinear_any(8, x, M, K, R, w, w_scale, bias, N, y, dbg, workspace, workspace_bytes, stream);
}

size_t qlinear_noalloc_max_bytes(void) { return QL_NOALLOC_SCRATCH_BYTES; }

int qlinear_w8a8_noalloc(const void *x, int64_t M, int64_t K, int64_t R, const void *w, const void *w_scale,
                         const void *bias, int64_t N, void *y, void *stream)
{
    int rc = check_layer_ptrs(x, w, w_scale, bias, y, nullptr, 8);
    if (rc) return rc;
    rc = check_shape(M, K, R, N);
    if (rc) return rc;
    if (layer_ws(M, K, R, Scratch::atomic).total > QL_NOALLOC_SCRATCH_BYTES) return QL_ERR_WORKSPACE;
    void *ws = nullptr;
    rc = noalloc_scratch(&ws);
    if (rc) return rc;
    // nothing in the scratch has to start at zero: codes, scales and partial maxima are written before they are read
    // (the atomic-maximum fallback of the DAQ pass clears its block maxima with a fill kernel of its own)
    return run_layer(x, M, K, R, 8, w, w_scale, bias, N, y, nullptr, ws, QL_NOALLOC_SCRATCH_BYTES, static_cast<hipStream_t>(stream));
}

int qlinear_w4a8(const void *x, int64_t M, int64_t K, int64_t R, const void *w4, const void *w_scale,
                 const void *bias, int64_t N, void *y, const ql_debug *dbg, void *workspace, size_t workspace_bytes,
                 void *stream)
{
    return qlinear_any(4, x, M, K, R, w4, w_scale, bias, N, y, dbg, workspace, workspace_bytes, stream);
}

int qlinear_w4a8_g(const void *x, int64_t M, int64_t K, int64_t R, const void *w4, const void *w_scale, int64_t group,
                   const void *bias, int64_t N, void *y, const ql_debug *dbg, void *workspace, size_t workspace_bytes,
                   void *stream)
{
    return qlinear_any(4, x, M, K, R, w4, w_scale, bias, N, y, dbg, workspace, workspace_bytes, stream, group);
}

int qlinear_w8a8_fused(const void *x, int64_t M, int64_t K, int64_t R, const void *w, const void *w_scale, const void *bias,
                       int64_t N, const ql_fusion *fusion, void *y, void *workspace, size_t workspace_bytes, void *stream)
{
    return qlinear_any(8, x, M, K, R, w, w_scale, bias, N, y, nullptr, workspace, workspace_bytes, stream, 128, fusion);
}

int qlinear_w4a8_fused(const void *x, int64_t M, int64_t K, int64_t R, const void *w4, const void *w_scale, int64_t group,
                       const void *bias, int64_t N, const ql_fusion *fusion, void *y, void *workspace,
                       size_t workspace_bytes, void *stream)
{
    return qlinear_any(4, x, M, K, R, w4, w_scale, bias, N, y, nullptr, workspace, workspace_bytes, stream, group, fusion);
}

int qlinear_f16(const void *x, int64_t M, int64_t K, const void *w, const void *bias, int64_t N, const ql_fusion *fusion,
                void *y, void *stream)
{
    if (!x || !w || !y) return QL_ERR_NULL;
    if (misaligned(x, 2) || misaligned(w, 2) || misaligned(y, 2) || misaligned(bias, 2)) return QL_ERR_ALIGN;
    int rc = check_shape(M, K, 1, N);
    if (rc) return rc;
    rc = check_fusion(fusion, M);
    if (rc) return rc;
    return run_layer(x, M, K, 1, 16, w, nullptr, bias, N, y, nullptr, nullptr, 0, static_cast<hipStream_t>(stream), nullptr, 128,
                     fusion);
}

int qgemm_w4a8_g(const void *q, const void *a_scales, int64_t M, int64_t K, int64_t R, const void *w4,
                 const void *w_scale, int64_t group, const void *bias, int64_t N, void *y, void *acc, void *stream)
{
    return qgemm_any(4, q, a_scales, M, K, R, w4, w_scale, bias, N, y, acc, stream, group);
}

int qgemm_w8a8(const void *q, const void *a_scales, int64_t M, int64_t K, int64_t R, const void *w,
               const void *w_scale, const void *bias, int64_t N, void *y, void *acc, void *stream)
{
    return qgemm_any(8, q, a_scales, M, K, R, w, w_scale, bias, N, y, acc, stream);
}

int qgemm_w4a8(const void *q, const void *a_scales, int64_t M, int64_t K, int64_t R, const void *w4,
               const void *w_scale, const void *bias, int64_t N, void *y, void *acc, void *stream)
{
    return qgemm_any(4, q, a_scales, M, K, R, w4, w_scale, bias, N, y, acc, stream);
}

int ql_pack_w4_host(const int8_t *codes, int64_t N, int64_t K, uint8_t *packed)
{
    if (!codes || !packed) return QL_ERR_NULL;
    if (N < 1 || K < 1 || K % 8 != 0) return QL_ERR_SHAPE;
    for (int64_t n = 0; n < N; ++n) {
        const int8_t *src = codes + n * K;
        uint8_t *dst = packed + n * (K / 2);
        for (int64_t blk = 0; blk < K / 8; ++blk)
            for (int j = 0; j < 4; ++j) {
                const int lo = src[8 * blk + j], hi = src[8 * blk + 4 + j];
                if (lo < -8 || lo > 7 || hi < -8 || hi > 7) return QL_ERR_SHAPE;
                dst[4 * blk + j] = (uint8_t)((lo & 0xf) | ((hi & 0xf) << 4));
            }
    }
    return QL_OK;
}

int ql_repack_w4_pairs_host(const uint8_t *pairs, int64_t N, int64_t K, uint8_t *packed)
{
    if (!pairs || !packed) return QL_ERR_NULL;
    if (pairs == packed) return QL_ERR_UNSUPPORTED;
    if (N < 1 || K < 1 || K % 8 != 0) return QL_ERR_SHAPE;
    for (int64_t n = 0; n < N; ++n) {
        const uint8_t *src = pairs + n * (K / 2);   // byte i: k = 2i in the low nibble, k = 2i+1 in the high nibble
        uint8_t *dst = packed + n * (K / 2);
        auto nib = [&](int64_t k) { return (uint8_t)((k & 1) ? (src[k / 2] >> 4) : (src[k / 2] & 0xf)); };
        for (int64_t blk = 0; blk < K / 8; ++blk)
            for (int j = 0; j < 4; ++j) dst[4 * blk + j] = (uint8_t)(nib(8 * blk + j) | (nib(8 * blk + 4 + j) << 4));
    }
    return QL_OK;
}

int ql_prepack_w4(const void *pairs, int64_t N, int64_t K, void *packed, void *stream)
{
    if (!pairs || !packed) return QL_ERR_NULL;
    if (pairs == packed) return QL_ERR_UNSUPPORTED;
    if (N < 1 || K < 1 || K % 8 != 0 || N * K / 8 > ((int64_t)1 << 31) * 256 - 256) return QL_ERR_SHAPE;
    if (misaligned(pairs, 4) || misaligned(packed, 4)) return QL_ERR_ALIGN;
    return device_status(ql::launch_prepack_w4(pairs, packed, N * K / 8, static_cast<hipStream_t>(stream)));
}

int ql_plan_create(const ql_layer_desc *layers, int32_t n_layers, int64_t M_max, ql_plan **plan_out)
{
    if (!layers || !plan_out) return QL_ERR_NULL;
    *plan_out = nullptr;
    if (n_layers < 1 || M_max < 1) return QL_ERR_SHAPE;
    int64_t widest = 0;
    for (int32_t l = 0; l < n_layers; ++l) {
        const ql_layer_desc &d = layers[l];
        if (d.w_bits != 8 && d.w_bits != 4 && d.w_bits != 16) return QL_ERR_UNSUPPORTED;
        if (d.w_bits != 4 && d.group != 0) return QL_ERR_UNSUPPORTED;
        if (!d.w || (!d.w_scale && d.w_bits != 16)) return QL_ERR_NULL;
        if (d.w_bits == 16 && misaligned(d.w, 2)) return QL_ERR_ALIGN;
        int rc = check_shape(M_max, d.K, 1, d.N);
        if (rc) return rc;
        if (d.w_bits == 4) {
            rc = check_group(d.K, d.group);
            if (rc) return rc;
        }
        if ((d.w_bits != 16 && misaligned(d.w_scale, d.w_bits == 8 ? 4 : 2)) || misaligned(d.bias, 2)) return QL_ERR_ALIGN;
        widest = d.K > widest ? d.K : widest;
    }
    ql_plan *p = new (std::nothrow) ql_plan;
    if (!p) return QL_ERR_WORKSPACE;
    p->layers.assign(layers, layers + n_layers);
    p->M_max = M_max;
    p->K_widest = widest;
    *plan_out = p;
    return QL_OK;
}

void ql_plan_destroy(ql_plan *plan) { delete plan; }

int32_t ql_plan_num_layers(const ql_plan *plan) { return plan ? (int32_t)plan->layers.size() : 0; }

size_t ql_plan_workspace_bytes(const ql_plan *plan, int64_t M, int64_t R)
{
    if (!plan || M < 1 || R < 1 || M % R != 0 || M > plan->M_max) return 0;
    // the widest layer's, unless a narrower one cuts its scale blocks into parts and the widest (K % 8 != 0) does not
    size_t most = 0;
    for (const ql_layer_desc &d : plan->layers) most = d.w_bits != 16 || d.K == plan->K_widest ? std::max(most, layer_ws(M, d.K, R).total) : most;
    return most;
}

// the launches of a window
static int plan_run_window(ql::PlanWindow &w, bool robust, hipStream_t stream)
{
    int rc = device_status(robust ? ql::launch_daq_robust_many(w.daq, stream) : ql::launch_daq_many(w.daq, stream));
    if (w.count && rc == QL_OK) rc = device_status(ql::launch_qgemm_many(w.together, w.count, stream));
    for (int i = 0; i < w.n && rc == QL_OK; ++i) {
        bool done = false;
        for (int j = 0; j < w.count; ++j) done = done || w.together[j] == &w.g[i];
        if (!done) rc = device_status(ql::launch_qgemm(w.g[i], -1, stream));
    }
    return rc;
}

static int plan_run_any(const ql_plan *plan, const void *const *x_in, void *const *y_out, int64_t M, int64_t R,
                        const ql_daq_params *dp, void *workspace, size_t workspace_bytes, void *stream,
                        const ql_fusion *const *fusion = nullptr)
{
    if (!plan || !x_in || !y_out) return QL_ERR_NULL;
    if (M < 1 || R < 1 || M % R != 0 || M > plan->M_max) return QL_ERR_SHAPE;
    if (dp && (dp->p_ppm < 1 || dp->p_ppm > 1000000 || dp->a_bits < 2 || dp->a_bits > 8)) return QL_ERR_UNSUPPORTED;
    for (size_t l = 0; l < plan->layers.size(); ++l) {
        if (!x_in[l] || !y_out[l]) return QL_ERR_NULL;
        if (misaligned(x_in[l], 2) || misaligned(y_out[l], 2)) return QL_ERR_ALIGN;
    }
    int rc = check_workspace(workspace, workspace_bytes, layer_ws(M, plan->K_widest, R, Scratch::least).total);
    if (rc) return rc;
    if (fusion)
        for (size_t l = 0; l < plan->layers.size(); ++l) {
            rc = check_fusion(fusion[l], M);
            if (rc) return rc;
        }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool windows = !fusion && g_gemm_variant.load() < 0;
    for (size_t l = 0; l < plan->layers.size(); ++l) {
        if (windows) {
            ql::PlanWindow w;
            ql::plan_window(plan->layers.data(), plan->layers.size(), l, x_in, y_out, M, R, dp, workspace, workspace_bytes, w);
            if (w.n) {
                rc = plan_run_window(w, dp != nullptr, s);
                if (rc) return rc;
                l += (size_t)w.n - 1;
                continue;
            }
        }
        const ql_layer_desc &d = plan->layers[l];
        rc = run_layer(x_in[l], M, d.K, R, d.w_bits, d.w, d.w_scale, d.bias, d.N, y_out[l], nullptr, workspace, workspace_bytes, s, dp,
                       d.w_bits == 4 ? d.group : 128, fusion ? fusion[l] : nullptr);
        if (rc) return rc;
    }
    return QL_OK;
}

int qlinear_plan_run(const ql_plan *plan, const void *const *x_in, void *const *y_out, int64_t M, int64_t R,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    return plan_run_any(plan, x_in, y_out, M, R, nullptr, workspace, workspace_bytes, stream);
}

int qlinear_plan_run_ex(const ql_plan *plan, const void *const *x_in, void *const *y_out, int64_t M, int64_t R,
                        const ql_daq_params *params, const ql_fusion *const *fusion, void *workspace, size_t workspace_bytes,
                        void *stream)
{
    return plan_run_any(plan, x_in, y_out, M, R, params, workspace, workspace_bytes, stream, fusion);
}

int qlinear_plan_run_robust(const ql_plan *plan, const void *const *x_in, void *const *y_out, int64_t M, int64_t R,
                            const ql_daq_params *params, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!params) return QL_ERR_NULL;
    return plan_run_any(plan, x_in, y_out, M, R, params, workspace, workspace_bytes, stream);
}

int ql_set_gemm_variant(int variant)
{
    if (variant < -1 || variant > ql::num_gemm_variants()) return QL_ERR_UNSUPPORTED;
    g_gemm_variant.store(variant);
    return QL_OK;
}

int ql_num_gemm_variants(void) { return ql::num_gemm_variants(); }

const char *ql_gemm_variant_name(int variant) { return ql::gemm_variant_name(variant); }

}  // extern "C"
