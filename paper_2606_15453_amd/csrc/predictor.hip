// Spatio-temporal expert predictor (Section 4.2): Cross-layer Correlation
// Tables with 2-bit confidences and a per-layer History Table.
//
// Tables live in HBM and are small (for 94 layers x 128 experts x top-8:
// 94 KB of CCT indices and 94 KB of confidences), so the runtime kernels run
// as a single workgroup each: the update gives every selected expert's entry
// a lane group, one lane per slot, and the prediction sums K x K contributions
// into per-row score bins in LDS with integer atomics, which is exact and
// order-free.
#include <algorithm>
#include <memory>
#include <new>
#include <vector>

#include "gating_dev.h"
#include "predictor_dev.h"


namespace stmoe {
namespace {

using namespace pred;

constexpr int kThreads = 256;    // of the profiling kernels and the decode path's

// ---------------------------------------------------------------- profiling
constexpr int kCountThreads = 1024;
constexpr int kCountSlice = 8192;     // counts a workgroup holds in LDS

// Rows of Co_i one workgroup counts: as many as fit its LDS counts.
inline int count_rows(int E) { return std::min(E, kCountSlice / E); }

// Algorithm 1: one workgroup counts `rows` rows of Co_i (blockIdx.y = i) over a
// chunk of n profiling tokens, in LDS, and after the last chunk selects
// CCT_i[e] from them: the K largest counts of Co_i[e][*] (equal counts ->
// lower index), all with confidence "10", one wave per row.  Counting into
// global memory with an atomic per pair took 45 us (48 layers of 128 experts,
// 512 rows of top-8), clearing it 6 and a selection launch 17.5; this takes
// the place of all three.
__global__ __launch_bounds__(kCountThreads) void co_build_kernel(const int32_t* sel, int n, int B, int L, int E, int K,
                                                                 int rows, int first, int last, int32_t* co,
                                                                 size_t stride, uint8_t* idx, uint8_t* conf) {
    __shared__ int32_t cnt[kCountSlice];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = blockIdx.y;
    const int e0 = blockIdx.x * rows, nr = min(rows, E - e0);
    int32_t* out = co + (size_t(i) * E + e0) * E;
    for (int t = tid; t < nr * E; t += kCountThreads) cnt[t] = first ? 0 : out[t];
    __syncthreads();
    for (int t = tid; t < n * B * K; t += kCountThreads) {
        const int pb = t / K;
        const int32_t* row = sel + (size_t(pb) * L + i) * K;
        const int e = row[t - pb * K] - e0;
        if (e < 0 || e >= nr) continue;
        for (int s = 0; s < K; ++s) atomicAdd(&cnt[e * E + row[K + s]], 1);
    }
    __syncthreads();
    for (int t = tid; t < nr * E; t += kCountThreads) out[t] = cnt[t];
    if (!last) return;
    for (int r = wave; r < nr; r += kCountThreads / 64) {
        uint32_t key[gating::kKeyRegs];
        bool ok[gating::kKeyRegs], win[gating::kKeyRegs];
        int pos[gating::kKeyRegs];
#pragma unroll
        for (int v = 0; v < gating::kKeyRegs; ++v) {
            const int f = 64 * v + lane;
            ok[v] = f < E;
            key[v] = ok[v] ? uint32_t(cnt[r * E + f]) : 0u;
        }
        gating::topk_positions(key, ok, E, K, win, pos);
        const size_t at = size_t(i) * stride + size_t(e0 + r) * K;
#pragma unroll
        for (int v = 0; v < gating::kKeyRegs; ++v)
            if (win[v]) {
                idx[at + pos[v]] = uint8_t(64 * v + lane);
                conf[at + pos[v]] = uint8_t(kConfInit);
            }
    }
}

// Sort one K-row of distinct expert indices ascending into dst (by ranking).
__device__ __forceinline__ void sorted_row(const int32_t* src, int K, uint8_t* dst) {
    for (int k = threadIdx.x; k < K; k += kThreads) {
        const int v = src[k];
        int rank = 0;
        for (int j = 0; j < K; ++j) rank += src[j] < v;
        dst[rank] = uint8_t(v);
    }
}

__global__ __launch_bounds__(kThreads) void ht_init_kernel(const int32_t* sel_last, int B, int L,
                                                           int K, size_t stride, uint8_t* ht) {
    const int l = blockIdx.x, b = blockIdx.y;
    sorted_row(sel_last + (size_t(b) * L + l) * K, K, ht + size_t(l) * stride + size_t(b) * K);
}

// ------------------------------------------------------ update and predict
template <int T>
__global__ __launch_bounds__(T) void update_kernel(UpdateArgs a) {
    __shared__ TableShared sh;
    Seg g[kMaxSegs];
    update_init<T>(sh);
    stage<T>(g, update_segs(a, sh, g));
    update_body<T>(a, sh);
}

template <int T>
__global__ __launch_bounds__(T) void predict_kernel(PredictArgs a) {
    __shared__ TableShared sh;
    Seg g[kMaxSegs];
    stage<T>(g, predict_segs(a, sh, g));
    predict_body<T>(a, sh);
}

// The decode path's router tail, verify/update and next-layer prediction in
// one workgroup (after the router's logits launch).  One round of loads
// brings the logits and every table into LDS; softmax/top-K writes the
// selection there, and the update and the prediction run on it.
template <int T>
__global__ __launch_bounds__(T) void route_update_predict_kernel(gating::RouteArgs r, UpdateArgs u,
                                                                        PredictArgs p) {
    __shared__ TableShared sh;
    Seg g[kMaxSegs];
    u.sel_cur = nullptr;     // the selection is produced in LDS
    p.sel_cur = nullptr;
    int n = 0;
    g[n++] = seg(r.zbuf, sh.z, size_t(r.B) * r.E * sizeof(float));
    update_init<T>(sh);
    n += update_segs(u, sh, g + n);
    n += predict_segs(p, sh, g + n);
    stage<T>(g, n);
    gating::softmax_topk_tail<T>(r, sh.z, sh.sel);
    update_body<T>(u, sh);
    // with one layer the prediction reads the HT row the update just wrote
    if (p.ht_next && p.ht_next == u.ht)
        for (int i = threadIdx.x; i < r.B * r.K; i += T) sh.htn[i] = sh.htnew[i];
    __syncthreads();
    predict_body<T>(p, sh);
}

// The decode path's verify/update and next-layer prediction without the
// router (the selection is read from global memory): used where the router
// runs as its own launches and this work overlaps the expert FFN.
template <int T>
__global__ __launch_bounds__(T) void update_predict_kernel(UpdateArgs u, PredictArgs p) {
    __shared__ TableShared sh;
    Seg g[kMaxSegs];
    p.sel_cur = nullptr;     // the update's copy of the selection serves both
    int n = 0;
    update_init<T>(sh);
    n += update_segs(u, sh, g + n);
    n += predict_segs(p, sh, g + n);
    stage<T>(g, n);
    update_body<T>(u, sh);
    // with one layer the prediction reads the HT row the update just wrote
    if (p.ht_next && p.ht_next == u.ht)
        for (int i = threadIdx.x; i < u.B * u.K; i += T) sh.htn[i] = sh.htnew[i];
    __syncthreads();
    predict_body<T>(p, sh);
}

// One layer's arguments of the sequential kernel below.
struct UpdPred {
    UpdateArgs u;
    PredictArgs p;
};

// The verify/update and next-layer prediction of every layer of one token,
// in layer order, in one workgroup: each layer runs the steps of
// update_predict_kernel on the arguments built for it; the barrier between
// layers orders the tables one layer writes before the next layer stages
// them.
// The arguments are built for both prediction sources with the online
// update on; `use` and `online` select the ablation at launch time.
template <int T>
__global__ __launch_bounds__(T) void update_predict_seq_kernel(const UpdPred* args, int n, int use,
                                                                      int online) {
    __shared__ TableShared sh;
    for (int l = 0; l < n; ++l) {
        UpdateArgs u = args[l].u;
        PredictArgs p = args[l].p;
        u.online = online;
        if (!(use & STMOE_USE_CCT)) {
            p.cidx = nullptr;
            p.cconf = nullptr;
        }
        if (!(use & STMOE_USE_HT)) p.ht_next = nullptr;
        Seg g[kMaxSegs];
        p.sel_cur = nullptr;     // the update's copy of the selection serves both
        int k = 0;
        update_init<T>(sh);
        k += update_segs(u, sh, g + k);
        k += predict_segs(p, sh, g + k);
        stage<T>(g, k);
        update_body<T>(u, sh);
        if (p.ht_next && p.ht_next == u.ht)
            for (int i = threadIdx.x; i < u.B * u.K; i += T) sh.htn[i] = sh.htnew[i];
        __syncthreads();
        predict_body<T>(p, sh);
        __syncthreads();
    }
}

// Launch a standalone predictor kernel with the threads its shape takes.
#define STMOE_PRED_LAUNCH(kernel, B, K, stream, args)                                             \
    do {                                                                                          \
        if (wide(B, K)) hipLaunchKernelGGL((kernel<1024>), dim3(1), dim3(1024), 0, stream, args); \
        else hipLaunchKernelGGL((kernel<256>), dim3(1), dim3(256), 0, stream, args);              \
    } while (0)

int check_sel_host(const int32_t* sel, size_t rows, int E, int K) {
    for (size_t r = 0; r < rows; ++r) {
        const int32_t* row = sel + r * K;
        for (int k = 0; k < K; ++k) {
            STMOE_CHECK(row[k] >= 0 && row[k] < E, "selection index out of range");
            for (int j = 0; j < k; ++j) STMOE_CHECK(row[j] != row[k], "selection row has a repeated expert");
        }
    }
    return STMOE_OK;
}

}  // namespace
}  // namespace stmoe

using namespace stmoe;

namespace {

// Layout of a predictor's device workspace: every table at a 256-byte
// aligned offset, then the staging area of the profiling selections (at
// least one token's [B][L][K], at least 1 MiB).
struct PredLayout {
    size_t co, cct_idx, cct_conf, ht, pend, stats, stage, stage_bytes, total;
};

size_t align256(size_t n) { return (n + 255) / 256 * 256; }

PredLayout pred_layout(int L, int E, int K, int B) {
    PredLayout y{};
    const size_t pairs = size_t(L > 1 ? L - 1 : 1);
    size_t off = 0;
    auto take = [&](size_t n) { const size_t at = off; off = align256(off + n); return at; };
    y.co = take(pairs * E * E * sizeof(int32_t));
    y.cct_idx = take(pairs * round4(size_t(E) * K));
    y.cct_conf = take(pairs * round4(size_t(E) * K));
    y.ht = take(size_t(L) * round4(size_t(B) * K));
    y.pend = take(size_t(L) * round4(size_t(B) * E));
    y.stats = take(size_t(L) * 3 * sizeof(unsigned long long));
    const size_t token = size_t(B) * L * K * sizeof(int32_t);
    y.stage_bytes = std::max(token, size_t(1) << 20) / token * token;
    y.stage = take(y.stage_bytes);
    y.total = off;
    return y;
}

int check_shape(int L, int E, int K, int B) {
    STMOE_CHECK(L >= 1 && L <= 4096, "L must be in [1, 4096]");
    STMOE_CHECK(E >= 1 && E <= kMaxE, "E must be in [1, 256]");
    STMOE_CHECK(K >= 1 && K <= E && K <= kMaxK, "K must be in [1, min(E, 16)]");
    STMOE_CHECK(B >= 1 && B <= kMaxB, "B must be in [1, 16]");
    return STMOE_OK;
}

}  // namespace

extern "C" size_t stmoe_workspace_bytes(int L, int E, int K, int B) {
    if (check_shape(L, E, K, B) != STMOE_OK) return 0;
    return pred_layout(L, E, K, B).total;
}

extern "C" int stmoe_create(int L, int E, int K, int B, void* dev_ws, size_t ws_bytes, stmoe_predictor** out) {
    clear_error();
    STMOE_CHECK(out && dev_ws, "null pointer");
    if (int rc = check_shape(L, E, K, B)) return rc;
    const PredLayout y = pred_layout(L, E, K, B);
    STMOE_CHECK(ws_bytes >= y.total, "workspace smaller than stmoe_workspace_bytes()");
    STMOE_CHECK(reinterpret_cast<uintptr_t>(dev_ws) % 256 == 0, "workspace must be 256-byte aligned");
    char* base = static_cast<char*>(dev_ws);
    auto* p = new stmoe_predictor();
    p->L = L; p->E = E; p->K = K; p->B = B;
    p->profiled = false;
    p->cct_stride = round4(size_t(E) * K);
    p->ht_stride = round4(size_t(B) * K);
    p->pend_stride = round4(size_t(B) * E);
    p->co = reinterpret_cast<int32_t*>(base + y.co);
    p->cct_idx = reinterpret_cast<uint8_t*>(base + y.cct_idx);
    p->cct_conf = reinterpret_cast<uint8_t*>(base + y.cct_conf);
    p->ht = reinterpret_cast<uint8_t*>(base + y.ht);
    p->pend = reinterpret_cast<uint8_t*>(base + y.pend);
    p->stats = reinterpret_cast<unsigned long long*>(base + y.stats);
    p->stage = reinterpret_cast<int32_t*>(base + y.stage);
    p->stage_bytes = y.stage_bytes;
    hipError_t e = hipMemset(dev_ws, 0, y.stage);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        set_error(std::string("stmoe_create: ") + hipGetErrorString(e));
        delete p;
        return STMOE_EHIP;
    }
    *out = p;
    return STMOE_OK;
}

extern "C" int stmoe_destroy(stmoe_predictor* p) {
    delete p;       // the tables live in the caller's workspace
    return STMOE_OK;
}

extern "C" int stmoe_profile(stmoe_predictor* p, const int32_t* sel, int P) {
    clear_error();
    STMOE_CHECK(p && sel, "null pointer");
    STMOE_CHECK(P >= 1, "P must be >= 1");
    const int L = p->L, E = p->E, K = p->K, B = p->B;
    if (int rc = check_sel_host(sel, size_t(P) * B * L, E, K)) return rc;
    const size_t tok = size_t(B) * L * K;                 // int32 per profiling token
    const int chunk = int(p->stage_bytes / (tok * sizeof(int32_t)));
    const int rows = count_rows(E);
    // the legacy null stream orders the blocking copies and the kernels
    hipError_t e = hipMemset(p->pend, 0, size_t(L) * p->pend_stride);
    if (e == hipSuccess) e = hipMemset(p->stats, 0, size_t(L) * 3 * sizeof(unsigned long long));
    int last_at = 0;
    for (int t0 = 0; t0 < P && e == hipSuccess; t0 += chunk) {
        const int n = std::min(chunk, P - t0);
        e = hipMemcpy(p->stage, sel + size_t(t0) * tok, size_t(n) * tok * sizeof(int32_t), hipMemcpyHostToDevice);
        if (e == hipSuccess && L > 1) {
            hipLaunchKernelGGL(co_build_kernel, dim3(unsigned((E + rows - 1) / rows), unsigned(L - 1)),
                               dim3(kCountThreads), 0, 0, p->stage, n, B, L, E, K, rows, t0 == 0, t0 + n == P, p->co,
                               p->cct_stride, p->cct_idx, p->cct_conf);
            e = hipGetLastError();
        }
        last_at = P - 1 - t0;                             // the last token's row within the final chunk
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(ht_init_kernel, dim3(L, B), dim3(kThreads), 0, 0, p->stage + size_t(last_at) * tok,
                           B, L, K, p->ht_stride, p->ht);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        set_error(std::string("stmoe_profile: ") + hipGetErrorString(e));
        return STMOE_EHIP;
    }
    p->profiled = true;
    return STMOE_OK;
}

extern "C" int stmoe_update(stmoe_predictor* p, int layer, const int32_t* sel_prev,
                            const int32_t* sel_cur, int online, void* stream) {
    clear_error();
    STMOE_CHECK(p && sel_cur, "null pointer");
    STMOE_CHECK(layer >= 0 && layer < p->L, "layer out of range");
    STMOE_CHECK(layer == 0 || sel_prev, "sel_prev is required for layer >= 1");
    if (!p->profiled) {
        set_error("stmoe_update: predictor has not been profiled");
        return STMOE_ESTATE;
    }
    const UpdateArgs a = update_args(p, layer, sel_prev, sel_cur, online);
    STMOE_PRED_LAUNCH(update_kernel, p->B, p->K, as_stream(stream), a);
    STMOE_LAUNCHED();
    return STMOE_OK;
}

extern "C" int stmoe_predict(stmoe_predictor* p, int layer, const int32_t* sel_cur, int use,
                             uint8_t* score, uint8_t* mask, uint8_t* max_score, int32_t* ranked,
                             int32_t* n_ranked, void* stream) {
    clear_error();
    STMOE_CHECK(p, "null predictor");
    STMOE_CHECK(layer >= -1 && layer < p->L - 1, "layer must be in [-1, L-2]");
    STMOE_CHECK((use & ~STMOE_USE_BOTH) == 0, "use must be a STMOE_USE_* bit set");
    const bool cct = (use & STMOE_USE_CCT) && layer >= 0;
    STMOE_CHECK(!cct || sel_cur, "sel_cur is required when the CCT is used");
    if (!p->profiled) {
        set_error("stmoe_predict: predictor has not been profiled");
        return STMOE_ESTATE;
    }
    const PredictArgs a = predict_args(p, layer, sel_cur, use, score, mask, max_score, ranked, n_ranked);
    STMOE_PRED_LAUNCH(predict_kernel, p->B, p->K, as_stream(stream), a);
    STMOE_LAUNCHED();
    return STMOE_OK;
}

namespace stmoe {
int launch_route_logits(const gating::RouteArgs& a, hipStream_t s);

// Internal: router + verify/update at `layer` + prediction of the next layer
// (layer 0 of the next token after the last layer) in two launches.  The
// caller has validated the shapes; the routing workspace follows
// moe_route_workspace_bytes.
int fused_route_predict(const void* x, const void* w_gate, int H, int dtype, int renorm, int32_t* idx,
                        float* w, void* route_ws, stmoe_predictor* p, int layer, const int32_t* sel_prev,
                        int use, int online, int32_t* ranked, int32_t* n_ranked, uint8_t* max_score,
                        hipStream_t s) {
    if (!p->profiled) {
        set_error("moe_decode_layer: predictor has not been profiled");
        return STMOE_ESTATE;
    }
    gating::RouteArgs r;
    r.x = x;
    r.wg = w_gate;
    r.B = p->B;
    r.H = H;
    r.E = p->E;
    r.K = p->K;
    r.renorm = renorm ? 1 : 0;
    r.bf16 = dtype == STMOE_BF16;
    r.idx = idx;
    r.w = w;
    r.logits = nullptr;
    r.zbuf = reinterpret_cast<float*>(route_ws);
    const UpdateArgs u = update_args(p, layer, sel_prev, idx, online);
    const PredictArgs q = layer + 1 < p->L
                              ? predict_args(p, layer, idx, use, nullptr, nullptr, max_score, ranked, n_ranked)
                              : predict_args(p, -1, nullptr, use & STMOE_USE_HT, nullptr, nullptr, max_score,
                                             ranked, n_ranked);
    if (int rc = launch_route_logits(r, s)) return rc;
    hipLaunchKernelGGL((route_update_predict_kernel<kThreads>), dim3(1), dim3(kThreads), 0, s, r, u, q);
    STMOE_LAUNCHED();
    return STMOE_OK;
}
}  // namespace stmoe

extern "C" int stmoe_export(stmoe_predictor* p, int32_t* co, uint8_t* cct_idx, uint8_t* cct_conf,
                            int32_t* ht) {
    clear_error();
    STMOE_CHECK(p, "null predictor");
    const size_t pairs = size_t(p->L > 1 ? p->L - 1 : 0);
    STMOE_HIP(hipDeviceSynchronize());
    if (co && pairs)
        STMOE_HIP(hipMemcpy(co, p->co, pairs * p->E * p->E * sizeof(int32_t), hipMemcpyDeviceToHost));
    const size_t ek = size_t(p->E) * p->K, bk = size_t(p->B) * p->K;
    // a table whose rows lie close together comes in one copy; a pitched copy
    // to pageable memory goes row by row (48 layers of 128 experts,
    // batch 8: profile and export together 1668 us so, 564 in single copies)
    auto fetch = [&](uint8_t* dst, const uint8_t* src, size_t row, size_t stride, size_t n) -> int {
        if (row == stride) {
            STMOE_HIP(hipMemcpy(dst, src, n * row, hipMemcpyDeviceToHost));
            return STMOE_OK;
        }
        const std::unique_ptr<uint8_t[]> all(new (std::nothrow) uint8_t[n * stride]);
        if (!all) {
            set_error("stmoe_export: out of host memory");
            return STMOE_ENOMEM;
        }
        STMOE_HIP(hipMemcpy(all.get(), src, n * stride, hipMemcpyDeviceToHost));
        for (size_t i = 0; i < n; ++i) std::copy_n(all.get() + i * stride, row, dst + i * row);
        return STMOE_OK;
    };
    if (cct_idx && pairs)
        if (int rc = fetch(cct_idx, p->cct_idx, ek, p->cct_stride, pairs)) return rc;
    if (cct_conf && pairs)
        if (int rc = fetch(cct_conf, p->cct_conf, ek, p->cct_stride, pairs)) return rc;
    if (ht) {
        std::vector<uint8_t> h(size_t(p->L) * bk);
        if (int rc = fetch(h.data(), p->ht, bk, p->ht_stride, size_t(p->L))) return rc;
        for (size_t i = 0; i < h.size(); ++i) ht[i] = h[i];
    }
    return STMOE_OK;
}

extern "C" int stmoe_import(stmoe_predictor* p, const uint8_t* cct_idx, const uint8_t* cct_conf,
                            const int32_t* ht) {
    clear_error();
    STMOE_CHECK(p && cct_idx && cct_conf && ht, "null pointer");
    const int E = p->E, K = p->K;
    const size_t pairs = size_t(p->L > 1 ? p->L - 1 : 0);
    // an entry names K distinct experts (Algorithm 1 builds it so and Algorithm 3
    // keeps it so), which bounds every Eq. 1 score by 3K + 2
    for (size_t r = 0; r < pairs * E; ++r) {
        const uint8_t* row = cct_idx + r * K;
        for (int k = 0; k < K; ++k) {
            STMOE_CHECK(row[k] < E, "CCT index out of range");
            STMOE_CHECK(cct_conf[r * K + k] <= 3, "CCT confidence out of range");
            for (int j = 0; j < k; ++j) STMOE_CHECK(row[j] != row[k], "CCT entry repeats an expert");
        }
    }
    const size_t bk = size_t(p->B) * K;
    std::vector<uint8_t> h(size_t(p->L) * bk);
    for (size_t r = 0; r < size_t(p->L) * p->B; ++r) {
        const int32_t* row = ht + r * K;
        for (int k = 0; k < K; ++k) {
            STMOE_CHECK(row[k] >= 0 && row[k] < E, "HT index out of range");
            for (int j = 0; j < k; ++j) STMOE_CHECK(row[j] != row[k], "HT row repeats an expert");
        }
        // HT rows are kept sorted ascending
        std::vector<int32_t> v(row, row + K);
        std::sort(v.begin(), v.end());
        for (int k = 0; k < K; ++k) h[r * K + k] = uint8_t(v[size_t(k)]);
    }
    STMOE_HIP(hipDeviceSynchronize());
    const size_t ek = size_t(E) * K;
    if (pairs) {
        STMOE_HIP(hipMemcpy2D(p->cct_idx, p->cct_stride, cct_idx, ek, ek, pairs, hipMemcpyHostToDevice));
        STMOE_HIP(hipMemcpy2D(p->cct_conf, p->cct_stride, cct_conf, ek, ek, pairs, hipMemcpyHostToDevice));
    }
    STMOE_HIP(hipMemcpy2D(p->ht, p->ht_stride, h.data(), bk, bk, p->L, hipMemcpyHostToDevice));
    p->profiled = true;
    return STMOE_OK;
}

extern "C" int stmoe_stats(stmoe_predictor* p, int64_t* out) {
    clear_error();
    STMOE_CHECK(p && out, "null pointer");
    STMOE_HIP(hipDeviceSynchronize());
    STMOE_HIP(hipMemcpy(out, p->stats, size_t(p->L) * 3 * sizeof(int64_t), hipMemcpyDeviceToHost));
    return STMOE_OK;
}

namespace stmoe {
// Internal: verify/update at `layer` from the selection sel_cur (device
// [B][K]) + prediction of the next layer, one launch on `s`.  The caller has
// validated the shapes.
int update_predict(stmoe_predictor* p, int layer, const int32_t* sel_prev, const int32_t* sel_cur,
                   int use, int online, int32_t* ranked, int32_t* n_ranked, uint8_t* max_score,
                   hipStream_t s) {
    if (!p->profiled) {
        set_error("moe_decode_layer: predictor has not been profiled");
        return STMOE_ESTATE;
    }
    const UpdateArgs u = update_args(p, layer, sel_prev, sel_cur, online);
    const PredictArgs q = layer + 1 < p->L
                              ? predict_args(p, layer, sel_cur, use, nullptr, nullptr, max_score, ranked, n_ranked)
                              : predict_args(p, -1, nullptr, use & STMOE_USE_HT, nullptr, nullptr, max_score,
                                             ranked, n_ranked);
    hipLaunchKernelGGL((update_predict_kernel<kThreads>), dim3(1), dim3(kThreads), 0, s, u, q);
    STMOE_LAUNCHED();
    return STMOE_OK;
}
}  // namespace stmoe

namespace stmoe {
// Internal: device bytes of the per-layer arguments of update_predict_seq.
size_t update_predict_seq_bytes(int L) { return size_t(L) * sizeof(UpdPred); }

// Internal: build the arguments of every layer for the selections idx_all
// (device [L][B][K]) into dev_args (device, update_predict_seq_bytes(L)),
// for both prediction sources with the online update on; synchronous.
int update_predict_seq_args(stmoe_predictor* p, const int32_t* idx_all, void* dev_args) {
    std::vector<UpdPred> v(size_t(p->L));
    const size_t bk = size_t(p->B) * p->K;
    for (int l = 0; l < p->L; ++l) {
        const int32_t* cur = idx_all + size_t(l) * bk;
        const int32_t* prev = l > 0 ? idx_all + size_t(l - 1) * bk : nullptr;
        v[size_t(l)].u = update_args(p, l, prev, cur, 1);
        v[size_t(l)].p = l + 1 < p->L
                             ? predict_args(p, l, cur, STMOE_USE_BOTH, nullptr, nullptr, nullptr, nullptr, nullptr)
                             : predict_args(p, -1, nullptr, STMOE_USE_HT, nullptr, nullptr, nullptr, nullptr,
                                            nullptr);
    }
    STMOE_HIP(hipMemcpy(dev_args, v.data(), v.size() * sizeof(UpdPred), hipMemcpyHostToDevice));
    return STMOE_OK;
}

// Internal: one token's verify/update and predictions for every layer, in
// layer order, one launch on `s` (the arguments from update_predict_seq_args).
int update_predict_seq(stmoe_predictor* p, const void* dev_args, int use, int online, hipStream_t s) {
    if (!p->profiled) {
        set_error("moe_decode_token: predictor has not been profiled");
        return STMOE_ESTATE;
    }
    hipLaunchKernelGGL((update_predict_seq_kernel<kThreads>), dim3(1), dim3(kThreads), 0, s,
                       static_cast<const UpdPred*>(dev_args), p->L, use, online ? 1 : 0);
    STMOE_LAUNCHED();
    return STMOE_OK;
}

// Internal: the shape a predictor was created with (checked by moe_ctx_create).
void stmoe_shape(const stmoe_predictor* p, int* L, int* E, int* K, int* B) {
    *L = p->L;
    *E = p->E;
    *K = p->K;
    *B = p->B;
}
}  // namespace stmoe
