// extern "C" boundary of the PM-LSH library: argument validation (before any
// HIP call), error codes, the thread-local error message, and the host-side
// orchestration of the ANN batches.

#include <algorithm>
#include <cmath>
#include <cstring>

#include "internal.hpp"

namespace pmlsh {

pmlsh_index* index_build(const pmlsh_build_args* a);
void index_release(pmlsh_index* x);
double index_default_r_min(const pmlsh_index* x, int64_t budget);
void run_acp(const pmlsh_index* x, int k, double c, double confidence, double beta,
             int64_t* out_pairs, float* out_dist, pmlsh_acp_stats* stats,
             hipStream_t stream);
void run_acp_bb(const pmlsh_index* x, int k, double c, double confidence, double beta,
                int64_t* out_pairs, float* out_dist, pmlsh_acp_stats* stats,
                hipStream_t stream);
void run_acp_lca(const pmlsh_index* x, int k, double c, double confidence, double beta,
                 double gamma, int64_t* out_pairs, float* out_dist, pmlsh_acp_stats* stats,
                 double* gamma_used, hipStream_t st);
void export_nodes(const pmlsh_index* x, int32_t* level, int32_t* first_leaf, int32_t* end_leaf,
                  float* radius);

namespace {
thread_local std::string g_error;
}

void set_error(const std::string& msg) { g_error = msg; }
void clear_error() { g_error.clear(); }
const char* error_cstr() { return g_error.c_str(); }
[[noreturn]] void fail(int code, const std::string& msg) { throw Error{code, msg}; }

// Per-query workspace bytes of the ANN kernel and the batch that fits a cap.
constexpr int64_t kWorkspaceCap = int64_t(4) << 30;

namespace {

// Workspace layout sizes of one ANN call: per query: projection, FP16 scan
// row, C, top-k scratch, and for the batched path three counters, a
// candidate region and the lower distance bounds of C; plus, for the batched
// path, the chunk distances, chosen chunks and the chunk x query mask (a
// 64-bit word per chunk and 64 queries, both layouts); plus the frontier
// lists of the per-query kernel's workgroups.
// All: budgets above kLeanBudget take the batched path too, and long candidate
// lists keep their pd^2 bits in memory. Short: neither. Least: besides, the pools
// hold what an exact filter needs.
enum class Pools { All, Short, Least };
struct AnnWorkspace {
    int64_t B, pool_q, per_query, nchunk, batch, slots, bytes;
    Pools pools;
    bool fast;
    bool vals;   // pd^2 bits kept per pool entry
};

// Most workgroups of the per-query kernel, each with its own pair of frontier
// lists: few on the batched path, which hands single queries over; more when
// every query takes the per-query path, and for large budgets, whose queries
// are handed over all together where the filter's widened radius overflows
// their pools (1M x 256 without contrast, BF16 filter, 1,024 queries of B =
// 5,000: 64 ms a call with 2,048 workgroups, 105 with 256).
int64_t front_slots_most(const AnnWorkspace& w) {
    return w.fast && w.B <= kLeanBudget ? 256 : 2048;
}
int64_t front_slots(const pmlsh_index* x, const AnnWorkspace& w, int64_t batch) {
    const int64_t by_memory = std::max<int64_t>(1, (int64_t(1) << 30) / (8 * x->n_leaves));
    return std::min<int64_t>({batch, front_slots_most(w), by_memory});
}

// Bytes of the workspace layout for batches of `batch` queries and `slots`
// frontier-list pairs (unrounded).
int64_t ann_layout_bytes(const pmlsh_index* x, const AnnWorkspace& w, int64_t batch,
                         int64_t slots) {
    const int64_t mask_bytes =
        w.fast ? batch * 8 + 2 * cdist_elems(batch, w.nchunk) +
                     (w.nchunk + 255) / 256 * 256 * ((batch + 63) / 64) * 8 + 64
               : 0;
    return batch * w.per_query + mask_bytes + slots * 2 * x->n_leaves * 4;
}

AnnWorkspace ann_workspace_base(const pmlsh_index* x, int k, int64_t B, Pools pools = Pools::All) {
    const bool wide = pools == Pools::All;
    AnnWorkspace w{};
    w.B = B;
    w.pools = pools;
    // the batched path, unless the budget exceeds its limit, the index's scan rows
    // cannot be formed or the plain FP32 path is switched on (read once per
    // call: layout and launch agree)
    w.fast = ann_fast_path(B) && x->scan_ok && tune_get(PMLSH_TUNE_FP32_PATH) == 0 &&
             (wide || B <= kLeanBudget);
    w.vals = w.fast && wide;
    w.pool_q = w.fast ? ann_pool_per_query(*x, B, pools == Pools::Least) : 0;
    w.per_query = (int64_t)MP * 8 + 64 + B * 8 + 3 * (int64_t)k * 4 +
                  (w.fast ? 4 * 4 + w.pool_q * (w.vals ? 8 : 4) + B * 4 : 0) +
                  (w.fast && x->filter_gemm ? (MP + 1) * 4 : 0);
    w.nchunk = x->n_pad16 / 64;
    return w;
}

// The batch, the frontier lists and the bytes of a layout.
void ann_workspace_size(const pmlsh_index* x, int64_t batch, AnnWorkspace* w) {
    w->batch = std::min<int64_t>(batch, 65535);
    w->slots = front_slots(x, *w, w->batch);
    w->bytes = ann_layout_bytes(x, *w, w->batch, w->slots);
    // sizes rounded up (to 1 MiB, or 64 MiB above 256 MiB) so that calls of
    // different batch sizes reuse the same pool blocks
    const int64_t q = w->bytes > (int64_t(256) << 20) ? int64_t(64) << 20 : int64_t(1) << 20;
    w->bytes = (w->bytes + q - 1) / q * q;
}

// The layout that a launch of nq queries starts from. Budgets above kLeanBudget of a
// few thousand points hold most of them: many such queries are faster one workgroup
// each on the per-query kernel (batched / per-query, us: 2,500 x 256, B = 2,060, 1,000
// queries 295 / 180, 30 queries 103 / 85; without contrast 320 / 389 and 101 / 162; 3,000
// x 16, B = 3,000 315 / 261 and 99 / 127; 4,000 x 16, B = 2,500 289 / 282 and 98 / 159,
// without contrast 305 / 305 and 100 / 149).
Pools pools_of(const pmlsh_index* x, int64_t nq, int64_t B) {
    return B > kLeanBudget && x->n <= 3072 && nq > 256 ? Pools::Short : Pools::All;
}

AnnWorkspace ann_workspace(const pmlsh_index* x, int64_t nq, int k, int64_t B, Pools pools) {
    AnnWorkspace w = ann_workspace_base(x, k, B, pools);
    // per query, with the distance blocks of a 64-query band spread over it
    const int64_t per_query_all =
        w.per_query + (w.fast ? 8 + 2 * (64 * cdist_groups(w.nchunk) + cdist_gmin_len(w.nchunk)) +
                                    (w.nchunk + 7) / 8
                              : 0);
    ann_workspace_size(x, std::max<int64_t>(1, std::min<int64_t>(nq, kWorkspaceCap / per_query_all)),
                       &w);
    return w;
}

// The next smaller layout, for a device that has no memory for w: half the
// queries per batch, then shorter pools. False when there is none.
bool ann_workspace_smaller(const pmlsh_index* x, int k, AnnWorkspace* w) {
    if (w->batch > 1) {
        ann_workspace_size(x, w->batch / 2, w);
        return true;
    }
    if (!w->fast || w->pools == Pools::Least) return false;
    *w = ann_workspace_base(x, k, w->B, w->vals ? Pools::Short : Pools::Least);
    ann_workspace_size(x, 1, w);
    return true;
}

// The workspace of one call, as large a layout as the device has memory for.
void* ann_workspace_alloc(const pmlsh_index* x, int64_t nq, int k, int64_t B, Pools pools,
                          hipStream_t st, AnnWorkspace* w) {
    *w = ann_workspace(x, nq, k, B, pools);
    return ws_alloc_least(
        w->bytes, st, [&](int64_t* bytes) {
            const bool more = ann_workspace_smaller(x, k, w);
            *bytes = w->bytes;
            return more;
        });
}

// Layout that fits a fixed region of cap bytes: at most a quarter of it for
// the frontier lists, the largest batch that fits in the rest. batch = 0
// when not even one query fits.
AnnWorkspace ann_workspace_in(const pmlsh_index* x, int64_t nq, int k, int64_t B, int64_t cap,
                              Pools pools) {
    AnnWorkspace w = ann_workspace_base(x, k, B, pools);
    const int64_t per_slot = 2 * x->n_leaves * 4;
    int64_t slots = std::min<int64_t>(front_slots_most(w), (cap / 4) / per_slot);
    slots = std::max<int64_t>(slots, 1);
    int64_t lo = 0, hi = std::min<int64_t>(nq, 65535);
    while (lo < hi) {   // largest batch with bytes <= cap
        const int64_t mid = (lo + hi + 1) / 2;
        if (ann_layout_bytes(x, w, mid, std::min(slots, mid)) <= cap) lo = mid;
        else hi = mid - 1;
    }
    w.batch = lo;
    w.slots = std::min(slots, std::max<int64_t>(lo, 1));
    w.bytes = lo > 0 ? ann_layout_bytes(x, w, w.batch, w.slots) : 0;
    return w;
}

// As ann_workspace_in for a region of a launch; shorter pools where those leave no
// room for a single query.
AnnWorkspace ann_workspace_region(const pmlsh_index* x, int64_t nq, int k, int64_t B, int64_t bytes,
                                  Pools pools) {
    AnnWorkspace w = ann_workspace_in(x, nq, k, B, bytes, pools);
    if (w.batch < 1 && pools == Pools::All) w = ann_workspace_in(x, nq, k, B, bytes, Pools::Short);
    if (w.batch < 1) w = ann_workspace_in(x, nq, k, B, bytes, Pools::Least);
    return w;
}

}  // namespace

void validate_ann(const pmlsh_index* index, const float* queries, int64_t nq, int k,
                  const int64_t* out_ids, const float* out_dist, double r_min) {
    if (!index) fail(PMLSH_EINVAL, "index is NULL");
    if (nq < 0) fail(PMLSH_EINVAL, "nq must be >= 0");
    if (nq > 0 && (!queries || !out_ids || !out_dist))
        fail(PMLSH_EINVAL, "queries and outputs must not be NULL");
    if (k < 1) fail(PMLSH_EINVAL, "k must be >= 1");
    if (k > index->n) fail(PMLSH_EINVAL, "k must be <= n");
    if (k > PMLSH_MAX_K) fail(PMLSH_EUNSUPPORTED, "k above PMLSH_MAX_K");
    if (index->d_pad > 8192) fail(PMLSH_EUNSUPPORTED, "ANN supports d <= 8192");
    if (std::isnan(r_min)) fail(PMLSH_EINVAL, "r_min is NaN");
}

int64_t ann_workspace_bytes(const pmlsh_index* x, int64_t nq, int k, double c,
                            double confidence, double beta) {
    pmlsh_plan plan;
    plan_params(x->n, x->m, k, c, confidence, beta, &plan);
    return nq > 0 ? ann_workspace(x, nq, k, plan.budget, pools_of(x, nq, plan.budget)).bytes : 0;
}

namespace {

// Parameters of one ANN call: the same for every query, or per query from
// the device array qpar (then k and budget are the largest of the call).
struct AnnCall {
    int k;
    int64_t budget;
    double c, t, r_min;
    const AnnQueryParams* qpar;
    int out_stride;
    int max_rounds;
    double ball_most = 0.0;   // as in AnnLaunch
};

// The batches of one ANN call over the workspace region ws laid out by w.
void run_ann_region(const pmlsh_index* x, const float* queries, int64_t nq, const AnnCall& call,
                    int64_t* out_ids, float* out_dist, int32_t* out_stats, hipStream_t st,
                    const AnnWorkspace& w, void* ws) {
    const int k = call.k;
    const int stride = call.out_stride > 0 ? call.out_stride : k;
    const int64_t B = w.B, pool_q = w.pool_q, nchunk = w.nchunk, batch = w.batch;
    const bool fast = w.fast;
    char* base = static_cast<char*>(ws);
    // projections and FP16 scan rows first: every row starts on a 64-byte
    // boundary
    float* qproj = reinterpret_cast<float*>(base);
    float* qproj_lo = qproj + batch * MP;
    uint16_t* qaug = reinterpret_cast<uint16_t*>(qproj_lo + batch * MP);
    uint16_t* cdist2 = qaug + batch * 32;
    uint16_t* cgmin = cdist2 + (fast ? cdist_block_elems(batch, nchunk) : 0);
    float2* qtest = reinterpret_cast<float2*>(cdist2 + (fast ? cdist_elems(batch, nchunk) : 0));
    uint64_t* cmask = reinterpret_cast<uint64_t*>(qtest + (fast ? batch : 0));
    uint32_t* list = reinterpret_cast<uint32_t*>(
        cmask + (fast ? (nchunk + 255) / 256 * 256 * ((batch + 63) / 64) : 0));
    uint32_t* vals = list + batch * pool_q;
    int32_t* front = reinterpret_cast<int32_t*>(vals + (w.vals ? batch * pool_q : 0));
    int32_t* cpos = front + w.slots * 2 * x->n_leaves;
    float* cdist = reinterpret_cast<float*>(cpos + batch * B);
    int32_t* topk = reinterpret_cast<int32_t*>(cdist + batch * B);
    float* clo = reinterpret_cast<float*>(topk + batch * 3 * (int64_t)k);
    int32_t* q_flag = reinterpret_cast<int32_t*>(clo + (fast ? batch * B : 0));
    int32_t* q_order = q_flag + batch;
    uint32_t* q_scanned = reinterpret_cast<uint32_t*>(q_order + batch);
    // count, then the queries the batched path hands to the per-query kernel
    uint32_t* pq_list = q_scanned + batch;
    // low-precision query projections and their bounds (filter_gemm)
    float* qlp = reinterpret_cast<float*>(pq_list + batch + 1);
    float* qeps = qlp + batch * MP;
    const bool lp = fast && x->filter_gemm != 0;
    for (int64_t q0 = 0; q0 < nq; q0 += batch) {
        const int64_t nb = std::min(batch, nq - q0);
        const float* qb = queries + q0 * x->d;
        {
            StageTimer tm(PMLSH_STAGE_PROJECT, st);
            launch_project(qb, nb, x->d, x->d, x->hash, qproj, qproj_lo, st);
            if (lp) launch_project_lp(qb, nb, x->d, x->d, x->hash, x->filter_gemm, qlp, qeps, st);
        }
        AnnLaunch L{};
        L.idx = x;
        L.queries = qb;
        L.qproj = qproj;
        L.qproj_lo = qproj_lo;
        L.nq = nb;
        L.k = k;
        L.c = call.c;
        L.t = call.t;
        L.r_min = call.r_min;
        L.max_rounds = call.max_rounds;
        L.budget = B;
        L.qpar = call.qpar ? call.qpar + q0 : nullptr;
        L.out_stride = stride;
        L.fast = fast;
        L.ball_most = call.ball_most;
        L.ws_front = front;
        L.front_slots = std::min<int64_t>(w.slots, nb);
        L.ws_cpos = cpos;
        L.ws_cdist = cdist;
        L.ws_topk = topk;
        if (fast) {
            L.ws_qaug = qaug;
            L.ws_qtest = qtest;
            L.ws_clo = clo;
            L.ws_cmask = cmask;
            L.ws_cdist2 = cdist2;
            L.ws_cgmin = cgmin;
            L.q_flag = q_flag;
            L.q_order = q_order;
            L.q_scanned = q_scanned;
            L.pq_list = pq_list;
            L.ws_qlp = lp ? qlp : nullptr;
            L.ws_qeps = lp ? qeps : nullptr;
            L.l_list = list;
            L.pool_cap = pool_q;
            L.l_val = w.vals ? vals : nullptr;
        }
        L.out_ids = out_ids + q0 * stride;
        L.out_dist = out_dist + q0 * stride;
        L.out_stats = out_stats ? out_stats + q0 * 4 : nullptr;
        launch_ann(L, st);
    }
}

// Per-query parameters to the device by a kernel that reads them from pinned
// memory, 16 bytes a thread. A copy from pageable memory had to be waited for,
// with all the work queued before it; this leaves the call asynchronous.
__global__ __launch_bounds__(256) void fetch_params_kernel(const uint4* __restrict__ host,
                                                           uint4* __restrict__ out, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = host[i];
}
static_assert(sizeof(AnnQueryParams) % sizeof(uint4) == 0, "parameters are copied 16 bytes at a time");

void fetch_params(const std::vector<AnnQueryParams>& params, AnnQueryParams* out, hipStream_t st) {
    const size_t bytes = params.size() * sizeof(AnnQueryParams);
    const int64_t n = (int64_t)(bytes / sizeof(uint4));
    void* host = pinned_alloc(bytes);
    std::memcpy(host, params.data(), bytes);
    void* dev = nullptr;
    hipError_t e = hipHostGetDevicePointer(&dev, host, 0);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(fetch_params_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                           static_cast<const uint4*>(dev), reinterpret_cast<uint4*>(out), n);
        e = hipGetLastError();
    }
    pinned_free(host, st);
    PMLSH_HIP(e);
}

// Plan and first radius of one ANN call (host only).
double ann_plan(const pmlsh_index* x, int k, double c, double confidence, double beta,
                double r_min, pmlsh_plan* plan) {
    plan_params(x->n, x->m, k, c, confidence, beta, plan);
    if (!(r_min > 0.0)) r_min = index_default_r_min(x, plan->budget);
    if (!std::isfinite(r_min)) fail(PMLSH_EINVAL, "r_min must be finite");
    return r_min;
}

// The radius up to which the rounds of a large budget are answered from the points of
// one ball (0: none): the ball that the sampled distances expect to hold fewer points.
// (r,c)-BC has one round; of Algorithm 2 those that a small r_min puts before the
// budget's radius, at most 0.3 of it where there are any, since queries with k
// neighbours near by end there. The rule leaves room for queries whose balls hold many
// more than the sample's: lists that outgrow the pools cost a second pass, or in
// (r,c)-BC the per-query kernel.
// us per call of 1,000 queries for the budget alone / with the ball / on the per-query
// kernel, by the first radius in units of the budget's:
//   (r,c)-BC   30,000 x 32, B = 2,902               0.25     239 /    136 /    126
//                                                   0.5      245 /    145 /    161
//              1M x 128, B = 96,695                 0.25   3,812 /    224 /  1,073
//                                                   0.5    3,837 /    284 /  2,404
//                                                   0.8    6,467 / 23,324 / 24,972
//              1M x 128 without contrast, B = 3,001 0.5      643 /    227 / 16,668
//                                                   0.65     700 / 23,720 / 29,888
//   ANN        100,000 x 64, B = 9,680, copies of   0.01     393 /    149 /     82
//              the queries among the points         0.1      390 /    154 /    101
//              1M x 128, B = 96,704, the same       0.01   3,766 /    284 /    162
//              ordinary queries                     0.01  19,697 /    440 /  1,069
//                                                   0.6    3,981 /    555 /  4,339
double ball_limit(const pmlsh_index* x, int64_t budget, double r_min, int max_rounds) {
    if (budget <= kLeanBudget) return 0.0;
    const double full = index_default_r_min(x, budget);
    double most = (budget * 100 >= x->n ? 0.7 : 0.6) * full;
    if (max_rounds != 1 && r_min < 0.3 * full) most = 0.3 * full;
    return r_min < most ? most : 0.0;
}

}  // namespace

void run_ann(const pmlsh_index* x, const float* queries, int64_t nq, int k, double c,
             double confidence, double beta, double r_min, int64_t* out_ids,
             float* out_dist, int32_t* out_stats, hipStream_t st, int max_rounds) {
    pmlsh_plan plan;
    r_min = ann_plan(x, k, c, confidence, beta, r_min, &plan);
    if (nq == 0) return;
    // (r,c)-BC by a few queries with a ball far below the budget's in a small index with
    // contrast: few nodes of the tree lie near it, and one launch finds them (batched /
    // per-query, us: 30,000 x 32, B = 2,902, a tenth of the budget's radius, 1 query 54 / 41,
    // 500 queries 80 / 53, 3,000 queries 186 / 187; 200,000 x 64, 500 queries 84 / 75; without
    // contrast 69 / 699)
    Pools pools = pools_of(x, nq, plan.budget);
    if (max_rounds == 1 && plan.budget > kLeanBudget && nq <= 512 && x->n <= 65536 && !x->low_contrast &&
        r_min < 0.2 * index_default_r_min(x, plan.budget))
        pools = Pools::Short;
    AnnWorkspace w;
    const AnnCall call{k, plan.budget, c, plan.t, r_min, nullptr, k, max_rounds,
                       ball_limit(x, plan.budget, r_min, max_rounds)};
    void* ws = ann_workspace_alloc(x, nq, k, plan.budget, pools, st, &w);
    try {
        run_ann_region(x, queries, nq, call, out_ids, out_dist, out_stats, st, w, ws);
    } catch (...) {
        ws_free(ws, st);
        throw;
    }
    ws_free(ws, st);
}

void run_ann_in(const pmlsh_index* x, const float* queries, int64_t nq, int k, double c,
                double confidence, double beta, double r_min, int64_t* out_ids,
                float* out_dist, int32_t* out_stats, hipStream_t st,
                const std::function<void*()>& region_of_device, int64_t region_bytes) {
    pmlsh_plan plan;
    r_min = ann_plan(x, k, c, confidence, beta, r_min, &plan);
    if (nq == 0) return;
    // a small fixed region holds most queries without the lists' pd^2 bits; a
    // large budget whose candidate pool does not fit takes the per-query path
    const AnnWorkspace w = ann_workspace_region(x, nq, k, plan.budget, region_bytes,
                                                plan.budget > kLeanBudget ? pools_of(x, nq, plan.budget) : Pools::Short);
    if (w.batch < 1) {
        const AnnWorkspace one = ann_workspace_in(x, 1, k, plan.budget, int64_t(1) << 62, Pools::Least);
        fail(PMLSH_EUNSUPPORTED,
             "one query of this index needs " + std::to_string(one.bytes) +
                 " bytes of workspace; the fixed region holds " + std::to_string(region_bytes));
    }
    const AnnCall call{k, plan.budget, c, plan.t, r_min, nullptr, k, 0,
                       ball_limit(x, plan.budget, r_min, 0)};
    run_ann_region(x, queries, nq, call, out_ids, out_dist, out_stats, st, w, region_of_device());
}

void plan_queries(const pmlsh_index* x, const pmlsh_query_args* args, int64_t nq,
                  std::vector<AnnQueryParams>* out, int* kmax, int64_t* bmax, double* ball_most) {
    out->resize((size_t)nq);
    *kmax = 1;
    *bmax = 1;
    *ball_most = 0.0;
    std::vector<int64_t> seen;   // the first queries of distinct parameters
    for (int64_t i = 0; i < nq; ++i) {
        const pmlsh_query_args& q = args[i];
        // queries of equal parameters share a plan (a plan solves for a chi-square
        // quantile, about 3 us)
        bool known = false;
        for (int64_t j : seen) {
            if (std::memcmp(&args[j], &q, sizeof(q)) != 0) continue;
            (*out)[(size_t)i] = (*out)[(size_t)j];
            known = true;
            break;
        }
        if (known) continue;
        if (seen.size() < 64) seen.push_back(i);
        try {
            validate_ann(x, nullptr, 0, q.k, nullptr, nullptr, q.r_min);
            pmlsh_plan plan;
            plan_params(x->n, x->m, q.k, q.c, q.confidence, q.beta, &plan);
            double r_min = q.r_min;
            if (!(r_min > 0.0)) r_min = index_default_r_min(x, plan.budget);
            if (!std::isfinite(r_min)) fail(PMLSH_EINVAL, "r_min must be finite");
            AnnQueryParams& p = (*out)[(size_t)i];
            p.c = q.c;
            p.t = plan.t;
            p.r_min = r_min;
            p.k = q.k;
            p.budget = (int32_t)plan.budget;
            *kmax = std::max(*kmax, q.k);
            *bmax = std::max<int64_t>(*bmax, plan.budget);
            const double ball = ball_limit(x, plan.budget, r_min, 0);
            if (ball > 0.0 && !(*ball_most > 0.0 && *ball_most < ball)) *ball_most = ball;
        } catch (const Error& e) {
            fail(e.code, "query " + std::to_string(i) + ": " + e.msg);
        }
    }
}

void run_ann_planned(const pmlsh_index* x, const float* queries, int64_t nq,
                     const AnnQueryParams& p, int64_t* out_ids, float* out_dist, hipStream_t st,
                     void* region, int64_t region_bytes) {
    if (nq == 0) return;
    const AnnWorkspace w = ann_workspace_region(x, nq, p.k, p.budget, region_bytes,
                                                pools_of(x, nq, p.budget));
    if (w.batch < 1) fail(PMLSH_ENOMEM, "the workspace region holds no query");
    const AnnCall call{p.k, p.budget, p.c, p.t, p.r_min, nullptr, p.k, 0,
                       ball_limit(x, p.budget, p.r_min, 0)};
    run_ann_region(x, queries, nq, call, out_ids, out_dist, nullptr, st, w, region);
}

int64_t ann_workspace_bytes_mixed(const pmlsh_index* x, int64_t nq, int kmax, int64_t bmax) {
    return nq > 0 ? ann_workspace(x, nq, kmax, bmax, pools_of(x, nq, bmax)).bytes : 0;
}

int64_t ann_workspace_bytes_least(const pmlsh_index* x, int kmax, int64_t bmax) {
    AnnWorkspace w = ann_workspace_base(x, kmax, bmax, Pools::Least);
    ann_workspace_size(x, 1, &w);
    return w.bytes;
}

void run_ann_mixed(const pmlsh_index* x, const float* queries, int64_t nq,
                   const AnnQueryParams* qpar, int kmax, int64_t bmax, double ball_most, int out_stride,
                   int64_t* out_ids, float* out_dist, int32_t* out_stats, hipStream_t st,
                   void* region, int64_t region_bytes) {
    if (nq == 0) return;
    const AnnCall call{kmax, bmax, 0.0, 0.0, 0.0, qpar, out_stride, 0, ball_most};
    if (region) {
        const AnnWorkspace w = ann_workspace_region(x, nq, kmax, bmax, region_bytes,
                                                    pools_of(x, nq, bmax));
        if (w.batch < 1) fail(PMLSH_ENOMEM, "the workspace region holds no query");
        run_ann_region(x, queries, nq, call, out_ids, out_dist, out_stats, st, w, region);
        return;
    }
    AnnWorkspace w;
    void* ws = ann_workspace_alloc(x, nq, kmax, bmax, pools_of(x, nq, bmax), st, &w);
    try {
        run_ann_region(x, queries, nq, call, out_ids, out_dist, out_stats, st, w, ws);
    } catch (...) {
        ws_free(ws, st);
        throw;
    }
    ws_free(ws, st);
}

}  // namespace pmlsh

using namespace pmlsh;

extern "C" {

int pmlsh_build(const pmlsh_build_args* args, pmlsh_index** out) {
    return guarded([&] {
        if (!out) fail(PMLSH_EINVAL, "out is NULL");
        *out = index_build(args);
    });
}

void pmlsh_free(pmlsh_index* index) { index_release(index); }

int pmlsh_plan_params(int64_t n, int32_t m, int32_t k, double c, double confidence,
                      double beta, pmlsh_plan* out) {
    return guarded([&] {
        if (!out) fail(PMLSH_EINVAL, "out is NULL");
        pmlsh_plan p;
        plan_params(n, m, k, c, confidence, beta, &p);
        *out = p;
    });
}

int pmlsh_default_r_min(const pmlsh_index* index, int64_t budget, double* r_min) {
    return guarded([&] {
        if (!index || !r_min) fail(PMLSH_EINVAL, "NULL argument");
        if (budget < 1) fail(PMLSH_EINVAL, "budget must be >= 1");
        *r_min = index_default_r_min(index, budget);
    });
}

int pmlsh_ann(const pmlsh_index* index, const float* queries, int64_t nq, int32_t k,
              double c, double confidence, double beta, double r_min, int64_t* out_ids,
              float* out_dist, int32_t* out_stats, void* stream) {
    return guarded([&] {
        validate_ann(index, queries, nq, k, out_ids, out_dist, r_min);
        run_ann(index, queries, nq, k, c, confidence, beta, r_min, out_ids, out_dist,
                out_stats, static_cast<hipStream_t>(stream));
    });
}

int pmlsh_ann_mixed(const pmlsh_index* index, const float* queries, int64_t nq,
                    const pmlsh_query_args* args, int32_t out_stride, int64_t* out_ids,
                    float* out_dist, int32_t* out_stats, void* stream) {
    return guarded([&] {
        if (!index) fail(PMLSH_EINVAL, "index is NULL");
        if (nq < 0) fail(PMLSH_EINVAL, "nq must be >= 0");
        if (nq == 0) return;
        if (!queries || !args || !out_ids || !out_dist)
            fail(PMLSH_EINVAL, "queries, args and outputs must not be NULL");
        std::vector<AnnQueryParams> params;
        int kmax = 1;
        int64_t bmax = 1;
        double ball_most = 0.0;
        plan_queries(index, args, nq, &params, &kmax, &bmax, &ball_most);
        if (out_stride < kmax) fail(PMLSH_EINVAL, "out_stride must be >= every k");
        hipStream_t st = static_cast<hipStream_t>(stream);
        // a captured graph would read the host parameters on every replay
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        PMLSH_HIP(hipStreamIsCapturing(st, &cap));
        if (cap != hipStreamCaptureStatusNone)
            fail(PMLSH_EDEVICE, "pmlsh_ann_mixed copies host parameters and cannot be captured");
        void* dp = ws_alloc(params.size() * sizeof(AnnQueryParams), st);
        try {
            fetch_params(params, static_cast<AnnQueryParams*>(dp), st);
            run_ann_mixed(index, queries, nq, static_cast<const AnnQueryParams*>(dp), kmax, bmax,
                          ball_most, out_stride, out_ids, out_dist, out_stats, st, nullptr, 0);
        } catch (...) {
            ws_free(dp, st);
            throw;
        }
        ws_free(dp, st);
    });
}

int pmlsh_bc(const pmlsh_index* index, const float* queries, int64_t nq, double r, double c,
             double confidence, double beta, int64_t* out_ids, float* out_dist,
             int32_t* out_stats, void* stream) {
    return guarded([&] {
        validate_ann(index, queries, nq, 1, out_ids, out_dist, r);
        if (!(r > 0.0) || !std::isfinite(r)) fail(PMLSH_EINVAL, "r must be positive and finite");
        pmlsh_plan plan;
        plan_params(index->n, index->m, 1, c, confidence, beta, &plan);
        if (nq == 0) return;
        hipStream_t st = static_cast<hipStream_t>(stream);
        int32_t* stats = out_stats;
        void* tmp = nullptr;
        if (!stats) {
            tmp = ws_alloc((size_t)nq * 4 * sizeof(int32_t), st);
            stats = static_cast<int32_t*>(tmp);
        }
        try {
            run_ann(index, queries, nq, 1, c, confidence, beta, r, out_ids, out_dist, stats, st, 1);
            launch_bc_finalize(out_ids, out_dist, stats, nq, (float)(c * r), st);
        } catch (...) {
            ws_free(tmp, st);
            throw;
        }
        ws_free(tmp, st);
    });
}

int pmlsh_acp(const pmlsh_index* index, int32_t k, double c, double confidence,
              double beta, int64_t* out_pairs, float* out_dist, pmlsh_acp_stats* stats,
              void* stream) {
    return guarded([&] {
        if (!index) fail(PMLSH_EINVAL, "index is NULL");
        if (!out_pairs || !out_dist) fail(PMLSH_EINVAL, "outputs must not be NULL");
        if (index->n < 2) fail(PMLSH_EINVAL, "ACP needs n >= 2");
        if (k < 1) fail(PMLSH_EINVAL, "k must be >= 1");
        const double pairs = (double)index->n * (double)(index->n - 1) / 2.0;
        if ((double)k > pairs) fail(PMLSH_EINVAL, "k must be <= n(n-1)/2");
        if (k > PMLSH_MAX_K) fail(PMLSH_EUNSUPPORTED, "k above PMLSH_MAX_K");
        run_acp(index, k, c, confidence, beta, out_pairs, out_dist, stats,
                static_cast<hipStream_t>(stream));
    });
}

int pmlsh_acp_bb(const pmlsh_index* index, int32_t k, double c, double confidence,
                 double beta, int64_t* out_pairs, float* out_dist, pmlsh_acp_stats* stats,
                 void* stream) {
    return guarded([&] {
        if (!index) fail(PMLSH_EINVAL, "index is NULL");
        if (!out_pairs || !out_dist) fail(PMLSH_EINVAL, "outputs must not be NULL");
        if (index->n < 2) fail(PMLSH_EINVAL, "ACP needs n >= 2");
        if (k < 1) fail(PMLSH_EINVAL, "k must be >= 1");
        const double pairs = (double)index->n * (double)(index->n - 1) / 2.0;
        if ((double)k > pairs) fail(PMLSH_EINVAL, "k must be <= n(n-1)/2");
        if (k > PMLSH_MAX_K) fail(PMLSH_EUNSUPPORTED, "k above PMLSH_MAX_K");
        run_acp_bb(index, k, c, confidence, beta, out_pairs, out_dist, stats,
                   static_cast<hipStream_t>(stream));
    });
}

int pmlsh_acp_lca(const pmlsh_index* index, int32_t k, double c, double confidence,
                  double beta, double gamma, int64_t* out_pairs, float* out_dist,
                  pmlsh_acp_stats* stats, double* gamma_used, void* stream) {
    return guarded([&] {
        if (!index) fail(PMLSH_EINVAL, "index is NULL");
        if (!out_pairs || !out_dist) fail(PMLSH_EINVAL, "outputs must not be NULL");
        if (index->n < 2) fail(PMLSH_EINVAL, "ACP needs n >= 2");
        if (k < 1) fail(PMLSH_EINVAL, "k must be >= 1");
        const double pairs = (double)index->n * (double)(index->n - 1) / 2.0;
        if ((double)k > pairs) fail(PMLSH_EINVAL, "k must be <= n(n-1)/2");
        if (k > PMLSH_MAX_K) fail(PMLSH_EUNSUPPORTED, "k above PMLSH_MAX_K");
        if (std::isnan(gamma) || std::isinf(gamma)) fail(PMLSH_EINVAL, "gamma must be finite");
        run_acp_lca(index, k, c, confidence, beta, gamma, out_pairs, out_dist, stats, gamma_used,
                    static_cast<hipStream_t>(stream));
    });
}

int pmlsh_index_export_nodes(const pmlsh_index* index, int32_t* level, int32_t* first_leaf,
                             int32_t* end_leaf, float* radius) {
    return guarded([&] {
        if (!index || !level || !first_leaf || !end_leaf || !radius)
            fail(PMLSH_EINVAL, "NULL argument");
        export_nodes(index, level, first_leaf, end_leaf, radius);
    });
}

int pmlsh_get_index_info(const pmlsh_index* index, pmlsh_index_info* out) {
    return guarded([&] {
        if (!index || !out) fail(PMLSH_EINVAL, "NULL argument");
        pmlsh_index_info i{};
        i.n = index->n;
        i.d = index->d;
        i.m = index->m;
        i.leaf_size = index->leaf_size;
        i.fanout = index->fanout;
        i.num_pivots = index->num_pivots;
        i.levels = index->levels;
        i.n_leaves = index->n_leaves;
        i.n_nodes = index->n_nodes;
        i.sample_size = (int64_t)index->sample_sorted.size();
        i.device_bytes = index->device_bytes;
        i.filter_gemm = index->filter_gemm;
        i.eps_max = index->eps_max;
        *out = i;
    });
}

int pmlsh_index_filter_projection(const pmlsh_index* index, float* proj, float* eps) {
    return guarded([&] {
        if (!index || !proj || !eps) fail(PMLSH_EINVAL, "NULL argument");
        if (!index->filter_gemm) fail(PMLSH_EINVAL, "the index was built with filter_gemm = 0");
        const int64_t n = index->n;
        PMLSH_HIP(hipSetDevice(index->device));
        struct Buf {
            float* p = nullptr;
            ~Buf() { if (p) (void)hipFree(p); }
        } dp, de;
        PMLSH_HIP(hipMalloc(&dp.p, (size_t)n * MP * sizeof(float)));
        PMLSH_HIP(hipMalloc(&de.p, (size_t)n * sizeof(float)));
        launch_project_lp(index->data, n, index->d, index->d_pad, index->hash,
                          index->filter_gemm, dp.p, de.p, nullptr);
        std::vector<float> hp((size_t)n * MP), he((size_t)n);
        PMLSH_HIP(hipMemcpy(hp.data(), dp.p, hp.size() * sizeof(float), hipMemcpyDeviceToHost));
        PMLSH_HIP(hipMemcpy(he.data(), de.p, he.size() * sizeof(float), hipMemcpyDeviceToHost));
        // leaf order -> id order
        const int m = index->m;
        for (int64_t j = 0; j < n; ++j) {
            const int64_t id = index->perm_host[(size_t)j];
            for (int i = 0; i < m; ++i) proj[id * m + i] = hp[(size_t)j * MP + i];
            eps[id] = he[(size_t)j];
        }
    });
}

int pmlsh_index_export_leaves(const pmlsh_index* index, int32_t* perm, int64_t* offsets) {
    return guarded([&] {
        if (!index || !perm || !offsets) fail(PMLSH_EINVAL, "NULL argument");
        std::memcpy(perm, index->perm_host.data(), index->perm_host.size() * sizeof(int32_t));
        const int64_t L = index->leaf_size;
        for (int64_t b = 0; b <= index->n_leaves; ++b) offsets[b] = std::min(index->n, b * L);
    });
}

int pmlsh_ann_timing_enable(int stage_mask) {
    return guarded([&] {
        if (stage_mask < 0 || stage_mask >= (1 << PMLSH_N_STAGES))
            fail(PMLSH_EINVAL, "stage_mask must be a mask of the PMLSH_N_STAGES stages");
        timing_set((unsigned)stage_mask);
    });
}

int pmlsh_ann_timing_read(pmlsh_ann_timing* out, int reset) {
    return guarded([&] {
        if (!out) fail(PMLSH_EINVAL, "out is NULL");
        timing_read(out, reset != 0);
    });
}

int pmlsh_tune(int key, int64_t value) {
    return guarded([&] {
        if (key < 0 || key >= PMLSH_N_TUNE) fail(PMLSH_EINVAL, "unknown tuning key");
        if (value == -1) value = tune_default(key);
        const int64_t hi = key == PMLSH_TUNE_GROUP_LIST      ? 2048
                           : key == PMLSH_TUNE_ACP_FIRST_CAP ? (int64_t(1) << 20)
                           : key == PMLSH_TUNE_SCAN_SHAPE    ? 2
                                                             : 1;
        if (value < 0 || value > hi) fail(PMLSH_EINVAL, "tuning value out of range");
        tune_set(key, value);
    });
}

const char* pmlsh_last_error(void) { return error_cstr(); }

}  // extern "C"
