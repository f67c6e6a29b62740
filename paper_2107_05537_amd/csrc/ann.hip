// (c,k)-ANN query kernel (gfx950): Algorithm 2 of PM-LSH, one workgroup per
// query, all rounds on the device.
//
// Per round i (radius r_i = r_min * c^i):
//   1. from the second round on, count the verified candidates within c*r_i
//      of q and stop when there are at least k (the stopping test of Algorithm 2);
//   2. walk the flattened PM-tree level by level, keeping the nodes that pass
//      the PM-tree access test of Eq. 5 for the range query (q', t*r_i); the
//      surviving leaves go to a per-query list in global memory;
//   3. scan those leaves: every point of the new shell t*r_{i-1} < pd <= t*r_i
//      is counted and histogrammed on its 64-bit key (pd^2 bits, id);
//   4. if the ball holds at least B points, the B - |C| smallest keys of the
//      shell are added to C (exact radix select, see block_select); otherwise
//      the whole shell is added and r grows by c;
//   5. the new members of C are verified: exact FP32 squared distance to q,
//      by direct differences (never by the |q|^2 + |o|^2 - 2 q.o expansion).
// The answer is the k members of C with the smallest (distance, id).
//
// Candidate membership and ordering are decided on bit patterns of FP32 values
// computed by one inlined routine with explicit fused multiply-adds, so every
// scan pass recomputes bit-identical projected distances and the counts of
// different passes agree exactly.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cstddef>
#include <cstdint>

#include "internal.hpp"

namespace pmlsh {
namespace {

constexpr int WG = 256;
constexpr int NWAVE = WG / 64;
constexpr int kMaxWaves = 16;   // waves of the largest workgroup (1,024 threads)
constexpr int NB = 2048;    // histogram bins of one radix-select step
constexpr int CAP = 2048;   // keys sorted in LDS at once (power of two)
constexpr int64_t kWideBudget = PMLSH_BATCHED_BUDGET;
constexpr int64_t kSelMax = 8192;         // most chunks the bound chooses per query
static_assert(kSelMax * 64 >= 2 * kWideBudget + 128, "the chosen chunks must hold 2 * budget points");
constexpr int MAX_LEVELS = 16;
constexpr int MAX_ROUNDS = 1000;
static_assert(kLeanBudget == CAP, "a lean budget's members fit the sorted LDS keys");
constexpr int64_t kScanBlocks = 1024;   // scan workgroups if the occupancy query fails

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));

struct AnnArgs {
    const float* data;
    const float* proj;
    const int32_t* perm;
    const float* ncen;
    const float* nrad;
    const float* hrmin;
    const float* hrmax;
    const int32_t* cb;
    const int32_t* ce;
    const int32_t* npts;
    const float* piv;
    int64_t n_nodes;
    int64_t n_leaves;
    int levels;
    int s;
    int d, d_pad;
    int32_t level_begin[MAX_LEVELS + 1];
    float coord_scale;
    float scan_scale;           // bound on |o' - scen| over the scan rows
    float scen[MP];             // centre of the scan rows
    const float* qlp;           // low-precision query projections of the filter, or null
    const float* qeps;          // their bounds
    float eps_max;              // largest bound of the points' scan-row projections
    const float* q;
    const float* qp;
    const float* qp_lo;         // FP32 rounding of (projection - qp)
    const float* proj_lo;       // the same for the data, leaf order
    // Algorithm 2's parameters, the same for every query of the launch, or
    // per query from qpar (then k and budget here are the largest of the
    // launch and serve as strides of the per-query workspace)
    int k;
    int32_t budget;
    double c, t, r_min;
    const AnnQueryParams* qpar;
    int out_stride;             // row stride of out_ids / out_dist (>= every k)
    int max_rounds;             // range queries per query at most ((r,c)-BC: 1)
    int32_t* ws_front;
    int32_t* ws_cpos;
    float* ws_cdist;
    int32_t* ws_topk;
    int64_t* out_ids;
    float* out_dist;
    int32_t* out_stats;
    // leaf-major fast path (per query): members of L in the first ball (-1: the
    // per-query kernel answers), candidate count, scanned points, candidate list
    int32_t* q_flag;
    uint32_t* pq_list;          // count, then the queries flagged for the per-query kernel
    uint32_t* l_count;          // candidates per query: entry q * l_stride
    int64_t l_stride;
    uint32_t* q_scanned;
    uint32_t* l_list;           // nq x q_cap leaf positions (candidate pool)
    int q_cap;
    int nq;
    int64_t n;
    // matrix-core scan: FP16 point rows, their count (padded to 64), scale,
    // and the per-query FP16 rows
    const uint16_t* proj16;
    int64_t n_pad16;
    float scale16;
    uint16_t* qaug;
    // chunk balls, and per query the radius tq of their test (Eq. 5) and
    // the margin of the stored squared distances, from the bound kernel
    const float* chunk_cen;
    const float* chunk_rad;
    float2* qtest;
    // the same mask chunk-major, in blocks of 256 chunks: word (chunk c, query
    // band qb) at cmask_at(c, qb), cwords = ceil(nq / 64) bands
    uint64_t* cmask;
    int cwords;
    // squared distances from every query to every chunk centre, as bf16 bit
    // patterns rounded toward zero (lower bounds), in blocks of 64 queries x
    // 64 chunks (cdist_at); the minimum of each group of 64 chunks (row
    // stride gld)
    uint16_t* cdist;
    uint16_t* cgmin;
    int64_t cgroups, gld;
    int glds;                   // bound kernel: group minima copied to LDS
    int ordered;                // the pool kernels take the queries in the order q_order,
    int32_t* q_order;           // which mask_kernel writes
    int grp_cap;                // bound kernel: most groups or blocks listed (<= kGrpCap)
    // bounded verification: FP16 rows (stride d16), their scales and error
    // bounds, and per C member a lower bound of its squared distance (the
    // upper bound goes to ws_cdist; equal bounds mean the exact value)
    const uint16_t* data16;
    const float2* d16_se;       // per row its scale and error bound
    int d16;
    float* ws_clo;
    // pd^2 bits of the pool entries (or null: long lists compute them again in
    // every pass), and the members of L per verify workgroup
    uint32_t* l_val;
    int vslice;
    // bound kernel: points sampled per budget point, chunks it may choose
    int sample, sel_cap;
    // Pass::Ball: no round of a larger radius has its ball listed, and whether
    // Pass::Rest follows
    double ball_most;
    int staged;
};

// Element (query q, chunk c) of the blocked chunk-distance matrix.
__device__ __forceinline__ int64_t cdist_at(const AnnArgs& a, int64_t q, int64_t c) {
    return (((q >> 6) * a.cgroups + (c >> 6)) << 12) + ((q & 63) << 6) + (c & 63);
}

// Mask word of chunk c and query band qb (queries 64 qb .. 64 qb + 63): the
// 256 words of one band and one block of 256 chunks are contiguous.
__device__ __forceinline__ int64_t cmask_at(const AnnArgs& a, int64_t c, int64_t qb) {
    return (((c >> 8) * a.cwords + qb) << 8) + (c & 255);
}

// skey and spos come last: the bound kernel uses only the fields before
// them and keeps its row of centre distances in their place.
struct Smem {
    uint32_t hist[NB];
    int32_t red[kMaxWaves * 2];
    int32_t cnt0, cnt1, cnt2;
    int32_t thr_bin, thr_below, thr_in;
    uint32_t near;
    int32_t pad_;
    uint64_t skey[CAP];
    int32_t spos[CAP];
};
static_assert(offsetof(Smem, skey) % 16 == 0, "row area must be 16-byte aligned");

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// The parameters of query qi of the launch.
__device__ __forceinline__ AnnQueryParams query_params(const AnnArgs& a, int64_t qi) {
    if (a.qpar) return a.qpar[qi];
    AnnQueryParams p;
    p.c = a.c;
    p.t = a.t;
    p.r_min = a.r_min;
    p.k = a.k;
    p.budget = a.budget;
    return p;
}

__device__ __forceinline__ uint64_t lanemask_lt() {
    return (1ull << lane_id()) - 1ull;
}

// Slot for each lane with take == true, one LDS atomic per wave.
__device__ __forceinline__ int wave_append(bool take, int32_t* counter) {
    const uint64_t m = __ballot(take);
    if (m == 0) return -1;
    const int leader = __ffsll((unsigned long long)m) - 1;
    int base = 0;
    if (lane_id() == leader) base = atomicAdd(counter, __popcll(m));
    base = __shfl(base, leader);
    return base + __popcll(m & lanemask_lt());
}

template <int T = WG>
__device__ __forceinline__ int block_sum(int v, Smem& sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane_id() == 0) sh.red[threadIdx.x >> 6] = v;
    __syncthreads();
    int s = 0;
#pragma unroll
    for (int w = 0; w < (T / 64); ++w) s += sh.red[w];
    __syncthreads();
    return s;
}

// Sum over each 16 lanes in all of them, by rotations of the lanes within the
// vector unit rather than exchanges through the LDS: the value that adding the
// lane 8, 4, 2 and 1 apart gives (a rotation by r reaches that lane or one
// that holds the same partial sum).
__device__ __forceinline__ float sum16(float x) {
    auto turned = [](float v, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
            0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xf, 0xf, false));
    };
    x += turned(x, std::integral_constant<int, 0x128>{});   // row_ror:8
    x += turned(x, std::integral_constant<int, 0x124>{});   // row_ror:4
    x += turned(x, std::integral_constant<int, 0x122>{});   // row_ror:2
    x += turned(x, std::integral_constant<int, 0x121>{});   // row_ror:1
    return x;
}

// Inclusive prefix sum over the wave (row shifts, then the row totals).
__device__ __forceinline__ int wave_inclusive_scan(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 to rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 to rows 2, 3
    return x;
}

// Exclusive prefix sum over the workgroup.
template <int T = WG>
__device__ __forceinline__ int block_exclusive_scan(int v, Smem& sh) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    int x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) sh.red[(T / 64) + wave] = x;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += sh.red[(T / 64) + w];
    __syncthreads();
    return before + x - v;
}

// Squared projected distance, always the same operation sequence.
__device__ __forceinline__ float proj_dist2(const float* __restrict__ o, const float* qp) {
    const float4* o4 = reinterpret_cast<const float4*>(o);
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < MP / 4; ++j) {
        const float4 v = o4[j];
        float t;
        t = __fsub_rn(qp[4 * j + 0], v.x); acc = __fmaf_rn(t, t, acc);
        t = __fsub_rn(qp[4 * j + 1], v.y); acc = __fmaf_rn(t, t, acc);
        t = __fsub_rn(qp[4 * j + 2], v.z); acc = __fmaf_rn(t, t, acc);
        t = __fsub_rn(qp[4 * j + 3], v.w); acc = __fmaf_rn(t, t, acc);
    }
    return acc;
}

__device__ __forceinline__ float node_dist(const AnnArgs& a, int node, const float* qp) {
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < MP; ++j) {
        const float t = qp[j] - a.ncen[(int64_t)j * a.n_nodes + node];
        acc = fmaf(t, t, acc);
    }
    return sqrtf(acc);
}

// Eq. 5: the node is accessed iff its covering ball and every pivot ring can
// hold a point within R of q'. `slack` absorbs FP32 rounding (conservative).
// All of the node's data is loaded before any test, so the loads overlap.
__device__ __forceinline__ bool node_pass(const AnnArgs& a, int node, const float* qp,
                                          const float* qpiv, float R, float slack) {
    float hmn[PMLSH_MAX_PIVOTS], hmx[PMLSH_MAX_PIVOTS];
#pragma unroll
    for (int i = 0; i < PMLSH_MAX_PIVOTS; ++i) {
        hmn[i] = hmx[i] = 0.f;
        if (i < a.s) {
            hmn[i] = a.hrmin[(int64_t)i * a.n_nodes + node];
            hmx[i] = a.hrmax[(int64_t)i * a.n_nodes + node];
        }
    }
    const float rad = a.nrad[node];
    bool pass = node_dist(a, node, qp) <= rad + R + slack;
#pragma unroll
    for (int i = 0; i < PMLSH_MAX_PIVOTS; ++i)
        if (i < a.s)
            pass = pass & (qpiv[i] - R <= hmx[i] + slack) & (qpiv[i] + R >= hmn[i] - slack);
    return pass;
}

__device__ __forceinline__ int shift_for(uint64_t lo, uint64_t hi) {
    const uint64_t span = hi - lo;
    if (span < (uint64_t)NB) return 0;
    const int bits = 64 - __clzll((long long)span);
    return bits - 11;
}

template <int T = WG>
__device__ __forceinline__ void clear_hist(Smem& sh) {
    for (int i = threadIdx.x; i < NB; i += T) sh.hist[i] = 0;
    __syncthreads();
}

// Finds the bin where the running count of the histogram reaches `need`.
template <int T = WG>
__device__ void find_threshold(int need, Smem& sh) {
    constexpr int PER = NB / T;
    const int base = threadIdx.x * PER;
    int local[PER];
    int s = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) { local[j] = (int)sh.hist[base + j]; s += local[j]; }
    const int excl = block_exclusive_scan<T>(s, sh);
    if (excl < need && excl + s >= need) {
        int acc = excl;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (acc + local[j] >= need) {
                sh.thr_bin = base + j;
                sh.thr_below = acc;
                sh.thr_in = local[j];
                break;
            }
            acc += local[j];
        }
    }
    __syncthreads();
}

// Histogram bin of a non-negative radius below R: 256 bins per octave over
// [R / 2^8, R], everything smaller in bin 0.
__device__ __forceinline__ int radius_bin(float v, uint32_t base) {
    const uint32_t b = __float_as_uint(v) >> 15;
    return b <= base ? 0 : (int)(b - base);
}

// Level-by-level traversal with Eq. 5; returns the number of leaves that pass
// and leaves their ids in fa (the first of the two per-query buffers).
//
// With `shrink`, the radius R (in/out) is lowered level by level to an upper
// bound tau on the budget-th smallest projected distance: the passing nodes
// whose every point lies within dist(q', centre) + radius <= tau hold at least
// `budget` points. Then every point of the final ball of radius tau lies in a
// kept leaf, the ball holds at least `budget` points, and its `budget`
// nearest points are those of the ball of the original radius.
__device__ int traverse(const AnnArgs& a, const float* qp, const float* qpiv, float& R,
                        float slack, bool shrink, int budget, int32_t* fa, int32_t* fb,
                        Smem& sh) {
    int ncur = a.level_begin[1] - a.level_begin[0];
    for (int l = 0; l < a.levels; ++l) {
        const bool leaf_level = (l == a.levels - 1);
        // A: test the candidates of this level at R; the passing ones go to fb
        if (threadIdx.x == 0) sh.cnt0 = 0;
        __syncthreads();
        for (int base = 0; base < ncur; base += WG) {
            const int i = base + threadIdx.x;
            bool pass = false;
            int node = 0;
            if (i < ncur) {
                node = (l == 0) ? a.level_begin[0] + i : fa[i];
                // entries always lie in this level; the check only keeps a
                // corrupted list from reading outside the node arrays
                if (node >= a.level_begin[l] && node < a.level_begin[l + 1])
                    pass = node_pass(a, node, qp, qpiv, R, slack);
            }
            const int slot = wave_append(pass, &sh.cnt0);
            if (pass && slot < a.n_leaves) fb[slot] = node;
        }
        __syncthreads();
        const int np = sh.cnt0 < a.n_leaves ? sh.cnt0 : (int)a.n_leaves;
        __syncthreads();
        // B: weighted histogram of the nodes' distance upper bounds -> tau
        float Rn = R;
        if (shrink) {
            const uint32_t hb = __float_as_uint(R) >> 15;
            const uint32_t base = hb > (uint32_t)(NB - 1) ? hb - (uint32_t)(NB - 1) : 0u;
            clear_hist(sh);
            int loc = 0;
            for (int i = threadIdx.x; i < np; i += WG) {
                const int node = fb[i];
                const float ub = node_dist(a, node, qp) + a.nrad[node] + slack;
                if (ub <= R) {
                    atomicAdd(&sh.hist[radius_bin(ub, base)], (uint32_t)a.npts[node]);
                    loc += a.npts[node];
                }
            }
            __syncthreads();
            if (block_sum(loc, sh) >= budget) {
                if (threadIdx.x == 0) sh.thr_bin = NB - 1;
                __syncthreads();
                find_threshold(budget, sh);
                // upper edge of the threshold bin: every counted ub is below it
                const float tau = __uint_as_float((base + (uint32_t)sh.thr_bin + 1u) << 15);
                Rn = tau < R ? tau : R;
            }
            __syncthreads();
        }
        // C: keep what passes at the lowered radius; expand inner nodes into fa
        if (threadIdx.x == 0) sh.cnt1 = 0;
        __syncthreads();
        for (int base = 0; base < np; base += WG) {
            const int i = base + threadIdx.x;
            bool keep = false;
            int node = 0;
            if (i < np) {
                node = fb[i];
                keep = Rn == R || node_pass(a, node, qp, qpiv, Rn, slack);
            }
            if (leaf_level) {
                const int slot = wave_append(keep, &sh.cnt1);
                if (keep && slot < a.n_leaves) fa[slot] = node;
            } else if (keep) {
                const int b = a.cb[node], e = a.ce[node];
                const int slot = atomicAdd(&sh.cnt1, e - b);
                if (slot + (e - b) <= a.n_leaves)
                    for (int j = b; j < e; ++j) fa[slot + (j - b)] = j;
            }
        }
        __syncthreads();
        ncur = sh.cnt1 < a.n_leaves ? sh.cnt1 : (int)a.n_leaves;
        R = Rn;
        __syncthreads();
    }
    return ncur;
}

// Calls f(valid, pos, pd2) for every point of the listed leaves; wave-uniform.
template <class F>
__device__ __forceinline__ void scan_leaves(const AnnArgs& a, const int32_t* leaves, int nl,
                                            const float* qp, F&& f) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int li = wave; li < nl; li += NWAVE) {
        const int leaf = leaves[li];
        const int p0 = a.cb[leaf], p1 = a.ce[leaf];
        for (int base = p0; base < p1; base += 64) {
            const int pos = base + lane;
            const bool valid = pos < p1;
            const float pd2 = valid ? proj_dist2(a.proj + (int64_t)pos * MP, qp) : FLT_MAX;
            f(valid, pos, pd2);
        }
    }
}

template <int T = WG>
__device__ void bitonic_sort(int count, Smem& sh) {
    int P = 1;
    while (P < count) P <<= 1;
    for (int i = count + threadIdx.x; i < P; i += T) { sh.skey[i] = ~0ull; sh.spos[i] = -1; }
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < P; i += T) {
                const int ixj = i ^ j;
                if (ixj > i) {
                    const bool up = (i & k) == 0;
                    const uint64_t x = sh.skey[i], y = sh.skey[ixj];
                    if ((x > y) == up) {
                        sh.skey[i] = y; sh.skey[ixj] = x;
                        const int32_t t = sh.spos[i]; sh.spos[i] = sh.spos[ixj]; sh.spos[ixj] = t;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// The need-th smallest (need in [1, n]) of the n <= CAP distinct 64-bit keys
// in sh.skey: NB-bin histogram passes over LDS, each narrowing the key range
// to the bin that holds it.
template <int T = WG>
__device__ uint64_t lds_select(int n, int need, Smem& sh) {
    uint64_t lo = ~0ull, hi = 0ull;
    for (int i = threadIdx.x; i < n; i += T) {
        const uint64_t k = sh.skey[i];
        lo = k < lo ? k : lo;
        hi = k > hi ? k : hi;
    }
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t l2 = __shfl_xor(lo, off), h2 = __shfl_xor(hi, off);
        lo = l2 < lo ? l2 : lo;
        hi = h2 > hi ? h2 : hi;
    }
    uint64_t* red = reinterpret_cast<uint64_t*>(sh.hist);
    if (lane_id() == 0) {
        red[threadIdx.x >> 6] = lo;
        red[(T / 64) + (threadIdx.x >> 6)] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < (T / 64); ++w) {
        lo = red[w] < lo ? red[w] : lo;
        hi = red[(T / 64) + w] > hi ? red[(T / 64) + w] : hi;
    }
    __syncthreads();
    for (;;) {
        const int sft = shift_for(lo, hi);
        clear_hist<T>(sh);
        for (int i = threadIdx.x; i < n; i += T) {
            const uint64_t k = sh.skey[i];
            if (k >= lo && k <= hi) atomicAdd(&sh.hist[(int)((k - lo) >> sft)], 1u);
        }
        __syncthreads();
        if (threadIdx.x == 0) sh.thr_bin = NB - 1;
        __syncthreads();
        find_threshold<T>(need, sh);
        const int tb = sh.thr_bin, below = sh.thr_below, inT = sh.thr_in;
        const uint64_t nlo = lo + ((uint64_t)tb << sft);
        const uint64_t span = (1ull << sft) - 1ull;
        const uint64_t nhi = hi - nlo > span ? nlo + span : hi;
        __syncthreads();
        if (sft == 0) return nlo;
        if (inT == 1) {
            // the bin holds one key: that key
            for (int i = threadIdx.x; i < n; i += T) {
                const uint64_t k = sh.skey[i];
                if (k >= nlo && k <= nhi) red[0] = k;
            }
            __syncthreads();
            const uint64_t key = red[0];
            __syncthreads();
            return key;
        }
        need -= below;
        lo = nlo;
        hi = nhi;
    }
}

// Exact selection of the `need` smallest 64-bit keys among the members of a
// source with key in [lo, hi] (radix select with NB-bin steps). src(v) calls
// v(valid, key, payload) wave-uniformly over all members; emit(payload, slot)
// receives every selected payload exactly once, slot in [0, need).
// If hist_ready, sh.hist already holds the histogram of [lo, hi] at
// shift_for(lo, hi) and `total` is the member count in [lo, hi].
template <int T = WG, class Src, class Emit>
__device__ void block_select(Src&& src, Emit&& emit, uint64_t lo, uint64_t hi, int need,
                             bool hist_ready, int total, Smem& sh) {
    int emitted = 0;
    for (;;) {
        const int shift = shift_for(lo, hi);
        if (!hist_ready) {
            clear_hist<T>(sh);
            src([&](bool valid, uint64_t key, int32_t) {
                if (valid && key >= lo && key <= hi) atomicAdd(&sh.hist[(key - lo) >> shift], 1u);
            });
            __syncthreads();
            int loc = 0;
            for (int i = threadIdx.x; i < NB; i += T) loc += (int)sh.hist[i];
            total = block_sum<T>(loc, sh);
        }
        hist_ready = false;
        if (total <= CAP) {
            if (threadIdx.x == 0) sh.cnt1 = 0;
            __syncthreads();
            src([&](bool valid, uint64_t key, int32_t payload) {
                const bool take = valid && key >= lo && key <= hi;
                const int slot = wave_append(take, &sh.cnt1);
                if (take && slot < CAP) { sh.skey[slot] = key; sh.spos[slot] = payload; }
            });
            __syncthreads();
            bitonic_sort<T>(total, sh);
            for (int i = threadIdx.x; i < need; i += T) emit(sh.spos[i], emitted + i);
            __syncthreads();
            return;
        }
        if (threadIdx.x == 0) { sh.thr_bin = NB - 1; sh.thr_below = 0; sh.thr_in = 0; }
        __syncthreads();
        find_threshold<T>(need, sh);
        const int tb = sh.thr_bin, below = sh.thr_below, inT = sh.thr_in;
        if (threadIdx.x == 0) { sh.cnt1 = 0; sh.cnt2 = 0; }
        __syncthreads();
        const bool gather_T = inT <= CAP;
        src([&](bool valid, uint64_t key, int32_t payload) {
            const bool in = valid && key >= lo && key <= hi;
            const int bin = in ? (int)((key - lo) >> shift) : NB;
            const bool lower = in && bin < tb;
            const int s1 = wave_append(lower, &sh.cnt1);
            if (lower && s1 < below) emit(payload, emitted + s1);
            const bool at = gather_T && in && bin == tb;
            const int s2 = wave_append(at, &sh.cnt2);
            if (at && s2 < CAP) { sh.skey[s2] = key; sh.spos[s2] = payload; }
        });
        __syncthreads();
        emitted += below;
        need -= below;
        if (gather_T) {
            bitonic_sort<T>(inT, sh);
            for (int i = threadIdx.x; i < need; i += T) emit(sh.spos[i], emitted + i);
            __syncthreads();
            return;
        }
        const uint64_t nlo = lo + ((uint64_t)tb << shift);
        const uint64_t nhi = nlo + ((1ull << shift) - 1ull);
        lo = nlo;
        hi = nhi < hi ? nhi : hi;
    }
}

// Exact squared distances of C entries [v0, v1): 16 lanes per row, each
// 16-lane group keeping VR rows in flight (VR independent loads per column
// step) so the gather of 1 KB rows runs at HBM rate rather than at latency.
constexpr int VR = 4;

template <int T = WG>
__device__ void verify(const AnnArgs& a, const float* qs, const int32_t* cpos, float* cdist,
                       int v0, int v1) {
    const int g = threadIdx.x >> 4, l16 = threadIdx.x & 15;
    const int d4 = a.d_pad >> 2;
    const float4* q4 = reinterpret_cast<const float4*>(qs);
    constexpr int GROUPS = T / 16;
    for (int base = v0; base < v1; base += GROUPS * VR) {
        const float4* row[VR];
        bool ok[VR];
        float acc[VR];
#pragma unroll
        for (int r = 0; r < VR; ++r) {
            const int i = base + g + GROUPS * r;
            ok[r] = i < v1;
            row[r] = reinterpret_cast<const float4*>(a.data + (int64_t)cpos[ok[r] ? i : v0] * a.d_pad);
            acc[r] = 0.f;
        }
#pragma unroll 2
        for (int c = l16; c < d4; c += 16) {
            float4 x[VR];
#pragma unroll
            for (int r = 0; r < VR; ++r) x[r] = row[r][c];
            const float4 y = q4[c];
#pragma unroll
            for (int r = 0; r < VR; ++r) {
                float t;
                t = y.x - x[r].x; acc[r] = __fmaf_rn(t, t, acc[r]);
                t = y.y - x[r].y; acc[r] = __fmaf_rn(t, t, acc[r]);
                t = y.z - x[r].z; acc[r] = __fmaf_rn(t, t, acc[r]);
                t = y.w - x[r].w; acc[r] = __fmaf_rn(t, t, acc[r]);
            }
        }
#pragma unroll
        for (int r = 0; r < VR; ++r) {
            const float v = sum16(acc[r]);
            if (ok[r] && l16 == 0) cdist[base + g + GROUPS * r] = v;
        }
    }
}

// Exact squared distances (same operation sequence as verify) of the C
// members listed in idx[0, cnt); both bounds of each become the exact value.
template <int T = WG>
__device__ void verify_list(const AnnArgs& a, const float* qs, const int32_t* cpos,
                            const int32_t* idx, int cnt, float* lo2, float* hi2) {
    const int g = threadIdx.x >> 4, l16 = threadIdx.x & 15;
    const int d4 = a.d_pad >> 2;
    const float4* q4 = reinterpret_cast<const float4*>(qs);
    constexpr int GROUPS = T / 16;
    for (int base = 0; base < cnt; base += GROUPS * VR) {
        const float4* row[VR];
        bool ok[VR];
        float acc[VR];
        int mi[VR];
#pragma unroll
        for (int r = 0; r < VR; ++r) {
            const int j = base + g + GROUPS * r;
            ok[r] = j < cnt;
            mi[r] = idx[ok[r] ? j : 0];
            row[r] = reinterpret_cast<const float4*>(a.data + (int64_t)cpos[mi[r]] * a.d_pad);
            acc[r] = 0.f;
        }
        // two words of every row per lane and step, all loads issued before
        // the first use; the operations and their order are those of verify
        for (int c0 = l16; c0 < d4; c0 += 32) {
            float4 x[VR][2];
#pragma unroll
            for (int r = 0; r < VR; ++r) {
                x[r][0] = row[r][c0];
                x[r][1] = c0 + 16 < d4 ? row[r][c0 + 16] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int c = c0 + 16 * u;
                if (u == 1 && c >= d4) break;
                const float4 y = q4[c];
#pragma unroll
                for (int r = 0; r < VR; ++r) {
                    float t;
                    t = y.x - x[r][u].x; acc[r] = __fmaf_rn(t, t, acc[r]);
                    t = y.y - x[r][u].y; acc[r] = __fmaf_rn(t, t, acc[r]);
                    t = y.z - x[r][u].z; acc[r] = __fmaf_rn(t, t, acc[r]);
                    t = y.w - x[r][u].w; acc[r] = __fmaf_rn(t, t, acc[r]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < VR; ++r) {
            const float v = sum16(acc[r]);
            if (ok[r] && l16 == 0) {
                lo2[mi[r]] = v;
                hi2[mi[r]] = v;
            }
        }
    }
}

// Bounds on the exact FP32 squared distance (the value verify would compute)
// of C members [v0, v1), from the FP16 rows: with D16 the distance to the
// FP16 row (accumulated in FP32 like verify, relative error <= gamma) and eps
// the row's bound |x - s x16|, the true distance lies in [D16 - eps, D16 +
// eps] and the FP32 value within a further factor (1 +- gamma); every
// rounding of the bound arithmetic is covered by extra factors of a few u.
template <int T = WG>
__device__ void verify16(const AnnArgs& a, const float* qs, const int32_t* cpos,
                         float* lo2, float* hi2, int v0, int v1) {
    const int g = threadIdx.x >> 4, l16 = threadIdx.x & 15;
    const int d8 = a.d16 >> 3;
    constexpr int GROUPS = T / 16;
    const float u = 5.9604645e-08f;
    const float gam = 2.f * u * (float)(a.d16 / 16 + 8);
    // the positions of a step are loaded one step ahead, and a row's scale and
    // bound with the row, so a step waits for one memory round trip (with the
    // positions and, at its end, the bounds loaded in it, for three)
    if (v0 >= v1) return;
    int nx[VR];
#pragma unroll
    for (int r = 0; r < VR; ++r) nx[r] = cpos[min(v0 + g + GROUPS * r, v1 - 1)];
    for (int base = v0; base < v1; base += GROUPS * VR) {
        const uint4* row[VR];
        bool ok[VR];
        float acc[VR];
        float2 se[VR];
#pragma unroll
        for (int r = 0; r < VR; ++r) {
            const int i = base + g + GROUPS * r;
            ok[r] = i < v1;
            row[r] = reinterpret_cast<const uint4*>(a.data16 + (int64_t)nx[r] * a.d16);
            se[r] = a.d16_se[nx[r]];
            nx[r] = cpos[min(i + GROUPS * VR, v1 - 1)];
            acc[r] = 0.f;
        }
        // two 16-byte words of every row per lane and step, all loads issued
        // before the first use (words past the row read as zero halves, and
        // the query's zero padding makes their terms zero)
        for (int c0 = l16; c0 < d8; c0 += 32) {
            uint4 h[VR][2];
#pragma unroll
            for (int r = 0; r < VR; ++r) {
                h[r][0] = row[r][c0];
                h[r][1] = c0 + 16 < d8 ? row[r][c0 + 16] : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int c = c0 + 16 * u;
                if (u == 1 && c >= d8) break;
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) y[e] = qs[8 * c + e];
#pragma unroll
                for (int r = 0; r < VR; ++r) {
                    const uint32_t w[4] = {h[r][u].x, h[r][u].y, h[r][u].z, h[r][u].w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const uint16_t bits = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
                        const float xv = (float)__builtin_bit_cast(_Float16, bits);
                        const float t = __fmaf_rn(-se[r].x, xv, y[e]);
                        acc[r] = __fmaf_rn(t, t, acc[r]);
                    }
                }
            }
        }
#pragma unroll
        for (int r = 0; r < VR; ++r) {
            acc[r] = sum16(acc[r]);
        }
        // lane r of a group takes row r's bounds: one pass of this arithmetic
        // for the VR rows
        float v = acc[0], eps = se[0].y;
        bool mine = ok[0] && l16 == 0;
#pragma unroll
        for (int r = 1; r < VR; ++r) {
            v = l16 == r ? acc[r] : v;
            eps = l16 == r ? se[r].y : eps;
            mine = mine || (ok[r] && l16 == r);
        }
        if (mine) {
            const float dlo = sqrtf(v * (1.f - gam)) * (1.f - 4.f * u);
            const float dhi = sqrtf(v * (1.f + 2.f * gam)) * (1.f + 4.f * u);
            const float tlo = fmaxf((dlo - eps) * (1.f - 2.f * u), 0.f);
            const float thi = (dhi + eps) * (1.f + 2.f * u);
            const int i = base + g + GROUPS * l16;
            lo2[i] = tlo * tlo * (1.f - gam) * (1.f - 4.f * u);
            hi2[i] = thi * thi * (1.f + gam) * (1.f + 4.f * u);
        }
    }
}

// Loads the query into LDS (zero padded), its projection and pivot
// distances into registers.
struct QueryCtx {
    float qp[MP];
    float qpiv[PMLSH_MAX_PIVOTS];
    float qn2;
};

__device__ __forceinline__ void load_projection(const AnnArgs& a, int64_t qi, QueryCtx& c) {
#pragma unroll
    for (int j = 0; j < MP; ++j) c.qp[j] = a.qp[qi * MP + j];
    c.qn2 = 0.f;
#pragma unroll
    for (int j = 0; j < MP; ++j) c.qn2 = fmaf(c.qp[j], c.qp[j], c.qn2);
}

template <int T = WG>
__device__ __forceinline__ void load_query(const AnnArgs& a, int64_t qi, float* qs, QueryCtx& c) {
    const float* qrow = a.q + qi * a.d;
    if (qs)
        for (int j = threadIdx.x; j < a.d16; j += T) qs[j] = j < a.d ? qrow[j] : 0.f;
    load_projection(a, qi, c);
#pragma unroll
    for (int i = 0; i < PMLSH_MAX_PIVOTS; ++i) {
        float acc = 0.f;
        if (i < a.s) {
#pragma unroll
            for (int j = 0; j < MP; ++j) {
                const float t = c.qp[j] - a.piv[i * MP + j];
                acc = fmaf(t, t, acc);
            }
        }
        c.qpiv[i] = sqrtf(acc);
    }
}

// Writes the k members of C (the first n_ver entries, n_ver >= k) with the
// smallest (distance^2 bits, id), in that order, and the per-query statistics.
// Relative error bound of the FP32 squared distance that verify computes
// (16 lanes, d_pad / 16 terms each, four shuffle additions).
__device__ __forceinline__ float verify_gamma(const AnnArgs& a) {
    return 2.f * 5.9604645e-08f * (float)(a.d_pad / 16 + 8);
}

constexpr int kRerankCap = 512;   // members the FP64 re-rank takes at most

// FP64 re-rank of the top-k, for near ties of the FP32 distances: every
// member whose exact FP32 squared distance v32 is at most kth32 (1 + 4 gamma),
// kth32 the k-th smallest v32 (+inf with at most k members), gets its squared
// distance in FP64 from its FP32 row; since v32 is within a factor 1 +- gamma
// of that value, no member outside can be among the k nearest in FP64. The k
// smallest (FP64 value, id) are written, each distance as the FP32 rounding
// of the FP64 root. src(j, v32, member) gives the cnt candidates. Returns
// false, writing nothing, when more than kRerankCap members qualify.
template <int T = WG, class Src>
__device__ bool rerank_topk64(const AnnArgs& a, int64_t qi, const float* qs, const int32_t* cpos,
                              int cnt, float kth32, Src&& src, Smem& sh) {
    const int k = query_params(a, qi).k;
    double* d64 = reinterpret_cast<double*>(sh.hist);
    int32_t* mem = reinterpret_cast<int32_t*>(d64 + kRerankCap);
    int32_t* pid = mem + kRerankCap;
    static_assert(NB * sizeof(uint32_t) >= kRerankCap * 16, "re-rank lists must fit the histogram");
    const double lim = (double)kth32 * (1.0 + 4.0 * (double)verify_gamma(a));
    __syncthreads();
    if (threadIdx.x == 0) sh.cnt2 = 0;
    __syncthreads();
    for (int b0 = 0; b0 < cnt; b0 += T) {
        const int j = b0 + threadIdx.x;
        float v = 0.f;
        int mi = 0;
        if (j < cnt) src(j, v, mi);
        const bool take = j < cnt && (double)v <= lim;
        const int slot = wave_append(take, &sh.cnt2);
        if (take && slot < kRerankCap) {
            mem[slot] = mi;
            pid[slot] = a.perm[cpos[mi]];
        }
    }
    __syncthreads();
    const int np = sh.cnt2;
    if (np > kRerankCap) return false;
    // FP64 squared distances, 16 lanes per member (differences of FP32
    // values are exact in FP64)
    {
        const int g = threadIdx.x >> 4, l16 = threadIdx.x & 15;
        const int d4 = a.d_pad >> 2;
        const float4* q4 = reinterpret_cast<const float4*>(qs);
        for (int base = 0; base < np; base += T / 16) {
            const int j = base + g;
            double acc = 0.0;
            if (j < np) {
                const float4* row = reinterpret_cast<const float4*>(a.data + (int64_t)cpos[mem[j]] * a.d_pad);
                // four words per lane and step, loaded before their first use
                for (int c0 = l16; c0 < d4; c0 += 64) {
                    float4 x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        x[u] = c0 + 16 * u < d4 ? row[c0 + 16 * u] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (c0 + 16 * u >= d4) break;
                        const float4 y = q4[c0 + 16 * u];
                        double t;
                        t = (double)y.x - (double)x[u].x; acc = fma(t, t, acc);
                        t = (double)y.y - (double)x[u].y; acc = fma(t, t, acc);
                        t = (double)y.z - (double)x[u].z; acc = fma(t, t, acc);
                        t = (double)y.w - (double)x[u].w; acc = fma(t, t, acc);
                    }
                }
            }
            acc += __shfl_xor(acc, 8, 16);
            acc += __shfl_xor(acc, 4, 16);
            acc += __shfl_xor(acc, 2, 16);
            acc += __shfl_xor(acc, 1, 16);
            if (j < np && l16 == 0) d64[j] = acc;
        }
    }
    __syncthreads();
    // rank by (FP64 value, id); ids are distinct
    for (int j = threadIdx.x; j < np; j += T) {
        const double v = d64[j];
        const int32_t id = pid[j];
        int rank = 0;
        for (int y = 0; y < np; ++y) rank += d64[y] < v || (d64[y] == v && pid[y] < id);
        if (rank < k) {
            a.out_ids[qi * a.out_stride + rank] = (int64_t)id;
            a.out_dist[qi * a.out_stride + rank] = (float)sqrt(v);
        }
    }
    __syncthreads();
    return true;
}

template <int T = WG>
__device__ void write_topk(const AnnArgs& a, int64_t qi, const float* qs, const int32_t* cpos,
                           const float* cdist, int n_ver, int rounds, int exit_kind,
                           int64_t scanned, Smem& sh) {
    const int32_t* perm = a.perm;
    const int k = query_params(a, qi).k;
    bool done = false;
    if (n_ver <= CAP) {
        // the k-th smallest FP32 value, then the FP64 re-rank
        float kth32 = __int_as_float(0x7f800000);
        if (n_ver > k) {
            for (int i = threadIdx.x; i < n_ver; i += T)
                sh.skey[i] = ((uint64_t)__float_as_uint(cdist[i]) << 32) | (uint32_t)perm[cpos[i]];
            __syncthreads();
            kth32 = __uint_as_float((uint32_t)(lds_select<T>(n_ver, k, sh) >> 32));
        }
        done = rerank_topk64<T>(a, qi, qs, cpos, n_ver, kth32,
                             [&](int j, float& v, int& mi) { v = cdist[j]; mi = j; }, sh);
    }
    if (done) {
    } else if (n_ver <= CAP) {
        for (int i = threadIdx.x; i < n_ver; i += T)
            sh.skey[i] = ((uint64_t)__float_as_uint(cdist[i]) << 32) | (uint32_t)perm[cpos[i]];
        __syncthreads();
        int m = n_ver;
        if (n_ver > k) {
            const uint64_t kth = lds_select<T>(n_ver, k, sh);
            // the k smallest keys, gathered through the histogram space
            uint64_t* tmp = reinterpret_cast<uint64_t*>(sh.hist);
            static_assert(NB * sizeof(uint32_t) >= PMLSH_MAX_K * sizeof(uint64_t),
                          "top-k staging must fit the histogram");
            if (threadIdx.x == 0) sh.cnt1 = 0;
            __syncthreads();
            for (int b0 = 0; b0 < n_ver; b0 += T) {
                const int i = b0 + threadIdx.x;
                const bool take = i < n_ver && sh.skey[i] <= kth;
                const int slot = wave_append(take, &sh.cnt1);
                if (take) tmp[slot] = sh.skey[i];
            }
            __syncthreads();
            for (int j = threadIdx.x; j < k; j += T) sh.skey[j] = tmp[j];
            __syncthreads();
            m = k;
        }
        bitonic_sort<T>(m, sh);
        for (int j = threadIdx.x; j < k; j += T) {
            const uint64_t key = sh.skey[j];
            a.out_ids[qi * a.out_stride + j] = (int64_t)(uint32_t)key;
            a.out_dist[qi * a.out_stride + j] = sqrtf(__uint_as_float((uint32_t)(key >> 32)));
        }
    } else {
        auto c_src = [&](auto&& v) {
            for (int base = 0; base < n_ver; base += T) {
                const int i = base + threadIdx.x;
                const bool valid = i < n_ver;
                uint64_t key = 0;
                if (valid) key = ((uint64_t)__float_as_uint(cdist[i]) << 32) | (uint32_t)perm[cpos[i]];
                v(valid, key, i);
            }
        };
        int32_t* topk = a.ws_topk + qi * 3 * (int64_t)a.k;
        block_select<T>(c_src, [&](int32_t i, int slot) { if (slot < k) topk[slot] = i; }, 0ull,
                     ~0ull, k, false, 0, sh);
        __syncthreads();
        // the k-th smallest FP32 value (the largest of the k selected), then
        // the FP64 re-rank
        float kmax = 0.f;
        for (int j = threadIdx.x; j < k; j += T) kmax = fmaxf(kmax, cdist[topk[j]]);
        for (int off = 32; off > 0; off >>= 1) kmax = fmaxf(kmax, __shfl_xor(kmax, off));
        if (lane_id() == 0) sh.red[threadIdx.x >> 6] = __float_as_int(kmax);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < (T / 64); ++w) kmax = fmaxf(kmax, __int_as_float(sh.red[w]));
        __syncthreads();
        if (rerank_topk64<T>(a, qi, qs, cpos, n_ver, kmax,
                          [&](int j, float& v, int& mi) { v = cdist[j]; mi = j; }, sh))
            done = true;
    }
    if (!done && n_ver > CAP) {
        const int32_t* topk = a.ws_topk + qi * 3 * (int64_t)a.k;
        for (int j = threadIdx.x; j < k; j += T) {
            const int i = topk[j];
            sh.skey[j] = ((uint64_t)__float_as_uint(cdist[i]) << 32) | (uint32_t)perm[cpos[i]];
        }
        __syncthreads();
        bitonic_sort<T>(k, sh);
        for (int j = threadIdx.x; j < k; j += T) {
            const uint64_t key = sh.skey[j];
            a.out_ids[qi * a.out_stride + j] = (int64_t)(uint32_t)key;
            a.out_dist[qi * a.out_stride + j] = sqrtf(__uint_as_float((uint32_t)(key >> 32)));
        }
    }
    if (a.out_stats && threadIdx.x == 0) {
        int32_t* st = a.out_stats + qi * 4;
        st[0] = rounds;
        st[1] = n_ver;
        st[2] = exit_kind;
        st[3] = scanned > 0x7fffffffll ? 0x7fffffff : (int32_t)scanned;
    }
}

__device__ void ann_one(const AnnArgs& a, int64_t qi, int32_t* fa, int32_t* fb, float* qs,
                        Smem& sh);

__global__ __launch_bounds__(WG) void ann_kernel(AnnArgs args) {
    // the argument block read in place (constant memory): naming the
    // parameter itself lets the compiler copy all of it into scratch memory
    (void)args;
    const AnnArgs& a = *(const AnnArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Smem& sh = *reinterpret_cast<Smem*>(smem_raw);
    float* qs = reinterpret_cast<float*>(smem_raw + ((sizeof(Smem) + 15) & ~size_t(15)));

    // workgroup b answers queries b, b + G, b + 2G, ... with the frontier
    // lists of slot b (G = gridDim.x slots)
    int32_t* fa = a.ws_front + (int64_t)blockIdx.x * 2 * a.n_leaves;
    int32_t* fb = fa + a.n_leaves;
    // every query, or only those the batched path flagged (a.pq_list)
    const int64_t total = a.pq_list ? (int64_t)a.pq_list[0] : a.nq;
    for (int64_t j = blockIdx.x; j < total; j += gridDim.x) {
        __syncthreads();
        ann_one(a, a.pq_list ? (int64_t)a.pq_list[1 + j] : j, fa, fb, qs, sh);
    }
}

// The budget cut of the per-query path in the FP64 order, as cut_fp64 does
// for the batched path: the need members chosen from the shell (FP32 keys,
// in cpos[n_ver, n_ver + need)) are replaced by the shell's entries below a
// band of 2E around the largest chosen FP32 pd^2 and the first band entries
// by (FP64 pd^2, id). The band stays inside the shell (entries of earlier
// rounds are in C by ball membership). Nothing changes when the band holds
// more than 512 entries.
template <class BallSrc>
__device__ void shell_cut_fp64(const AnnArgs& a, int64_t qi, const QueryCtx& qc, BallSrc& ball_src,
                               uint32_t lo_hi, int n_ver, int need, int32_t* cpos, Smem& sh) {
    constexpr int kBandCap = 512;
    int32_t* bpos = reinterpret_cast<int32_t*>(sh.hist);
    uint32_t* bid = reinterpret_cast<uint32_t*>(sh.hist + kBandCap);
    double* b64 = reinterpret_cast<double*>(sh.hist + 2 * kBandCap);
    static_assert(NB >= 4 * kBandCap, "the band must fit the histogram");
    // the largest FP32 pd^2 among the chosen
    float kmax = 0.f;
    for (int j = threadIdx.x; j < need; j += WG)
        kmax = fmaxf(kmax, proj_dist2(a.proj + (int64_t)cpos[n_ver + j] * MP, qc.qp));
    for (int off = 32; off > 0; off >>= 1) kmax = fmaxf(kmax, __shfl_xor(kmax, off));
    if (lane_id() == 0) sh.red[threadIdx.x >> 6] = __float_as_int(kmax);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) kmax = fmaxf(kmax, __int_as_float(sh.red[w]));
    __syncthreads();
    const float big = sqrtf(qc.qn2) + a.coord_scale;
    const float e = 2.f * (2.384185791015625e-07f * sqrtf(kmax) * big + 1.9073486328125e-06f * kmax);
    const float blo = fmaxf(kmax - 2.f * e, __uint_as_float(lo_hi)), bhi = kmax + 2.f * e;
    if (threadIdx.x == 0) sh.cnt2 = 0;
    __syncthreads();
    int below = 0;
    ball_src([&](bool mem, uint64_t key, int32_t pos) {
        const float v = __uint_as_float((uint32_t)(key >> 32));
        below += mem && v < blo;
        const bool inb = mem && v >= blo && v <= bhi;
        const int slot = wave_append(inb, &sh.cnt2);
        if (inb && slot < kBandCap) {
            bpos[slot] = pos;
            bid[slot] = (uint32_t)key;
        }
    });
    below = block_sum(below, sh);
    const int nb = sh.cnt2;
    // a band that is taken whole leaves the FP32 choice as it is
    if (nb > kBandCap || below > need || below + nb <= need) return;
    for (int j = threadIdx.x; j < nb; j += WG) {
        const int64_t pos = bpos[j];
        double acc = 0.0;
#pragma unroll
        for (int t = 0; t < MP; ++t) {
            const double o = (double)a.proj[pos * MP + t] + (double)a.proj_lo[pos * MP + t];
            const double q = (double)a.qp[qi * MP + t] + (double)a.qp_lo[qi * MP + t];
            const double dd = q - o;
            acc = fma(dd, dd, acc);
        }
        b64[j] = acc;
    }
    __syncthreads();
    // C's shell part again: the entries below the band, then the band's
    // first need - below
    if (threadIdx.x == 0) sh.cnt2 = 0;
    __syncthreads();
    ball_src([&](bool mem, uint64_t key, int32_t pos) {
        const bool take = mem && __uint_as_float((uint32_t)(key >> 32)) < blo;
        const int slot = wave_append(take, &sh.cnt2);
        if (take) cpos[n_ver + slot] = pos;
    });
    __syncthreads();
    const int keep = need - below;
    for (int j = threadIdx.x; j < nb; j += WG) {
        const double v = b64[j];
        const uint32_t id = bid[j];
        int rank = 0;
        for (int y = 0; y < nb; ++y) rank += b64[y] < v || (b64[y] == v && bid[y] < id);
        if (rank < keep) cpos[n_ver + below + rank] = bpos[j];
    }
    __syncthreads();
}

// Algorithm 2 for query qi, round by round with PM-tree walks.
__device__ void ann_one(const AnnArgs& a, int64_t qi, int32_t* fa, int32_t* fb, float* qs,
                        Smem& sh) {
    QueryCtx qc;
    load_query(a, qi, qs, qc);
    const float* qp = qc.qp;
    const float* qpiv = qc.qpiv;
    const float qn2 = qc.qn2;
    __syncthreads();

    const AnnQueryParams qpar = query_params(a, qi);
    int32_t* cpos = a.ws_cpos + qi * (int64_t)a.budget;
    float* cdist = a.ws_cdist + qi * (int64_t)a.budget;
    const int32_t* perm = a.perm;
    const int B = qpar.budget;

    double r = qpar.r_min;
    int n_ver = 0;
    int rounds = 0;
    int exit_kind = 0;
    int64_t scanned = 0;
    uint32_t prev_hi = 0;     // bits of the previous squared radius
    bool first = true;

    for (;;) {
        if (rounds > 0) {
            const double cr = qpar.c * r;
            const float thr2 = (float)(cr * cr);
            int loc = 0;
            for (int i = threadIdx.x; i < n_ver; i += WG) loc += cdist[i] <= thr2;
            if (block_sum(loc, sh) >= qpar.k) { exit_kind = PMLSH_EXIT_NEAR; break; }
        }
        // the round after the cap is the last: every point whose projected
        // distance is a number lies in its ball, so only a query whose
        // distances are not (NaN or infinite coordinates) leaves it without
        // the budget's points
        const bool last = rounds >= MAX_ROUNDS;
        if (last) r = __longlong_as_double(0x7ff0000000000000ll);
        const double Rd = qpar.t * r;
        const float R = (float)Rd;
        const float R2 = (float)(Rd * Rd);
        ++rounds;
        const float slack = 1e-5f * (sqrtf(qn2) + a.coord_scale + R);

        // range query (q', R), shrunk to the budget when the ball is large
        float Rq = R;
        int nl = traverse(a, qp, qpiv, Rq, slack, true, B, fa, fb, sh);
        const int32_t* leaves = fa;
        const float R2q = Rq < R ? (float)((double)Rq * (double)Rq) : R2;

        // shell (prev, R2q] on the 64-bit keys (pd^2 bits << 32 | id)
        const uint32_t lo_hi = first ? 0u : prev_hi + 1u;
        uint32_t hi_hi = __float_as_uint(R2q);
        const uint64_t klo = (uint64_t)lo_hi << 32;
        uint64_t khi = ((uint64_t)hi_hi << 32) | 0xffffffffull;
        int sh0 = shift_for(klo, khi);
        auto ball_src = [&](auto&& v) {
            scan_leaves(a, leaves, nl, qp, [&](bool valid, int pos, float pd2) {
                const uint32_t b = __float_as_uint(pd2);
                const bool mem = valid && b >= lo_hi && b <= hi_hi;
                const uint64_t key = mem ? (((uint64_t)b << 32) | (uint32_t)perm[pos]) : 0ull;
                v(mem, key, pos);
            });
        };
        auto count_pass = [&]() {
            clear_hist(sh);
            int loc = 0, sc = 0;
            ball_src([&](bool mem, uint64_t key, int32_t) {
                if (mem) { ++loc; atomicAdd(&sh.hist[(key - klo) >> sh0], 1u); }
            });
            for (int li = threadIdx.x; li < nl; li += WG) sc += a.ce[leaves[li]] - a.cb[leaves[li]];
            scanned += block_sum(sc, sh);
            return block_sum(loc, sh);
        };
        int shell = count_pass();
        if (Rq < R && n_ver + shell < B) {
            // the lowered radius fell short (rounding at the bound): redo the
            // range query at the full radius
            Rq = R;
            nl = traverse(a, qp, qpiv, Rq, slack, false, B, fa, fb, sh);
            hi_hi = __float_as_uint(R2);
            khi = ((uint64_t)hi_hi << 32) | 0xffffffffull;
            sh0 = shift_for(klo, khi);
            shell = count_pass();
        }

        if (n_ver + shell >= B) {
            const int need = B - n_ver;
            block_select(ball_src,
                         [&](int32_t pos, int slot) {
                             if (slot < need) cpos[n_ver + slot] = pos;
                         },
                         klo, khi, need, true, shell, sh);
            __syncthreads();
            shell_cut_fp64(a, qi, qc, ball_src, lo_hi, n_ver, need, cpos, sh);
            verify(a, qs, cpos, cdist, n_ver, B);
            n_ver = B;
            exit_kind = PMLSH_EXIT_BUDGET;
            __syncthreads();
            break;
        }
        if (threadIdx.x == 0) sh.cnt1 = 0;
        __syncthreads();
        ball_src([&](bool mem, uint64_t, int32_t pos) {
            const int slot = wave_append(mem, &sh.cnt1);
            if (mem && n_ver + slot < B) cpos[n_ver + slot] = pos;
        });
        __syncthreads();
        verify(a, qs, cpos, cdist, n_ver, n_ver + shell);
        n_ver += shell;
        __syncthreads();
        prev_hi = hi_hi;
        first = false;
        if (last || rounds >= a.max_rounds) break;
        r = qpar.c * r;
    }

    write_topk(a, qi, qs, cpos, cdist, n_ver, rounds, exit_kind, scanned, sh);
    // places that no member fills
    __syncthreads();
    for (int j = n_ver + (int)threadIdx.x; j < qpar.k; j += WG) {
        a.out_ids[qi * a.out_stride + j] = -1;
        a.out_dist[qi * a.out_stride + j] = __int_as_float(0x7f800000);
    }
}

// ------------------------------------------------------------------------
// Batched path, for B <= kWideBudget.
//
// Every candidate set of Algorithm 2 is a prefix of the order of the data by
// (projected distance, id) (the ball of a round holds the points up to t*r;
// a budget exit keeps the B first), and "the ball holds at least B points"
// is "the B-th projected distance is <= t*r". So the list L of the B
// projected-nearest points, verified as far as the rounds need, decides
// every round. The path finds L in three kernels:
//   tau     per query: an upper bound tau on the B-th projected distance
//           from the tree alone (the traversal's budget shrink);
//   filter  per leaf block x query block: each leaf's points are loaded once
//           into registers and tested against every query of the block whose
//           range query (q', tau) reaches the leaf (Eq. 5); points with
//           pd^2 <= tau^2 are appended to the query's candidate list;
//   finish  per query: exact radix select of L from the list, the rounds of
//           Algorithm 2 on L with incremental verification, the top-k; or the
//           same in three kernels (pool_cut_kernel and its followers).
// Queries whose list overflows (or that fall outside the path) are flagged
// and answered by the per-query kernel above.

// Squared FP32 distances from every query of the batch to every chunk centre,
// as |q'|^2 + |c|^2 - 2 q'.c (clamped at 0), on the FP32 matrix cores: a
// workgroup takes 64 queries x 256 chunks in four sub-tiles of 64 chunks,
// each wave a strip of 16 queries x 64 chunks per sub-tile (four 16 x 16
// tiles of v_mfma_f32_16x16x4_f32, K = 16 in four steps; the next
// sub-tile's centres are loaded meanwhile); each sub-tile goes through LDS
// and leaves as one block of the matrix (64 queries x 64 chunks, 8 KB
// contiguous). The values are bf16 bit patterns, rounded toward zero (the
// FP32 value's upper half), so each stored value is at most the FP32 value
// and above it by less than a factor 1 + 2^-7. The expansion's rounding error, in any
// summation order of the 16 products, stays below 64 u (|q'| + S)^2 (S
// bounds every centre norm); the chunk-ball test adds that much to its
// threshold and tests the rounded-down value, and the choice of chunks for
// the bound needs no exactness.
constexpr int DQB = 64;    // queries per workgroup
constexpr int DCS = 64;    // chunks per sub-tile
constexpr int DCB = 256;   // chunks per workgroup (four sub-tiles)

__global__ __launch_bounds__(WG) void dist_kernel(AnnArgs a) {
    __shared__ float sq[DQB][MP + 1];
    __shared__ float sc[DCS][MP + 1];
    __shared__ float sqn[DQB], scn[DCS];
    __shared__ __align__(16) uint16_t tile[DQB][DCS];
    const int q0 = blockIdx.y * DQB;
    const int nch = (int)(a.n_pad16 >> 6);
    const int nqb = min(DQB, a.nq - q0);
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    // one centre coordinate quadruple per thread: centre e / 4, columns 4 (e % 4)
    const int ce = threadIdx.x >> 2, cq = (threadIdx.x & 3) * 4;
    auto load_cen = [&](int c0) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c0 + ce < nch) v = *reinterpret_cast<const float4*>(a.chunk_cen + (int64_t)(c0 + ce) * MP + cq);
        return v;
    };
    float4 cnext = load_cen(blockIdx.x * DCB);
    {
        // every load of the staging goes out before the LDS stores
        constexpr int PER = DQB * MP / WG;
        float v[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = threadIdx.x + u * WG, r = e / MP;
            v[u] = r < nqb ? a.qp[(int64_t)(q0 + r) * MP + e % MP] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = threadIdx.x + u * WG;
            sq[e / MP][e % MP] = v[u];
        }
    }
    __syncthreads();
    if (threadIdx.x < DQB) {
        float n2 = 0.f;
#pragma unroll
        for (int t = 0; t < MP; ++t) n2 = fmaf(sq[threadIdx.x][t], sq[threadIdx.x][t], n2);
        sqn[threadIdx.x] = n2;
    }
    // A operand (16 queries x 16): lane holds row li, columns lk, 4 + lk, ...
    float av[MP / 4];
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < MP / 4; ++kk) av[kk] = sq[16 * wave + li][4 * kk + lk];
    for (int sub = 0; sub < DCB / DCS; ++sub) {
        const int c0 = blockIdx.x * DCB + sub * DCS;
        if (c0 >= nch) break;
        sc[ce][cq] = cnext.x;
        sc[ce][cq + 1] = cnext.y;
        sc[ce][cq + 2] = cnext.z;
        sc[ce][cq + 3] = cnext.w;
        if (sub + 1 < DCB / DCS) cnext = load_cen(c0 + DCS);
        __syncthreads();
        if (threadIdx.x < DCS) {
            float n2 = 0.f;
#pragma unroll
            for (int t = 0; t < MP; ++t) n2 = fmaf(sc[threadIdx.x][t], sc[threadIdx.x][t], n2);
            scn[threadIdx.x] = n2;
        }
        // B (16 x 16 chunks): lane holds row lk, column li; result register v
        // of lane l is query 4 (l / 16) + v and chunk l % 16 of the tile
        float4_t acc[4] = {};
#pragma unroll
        for (int kk = 0; kk < MP / 4; ++kk)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[kk], sc[16 * t + li][4 * kk + lk],
                                                              acc[t], 0, 0, 0);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int cl = 16 * t + li;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int ql = 16 * wave + 4 * lk + v;
                const float d2 = fmaxf(fmaf(-2.f, acc[t][v], sqn[ql] + scn[cl]), 0.f);
                tile[ql][cl] = (uint16_t)(__float_as_uint(d2) >> 16);
            }
        }
        __syncthreads();
        // four threads per query row, 16 chunks (32 bytes) each: the sub-tile
        // (64 queries x 64 chunks) is one block of the matrix, written as
        // one contiguous 8 KB run
        const int ql = threadIdx.x >> 2, seg = (threadIdx.x & 3) * 16;
        uint32_t gm = 0xffffu;
        {
            const uint4* src = reinterpret_cast<const uint4*>(&tile[ql][seg]);
            const uint4 x0 = src[0], x1 = src[1];
            if (ql < nqb) {
                uint4* dst = reinterpret_cast<uint4*>(a.cdist + cdist_at(a, q0 + ql, c0 + seg));
                dst[0] = x0;
                dst[1] = x1;
            }
            const uint32_t w[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint32_t h = (e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xffffu);
                if (c0 + seg + e < nch) gm = min(gm, h);
            }
        }
        // the group minimum over the four threads of the row
        gm = min(gm, (uint32_t)__shfl_xor((int)gm, 1));
        gm = min(gm, (uint32_t)__shfl_xor((int)gm, 2));
        if ((threadIdx.x & 3) == 0 && ql < nqb)
            a.cgmin[(int64_t)(q0 + ql) * a.gld + (c0 >> 6)] = (uint16_t)gm;
    }
}

// float bits >> 19 of 2^-64: the first of the fixed centre-distance bins
constexpr uint32_t kCenBinBase = 63u << 4;
// Groups (and 256-chunk blocks) the bound kernel lists per query at most, and
// the largest LDS footprint of its group minima and group list (beyond it the
// minima are read from HBM in every pass).
constexpr int kGrpCap = 2048;
constexpr size_t kTauGroupLds = 64 * 1024;

// Upper bound tau on the budget-th smallest projected distance of one query,
// and the query's row of the chunk mask:
//   1. the squared distances from q' to every 64-point chunk centre (computed
//      by dist_kernel, bf16 lower bounds), read four chunks per thread, and
//      the minimum of every group of 64 chunks, which rules out the groups
//      that cannot hold a chosen chunk or a passing one;
//   2. the chunks nearest to q' that hold at least min(n, 2 * budget) points,
//      chosen with a histogram of those distances weighted by chunk sizes;
//   3. over the points of the chosen chunks, the budget-th smallest pd^2
//      (upper edge of its histogram bin) is tau^2;
//   4. the radius of the chunk-ball test of Eq. 5 (a chunk can hold a point
//      within tau of q' only if |q' - centre| <= radius + tau), applied to
//      every chunk by mask_kernel.
// The chosen points are data points, so the ball of radius tau holds at least
// `budget` points and therefore the budget nearest points by projected
// distance. The choice of chunks only affects how tight tau is, never its
// validity.
//
// Steps 1 to 3 are this function's, which returns tau^2.
__device__ __forceinline__ float budget_radius2(const AnnArgs& a, int64_t qi, const QueryCtx& qc,
                                                Smem& sh, unsigned char* smem_raw) {
    const int nch = (int)(a.n_pad16 >> 6);
    const int ng4 = (nch + 3) >> 2;
    const int ngr = (nch + 63) >> 6;
    // four bf16 distances per 8-byte element (element g: chunks 4 g .. 4 g + 3;
    // the 16 elements of a group of 64 chunks are contiguous)
    const uint2* cd4 = reinterpret_cast<const uint2*>(a.cdist + cdist_at(a, qi, 0));
    const int64_t band_stride4 = 1024;   // uint2 elements per block
    auto row4 = [&](int g) { return cd4[(int64_t)(g >> 4) * band_stride4 + (g & 15)]; };
    const uint16_t* grow16 = a.cgmin + qi * a.gld;
    // the group minima (copied to LDS when a.glds is set, else read in the
    // row), then the list of candidate groups and the list of chosen chunks
    unsigned char* lds_free = smem_raw + offsetof(Smem, skey);
    const uint16_t* gmin = grow16;
    if (a.glds) {
        uint16_t* g = reinterpret_cast<uint16_t*>(lds_free);
        // eight loads per thread go out before their LDS stores
        for (int j0 = threadIdx.x; j0 < ngr; j0 += 8 * WG) {
            uint16_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = j0 + u * WG;
                v[u] = j < ngr ? grow16[j] : (uint16_t)0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = j0 + u * WG;
                if (j < ngr) g[j] = v[u];
            }
        }
        gmin = g;
        lds_free += 2 * (size_t)((ngr + 7) & ~7);
    }
    int32_t* glist = reinterpret_cast<int32_t*>(lds_free);
    // the chunks chosen for the bound (step 2)
    int32_t* sel = glist + kGrpCap;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    // bf16 bit pattern k of an element (non-negative values: ordered as
    // unsigned integers)
    auto half_k = [](const uint2& v, int k) {
        const uint32_t w = k < 2 ? v.x : v.y;
        return (k & 1) ? (w >> 16) : (w & 0xffffu);
    };
    const uint32_t hbase = kCenBinBase;
    auto cbin = [&](uint32_t h) { return min(max(h >> 3, hbase) - hbase, (uint32_t)(NB - 1)); };
    const int32_t budget = query_params(a, qi).budget;
    const int64_t want = min((int64_t)a.n, (int64_t)a.sample * budget);
    const int wc = (int)min<int64_t>(min(nch, a.sel_cap), (want + 63) / 64 + 1);

    // b0 bounds the bin sought in step 1 from above: every group holds a
    // chunk at its minimum, so with wc groups whose minima lie in bins <= b0
    // at least wc chunks lie there, and only chunks in those bins need to be
    // counted. A group whose minimum lies above b0 holds none of them: the
    // passes visit only the ngl groups listed (the whole row when more than
    // a.grp_cap groups qualify).
    clear_hist(sh);
    // the nearest group besides, for the order that the queries finish in
    uint32_t near = 0xffffffffu;
    for (int j = threadIdx.x; j < ngr; j += WG) {
        const uint32_t h = gmin[j];
        atomicAdd(&sh.hist[cbin(h)], 1u);
        near = min(near, (h << 16) | (uint32_t)min(j, 0xffff));
    }
    if (threadIdx.x == 0) {
        sh.thr_bin = NB - 1;
        sh.cnt0 = 0;
        sh.near = 0xffffffffu;
    }
    __syncthreads();
    if (a.ordered) atomicMin(&sh.near, near);
    uint32_t b0 = NB - 1;
    if (ngr >= wc) {
        find_threshold(wc, sh);
        b0 = (uint32_t)sh.thr_bin;
    }
    for (int j0 = 0; j0 < ngr; j0 += WG) {
        const int j = j0 + threadIdx.x;
        const bool take = j < ngr && cbin(gmin[j]) <= b0;
        const int slot = wave_append(take, &sh.cnt0);
        if (take && slot < a.grp_cap) glist[slot] = j;
    }
    __syncthreads();
    const int ngl = sh.cnt0;
    const bool grp = ngl <= a.grp_cap;
    __syncthreads();
    // f(g, element g of the row) for every element of the listed groups, or
    // of the whole row (16 consecutive threads read a group's 128 bytes)
    auto for_elems = [&](auto&& f) {
        if (grp) {
            for (int e = threadIdx.x; e < 16 * ngl; e += WG) {
                const int g = 16 * glist[e >> 4] + (e & 15);
                if (g < ng4) f(g, row4(g));
            }
        } else {
            for (int g = threadIdx.x; g < ng4; g += WG) f(g, row4(g));
        }
    };

    // 1: histogram of the centre distances (chunk counts) on fixed bins: 16
    // per octave of the squared distance over [2^-64, 2^64), clamped at both
    // ends, so no range pass is needed. The chosen chunks are those of the
    // bins up to the one where the running count reaches wc = min(n_chunks,
    // ceil(want / 64) + 1) chunks, want = min(n, 2 * budget) points (the
    // extra chunk covers the one chunk with fewer than 64 points).
    clear_hist(sh);
    for_elems([&](int g, const uint2& v) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t b = cbin(half_k(v, k));
            if (4 * g + k < nch && b <= b0) atomicAdd(&sh.hist[b], 1u);
        }
    });
    __syncthreads();
    if (threadIdx.x == 0) sh.thr_bin = NB - 1;
    __syncthreads();
    find_threshold(wc, sh);
    const uint32_t tbin = (uint32_t)sh.thr_bin;
    const int nlow = sh.thr_below;         // chunks of the bins below tbin (< wc)
    const int need = wc - nlow;           // chunks still wanted from bin tbin
    const int in_bin = sh.thr_in;
    // every chunk with a stored value <= tlim is chosen: all of bin tbin, or,
    // when that bin holds more than eight chunks beyond those wanted, only
    // its sub-bins (the three low bits of the bf16 pattern) up to the one
    // where the count reaches `need` (the clamped end bins stay whole)
    uint32_t tlim = tbin == (uint32_t)(NB - 1) ? 0xffffu : ((tbin + hbase) << 3) | 7u;
    if (in_bin - need > 8 && tbin != 0u && tbin != (uint32_t)(NB - 1)) {
        __syncthreads();
        clear_hist(sh);
        for_elems([&](int g, const uint2& v) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t h = half_k(v, k);
                if (4 * g + k < nch && (h >> 3) == tbin + hbase) atomicAdd(&sh.hist[h & 7u], 1u);
            }
        });
        __syncthreads();
        if (threadIdx.x == 0) sh.thr_bin = NB - 1;
        __syncthreads();
        find_threshold(need, sh);
        tlim = ((tbin + hbase) << 3) | (uint32_t)sh.thr_bin;
    }
    if (threadIdx.x == 0) sh.cnt1 = 0;
    __syncthreads();

    // 2: the chosen chunks, and the largest distance bound over their points.
    // The list holds sel_cap >= wc chunks: those of the bins below tbin (fewer
    // than wc) come first, then as many of bin tbin's as fit, so its points
    // are at least budget and the bound stays valid
    if (threadIdx.x == 0) sh.cnt2 = 0;
    __syncthreads();
    float rmax = 0.f;
    for_elems([&](int g, const uint2& v) {
        bool tk[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) tk[k] = 4 * g + k < nch && half_k(v, k) <= tlim;
        if (tk[0] | tk[1] | tk[2] | tk[3]) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (tk[k]) {
                    const int i = 4 * g + k;
                    const uint32_t h = half_k(v, k);
                    const int slot = cbin(h) < tbin ? atomicAdd(&sh.cnt1, 1)
                                                    : nlow + atomicAdd(&sh.cnt2, 1);
                    if (slot < a.sel_cap) {
                        // the stored distance is low by less than a factor 1 + 2^-7
                        const float d = sqrtf(__uint_as_float(h << 16)) * 1.0079f;
                        rmax = fmaxf(rmax, d + a.chunk_rad[i]);
                        sel[slot] = i;
                    }
                }
            }
        }
    });
    for (int off = 32; off > 0; off >>= 1) rmax = fmaxf(rmax, __shfl_xor(rmax, off));
    if (lane == 0) sh.red[wave] = __float_as_int(rmax);
    __syncthreads();
    const int nsel = min(nlow + sh.cnt2, a.sel_cap);
    float R = 0.f;
#pragma unroll
    for (int w = 0; w < NWAVE; ++w) R = fmaxf(R, __int_as_float(sh.red[w]));
    __syncthreads();
    // every chosen point lies within R up to rounding; the margin keeps the
    // histogram range above all of them
    R = R * 1.0001f + 1e-5f * (sqrtf(qc.qn2) + a.coord_scale);
    float R2 = (float)((double)R * (double)R);

    // 3: histogram of pd^2 over the chosen points -> budget-th smallest
    const uint32_t hb2 = __float_as_uint(R2) >> 15;
    const uint32_t base2 = hb2 > (uint32_t)(NB - 1) ? hb2 - (uint32_t)(NB - 1) : 0u;
    clear_hist(sh);
    int cnt = 0;
    {
        // four points per thread in flight: their row loads go out together
        constexpr int PU = 4;
        for (int e0 = threadIdx.x; e0 < nsel * 64; e0 += PU * WG) {
            float pd2[PU];
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const int e = e0 + u * WG;
                const int64_t pos = e < nsel * 64 ? ((int64_t)sel[e >> 6] << 6) + (e & 63) : a.n;
                pd2[u] = pos < a.n ? proj_dist2(a.proj + pos * MP, qc.qp)
                                   : __int_as_float(0x7f800000);
            }
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                if (pd2[u] <= R2) {
                    atomicAdd(&sh.hist[radius_bin(pd2[u], base2)], 1u);
                    ++cnt;
                }
            }
        }
    }
    __syncthreads();
    if (block_sum(cnt, sh) >= budget) {
        if (threadIdx.x == 0) sh.thr_bin = NB - 1;
        __syncthreads();
        find_threshold(budget, sh);
        const float e2 = __uint_as_float((base2 + (uint32_t)sh.thr_bin + 1u) << 15);
        if (e2 < R2) R2 = e2;
    } else {
        // rounding left fewer than `budget` chosen points inside R: no bound
        R2 = __int_as_float(0x7f800000);
    }
    return R2;
}

// What a pass over a batch looks for. Budget: every query's budget. Ball: the points of
// one ball, where those are expected to be fewer than a budget above kLeanBudget: tau
// is its radius and no bound is needed. The lists answer the one range query of
// (r,c)-BC, or those rounds of Algorithm 2 whose balls they hold; queries that are
// undecided after those, or whose lists outgrow their pools, are the Rest, a pass for
// the budget that leaves the decided queries out.
enum class Pass { Budget, Ball, Rest };
constexpr int kDecided = -2, kUndecided = -3;   // in a query's flag, after Pass::Ball

// The radius of the last round whose ball a query's list holds in Pass::Ball (0: of none).
__device__ __forceinline__ double ball_radius(const AnnArgs& a, const AnnQueryParams& p) {
    double r = p.r_min;
    if (!(r < a.ball_most)) return 0.0;
    for (int i = 0; a.max_rounds != 1 && i < 64 && p.c * r <= a.ball_most; ++i) r = p.c * r;
    return r;
}

template <Pass PASS>
__global__ __launch_bounds__(WG) void tau_kernel(AnnArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Smem& sh = *reinterpret_cast<Smem*>(smem_raw);
    const int64_t qi = blockIdx.x;
    if constexpr (PASS == Pass::Rest) {
        if (a.q_flag[qi] != kUndecided) {
            if (threadIdx.x == 0) {
                a.qtest[qi] = make_float2(__int_as_float(0x7fc00000), 0.f);   // no chunk passes
                if (qi == 0) a.pq_list[0] = 0u;
            }
            return;
        }
    }
    QueryCtx qc;
    load_query(a, qi, nullptr, qc);
    float R2;
    if constexpr (PASS == Pass::Ball) {
        const AnnQueryParams p = query_params(a, qi);
        const double rd = p.t * ball_radius(a, p);
        R2 = rd > 0.0 ? (float)(rd * rd) : __int_as_float(0x7f800000);
    } else
        R2 = budget_radius2(a, qi, qc, sh, smem_raw);

    // 4: the radius of the chunk-ball test, which mask_kernel applies: it
    // covers the FP32 errors of pd^2 and of the test's own distance
    // (relative 2^-16 and 1e-5 (tau + S)); the margin covers the rounding
    // of the expanded squared distance (64 u (|q'| + S)^2)
    if (threadIdx.x == 0) {
        const float tq0 = sqrtf(R2);
        const float tq = tq0 * (1.f + 1.52587890625e-05f) + 1e-5f * (tq0 + a.coord_scale);
        const float big = sqrtf(qc.qn2) + a.coord_scale;
        a.qtest[qi] = make_float2(tq, 64.f * 5.9604645e-08f * big * big);
    }

    if (threadIdx.x == 0) {
        a.l_count[qi * a.l_stride] = 0u;
        a.q_scanned[qi] = 0u;   // mask_kernel adds 64 per passing chunk
        a.q_flag[qi] = a.ordered ? (int32_t)(sh.near & 0xffffu) : 0;
        if (qi == 0) a.pq_list[0] = 0u;   // the flagged list of the batch starts empty
        // The query's FP16 row of the matrix-core scan, q' taken relative to
        // the centre of the rows. thr = tau^2 - |q'|^2 plus 96 u (|q'| + S)^2
        // (S bounds every |o'| of a scan row) covers the FP32 errors of the
        // exact pd^2, of the centring and of |q'|^2; the further
        // 2^-15 (|q'| + S)^2 covers the FP32 accumulation of the scan and its
        // hi/lo splits. When the rows come from the low-precision projection,
        // q' is the query's own low-precision projection and tau grows by
        // eps(query) + eps_max, which bounds how far a point's low-precision
        // projected distance lies from its exact one.
        const float u = 5.9604645e-08f;   // 2^-24
        const float* qsrc = a.qlp ? a.qlp + qi * MP : qc.qp;
        float qv[MP];
        float qv2 = 0.f, R2s = R2;
#pragma unroll
        for (int t = 0; t < MP; ++t) {
            qv[t] = qsrc[t] - a.scen[t];
            qv2 = fmaf(qv[t], qv[t], qv2);
        }
        if (a.qlp) {
            const float tw = (sqrtf(R2) + (a.qeps[qi] + a.eps_max)) * (1.f + 2.384185791015625e-07f);
            R2s = tw * tw * (1.f + 2.384185791015625e-07f);
        }
        const float qn = sqrtf(qv2);
        const float big = qn + a.scan_scale;
        const float thr = (R2s + 96.f * u * big * big) - qv2 + 3.0517578e-05f * big * big;
        const float s = a.scale16;
        const float v = -(s * s) * thr;
        float qmax = 0.f;
#pragma unroll
        for (int t = 0; t < MP; ++t) qmax = fmaxf(qmax, fabsf(qv[t]));
        const bool ok = fabsf(v) < 30000.f && 2.f * s * qmax < 30000.f && s * qn < 30000.f;
        _Float16 w[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) w[i] = (_Float16)0.f;
        if (ok) {
#pragma unroll
            for (int t = 0; t < MP; ++t) w[t] = (_Float16)(-2.f * s * qv[t]);
            w[16] = (_Float16)1.f;
            w[17] = (_Float16)1.f;
            const _Float16 hi = (_Float16)v;
            w[18] = hi;
            w[19] = (_Float16)(v - (float)hi);
            w[20] = (_Float16)(-s * qn);
        } else {
            // outside the FP16 range (or no finite radius): every product is
            // +1, no candidate, and the per-query path answers the query
            w[18] = (_Float16)1.f;
            if constexpr (PASS == Pass::Ball) a.l_count[qi * a.l_stride] = 0xffffffffu;   // as a list too long
        }
        uint4* dst = reinterpret_cast<uint4*>(a.qaug + qi * 32);
        const uint4* src = reinterpret_cast<const uint4*>(w);
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[i] = src[i];
    }
}

// ---- The order that the three finishing kernels of pools take the queries in ----
//
// Queries near one another in the leaf order gather many of the same rows, and
// each XCD has an L2 of its own. Within a window of kOrderWindow queries they
// are ranked by the nearest group of 64 chunks (ties by index; the group is
// about 2 MB of FP16 rows at 256 dimensions, half an L2), and the workgroups
// of an XCD (every eighth one) take a run of consecutive ranks. Each answer
// stays where it belongs; only the time of the gathers changes. The bound
// kernel leaves the group's number in the query's flag, which the finishing
// kernels write later.
// us per call in order of index / of rank: 1,024 queries, 1M x 256 at B = 4,899
// 842 / 800; 256 queries, 200,000 x 128 at B = 19,349, 423 / 415. Up to
// kLeanBudget the rows are too few to pay for the detour (1M x 256, B = 875,
// 207 / 210; 10M x 128, B = 750, 466 / 498; 20,000 x 32 without contrast, B =
// 300, 107 / 113), and fewer than 64 queries share too little.
constexpr int kOrderWindow = 1024;

// The ranks of queries q0 + first, q0 + first + step, ... below q0 + nqb in
// their window, by one wave (nqb <= 64 and q0 a multiple of 64: one window).
__device__ void order_queries(const AnnArgs& a, int q0, int nqb, int first, int step) {
    if (first >= nqb) return;
    const int w0 = q0 / kOrderWindow * kOrderWindow;
    const int nw = min(kOrderWindow, a.nq - w0);
    const int lane = lane_id();
    int32_t key[kOrderWindow / 64];
#pragma unroll
    for (int u = 0; u < kOrderWindow / 64; ++u)
        key[u] = lane + 64 * u < nw ? a.q_flag[w0 + lane + 64 * u] : 0x7fffffff;
    for (int i = first; i < nqb; i += step) {
        const int me = q0 - w0 + i;
        const int32_t mine = a.q_flag[w0 + me];
        int rank = 0;
#pragma unroll
        for (int u = 0; u < kOrderWindow / 64; ++u)
            rank += __popcll(__ballot(key[u] < mine || (key[u] == mine && lane + 64 * u < me)));
        if (lane == 0) a.q_order[w0 + rank] = w0 + me;
    }
}

// Place `b` of `n` workgroups in an order whose runs of consecutive places go
// to one XCD each (workgroup b runs on XCD b % 8).
__device__ __forceinline__ uint32_t xcd_place(uint32_t b, uint32_t n) {
    const uint32_t x = b & 7u, rem = n & 7u;
    return x * (n >> 3) + min(x, rem) + (b >> 3);
}

// The query of a finishing kernel's place.
__device__ __forceinline__ int64_t query_of(const AnnArgs& a, uint32_t place) {
    return a.q_order[place];
}

// The chunk-ball test of Eq. 5 for every (query, chunk) pair of the batch,
// written as the chunk-major mask the scan reads: bit l of word qb of chunk
// c is query 64 qb + l. A workgroup takes 64 queries x 256 chunks: thread t
// holds the eight chunks 8 (t % 32) .. + 7 of its block and the eight
// queries 8 (t / 32) .. + 7, reads the eight stored squared centre distances
// of each of its query rows in one 16-byte load (eight threads cover a
// query's 128-byte row of a 64-chunk block) and tests d^2 <= (radius +
// tq)^2 + margin with the query's (tq, margin) from the bound kernel. The
// eight query bits of every chunk are one byte of its word, stored in LDS as
// one 8-byte run per thread and assembled per chunk; each query's passing
// chunks, 64 points each, are added to its scan count.
constexpr int MQB = 64;    // queries per workgroup (one mask word)
constexpr int MCH = 256;   // chunks per workgroup: eight per thread of a query octet
static_assert(MCH == 8 * 32 && MQB == 8 * (WG / 32), "thread t: chunk octet t % 32, query octet t / 32");

__global__ __launch_bounds__(WG) void mask_kernel(AnnArgs a) {
    __shared__ float2 qt[MQB];
    __shared__ __align__(16) uint8_t lb[MQB / 8][MCH];   // row qo: byte qo of every chunk's word
    __shared__ uint32_t cnt[MQB];
    const int nch = (int)(a.n_pad16 >> 6);
    const int q0 = blockIdx.y * MQB;
    const int nqb = min(MQB, a.nq - q0);
    const int co = threadIdx.x & 31, qo = threadIdx.x >> 5;
    const int c0 = blockIdx.x * MCH + 8 * co;   // the thread's first chunk
    if (threadIdx.x < MQB) {
        qt[threadIdx.x] = (int)threadIdx.x < nqb ? a.qtest[q0 + threadIdx.x] : make_float2(0.f, 0.f);
        cnt[threadIdx.x] = 0u;
    }
    // the eight rows' loads go out before any test
    uint4 w[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int q = 8 * qo + u;
        w[u] = q < nqb && c0 < nch
                   ? *reinterpret_cast<const uint4*>(a.cdist + cdist_at(a, q0 + q, c0))
                   : make_uint4(0u, 0u, 0u, 0u);
    }
    float rad[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) rad[e] = c0 + e < nch ? a.chunk_rad[c0 + e] : 0.f;
    __syncthreads();
    uint32_t bits[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};   // chunk e: the eight query bits
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int q = 8 * qo + u;
        const float2 t = qt[q];
        const uint32_t h[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
        uint32_t np = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t hb = (e & 1) ? (h[e >> 1] & 0xffff0000u) : (h[e >> 1] << 16);
            const float ra = rad[e] + t.x;
            const bool p = q < nqb && c0 + e < nch && __uint_as_float(hb) <= fmaf(ra, ra, t.y);
            bits[e] |= (uint32_t)p << u;
            np += p;
        }
        // the query's passing chunks over the 32 chunk octets (half a wave)
        np += (uint32_t)__shfl_xor((int)np, 1);
        np += (uint32_t)__shfl_xor((int)np, 2);
        np += (uint32_t)__shfl_xor((int)np, 4);
        np += (uint32_t)__shfl_xor((int)np, 8);
        np += (uint32_t)__shfl_xor((int)np, 16);
        if (co == 0 && np) cnt[q] = np;
    }
    // the eight chunks' bytes of this query octet in one 8-byte store
    *reinterpret_cast<uint2*>(&lb[qo][8 * co]) =
        make_uint2(bits[0] | (bits[1] << 8) | (bits[2] << 16) | (bits[3] << 24),
                   bits[4] | (bits[5] << 8) | (bits[6] << 16) | (bits[7] << 24));
    __syncthreads();
    for (int i = threadIdx.x; i < MCH; i += WG) {
        const int c = blockIdx.x * MCH + i;
        uint64_t wd = 0ull;
#pragma unroll
        for (int o = 0; o < MQB / 8; ++o) wd |= (uint64_t)lb[o][i] << (8 * o);
        if (c < nch) a.cmask[cmask_at(a, c, blockIdx.y)] = wd;
    }
    if (a.out_stats && (int)threadIdx.x < nqb && cnt[threadIdx.x])
        atomicAdd(&a.q_scanned[q0 + threadIdx.x], 64u * cnt[threadIdx.x]);
    if (a.ordered)
        order_queries(a, q0, nqb, blockIdx.x * NWAVE + (threadIdx.x >> 6), gridDim.x * NWAVE);
}

// ---- Matrix-core scan (the range filter of the batched path) ----
//
// For every (point, query) pair of the batch one FP16 MFMA dot product of
// 32-half rows decides whether the point can lie within tau of the query:
//   point row P: s*o'_0..s*o'_15, hi(s^2|o'|^2), lo(s^2|o'|^2), 1, 1,
//                cm*s*|o'|, zeros
//   query row Q: -2s*q'_0..-2s*q'_15, 1, 1, hi(-s^2 thr), lo(-s^2 thr),
//                -s*|q'|, zeros
// so P.Q = s^2 (|o'|^2 - 2 q'.o' - thr - cm |q'||o'|), accumulated in FP32.
// thr is tau^2 - |q'|^2 plus margins for the FP32 errors of the exact pd^2 and
// of the split terms; the FP16 rounding of the dot product is bounded by
// 2^-9 |q'||o'|, which the cm term covers pair by pair. Hence every point
// whose FP32 direct-difference pd^2 is within tau^2 gives P.Q < 0, and the
// pool also receives a few points just outside, which the finishing kernel
// removes with the exact pd^2. This is the PM-tree range query of the
// paper computed without the tree: the node tests of Eq. 5 only save work on
// a processor that compares one pair at a time, while the matrix cores
// compare all pairs of a batch at 16 x 16 x 32 per instruction.
//
// Grid: x strides over 64-point chunks, y over blocks of 512 or 1,024 queries;
// each wave of a workgroup owns two or four of the block's mask words (128 or 256
// queries).
// For each chunk a wave packs the queries whose chunk-ball test passed (the
// set bits of its mask words) into a list and runs the MFMA on groups of 16
// listed queries, so a group's 16 columns are all queries that may hold
// candidates in the chunk (the last group is padded with a row whose product
// with every point is positive). The FP16 rows of the block's queries sit in
// LDS as B operands (lane l: listed query 16 g + l % 16, halves
// 8 (l / 16) .. + 7); the chunk's four 16-point tiles are the A operands
// (lane l: point 16 t + l % 16, same halves). Halves 24..31 are zero in every
// point and query row: neither is stored, and lanes 48..63 hold zeros. A
// result register r of lane l holds point 4 (l / 16) + r of the tile and
// listed query l % 16.

// Two block shapes of the scan: 512 queries in four waves of 128 (four
// workgroups per compute unit) for indexes of fewer than kScanLargeChunks
// chunks, 1,024 in sixteen waves of 256 (one per compute unit) above: staging a
// block's query rows is a fixed cost per workgroup, and with 128 queries per
// wave a chunk's rows are read by twice as many waves (10M x 128, 1,024
// queries: 296 us against 187 with 256). Four waves per SIMD in either
// (128 VGPRs, two chunk slots in flight): the loop's query lists, matrix products
// and ballots wait on one another, and more waves hide more of that than deeper
// slots did. 1M x 256, 1,024 queries, us, three waves with four slots / four
// with three / four with two / four with one: B = 885 54 / 70 / 48 / 52;
// B = 4,899 139 / 145 / 127 / 132; 1M x 960 without contrast 284 / 239 / 226 / 230
// (with empty chunks skipped and the denser staging 43, 118 and 183 now).
struct ScanSmall { static constexpr int QB = 512, QW = 128, NW = 4, WGS = 4, STG = 512; };
struct ScanLarge { static constexpr int QB = 1024, QW = 256, NW = 16, WGS = 1, STG = 512; };
constexpr int64_t kScanLargeChunks = 32768;   // 2,097,152 points
// An index so small that waves of 128 queries would leave SIMDs idle is bound by
// one wave's chain of candidates and flushes (every point of its chunk may be a
// candidate of every query): waves of 64 queries with a longer stage. 1,000
// queries, whole calls, with ScanSmall / ScanFew: 200 x 16, B = 100 97 / 72 us;
// 1,000 x 32, B = 300 94 / 78; 5,000 x 64, B = 300 78 / 72.
struct ScanFew { static constexpr int QB = 256, QW = 64, NW = 4, WGS = 2, STG = 1024; };

// Query rows, then per-wave candidate stages: every wave packs, stages,
// counts and flushes its own candidates, so after the rows are loaded the
// scan needs no workgroup barrier. QB queries per block and NW waves of QW
// queries each, STG candidates staged per wave.
template <class S>
struct __align__(16) ScanShared {
    uint16_t qrow[S::QB + 1][kScanRow];   // FP16 query rows of the block, padding row last
    uint32_t pos[S::NW][S::STG];          // staged candidates: leaf position
    uint8_t qid[S::NW][S::STG];           // and query within the wave's range
    uint32_t hits[S::NW][S::QW], base[S::NW][S::QW];
    // queries of the wave passing the chunk, by column: slot 16 g + j of the
    // list is lcol[j][g]
    uint8_t lcol[S::NW][16][S::QW / 16];
};
template <class S>
constexpr bool scan_shape_ok() {
    return S::QW % 64 == 0 && S::QW <= 256 && S::QB % S::QW == 0 &&
           (S::QB / S::QW & (S::QB / S::QW - 1)) == 0 && S::NW % (S::QB / S::QW) == 0 &&
           sizeof(ScanShared<S>) * S::WGS <= 160 * 1024;
}
static_assert(scan_shape_ok<ScanSmall>() && scan_shape_ok<ScanLarge>() && scan_shape_ok<ScanFew>(),
              "a wave's queries are whole mask words (ids below 256), every query has the same "
              "number of waves, and the scan workgroups of a compute unit fit its LDS");

__device__ __forceinline__ half8_t load_half8(const uint16_t* p) {
    return __builtin_bit_cast(half8_t, *reinterpret_cast<const uint4*>(p));
}

__device__ __forceinline__ void scan_mfma(const half8_t (&av)[4], half8_t b, float4_t (&cc)[4]) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
        cc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[mt], b, float4_t{}, 0, 0, 0);
}

// Writes the wave's staged candidates to the pool with one reservation per
// query (queries qw0 .. qw0 + nqw - 1 of the batch) and empties the stage.
// Only this wave touches its part of the shared memory.
template <class S>
__device__ __forceinline__ void scan_flush(const AnnArgs& a, ScanShared<S>& ss, int wave, int lane,
                                           uint32_t& wn, int64_t qw0, int nqw) {
    uint32_t* hits = ss.hits[wave];
    uint32_t* base = ss.base[wave];
    for (uint32_t e = lane; e < wn; e += 64) atomicAdd(&hits[ss.qid[wave][e]], 1u);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int e = lane; e < nqw; e += 64) {
        const uint32_t h = hits[e];
        if (h) base[e] = atomicAdd(&a.l_count[(qw0 + e) * a.l_stride], h);
        hits[e] = 0u;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (uint32_t e = lane; e < wn; e += 64) {
        const int q = ss.qid[wave][e];
        const uint32_t slot = base[q] + atomicAdd(&hits[q], 1u);
        if (slot < (uint32_t)a.q_cap) a.l_list[(qw0 + q) * a.q_cap + slot] = ss.pos[wave][e];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int e = lane; e < nqw; e += 64) hits[e] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    wn = 0;
}

// Stages the negative results of one 64-point x 16-query group (q: the
// lane's query within the wave's range), flushing the stage first whenever
// a ballot's candidates would not fit, so no candidate is lost. The group is
// skipped when no result is negative; otherwise register r of the four tiles
// is tested together first, since most register positions hold no candidate.
template <class S>
__device__ __forceinline__ void scan_emit(const AnnArgs& a, ScanShared<S>& ss, int wave, int lane,
                                          uint32_t& wn, const float4_t (&cc)[4], int64_t p0, int q,
                                          int64_t qw0, int nqw) {
    // a result is a candidate when its sign bit is set: bit 4 t + r of the
    // lane's mask is register r of tile t
    uint32_t mk = 0u;
#pragma unroll
    for (int b = 15; b >= 0; --b)
        mk = __builtin_amdgcn_alignbit(mk, __float_as_uint(cc[b >> 2][b & 3]), 31);
    // a padding column has no query to write for, whatever its products
    mk = q < 0 ? 0u : mk;
    const uint32_t prow = (uint32_t)p0 + 4u * (uint32_t)(lane >> 4);
    // A step stages one candidate of every lane that has any left, at the count
    // of such lanes below it. Where some lane has many (chunks of a query's own
    // cluster: most points of a column), all of a lane's go to consecutive slots
    // instead, at the prefix sum of the lanes' counts: fewer instructions per
    // step, but the sum before the first.
    uint64_t m = __builtin_amdgcn_ballot_w64(mk != 0u);
    if (!m) return;
    const int own = __popc(mk);
    if (__builtin_amdgcn_ballot_w64(own > 3)) {
        const int upto = wave_inclusive_scan(own);
        const uint32_t nh = (uint32_t)__builtin_amdgcn_readlane(upto, 63);
        if (wn + nh > (uint32_t)S::STG && wn > 0u) scan_flush(a, ss, wave, lane, wn, qw0, nqw);
        if (wn + nh <= (uint32_t)S::STG) {   // else (a group can hold 1,024) the steps below
            uint32_t at = wn + (uint32_t)(upto - own);
            while (mk) {
                const uint32_t b = (uint32_t)__builtin_ctz(mk);
                mk &= mk - 1u;
                ss.pos[wave][at] = prow + ((b >> 2) << 4) + (b & 3u);
                ss.qid[wave][at] = (uint8_t)q;
                ++at;
            }
            wn += nh;
            return;
        }
    }
    do {
        const uint32_t nh = (uint32_t)__popcll(m);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (wn + nh > (uint32_t)S::STG) scan_flush(a, ss, wave, lane, wn, qw0, nqw);
        if (mk) {
            const uint32_t b = (uint32_t)__builtin_ctz(mk);
            ss.pos[wave][wn + rank] = prow + ((b >> 2) << 4) + (b & 3u);
            ss.qid[wave][wn + rank] = (uint8_t)q;
            mk &= mk - 1u;
        }
        wn += nh;
        m = __builtin_amdgcn_ballot_w64(mk != 0u);
    } while (m);
}

template <class S>
__global__ __launch_bounds__(64 * S::NW)
    __attribute__((amdgpu_waves_per_eu(S::NW * S::WGS / 4))) void scan_kernel(AnnArgs a) {
    constexpr int SQB = S::QB;        // queries per scan block
    constexpr int SQW = S::QW;        // queries per wave
    constexpr int NQ = SQB / SQW;     // waves that cover the block's queries
    constexpr int QPL = SQW / 64;     // queries per lane in the list building
    constexpr int SPAD = SQB;         // index of the padding row
    __shared__ ScanShared<S> ss;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lq = lane >> 4;
    const int q0 = blockIdx.y * SQB;
    const int nqb = min(SQB, a.nq - q0);
    const int nwq = (nqb + 63) >> 6;            // mask words of this query block
    // the waves that share the block's words (fewer when there are fewer words),
    // whole words each, and the chunks in work at once
    const int nqg = nwq >= NQ ? NQ : nwq <= 1 ? 1 : 1 << (32 - __builtin_clz(nwq - 1));
    const int nc = S::NW / nqg;
    const int wpw = (nwq + nqg - 1) / nqg;
    const int w0 = wave % nqg * wpw;            // first word of this wave
    const int nw = max(0, min(nwq - w0, wpw));
    const int64_t qw0 = (int64_t)q0 + w0 * 64;  // first query of this wave
    const int nqw = max(0, min(nqb - w0 * 64, nw * 64));   // its queries

    // the block's query rows (halves 0..23; 16 bytes per thread and step)
    for (int e = threadIdx.x; e < (SQB + 1) * 3; e += 64 * S::NW) {
        const int r = e / 3, part = e - 3 * r;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (r < nqb) {
            v = *reinterpret_cast<const uint4*>(a.qaug + (int64_t)(q0 + r) * 32 + part * 8);
        } else if (r == SPAD && part == 2) {
            v.y = 0x3c00u;   // half 18 = 1: the product with any point is >= 0
        }
        *reinterpret_cast<uint4*>(&ss.qrow[r][part * 8]) = v;
    }
    for (int e = lane; e < SQW; e += 64) ss.hits[wave][e] = 0u;
    __syncthreads();

    uint32_t wn = 0;
    // Point chunks, strided over the waves of a query range. Most chunks hold
    // points near none of a wave's queries (1M x 256, B = 885: 69 % of the
    // pairs of a chunk and 128 queries; 10M x 128: 75 % with 256), so a wave
    // loads the mask words of 64 of its chunks at once, one chunk per lane, and
    // visits the non-empty ones only. The rows of the next one are in flight
    // while one is in work.
    const int64_t nchunk = a.n_pad16 >> 6;
    const int64_t G = (int64_t)gridDim.x * nc;
    const int l16 = lane & 15;
    // lane i packs the QPL queries QPL i .. QPL i + QPL - 1 of the wave's
    // range, held in mask word i / (64 / QPL)
    const int pk_word = lane / (64 / QPL), pk_shift = QPL * (lane % (64 / QPL));
    // Every row load is unconditional (a load under a branch makes the compiler
    // wait for every load in flight): lanes 48..63, whose halves 24..31 of the A
    // operand are zero, read halves 16..23, cleared where the rows are used.
    const uint16_t* rbase = a.proj16 + (l16 * kScanRow + (lq < 3 ? lq : 2) * 8);
    const uint32_t rkeep = lq < 3 ? 0xffffffffu : 0u;

    struct Slot {
        half8_t r[4];
    };
    auto load = [&](int64_t cc, Slot& dst) {
        const uint16_t* rp = rbase + cc * (64 * kScanRow);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) dst.r[mt] = load_half8(rp + mt * 16 * kScanRow);
    };
    uint8_t (*lcol)[SQW / 16] = ss.lcol[wave];
    // cm: the mask word that holds the lane's queries
    auto chunk = [&](const Slot& cur, uint64_t cm, int64_t cc) {
        // the list of passing queries: each lane's set bits at the count of
        // set bits in the lanes below it
        const uint32_t pk = (uint32_t)(cm >> pk_shift) & ((1u << QPL) - 1u);
        int total = 0;
        uint32_t at = 0;
#pragma unroll
        for (int b = 0; b < QPL; ++b) {
            const uint64_t bb = __builtin_amdgcn_ballot_w64((pk >> b) & 1u);
            total += __popcll(bb);
            at += __builtin_amdgcn_mbcnt_hi((uint32_t)(bb >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)bb, 0u));
        }
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        half8_t av[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
            av[mt] = __builtin_bit_cast(half8_t, __builtin_bit_cast(u32x4, cur.r[mt]) & rkeep);
#pragma unroll
        for (int b = 0; b < QPL; ++b)
            if ((pk >> b) & 1u) {
                lcol[at & 15][at >> 4] = (uint8_t)(QPL * lane + b);
                ++at;
            }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        // room for a chunk's typical candidates (a fuller chunk flushes
        // inside the emit)
        if (wn > (uint32_t)(S::STG - 256)) scan_flush(a, ss, wave, lane, wn, qw0, nqw);
        const uint8_t* mycol = lcol[l16];
        // two groups per step: their row reads and matrix products go out
        // before either result is examined
        for (int g = 0; g < total; g += 32) {
            const bool two = g + 16 < total;
            const int qa = g + l16 < total ? (int)mycol[g >> 4] : -1;
            const int qb = two && g + 16 + l16 < total ? (int)mycol[(g >> 4) + 1] : -1;
            half8_t ba = half8_t{}, bb = half8_t{};
            if (lq < 3) {
                ba = load_half8(&ss.qrow[qa >= 0 ? w0 * 64 + qa : SPAD][lq * 8]);
                if (two) bb = load_half8(&ss.qrow[qb >= 0 ? w0 * 64 + qb : SPAD][lq * 8]);
            }
            float4_t ca[4], cb[4];
            scan_mfma(av, ba, ca);
            if (two) scan_mfma(av, bb, cb);
            scan_emit(a, ss, wave, lane, wn, ca, cc << 6, qa, qw0, nqw);
            if (two) scan_emit(a, ss, wave, lane, wn, cb, cc << 6, qb, qw0, nqw);
        }
    };
    const int64_t mband = (q0 >> 6) + (nw > 0 ? w0 : 0);
    for (int64_t cb = (int64_t)blockIdx.x * nc + wave / nqg; cb < nchunk; cb += 64 * G) {
        const int64_t mine = cb + lane * G;
        uint64_t m[QPL];
        uint64_t any = 0ull;
#pragma unroll
        for (int k = 0; k < QPL; ++k) {
            const uint64_t v = a.cmask[cmask_at(a, mine < nchunk ? mine : cb, mband + (k < nw ? k : 0))];
            m[k] = mine < nchunk && k < nw ? v : 0ull;
            any |= m[k];
        }
        uint64_t nz = __builtin_amdgcn_ballot_w64(any != 0ull);
        if (!nz) continue;
        // the lane's mask word of the chunk that lane b loaded
        auto word_of = [&](int b) {
            uint64_t cm = 0ull;
#pragma unroll
            for (int k = 0; k < QPL; ++k) {
                const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)m[k], b);
                const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(m[k] >> 32), b);
                if (pk_word == k) cm = ((uint64_t)hi << 32) | lo;
            }
            return cm;
        };
        int b = __builtin_ctzll(nz);
        Slot s0, s1;
        load(cb + b * G, s0);
        for (;;) {
            nz &= nz - 1;
            const int b1 = nz ? __builtin_ctzll(nz) : b;
            load(cb + b1 * G, s1);
            chunk(s0, word_of(b), cb + b * G);
            if (!nz) break;
            nz &= nz - 1;
            b = nz ? __builtin_ctzll(nz) : b1;
            load(cb + b * G, s0);
            chunk(s1, word_of(b1), cb + b1 * G);
            if (!nz) break;
        }
    }
    scan_flush(a, ss, wave, lane, wn, qw0, nqw);
}

// The budget cut of L in the FP64 order. The FP32 pd^2 of a pool entry
// (direct differences of the FP32 projections) is within
// E = 2^-22 pd (|q'| + S) + 2^-19 pd^2 of its value from the FP64 projections
// (the FP32 roundings of both projections and of the differences, and the
// FP32 sum of 16 squares), so only entries whose FP32 value lies within a
// band of 2E around the B-th value (kth) can be ordered differently in FP64.
// Their pd^2 is recomputed in FP64 from the hi and lo halves of both
// projections: the entries below the band are in L, the first B - below of
// the band by (FP64 pd^2, id) join them, everything else leaves (key ~0).
// Returns false, marking nothing, when the band holds more than 512 entries.
template <int T = WG>
__device__ bool cut_fp64(const AnnArgs& a, int64_t qi, const QueryCtx& qc, int n, int B,
                         uint64_t kth, Smem& sh) {
    constexpr int kBandCap = 512;
    int32_t* band = reinterpret_cast<int32_t*>(sh.hist);            // entry, ~entry if out
    uint32_t* bid = reinterpret_cast<uint32_t*>(sh.hist + kBandCap); // its id
    double* b64 = reinterpret_cast<double*>(sh.hist + 2 * kBandCap); // its FP64 pd^2
    static_assert(NB >= 4 * kBandCap, "the band must fit the histogram");
    const float k2 = __uint_as_float((uint32_t)(kth >> 32));
    const float big = sqrtf(qc.qn2) + a.coord_scale;
    const float e = 2.f * (2.384185791015625e-07f * sqrtf(k2) * big + 1.9073486328125e-06f * k2);
    const float blo = k2 - 2.f * e, bhi = k2 + 2.f * e;
    __syncthreads();
    if (threadIdx.x == 0) sh.cnt2 = 0;
    __syncthreads();
    int below = 0;
    for (int b0 = 0; b0 < n; b0 += T) {
        const int i = b0 + threadIdx.x;
        const float v = i < n ? __uint_as_float((uint32_t)(sh.skey[i] >> 32)) : __int_as_float(0x7f800000);
        below += i < n && v < blo;
        const bool inb = i < n && v >= blo && v <= bhi;
        const int slot = wave_append(inb, &sh.cnt2);
        if (inb && slot < kBandCap) band[slot] = i;
    }
    below = block_sum<T>(below, sh);
    const int nb = sh.cnt2;
    if (nb > kBandCap || below >= B || below + nb < B) return false;
    if (below + nb == B) {
        // the whole band is in L whatever its FP64 order
        for (int i = threadIdx.x; i < n; i += T)
            if (__uint_as_float((uint32_t)(sh.skey[i] >> 32)) > bhi) sh.skey[i] = ~0ull;
        __syncthreads();
        return true;
    }
    for (int j = threadIdx.x; j < nb; j += T) {
        const int64_t pos = sh.spos[band[j]];
        bid[j] = (uint32_t)a.perm[pos];
        double acc = 0.0;
#pragma unroll
        for (int t = 0; t < MP; ++t) {
            const double o = (double)a.proj[pos * MP + t] + (double)a.proj_lo[pos * MP + t];
            const double q = (double)a.qp[qi * MP + t] + (double)a.qp_lo[qi * MP + t];
            const double dd = q - o;
            acc = fma(dd, dd, acc);
        }
        b64[j] = acc;
    }
    __syncthreads();
    const int need = B - below;
    for (int j = threadIdx.x; j < nb; j += T) {
        const double v = b64[j];
        const uint32_t id = bid[j];
        int rank = 0;
        for (int y = 0; y < nb; ++y) rank += b64[y] < v || (b64[y] == v && bid[y] < id);
        if (rank >= need) band[j] = ~band[j];
    }
    __syncthreads();
    for (int j = threadIdx.x; j < nb; j += T)
        if (band[j] < 0) sh.skey[~band[j]] = ~0ull;
    for (int i = threadIdx.x; i < n; i += T)
        if (__uint_as_float((uint32_t)(sh.skey[i] >> 32)) > bhi) sh.skey[i] = ~0ull;
    __syncthreads();
    return true;
}

// L in LDS from a list of n <= CAP entries, B <= n: sh.skey holds the entries'
// keys (pd^2 bits above, the entry's number below, or ~0 outside L), sh.spos
// their positions. Ids are read only where they decide, in the FP64 band and
// for equal FP32 values at the cut when the band is too long (reading all of
// them costs a random 4-byte access per entry).
template <int T>
__device__ void lds_cut(const AnnArgs& a, int64_t qi, const QueryCtx& qc, const uint32_t* list,
                        int n, int B, Smem& sh) {
    // four entries per thread in flight: their list and projection loads are
    // issued together
    constexpr int PU = 4;
    for (int i0 = threadIdx.x; i0 < n; i0 += PU * T) {
        int32_t pos[PU];
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            const int i = i0 + u * T;
            pos[u] = (int32_t)list[i < n ? i : i0];
        }
        float pd2[PU];
#pragma unroll
        for (int u = 0; u < PU; ++u) pd2[u] = proj_dist2(a.proj + (int64_t)pos[u] * MP, qc.qp);
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            const int i = i0 + u * T;
            if (i < n) {
                sh.skey[i] = ((uint64_t)__float_as_uint(pd2[u]) << 32) | (uint32_t)i;
                sh.spos[i] = pos[u];
            }
        }
    }
    __syncthreads();
    if (n == B) return;
    uint64_t kth = lds_select<T>(n, B, sh);
    if (cut_fp64<T>(a, qi, qc, n, B, kth, sh)) return;
    // the FP32 order, ties by id
    for (int i = threadIdx.x; i < n; i += T)
        sh.skey[i] = (sh.skey[i] & 0xffffffff00000000ull) | (uint32_t)a.perm[sh.spos[i]];
    __syncthreads();
    kth = lds_select<T>(n, B, sh);
    for (int i = threadIdx.x; i < n; i += T)
        if (sh.skey[i] > kth) sh.skey[i] = ~0ull;
    __syncthreads();
}

// The need-th smallest (from 1) of the values get(i) in [lo, hi], i < n, of
// which there are at least need: histogram passes over ever narrower ranges,
// four values per thread in flight.
template <int T, class Get>
__device__ uint32_t select_u32(int n, int need, uint32_t lo, uint32_t hi, Get&& get, Smem& sh) {
    for (;;) {
        const uint32_t span = hi - lo;
        const int shift = span < (uint32_t)NB ? 0 : 32 - __clz((int)span) - 11;
        clear_hist<T>(sh);
        if (threadIdx.x == 0) {
            sh.thr_bin = NB - 1;
            sh.thr_below = sh.thr_in = 0;
        }
        for (int i0 = threadIdx.x; i0 < n; i0 += 4 * T) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = get(min(i0 + u * T, n - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + u * T < n && v[u] >= lo && v[u] <= hi)
                    atomicAdd(&sh.hist[(v[u] - lo) >> shift], 1u);
        }
        __syncthreads();
        find_threshold<T>(need, sh);
        const uint32_t nlo = lo + ((uint32_t)sh.thr_bin << shift);
        const bool one = sh.thr_in == 1;
        need -= sh.thr_below;
        __syncthreads();
        if (shift == 0) return nlo;
        const uint32_t top = (1u << shift) - 1u;
        hi = hi - nlo > top ? nlo + top : hi;
        lo = nlo;
        if (one) {
            // the bin holds one value: that value
            for (int i = threadIdx.x; i < n; i += T) {
                const uint32_t v = get(i);
                if (v >= lo && v <= hi) sh.hist[0] = v;
            }
            __syncthreads();
            const uint32_t v = sh.hist[0];
            __syncthreads();
            return v;
        }
    }
}

// L from a list of any length, which stays in memory: emit(take, position, pd^2
// bits), called by whole waves, gets the B of its n >= B entries, sh.cnt0 and
// sh.cnt1 being zero before the first. The B-th smallest pd^2 by radix passes;
// the FP64 order decides around it as in cut_fp64, so L is the same whichever
// kernel finishes a query and whatever queries it came with; the FP32 order with
// ties by id when more than kBandCap entries lie there.
template <int T, class Emit>
__device__ void pool_cut(const AnnArgs& a, int64_t qi, const QueryCtx& qc, const uint32_t* list,
                         int n, int B, Emit&& emit, Smem& sh) {
    // the pd^2 bits are computed once into l_val (or again in every pass, where
    // the workspace has no room for them)
    uint32_t* val = a.l_val ? a.l_val + qi * a.q_cap : nullptr;
    auto compute = [&](int i) {
        return __float_as_uint(proj_dist2(a.proj + (int64_t)(int32_t)list[i] * MP, qc.qp));
    };
    auto get = [&](int i) { return val ? val[i] : compute(i); };
    // f(valid, entry, bits) for every entry, wave-uniform, four loads in flight
    auto for_pool = [&](auto&& f) {
        for (int b0 = 0; b0 < n; b0 += 4 * T) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = get(min(b0 + u * T + (int)threadIdx.x, n - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = b0 + u * T + threadIdx.x;
                f(i < n, min(i, n - 1), v[u]);
            }
        }
    };
    // the bin of the B-th: 256 bins per octave up to the test radius, which at
    // least B entries do not exceed
    const float tq = a.qtest[qi].x;
    const uint32_t hb = __float_as_uint(tq * tq) >> 15;
    const uint32_t base = hb > (uint32_t)(NB - 1) ? hb - (uint32_t)(NB - 1) : 0u;
    clear_hist<T>(sh);
    if (threadIdx.x == 0) {
        sh.thr_bin = NB - 1;
        sh.thr_below = 0;
    }
    for (int b0 = 0; b0 < n; b0 += 4 * T) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = compute(min(b0 + u * T + (int)threadIdx.x, n - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = b0 + u * T + threadIdx.x;
            if (i >= n) break;
            if (val) val[i] = v[u];
            atomicAdd(&sh.hist[min(radius_bin(__uint_as_float(v[u]), base), NB - 1)], 1u);
        }
    }
    __syncthreads();
    find_threshold<T>(B, sh);
    const uint32_t tb = (uint32_t)sh.thr_bin;
    const int before = sh.thr_below;
    __syncthreads();
    const uint32_t k2 = select_u32<T>(
        n, B - before, tb == 0u ? 0u : (base + tb) << 15,
        tb == (uint32_t)(NB - 1) ? 0xffffffffu : ((base + tb + 1u) << 15) - 1u, get, sh);
    // the FP64 order decides inside the band of cut_fp64
    constexpr int kBandCap = 512;
    int32_t* band = reinterpret_cast<int32_t*>(sh.hist);              // entry
    uint32_t* bid = reinterpret_cast<uint32_t*>(sh.hist + kBandCap);  // its id
    double* b64 = reinterpret_cast<double*>(sh.hist + 2 * kBandCap);  // its FP64 pd^2
    const float kf = __uint_as_float(k2);
    const float big = sqrtf(qc.qn2) + a.coord_scale;
    const float e = 2.f * (2.384185791015625e-07f * sqrtf(kf) * big + 1.9073486328125e-06f * kf);
    const float blo = kf - 2.f * e, bhi = kf + 2.f * e;
    if (threadIdx.x == 0) sh.cnt2 = 0;
    __syncthreads();
    int below = 0, less = 0, equal = 0;
    for_pool([&](bool ok, int i, uint32_t b) {
        const float v = __uint_as_float(b);
        below += ok && v < blo;
        less += ok && b < k2;
        equal += ok && b == k2;
        const bool inb = ok && v >= blo && v <= bhi;
        const int slot = wave_append(inb, &sh.cnt2);
        if (inb && slot < kBandCap) {
            band[slot] = i;
            bid[slot] = (uint32_t)a.perm[list[i]];
        }
    });
    below = block_sum<T>(below, sh);
    less = block_sum<T>(less, sh);
    equal = block_sum<T>(equal, sh);
    const int nb = sh.cnt2;
    const bool by64 = nb <= kBandCap && below < B && below + nb >= B;
    float flim = bhi;          // by64: everything below blo, and the band or part of it
    uint32_t idlim = 0xffffffffu;
    if (by64 && below + nb > B) {
        for (int j = threadIdx.x; j < nb; j += T) {
            const int64_t pos = list[band[j]];
            double acc = 0.0;
#pragma unroll
            for (int t = 0; t < MP; ++t) {
                const double o = (double)a.proj[pos * MP + t] + (double)a.proj_lo[pos * MP + t];
                const double q = (double)a.qp[qi * MP + t] + (double)a.qp_lo[qi * MP + t];
                const double dd = q - o;
                acc = fma(dd, dd, acc);
            }
            b64[j] = acc;
        }
        flim = -1.f;   // the band's members are emitted from the list below
    } else if (!by64 && less + equal > B) {
        // more entries than wanted at the B-th value: the smallest ids of them
        idlim = select_u32<T>(
            n, B - less, 0u, 0x7fffffffu,
            [&](int i) { return get(i) == k2 ? (uint32_t)a.perm[list[i]] : 0xffffffffu; }, sh);
    }
    __syncthreads();
    if (threadIdx.x == 0) sh.cnt0 = sh.cnt1 = 0;
    __syncthreads();
    for_pool([&](bool ok, int i, uint32_t b) {
        const float v = __uint_as_float(b);
        bool take = ok && (by64 ? v < blo || v <= flim : b <= k2);
        if (idlim != 0xffffffffu && take && b == k2) take = (uint32_t)a.perm[list[i]] <= idlim;
        emit(take, take ? (int32_t)list[i] : 0, b);
    });
    if (by64 && flim < 0.f) {
        const int want = B - below;
        for (int b0 = 0; b0 < nb; b0 += T) {
            const int j = b0 + threadIdx.x;
            int rank = want;
            if (j < nb) {
                const double v = b64[j];
                const uint32_t id = bid[j];
                rank = 0;
                for (int y = 0; y < nb; ++y) rank += b64[y] < v || (b64[y] == v && bid[y] < id);
            }
            const bool take = rank < want;
            emit(take, take ? (int32_t)list[band[j]] : 0, take ? get(band[j]) : 0u);
        }
    }
}

// The answer from the bounds lo2 <= exact <= hi2 of the n_ver members i < lim of
// C with member(i): the top-k and the statistics.
template <int T, class Member>
__device__ void answer_members(const AnnArgs& a, int64_t qi, const float* qs, int32_t* cpos,
                               const float* lo2, float* hi2, int lim, Member&& member, int n_ver,
                               int rounds, int exit_kind, Smem& sh) {
    const int k = query_params(a, qi).k;
    __syncthreads();
    // Top-k: the k-th smallest upper bound hk; only members whose lower bound
    // is within a factor 1 + 4 gamma of it can be placed among the k nearest
    // by the FP64 order.
    float hk = __int_as_float(0x7f800000);
    if (n_ver > k) {
        // the bounds' bits, in LDS when they fit
        uint32_t* cache = reinterpret_cast<uint32_t*>(sh.skey);
        const bool cached = lim <= 2 * CAP;
        auto bits = [&](int i) { return member(i) ? __float_as_uint(hi2[i]) : 0xffffffffu; };
        uint32_t lo = 0xffffffffu, hi = 0u;
        for (int i = threadIdx.x; i < lim; i += T) {
            const uint32_t b = bits(i);
            if (cached) cache[i] = b;
            lo = min(lo, b);
            hi = b == 0xffffffffu ? hi : max(hi, b);
        }
        for (int off = 32; off > 0; off >>= 1) {
            lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
            hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
        }
        if (lane_id() == 0) {
            sh.red[threadIdx.x >> 6] = (int32_t)lo;
            sh.red[T / 64 + (threadIdx.x >> 6)] = (int32_t)hi;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < T / 64; ++w) {
            lo = min(lo, (uint32_t)sh.red[w]);
            hi = max(hi, (uint32_t)sh.red[T / 64 + w]);
        }
        hk = __uint_as_float(cached ? select_u32<T>(lim, k, lo, hi, [&](int i) { return cache[i]; }, sh)
                                    : select_u32<T>(lim, k, lo, hi, bits, sh));
    }
    const float hkw = (float)((double)hk * (1.0 + 4.0 * (double)verify_gamma(a)) * (1.0 + 1e-7));
    __syncthreads();
    if (threadIdx.x == 0) sh.cnt1 = 0;
    __syncthreads();
    for (int b0 = 0; b0 < lim; b0 += T) {
        const int i = b0 + threadIdx.x;
        const bool take = i < lim && member(i) && lo2[i] <= hkw;
        const int slot = wave_append(take, &sh.cnt1);
        if (take && slot < kRerankCap) sh.spos[slot] = i;
    }
    __syncthreads();
    const int m = sh.cnt1;
    __syncthreads();   // the counter is used again below
    if (m <= kRerankCap) {
        // the FP64 re-rank decides their order from their rows (no FP32 value
        // is needed)
        rerank_topk64<T>(
            a, qi, qs, cpos, m, __int_as_float(0x7f800000),
            [&](int j, float& v, int& mi) {
                v = 0.f;
                mi = sh.spos[j];
            },
            sh);
        if (a.out_stats && threadIdx.x == 0) {
            int32_t* st = a.out_stats + qi * 4;
            st[0] = rounds;
            st[2] = exit_kind;
            st[3] = (int32_t)a.q_scanned[qi];
        }
    } else {
        // too many: their exact FP32 values, moved to the front (a step reads
        // its T entries before any of them is written, and writes only slots
        // that have been read), then the top-k of exact values
        if (threadIdx.x == 0) sh.cnt1 = 0;
        __syncthreads();
        for (int b0 = 0; b0 < lim; b0 += T) {
            const int i = b0 + threadIdx.x;
            const bool take = i < lim && member(i) && lo2[i] <= hkw;
            const int32_t pos = take ? cpos[i] : 0;
            const int slot = wave_append(take, &sh.cnt1);
            __syncthreads();
            if (take) cpos[slot] = pos;
        }
        __syncthreads();
        verify<T>(a, qs, cpos, hi2, 0, m);
        __syncthreads();
        write_topk<T>(a, qi, qs, cpos, hi2, m, rounds, exit_kind, (int64_t)a.q_scanned[qi], sh);
    }
    if (a.out_stats && threadIdx.x == 0) a.out_stats[qi * 4 + 1] = n_ver;
}

template <int T>
__global__ __launch_bounds__(T) void finish_kernel(AnnArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Smem& sh = *reinterpret_cast<Smem*>(smem_raw);
    float* qs = reinterpret_cast<float*>(smem_raw + ((sizeof(Smem) + 15) & ~size_t(15)));
    const int64_t qi = blockIdx.x;
    const AnnQueryParams qpar = query_params(a, qi);
    const int B = qpar.budget;
    const int k = qpar.k;
    const uint32_t cnt = a.l_count[qi * a.l_stride];
    if (cnt > (uint32_t)a.q_cap || cnt < (uint32_t)B) {
        // list overflow, or the bound fell short: the per-query kernel answers
        if (threadIdx.x == 0) {
            a.q_flag[qi] = -1;
            a.pq_list[1 + atomicAdd(&a.pq_list[0], 1u)] = (uint32_t)qi;
        }
        return;
    }
    QueryCtx qc;
    load_query<T>(a, qi, qs, qc);
    int32_t* cpos = a.ws_cpos + qi * (int64_t)a.budget;
    float* cdist = a.ws_cdist + qi * (int64_t)a.budget;
    const uint32_t* list = a.l_list + qi * a.q_cap;
    const int n = (int)cnt;

    // L: the B smallest (pd^2, id) of the list, kept in LDS as keys (pd^2 bits,
    // the entry's number) and leaf positions (entries outside L get the key ~0). Every ball of the
    // rounds below holds the members of L with pd^2 bits <= its radius bits,
    // which is the prefix of L in (pd^2, id) order, so L needs no sorting.
    int nl;
    __syncthreads();
    if (n <= CAP) {
        lds_cut<T>(a, qi, qc, list, n, B, sh);
        nl = n;
    } else {
        pool_cut<T>(
            a, qi, qc, list, n, B,
            [&](bool take, int32_t pos, uint32_t) {
                const int slot = wave_append(take, &sh.cnt0);
                if (take && slot < B) cpos[slot] = pos;
            },
            sh);
        __syncthreads();
        for (int j = threadIdx.x; j < B; j += T) {
            const int32_t pos = cpos[j];
            sh.skey[j] = ((uint64_t)__float_as_uint(proj_dist2(a.proj + (int64_t)pos * MP, qc.qp)) << 32) |
                         (uint32_t)j;
            sh.spos[j] = pos;
        }
        __syncthreads();
        nl = B;
    }

    // Verification keeps, per member of C, bounds lo2 <= exact <= hi2 on the
    // FP32 squared distance that verify would compute (FP16 rows, verify16);
    // a decision that the bounds cannot settle reads the FP32 rows of the
    // members concerned (verify_list), so every decision equals the one
    // taken on exact values. The index lists live in the histogram space.
    float* lo2 = a.ws_clo + qi * (int64_t)a.budget;
    float* hi2 = cdist;
    int32_t* ilist = reinterpret_cast<int32_t*>(sh.hist);
    double r = qpar.r_min;
    int n_ver = 0, rounds = 0, exit_kind = 0;
    uint32_t prev_bits = 0;
    for (;;) {
        if (rounds > 0) {
            // the c r stop: at least k verified members within c r
            const double cr = qpar.c * r;
            const float thr2 = (float)(cr * cr);
            int sure = 0, maybe = 0;
            for (int i = threadIdx.x; i < n_ver; i += T) {
                sure += hi2[i] <= thr2;
                maybe += lo2[i] <= thr2 && hi2[i] > thr2;
            }
            sure = block_sum<T>(sure, sh);
            maybe = block_sum<T>(maybe, sh);
            if (sure < k && sure + maybe >= k) {
                if (threadIdx.x == 0) sh.cnt1 = 0;
                __syncthreads();
                for (int b0 = 0; b0 < n_ver; b0 += T) {
                    const int i = b0 + threadIdx.x;
                    const bool take = i < n_ver && lo2[i] <= thr2 && hi2[i] > thr2;
                    const int slot = wave_append(take, &sh.cnt1);
                    if (take) ilist[slot] = i;
                }
                __syncthreads();
                verify_list<T>(a, qs, cpos, ilist, sh.cnt1, lo2, hi2);
                __syncthreads();
                int loc = 0;
                for (int i = threadIdx.x; i < n_ver; i += T) loc += hi2[i] <= thr2;
                sure = block_sum<T>(loc, sh);
            }
            if (sure >= k) { exit_kind = PMLSH_EXIT_NEAR; break; }
        }
        if (rounds >= MAX_ROUNDS) r = __longlong_as_double(0x7ff0000000000000ll);
        const double Rd = qpar.t * r;
        const uint32_t r2bits = __float_as_uint((float)(Rd * Rd));
        // members of L that the ball gains this round go to C after the
        // n_ver verified ones
        if (threadIdx.x == 0) sh.cnt1 = n_ver;
        __syncthreads();
        for (int b0 = 0; b0 < nl; b0 += T) {
            const int i = b0 + threadIdx.x;
            bool take = false;
            if (i < nl) {
                const uint64_t key = sh.skey[i];
                const uint32_t kb = (uint32_t)(key >> 32);
                take = key != ~0ull && kb <= r2bits && (rounds == 0 || kb > prev_bits);
            }
            const int slot = wave_append(take, &sh.cnt1);
            if (take && slot < B) cpos[slot] = sh.spos[i];
        }
        __syncthreads();
        const int nb = sh.cnt1 < B ? sh.cnt1 : B;
        ++rounds;
        verify16<T>(a, qs, cpos, lo2, hi2, n_ver, nb);
        n_ver = nb;
        prev_bits = r2bits;
        __syncthreads();
        if (nb == B) { exit_kind = PMLSH_EXIT_BUDGET; break; }
        if (rounds >= a.max_rounds) break;
        r = qpar.c * r;
    }

    answer_members<T>(a, qi, qs, cpos, lo2, hi2, n_ver, [](int) { return true; }, n_ver, rounds,
                       exit_kind, sh);
}

// ---- The candidate list in three kernels ----
//
// The pool of a query becomes its answer in three steps of different shape:
//   cut     one workgroup per query: L, the B pool entries of smallest
//           (pd^2, id), written as positions and pd^2 bits, the members of
//           the first round's ball in front;
//   verify  one workgroup per slice of a query's members: distance bounds
//           from the FP16 rows, with no step that waits for another slice;
//   answer  one workgroup per query: the rounds of Algorithm 2 on the bounds,
//           the top-k.
// No step holds a whole list in LDS, so they take any budget up to
// kWideBudget. Budgets above kLeanBudget used to go to the per-query kernel,
// whose tree walk and leaf scans run query by query: 1M x 256, 1,024 queries
// of B = 4,899 26.6 ms (now cut 118 us, verify 348 us, answer 79 us, 0.80 ms
// in all); 200,000 x 128, 256 queries of B = 19,349 4.7 ms (66, 144, 44 us,
// 0.41 ms). The cut is bound by the 64-byte projection rows of the pool
// (gathered through 128-byte lines), the verification by HBM (the FP16 rows of
// all members), the answer by the latency of its passes.

// Bits of the squared radius of the first range query.
__device__ __forceinline__ uint32_t first_radius_bits(const AnnQueryParams& p) {
    const double rd = p.t * p.r_min;
    return __float_as_uint((float)(rd * rd));
}

template <int T, Pass PASS>
__global__ __launch_bounds__(T) void pool_cut_kernel(AnnArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Smem& sh = *reinterpret_cast<Smem*>(smem_raw);
    const int64_t qi = a.ordered ? query_of(a, xcd_place(blockIdx.x, gridDim.x)) : blockIdx.x;
    const AnnQueryParams qpar = query_params(a, qi);
    const int B = qpar.budget;
    constexpr bool BALL = PASS == Pass::Ball;
    if constexpr (PASS == Pass::Rest) {
        if (a.q_flag[qi] < 0) return;
    }
    const uint32_t cnt = a.l_count[qi * a.l_stride];
    if (cnt > (uint32_t)a.q_cap || (!BALL && cnt < (uint32_t)B)) {
        // list overflow, or the bound fell short: the per-query kernel answers
        if (BALL && a.staged) {
            if (threadIdx.x == 0) a.q_flag[qi] = kUndecided;
        } else if (threadIdx.x == 0) {
            a.q_flag[qi] = -1;
            a.pq_list[1 + atomicAdd(&a.pq_list[0], 1u)] = (uint32_t)qi;
        }
        return;
    }
    QueryCtx qc;
    load_projection(a, qi, qc);
    int32_t* cpos = a.ws_cpos + qi * (int64_t)a.budget;
    const uint32_t* list = a.l_list + qi * a.q_cap;
    const int n = (int)cnt;
    const int nl = BALL ? min(n, B) : B;   // a ball's list is L however short
    const uint32_t first = first_radius_bits(qpar);
    // members of L: the first ball's from the front, the others from the back
    auto emit = [&](bool take, int32_t pos, uint32_t bits) {
        const bool in = take && bits <= first;
        const int s0 = wave_append(in, &sh.cnt0);
        const int s1 = wave_append(take && !in, &sh.cnt1);
        const int slot = in ? s0 : nl - 1 - s1;
        if (take && slot >= 0 && slot < nl) cpos[slot] = pos;
    };
    if (BALL && threadIdx.x == 0) a.q_order[qi] = nl;
    if (BALL && n <= B) {
        // every entry is in L
        if (threadIdx.x == 0) sh.cnt0 = sh.cnt1 = 0;
        __syncthreads();
        for (int b0 = 0; b0 < n; b0 += T) {
            const int i = b0 + threadIdx.x;
            const int32_t pos = i < n ? (int32_t)list[i] : 0;
            const float pd2 = i < n ? proj_dist2(a.proj + (int64_t)pos * MP, qc.qp) : 0.f;
            emit(i < n, pos, __float_as_uint(pd2));
        }
        __syncthreads();
        if (threadIdx.x == 0) a.q_flag[qi] = sh.cnt0;
        return;
    }
    if (n <= CAP) {
        lds_cut<T>(a, qi, qc, list, n, B, sh);
        if (threadIdx.x == 0) sh.cnt0 = sh.cnt1 = 0;
        __syncthreads();
        for (int b0 = 0; b0 < n; b0 += T) {
            const int i = b0 + threadIdx.x;
            const uint64_t key = i < n ? sh.skey[i] : ~0ull;
            emit(key != ~0ull, i < n ? sh.spos[i] : 0, (uint32_t)(key >> 32));
        }
        __syncthreads();
        if (threadIdx.x == 0) a.q_flag[qi] = sh.cnt0;
        return;
    }
    pool_cut<T>(a, qi, qc, list, n, B, emit, sh);
    __syncthreads();
    if (threadIdx.x == 0) a.q_flag[qi] = sh.cnt0;
}

// Distance bounds of the members in the first ball: slices of a.vslice members
// of each query (blockIdx.x and .y, placed like the other kernels' queries, so
// that all slices of a run of queries are one XCD's).
__global__ __launch_bounds__(WG) void pool_verify_kernel(AnnArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    float* qs = reinterpret_cast<float*>(smem_raw);
    uint32_t at = blockIdx.y * gridDim.x + blockIdx.x;
    if (a.ordered) at = xcd_place(at, gridDim.x * gridDim.y);
    const int64_t qi = a.ordered ? query_of(a, at / gridDim.x) : at / gridDim.x;
    const int n1 = a.q_flag[qi];
    const int v0 = (int)(at % gridDim.x) * a.vslice;
    if (v0 >= n1) return;
    const float* qrow = a.q + qi * a.d;
    for (int j = threadIdx.x; j < a.d16; j += WG) qs[j] = j < a.d ? qrow[j] : 0.f;
    __syncthreads();
    const int64_t row = qi * (int64_t)a.budget;
    verify16(a, qs, a.ws_cpos + row, a.ws_clo + row, a.ws_cdist + row, v0, min(n1, v0 + a.vslice));
}

template <int T, Pass PASS>
__global__ __launch_bounds__(T) void pool_answer_kernel(AnnArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Smem& sh = *reinterpret_cast<Smem*>(smem_raw);
    float* qs = reinterpret_cast<float*>(smem_raw + ((sizeof(Smem) + 15) & ~size_t(15)));
    const int64_t qi = a.ordered ? query_of(a, xcd_place(blockIdx.x, gridDim.x)) : blockIdx.x;
    const int n1 = a.q_flag[qi];
    if (n1 < 0) return;   // the per-query kernel's (or decided already, or the rest's)
    const AnnQueryParams qpar = query_params(a, qi);
    const int B = qpar.budget;
    const int nl = PASS == Pass::Ball ? a.q_order[qi] : B;   // members of L
    const int k = qpar.k;
    const float* qrow = a.q + qi * a.d;
    for (int j = threadIdx.x; j < a.d16; j += T) qs[j] = j < a.d ? qrow[j] : 0.f;
    const int64_t row = qi * (int64_t)a.budget;
    int32_t* cpos = a.ws_cpos + row;
    float* lo2 = a.ws_clo + row;
    float* hi2 = a.ws_cdist + row;
    int32_t* ilist = reinterpret_cast<int32_t*>(sh.hist);
    __syncthreads();

    // The rounds. C is the members of L with pd^2 bits <= cbits: after the
    // first range query the n1 in front, whose bounds the verify kernel wrote;
    // the others get theirs here when a second one is needed, and their pd^2
    // is computed again where it is asked for.
    double r = qpar.r_min;
    const double last = PASS == Pass::Ball ? ball_radius(a, qpar) : 0.0;
    uint32_t cbits = first_radius_bits(qpar);
    int lim = n1, n_ver = n1, rounds = 1, exit_kind = n1 == B ? PMLSH_EXIT_BUDGET : 0;
    auto member = [&](int i) {
        return i < n1 ||
               __float_as_uint(proj_dist2(a.proj + (int64_t)cpos[i] * MP, a.qp + qi * MP)) <= cbits;
    };
    while (exit_kind == 0 && rounds < a.max_rounds) {
        r = qpar.c * r;
        // the c r stop: at least k verified members within c r; a decision
        // that the bounds leave open reads the FP32 rows of the members
        // concerned, so it equals the one taken on exact values
        const double cr = qpar.c * r;
        const float thr2 = (float)(cr * cr);
        int sure = 0, maybe = 0;
        for (int i = threadIdx.x; i < lim; i += T) {
            const bool in = member(i);
            sure += in && hi2[i] <= thr2;
            maybe += in && lo2[i] <= thr2 && hi2[i] > thr2;
        }
        sure = block_sum<T>(sure, sh);
        maybe = block_sum<T>(maybe, sh);
        if (sure < k && sure + maybe >= k) {
            for (int b0 = 0; b0 < lim; b0 += NB) {
                if (threadIdx.x == 0) sh.cnt1 = 0;
                __syncthreads();
                for (int i0 = b0; i0 < min(lim, b0 + NB); i0 += T) {
                    const int i = i0 + threadIdx.x;
                    const bool take = i < lim && member(i) && lo2[i] <= thr2 && hi2[i] > thr2;
                    const int slot = wave_append(take, &sh.cnt1);
                    if (take) ilist[slot] = i;
                }
                __syncthreads();
                verify_list<T>(a, qs, cpos, ilist, sh.cnt1, lo2, hi2);
                __syncthreads();
            }
            int loc = 0;
            for (int i = threadIdx.x; i < lim; i += T) loc += member(i) && hi2[i] <= thr2;
            sure = block_sum<T>(loc, sh);
        }
        if (sure >= k) { exit_kind = PMLSH_EXIT_NEAR; break; }
        if (PASS == Pass::Ball && r > last) {
            if (threadIdx.x == 0) a.q_flag[qi] = kUndecided;
            return;
        }
        if (rounds >= MAX_ROUNDS) r = __longlong_as_double(0x7ff0000000000000ll);
        const double rd = qpar.t * r;
        cbits = __float_as_uint((float)(rd * rd));
        if (lim < nl) {
            verify16<T>(a, qs, cpos, lo2, hi2, lim, nl);
            lim = nl;
            __syncthreads();
        }
        int loc = 0;
        for (int i = threadIdx.x; i < nl; i += T) loc += member(i);
        n_ver = block_sum<T>(loc, sh);
        ++rounds;
        if (n_ver == B) exit_kind = PMLSH_EXIT_BUDGET;
    }

    answer_members<T>(a, qi, qs, cpos, lo2, hi2, lim, member, n_ver, rounds, exit_kind, sh);
    if (PASS == Pass::Ball && threadIdx.x == 0) a.q_flag[qi] = kDecided;
}

}  // namespace

// Pool entries per query: the bound leaves up to about 1.3 B candidates on
// clustered data and 5 to 8 B on data without contrast (fewer for large B). The
// radius that filter_gemm widens by its bounds passes more of them, and the
// queries that overflow cost milliseconds on the per-query kernel. 1,024 queries of
// a call, ms, with the entries of the exact filter / 2 / 4 / 8 / 16 times as many:
//   FP16, 1M x 256 without contrast, B = 2,500   19  / 1.0
//   BF16, 1M x 256, B = 885                      1.4 / 1.4 / 0.32
//                   B = 4,910                    33  / 14  / 1.6 / 1.6
//   BF16, 1M x 256 without contrast, B = 1,010   63  / 63  / 63  / 19  / 2.2
//                                    B = 5,010   105 / 64  / 19  / 3.7 / 4.3
//   BF16, 1M x 960 without contrast, B = 2,010   73  / 74  / 74  / 74  / 56
//                                    B = 5,010   108 / 68  / 68  / 63  / 11
// least: the exact filter's, where memory is short.
int64_t ann_pool_per_query(const pmlsh_index& x, int64_t budget, bool least) {
    const bool bf16 = x.filter_gemm == PMLSH_FILTER_GEMM_BF16;
    const int64_t f = least || !x.filter_gemm ? 1 : !bf16 ? 2 : x.low_contrast ? 16 : 4;
    const int64_t want = std::max(std::min<int64_t>(f * 8 * budget, f * 65536),
                                  std::min<int64_t>(f + 2, 4) * budget);
    return std::min(x.n, std::max<int64_t>(want, 16384));
}

namespace {

// (r,c)-BC answer from one round of Algorithm 2 with k = 1 (Algorithm 1):
// when the ball fell short of the budget, the nearest candidate is the
// answer only if it lies within c r; otherwise (and for an empty ball) the
// answer is "nothing", id -1 and distance +inf.
__global__ __launch_bounds__(WG) void bc_finalize_kernel(int64_t* ids, float* dist,
                                                         const int32_t* stats, int64_t nq,
                                                         float cr) {
    const int64_t q = (int64_t)blockIdx.x * WG + threadIdx.x;
    if (q >= nq) return;
    const int32_t n_cand = stats[q * 4 + 1], exit_kind = stats[q * 4 + 2];
    if (exit_kind == PMLSH_EXIT_BUDGET) return;
    if (n_cand == 0 || !(dist[q] <= cr)) {
        ids[q] = -1;
        dist[q] = __int_as_float(0x7f800000);
    }
}

}  // namespace

void launch_bc_finalize(int64_t* ids, float* dist, const int32_t* stats, int64_t nq, float cr,
                        hipStream_t stream) {
    if (nq <= 0) return;
    hipLaunchKernelGGL(bc_finalize_kernel, dim3((unsigned)((nq + WG - 1) / WG)), dim3(WG), 0,
                       stream, ids, dist, stats, nq, cr);
    PMLSH_HIP(hipGetLastError());
}

bool ann_fast_path(int64_t budget) { return budget <= kWideBudget; }

int ann_lds_bytes(int d_pad) {
    return (int)(((sizeof(Smem) + 15) & ~size_t(15)) + (size_t)d_pad * sizeof(float));
}

namespace {

template <int T, Pass PASS = Pass::Budget>
void launch_pool(AnnArgs& a, const AnnLaunch& L, int lds_cut, int lds_answer, hipStream_t stream) {
    // members of L per verify workgroup: enough workgroups to fill the chip a few
    // times over, at least the 64 rows that one has in flight
    const int64_t per = (L.budget * L.nq + 4095) / 4096;
    a.vslice = (int)std::min<int64_t>(512, std::max<int64_t>(64, (per + 63) / 64 * 64));
    PMLSH_HIP(hipFuncSetAttribute((const void*)pool_cut_kernel<T, PASS>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds_cut));
    auto* answer = pool_answer_kernel<T, PASS == Pass::Ball ? PASS : Pass::Budget>;
    PMLSH_HIP(hipFuncSetAttribute((const void*)answer,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds_answer));
    hipLaunchKernelGGL((pool_cut_kernel<T, PASS>), dim3((unsigned)L.nq), dim3(T), (unsigned)lds_cut,
                       stream, a);
    const dim3 vgrid((unsigned)((L.budget + a.vslice - 1) / a.vslice), (unsigned)L.nq);
    hipLaunchKernelGGL(pool_verify_kernel, vgrid, dim3(WG), (unsigned)(4 * a.d16), stream, a);
    hipLaunchKernelGGL(answer, dim3((unsigned)L.nq), dim3(T), (unsigned)lds_answer, stream, a);
}

template <int T>
void launch_finish(const AnnArgs& a, const AnnLaunch& L, int lds, hipStream_t stream) {
    PMLSH_HIP(hipFuncSetAttribute((const void*)finish_kernel<T>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    hipLaunchKernelGGL(finish_kernel<T>, dim3((unsigned)L.nq), dim3(T), (unsigned)lds, stream, a);
}

// Points sampled per budget point by the bound kernel. Where the chunks are
// wider than the spread of their centres, points of every chunk lie inside the
// ball and the nearest chunks' 2 B points bound its radius poorly: at 1M
// points and B = 1,000 the ball then holds 14 B (up to 25 B) candidates, from
// 4 B points 5 B (up to 8 B). On clustered data 2 B points leave 1.0 to 1.3 B.
int ann_bound_sample(const pmlsh_index& x) { return x.low_contrast ? 4 : 2; }

}  // namespace

void launch_ann(const AnnLaunch& L, hipStream_t stream) {
    const pmlsh_index& x = *L.idx;
    if (L.nq <= 0) return;
    if (x.levels > MAX_LEVELS) fail(PMLSH_EUNSUPPORTED, "tree deeper than 16 levels");
    AnnArgs a{};
    a.data = x.data;
    a.proj = x.proj_hi;
    a.perm = x.perm;
    a.ncen = x.tree.centre;
    a.nrad = x.tree.radius;
    a.hrmin = x.tree.hr_min;
    a.hrmax = x.tree.hr_max;
    a.cb = x.tree.child_begin;
    a.ce = x.tree.child_end;
    a.npts = x.tree.npts;
    a.piv = x.tree.pivots;
    a.n_nodes = x.n_nodes;
    a.n_leaves = x.n_leaves;
    a.levels = x.levels;
    a.s = x.num_pivots;
    a.d = x.d;
    a.d_pad = x.d_pad;
    for (int l = 0; l <= x.levels; ++l) a.level_begin[l] = (int32_t)x.level_begin[l];
    a.coord_scale = x.coord_scale;
    a.scan_scale = x.scan_scale;
    for (int t = 0; t < MP; ++t) a.scen[t] = x.scan_centre[t];
    a.eps_max = x.eps_max;
    a.qlp = nullptr;
    a.qeps = nullptr;
    a.q = L.queries;
    a.qp = L.qproj;
    a.qp_lo = L.qproj_lo;
    a.proj_lo = x.proj_lo;
    a.qpar = L.qpar;
    a.out_stride = L.out_stride > 0 ? L.out_stride : L.k;
    a.k = L.k;
    a.budget = (int32_t)L.budget;
    a.c = L.c;
    a.t = L.t;
    a.r_min = L.r_min;
    a.max_rounds = L.max_rounds > 0 ? L.max_rounds : 0x7fffffff;
    const bool ball = L.fast && L.ball_most > 0.0;
    a.ball_most = L.ball_most;
    a.staged = ball && a.max_rounds != 1;
    a.ws_front = L.ws_front;
    a.ws_cpos = L.ws_cpos;
    a.ws_cdist = L.ws_cdist;
    a.ws_topk = L.ws_topk;
    a.out_ids = L.out_ids;
    a.out_dist = L.out_dist;
    a.out_stats = L.out_stats;
    a.nq = (int)L.nq;
    a.n = x.n;
    a.proj16 = x.proj16;
    a.n_pad16 = x.n_pad16;
    a.scale16 = x.scale16;
    a.chunk_cen = x.chunk_cen;
    a.chunk_rad = x.chunk_rad;
    a.data16 = x.data16;
    a.d16_se = x.data16_se;
    a.d16 = x.d16;
    const int lds = ann_lds_bytes(x.d16);
    PMLSH_HIP(hipFuncSetAttribute((const void*)ann_kernel,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    if (L.fast) {
        a.qaug = L.ws_qaug;
        a.qlp = L.ws_qlp;
        a.qeps = L.ws_qeps;
        a.qtest = L.ws_qtest;
        a.cmask = L.ws_cmask;
        a.cwords = (int)((L.nq + 63) / 64);
        a.cdist = L.ws_cdist2;
        a.cgmin = L.ws_cgmin;
        a.cgroups = cdist_groups(x.n_pad16 / 64);
        a.gld = cdist_gmin_len(x.n_pad16 / 64);
        a.ws_clo = L.ws_clo;
        a.l_val = L.l_val;
        a.q_flag = L.q_flag;
        a.q_order = L.q_order;
        a.pq_list = L.pq_list;
        // A query's candidate count sits where its members go later, so that
        // the counts of different queries are on lines of their own: the
        // scan's reservations on packed counts queued up at 64 lines.
        a.l_count = reinterpret_cast<uint32_t*>(L.ws_cpos);
        a.l_stride = L.budget;
        a.q_scanned = L.q_scanned;
        a.l_list = L.l_list;
        a.q_cap = (int)L.pool_cap;
        const int lds0 = ann_lds_bytes(0);
        const int64_t nchunk = x.n_pad16 / 64;
        {
            StageTimer tm(PMLSH_STAGE_DIST, stream);
            dim3 dgrid((unsigned)((nchunk + DCB - 1) / DCB), (unsigned)((L.nq + DQB - 1) / DQB));
            hipLaunchKernelGGL(dist_kernel, dgrid, dim3(WG), 0, stream, a);
            PMLSH_HIP(hipGetLastError());
        }
        auto bound_and_mask = [&](Pass pass) {
            StageTimer tm(PMLSH_STAGE_TAU, stream);
            const int64_t ngr = (nchunk + 63) / 64;
            a.sample = ann_bound_sample(x);
            a.ordered = L.nq >= 64 && L.budget > kLeanBudget && pass == Pass::Budget;
            a.sel_cap = (int)std::min<int64_t>(kSelMax, std::max<int64_t>(kSelCap, (a.sample * L.budget + 63) / 64 + 1));
            a.grp_cap = (int)std::min<int64_t>(kGrpCap, std::max<int64_t>(0, tune_get(PMLSH_TUNE_GROUP_LIST)));
            const size_t min_bytes = 2 * (size_t)((ngr + 7) & ~7);
            a.glds = tune_get(PMLSH_TUNE_GROUP_MINIMA_LDS) != 0 &&
                     min_bytes + 4 * (size_t)(kGrpCap + a.sel_cap - kSelCap) <= kTauGroupLds;
            const size_t lds_t = std::max((size_t)lds0, offsetof(Smem, skey) +
                                          (a.glds ? min_bytes : 0) +
                                          4 * (size_t)(kGrpCap + a.sel_cap));
            auto* tau_fn = pass == Pass::Ball   ? tau_kernel<Pass::Ball>
                           : pass == Pass::Rest ? tau_kernel<Pass::Rest>
                                                : tau_kernel<Pass::Budget>;
            PMLSH_HIP(hipFuncSetAttribute((const void*)tau_fn,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_t));
            hipLaunchKernelGGL(tau_fn, dim3((unsigned)L.nq), dim3(WG), (unsigned)lds_t, stream, a);
            PMLSH_HIP(hipGetLastError());
            dim3 mgrid((unsigned)((nchunk + MCH - 1) / MCH), (unsigned)((L.nq + MQB - 1) / MQB));
            hipLaunchKernelGGL(mask_kernel, mgrid, dim3(WG), 0, stream, a);
            PMLSH_HIP(hipGetLastError());
        };
        // one resident wave of workgroups striding over the chunks, in the
        // block shape that suits the index's size
        const int64_t shape = tune_get(PMLSH_TUNE_SCAN_SHAPE);
        const bool large = shape == 0 ? nchunk >= kScanLargeChunks : shape == 2;
        const bool few = shape == 0 && nchunk * ((L.nq + ScanSmall::QW - 1) / ScanSmall::QW) < 1024;
        auto* scan_fn = large ? scan_kernel<ScanLarge> : few ? scan_kernel<ScanFew> : scan_kernel<ScanSmall>;
        const int sqb = large ? ScanLarge::QB : few ? ScanFew::QB : ScanSmall::QB;
        const int swg = 64 * (large ? ScanLarge::NW : few ? ScanFew::NW : ScanSmall::NW);
        static thread_local int scan_slots[64][3] = {};
        int& slots = scan_slots[x.device & 63][large ? 1 : few ? 2 : 0];
        if (slots == 0) {
            int per_cu = 0, cus = 0;
            PMLSH_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)scan_fn, swg, 0));
            PMLSH_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, x.device));
            slots = per_cu > 0 && cus > 0 ? per_cu * cus : (int)kScanBlocks;
        }
        const int64_t ny = (L.nq + sqb - 1) / sqb;
        int64_t gx = std::max<int64_t>(1, slots / ny);
        gx = std::min(gx, nchunk);   // at least one chunk per workgroup on average
        dim3 sgrid((unsigned)gx, (unsigned)ny);
        auto scan = [&] {
            StageTimer tm(PMLSH_STAGE_FILTER, stream);
            hipLaunchKernelGGL(scan_fn, sgrid, dim3((unsigned)swg), 0, stream, a);
            PMLSH_HIP(hipGetLastError());
        };
        if (ball) {
            bound_and_mask(Pass::Ball);
            scan();
            StageTimer tm(PMLSH_STAGE_FINISH, stream);
            launch_pool<1024, Pass::Ball>(a, L, lds0, lds, stream);
        }
        if (!ball || a.staged) {
            bound_and_mask(ball ? Pass::Rest : Pass::Budget);
            scan();
        }
        StageTimer tm(PMLSH_STAGE_FINISH, stream);
        // Which kernels finish a budget of at most kLeanBudget. One workgroup of
        // 256 threads per query suits more than 512 queries: four are resident
        // per compute unit. With fewer queries the chip has room, and a query's
        // chain of row gathers (64 rows in flight per 256 threads) sets the time:
        // 512 threads up to 512 queries, 1,024 up to 256, but 256 where there are
        // so few rows that the barriers of a larger workgroup cost more. The three
        // kernels spread one query's rows over many workgroups for two launches
        // more: that pays for a few queries of many wide rows only. us per call,
        // threads 256 / 512 / 1,024 / three kernels:
        //   5,000 x 64          100 queries, B = 150    58 /  59 /  62 /  68
        //   20,000 x 32 (*)     256 queries, B = 20     58 /  59 /  62 /  67
        //   1M x 128              1 query,   B = 20     56 /  58 /  61 /  62
        //                       256 queries, B = 520    85 /  83 /  84 /  90
        //   1M x 256              1 query,   B = 885     - /   - /  70 /  68
        //                       32 queries, B = 900    89 /  82 /  80 /  80
        //                       256 queries, B = 1,900 211 / 181 / 170 / 198
        //                       512 queries, B = 1,900 266 / 243 / 262 / 271
        //                     1,024 queries, B = 900   212 / 229 / 269 / 227
        //                     1,024 queries, B = 2,040 418 / 427 / 471 / 424
        //   1M x 960 (*)          1 query,   B = 1,020 179 / 152 / 144 / 138
        //                     1,024 queries, B = 1,020 747 / 769 / 819 / 758
        //   20,000 x 900         32 queries, B = 900   126 / 106 / 105 /  93
        // (*) data without contrast.
        const int64_t B = L.budget, nq = L.nq;
        if (a.staged)
            launch_pool<1024, Pass::Rest>(a, L, lds0, lds, stream);
        else if (ball)
            ;
        else if (B > kLeanBudget)
            launch_pool<1024>(a, L, lds0, lds, stream);
        else if (nq <= 32 && B >= 768 && x.d16 >= 256)
            launch_pool<WG>(a, L, lds0, lds, stream);
        else if (nq > 512 || B < 128)
            launch_finish<WG>(a, L, lds, stream);
        else if (nq > 256 || B < 512)
            launch_finish<512>(a, L, lds, stream);
        else
            launch_finish<1024>(a, L, lds, stream);
        PMLSH_HIP(hipGetLastError());
    }
    // per-query path: every query when the fast path does not apply, else only
    // the queries the fast path flagged
    StageTimer tm(PMLSH_STAGE_PERQUERY, stream);
    const int64_t slots = std::max<int64_t>(1, std::min<int64_t>(L.front_slots, L.nq));
    hipLaunchKernelGGL(ann_kernel, dim3((unsigned)slots), dim3(WG), lds, stream, a);
    PMLSH_HIP(hipGetLastError());
}

}  // namespace pmlsh
