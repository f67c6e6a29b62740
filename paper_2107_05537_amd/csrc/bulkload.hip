// Device bulk-load of the leaf order of the PM-tree (Section 4.1): the
// recursive gap-aware splits of the whole point set, computed level by level
// on the GPU. Every node with more than leaf_size points is cut along its
// principal direction (power iteration on the 16 x 16 covariance of its
// projected points, started from the coordinate axis of largest variance)
// at a whole-leaf boundary within the middle 60 % of its leaves, where the
// sorted projections onto that direction show the widest gap, so cuts fall
// between clusters rather than through them.
//
// Per level, for all nodes being cut at once: FP64 coordinate sums and
// centred second moments over pieces of at most kPiece points (one
// workgroup per piece, reduced per node in a fixed order, so a build is
// deterministic), one wave per node for the power iteration, FP64 keys
// (direction . point), a sort of the nodes' points by (key, position), so
// equal keys keep their order, and one wave per node for the cut. The host
// only keeps the list of nodes and their children.

#include <algorithm>

#include "internal.hpp"

namespace pmlsh {
namespace {

constexpr int kPiece = 8192;     // points per moment workgroup
constexpr int kCov = MP * (MP + 1) / 2;   // upper triangle of the covariance

struct Piece {
    int32_t seg;                 // node (index into the level's list)
    int32_t b, e;                // positions [b, e) of the leaf order
};

// Coordinate sums of every piece (four waves, shuffle then LDS, fixed order);
// positions are ids when perm is null. The pieces of leaves fill one wave: the
// others skip the sums, which took longer than the rows (15,625 leaves: 140 us
// before, 80 now); of the large pieces the gathers are the bound (32 us
// a level of 1M points before, 28 now).
constexpr int kSumAhead = 4;
__global__ __launch_bounds__(256) void bl_sum_kernel(const float* __restrict__ proj,
                                                      const int32_t* perm,
                                                      const Piece* __restrict__ pieces,
                                                      double* __restrict__ part) {
    const Piece pc = pieces[blockIdx.x];
    __shared__ double red[4][MP];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (pc.b + 64 * w < pc.e) {
        double acc[MP];
#pragma unroll
        for (int j = 0; j < MP; ++j) acc[j] = 0.0;
        // kSumAhead rows in flight per thread, added in their order
        for (int i = pc.b + (int)threadIdx.x; i < pc.e; i += 256 * kSumAhead) {
            float4 v[kSumAhead][MP / 4];
#pragma unroll
            for (int u = 0; u < kSumAhead; ++u) {
                const int at = min(i + 256 * u, pc.e - 1);
                const int64_t row = perm ? (int64_t)perm[at] : (int64_t)at;
                const float4* p = reinterpret_cast<const float4*>(proj + row * MP);
#pragma unroll
                for (int q = 0; q < MP / 4; ++q) v[u][q] = p[q];
            }
#pragma unroll
            for (int u = 0; u < kSumAhead; ++u) {
                if (i + 256 * u >= pc.e) break;
#pragma unroll
                for (int q = 0; q < MP / 4; ++q) {
                    acc[4 * q] += v[u][q].x;
                    acc[4 * q + 1] += v[u][q].y;
                    acc[4 * q + 2] += v[u][q].z;
                    acc[4 * q + 3] += v[u][q].w;
                }
            }
        }
        // the sums over the wave, lanes 32, 16, 8, 4, 2 and 1 apart in turn;
        // while more than one coordinate is left each lane keeps half of them
        // and hands the other half over
#pragma unroll
        for (int h = MP / 2; h > 0; h >>= 1) {
            const int off = 4 * h;
            const bool up = (lane & off) != 0;
#pragma unroll
            for (int j = 0; j < h; ++j) {
                const double give = up ? acc[j] : acc[j + h];
                const double keep = up ? acc[j + h] : acc[j];
                acc[j] = keep + __shfl_xor(give, off);
            }
        }
        acc[0] += __shfl_xor(acc[0], 2);
        acc[0] += __shfl_xor(acc[0], 1);
        if ((lane & 3) == 0) red[w][lane >> 2] = acc[0];
    } else if (lane < MP) {
        red[w][lane] = 0.0;
    }
    __syncthreads();
    if (threadIdx.x < MP) {
        const int j = threadIdx.x;
        part[(int64_t)blockIdx.x * MP + j] = ((red[0][j] + red[1][j]) + red[2][j]) + red[3][j];
    }
}

// The value that lane (l + N) & 15 of the lane's row of 16 holds.
template <int N>
__device__ __forceinline__ double lane_ahead(double v) {
    if constexpr (N == 0) return v;
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + 16 - N,
                                                              0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32),
                                                              0x120 + 16 - N, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Centred second moments (upper triangle) of every piece about its node's
// mean, on the FP64 matrix cores. v_mfma_f64_4x4x4 adds four points to four
// 4 x 4 blocks of the matrix, each entry as four fused multiply-adds in the
// order of the points, so an entry is the same chain of roundings over its
// piece as a loop of fma would give. Lane 16 k + 4 b + i holds coordinate
// 4 b + i of point k: as it stands that is block row b of the left operand,
// and turned by 4 w lanes within each 16 the block column (b + w) & 3 of the
// right one, so wave w = 0, 1, 2 of a workgroup forms the blocks w off the
// diagonal (of the last two pairs each comes twice) from one load per lane.
//
// What it was bound by: two LDS reads per multiply-add and point, 64 dependent
// steps between loads that nothing overlapped. Now the gathers of the rows
// (64 bytes each) bound it, kCovAhead x 64 of them in flight per wave; the
// chain takes 22 clocks per four points. A level of 1M points: 206 to 278 us
// before, 81 to 119 now (3.8 and 1.7 ms a build).
constexpr int kCovAhead = 4;     // chunks of 64 points in flight
static_assert(MP == 16, "a row is a lane's row of 16");
template <int W>
__device__ void cov_wave(const float* __restrict__ proj, const int32_t* __restrict__ perm,
                         const Piece& pc, const double* __restrict__ mean,
                         double* __restrict__ part) {
    const int lane = threadIdx.x & 63, k = lane >> 4, c = lane & 15;
    const double mu = mean[(int64_t)pc.seg * MP + c];
    double acc = 0.0;
    float v[kCovAhead][16];
    auto ids = [&](int base) { return perm[min(base + lane, pc.e - 1)]; };
    // step u of a chunk takes its points 4 u .. 4 u + 3
    auto fetch = [&](float (&to)[16], int32_t id) {
#pragma unroll
        for (int u = 0; u < 16; ++u)
            to[u] = proj[(int64_t)__shfl(id, 4 * u + k) * MP + c];
    };
    auto add = [&](const float (&from)[16], int base) {
        if (base + 64 <= pc.e) {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double x = (double)from[u] - mu;
                acc = __builtin_amdgcn_mfma_f64_4x4x4f64(x, lane_ahead<4 * W>(x), acc, 0, 0, 0);
            }
        } else {
            // points past the piece add a product of zeros
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double x = base + 4 * u + k < pc.e ? (double)from[u] - mu : 0.0;
                acc = __builtin_amdgcn_mfma_f64_4x4x4f64(x, lane_ahead<4 * W>(x), acc, 0, 0, 0);
            }
        }
    };
    int32_t next[kCovAhead];
#pragma unroll
    for (int s = 0; s < kCovAhead; ++s) next[s] = ids(pc.b + 64 * s);
#pragma unroll
    for (int s = 0; s < kCovAhead; ++s) {
        fetch(v[s], next[s]);
        next[s] = ids(pc.b + 64 * (s + kCovAhead));
    }
    for (int base = pc.b; base < pc.e; base += 64 * kCovAhead) {
#pragma unroll
        for (int s = 0; s < kCovAhead; ++s) {
            const int at = base + 64 * s;
            if (at < pc.e) add(v[s], at);
            fetch(v[s], next[s]);
            next[s] = ids(at + 64 * 2 * kCovAhead);
        }
    }
    // lane 16 i + 4 b + j: entry (i, j) of block (b, (b + W) & 3)
    const int b = (lane >> 2) & 3;
    const int r0 = 4 * b + k, c0 = 4 * ((b + W) & 3) + (lane & 3);
    const int r = min(r0, c0), q = max(r0, c0);
    const bool mine = W == 0 ? r0 <= c0 : W == 1 || b < 2;
    if (mine) part[(int64_t)blockIdx.x * kCov + r * MP - r * (r - 1) / 2 + (q - r)] = acc;
}

__global__ __launch_bounds__(192) void bl_cov_kernel(const float* __restrict__ proj,
                                                      const int32_t* __restrict__ perm,
                                                      const Piece* __restrict__ pieces,
                                                      const double* __restrict__ mean,
                                                      double* __restrict__ part) {
    const Piece pc = pieces[blockIdx.x];
    switch (threadIdx.x >> 6) {
        case 0: cov_wave<0>(proj, perm, pc, mean, part); break;
        case 1: cov_wave<1>(proj, perm, pc, mean, part); break;
        default: cov_wave<2>(proj, perm, pc, mean, part); break;
    }
}

// Per node and entry, the sum of its pieces' partial values in piece order,
// divided by `div[node]` when div is given.
__global__ void bl_reduce_kernel(const double* __restrict__ part, int width,
                                 const int32_t* __restrict__ piece_begin, int m,
                                 const int32_t* __restrict__ div, double* __restrict__ out) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)m * width) return;
    const int s = (int)(t / width), w = (int)(t % width);
    double v = 0.0;
    for (int p = piece_begin[s]; p < piece_begin[s + 1]; ++p) v += part[(int64_t)p * width + w];
    out[t] = div ? v / (double)div[s] : v;
}

// Principal direction of every node: 30 steps of the power iteration on its
// covariance (lane l < 16 holds row l), started from the axis of largest
// variance (the first one on ties); kept where the product vanishes.
__global__ __launch_bounds__(256) void bl_direction_kernel(const double* __restrict__ cov, int m,
                                                            double* __restrict__ dir_out) {
    const int s = (int)(((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (s >= m) return;
    const double* c = cov + (int64_t)s * kCov;
    const int l = lane & (MP - 1);
    double row[MP];
#pragma unroll
    for (int k = 0; k < MP; ++k) {
        const int a = min(l, k), b = max(l, k);
        // index of (a, b) in the upper triangle
        row[k] = c[a * MP - a * (a - 1) / 2 + (b - a)];
    }
    int ax = 0;
    double best = c[0];
    for (int j = 1; j < MP; ++j) {
        const double v = c[j * MP - j * (j - 1) / 2];
        if (v > best) { best = v; ax = j; }
    }
    double dir[MP];
#pragma unroll
    for (int k = 0; k < MP; ++k) dir[k] = k == ax ? 1.0 : 0.0;
    for (int it = 0; it < 30; ++it) {
        double nd = 0.0;
#pragma unroll
        for (int k = 0; k < MP; ++k) nd += row[k] * dir[k];
        double n2 = nd * nd;
        // sum over the 16 lanes of the row block (each block of 16 lanes
        // holds the same rows), in a fixed order
        for (int off = 8; off > 0; off >>= 1) n2 += __shfl_xor(n2, off, 16);
        const double nrm = sqrt(n2);
        if (!(nrm > 0.0)) break;
        const double v = nd / nrm;
#pragma unroll
        for (int k = 0; k < MP; ++k) dir[k] = __shfl(v, k, 16);
    }
    if (lane < MP) dir_out[(int64_t)s * MP + lane] = dir[lane];
}

// FP64 key direction . point of every position of the pieces, and the
// sort's values (the ids at those positions).
__global__ __launch_bounds__(256) void bl_keys_kernel(const float* __restrict__ proj,
                                                       const int32_t* __restrict__ perm,
                                                       const Piece* __restrict__ pieces,
                                                       const double* __restrict__ dir,
                                                       double* __restrict__ key) {
    const Piece pc = pieces[blockIdx.x];
    __shared__ double dv[MP];
    if (threadIdx.x < MP) dv[threadIdx.x] = dir[(int64_t)pc.seg * MP + threadIdx.x];
    __syncthreads();
    for (int i = pc.b + (int)threadIdx.x; i < pc.e; i += 256) {
        const float* p = proj + (int64_t)perm[i] * MP;
        double v = 0.0;
#pragma unroll
        for (int j = 0; j < MP; ++j) v += dv[j] * (double)p[j];
        key[i] = v;
    }
}

// ---- The sort of a level: every node's positions by (key, position) ----
//
// A range of at most kSortCap positions is sorted by one workgroup in LDS. A
// longer one is first cut into about one bucket per kBucket positions: splitters
// from a sorted sample of kOver positions per bucket, a count of every bucket,
// and a scatter of (key, position) in any order within the bucket. Buckets above
// kSortCap (ranges of more than kMaxBuckets buckets) go through this again.
// Keys are compared together with their positions, so all are distinct: the
// result does not depend on the scatter's order, equal keys keep theirs and
// never gather in one bucket. One workgroup per node, as a segmented sort has
// it, leaves the chip idle at the top of the tree: at 1M points it took 5.4 ms
// per level on average (146 of the build's 195 ms); this takes 0.1 ms (sorting
// 0.05, samples 0.016, buckets and scatter 0.03), bound by the LDS passes of the
// bitonic network (256 / 512 / 1,024 threads with one step per pass: 91 / 66 /
// 64 us per launch; ranges of 2,048 cost more bucket passes than they save).
// 10M points: 1.74 s of sorts per build before.
constexpr int kSortCap = 4096;
constexpr int kBucket = 1536;
constexpr int kOver = 16;
constexpr int kMaxBuckets = 512;
constexpr int kSampleWg = 1024;
constexpr int kSortWg = 512;

// A range of positions to sort, from the scattered copies (or the keys).
struct SortRange {
    int32_t b, e;
    int32_t scattered;
};
// A range to cut into k buckets, whose splitters, counts and cursors start at
// entry first (k entries; the last splitter is not used).
struct CutRange {
    int32_t b, e;
    int32_t scattered;
    int32_t k, first;
};

struct SortKey {
    uint64_t k;   // ordered like the FP64 key
    uint32_t p;   // position before the sort
};
__device__ __forceinline__ bool key_less(uint64_t ak, uint32_t ap, uint64_t bk, uint32_t bp) {
    return ak < bk || (ak == bk && ap < bp);
}
__device__ __forceinline__ uint64_t ordered_bits(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    return (u >> 63) ? ~u : u | (1ull << 63);
}
__device__ __forceinline__ double from_ordered_bits(uint64_t u) {
    return __longlong_as_double((long long)((u >> 63) ? u & ~(1ull << 63) : ~u));
}
__device__ __forceinline__ SortKey load_key(const double* key, const uint64_t* skey,
                                            const uint32_t* spos, int32_t scattered, int32_t i) {
    SortKey r;
    if (scattered) {
        r.k = skey[i];
        r.p = spos[i];
    } else {
        r.k = ordered_bits(key[i]);
        r.p = (uint32_t)i;
    }
    return r;
}

// Element i of a list sorted in LDS: one free place after every 16, so that
// lanes eight elements apart do not meet in one bank.
__device__ __forceinline__ int lds_at(int i) { return i + (i >> 4); }
constexpr int lds_places(int n) { return n + n / 16; }

// The steps of distances h 2^(S-1), ..., 2 h, h of a bitonic merge of runs of k,
// 2^S elements in registers per thread and pass.
template <int T, int S>
__device__ __forceinline__ void merge_steps(uint64_t* sk, uint32_t* sp, int P, int k, int h) {
    constexpr int E = 1 << S;
    for (int t = threadIdx.x; t < P >> S; t += T) {
        const int base = ((t & ~(h - 1)) << S) | (t & (h - 1));
        const bool up = (base & k) == 0;
        uint64_t a[E];
        uint32_t b[E];
#pragma unroll
        for (int m = 0; m < E; ++m) {
            a[m] = sk[lds_at(base + m * h)];
            b[m] = sp[lds_at(base + m * h)];
        }
#pragma unroll
        for (int q = S - 1; q >= 0; --q) {
#pragma unroll
            for (int m = 0; m < E; ++m) {
                const int x = m | (1 << q);
                if (x == m) continue;
                const bool swap = key_less(a[x], b[x], a[m], b[m]) == up;
                const uint64_t ta = a[m];
                const uint32_t tb = b[m];
                a[m] = swap ? a[x] : ta;
                b[m] = swap ? b[x] : tb;
                a[x] = swap ? ta : a[x];
                b[x] = swap ? tb : b[x];
            }
        }
#pragma unroll
        for (int m = 0; m < E; ++m) {
            sk[lds_at(base + m * h)] = a[m];
            sp[lds_at(base + m * h)] = b[m];
        }
    }
    __syncthreads();
}

// Sorts n elements (at lds_at(0) .. lds_at(n - 1), lds_places of the next power
// of two reserved) by (key, position). Three steps of the bitonic network per
// pass over the LDS: 26 passes and barriers for 2,048 elements instead of 66,
// which is what it is bound by (1M points: 66 us per launch of the ranges' sorts
// with one step per pass, 38 now; the largest samples 118, 60).
template <int T>
__device__ void sort_lds(uint64_t* sk, uint32_t* sp, int n) {
    int P = 2;
    while (P < n) P <<= 1;
    for (int i = n + (int)threadIdx.x; i < P; i += T) {
        sk[lds_at(i)] = ~0ull;
        sp[lds_at(i)] = ~0u;
    }
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
        int j = k >> 1;
        for (; j >= 4; j >>= 3) merge_steps<T, 3>(sk, sp, P, k, j >> 2);
        if (j == 2)
            merge_steps<T, 2>(sk, sp, P, k, 1);
        else if (j == 1)
            merge_steps<T, 1>(sk, sp, P, k, 1);
    }
}

// Splitters of one range per workgroup, and its counters cleared.
__global__ __launch_bounds__(kSampleWg) void bl_sample_kernel(
    const CutRange* __restrict__ ranges, const double* __restrict__ key,
    const uint64_t* __restrict__ skey, const uint32_t* __restrict__ spos,
    uint64_t* __restrict__ split_k, uint32_t* __restrict__ split_p, int32_t* __restrict__ count) {
    extern __shared__ __align__(16) unsigned char smem[];
    const CutRange r = ranges[blockIdx.x];
    const int ns = r.k * kOver;
    uint64_t* sk = reinterpret_cast<uint64_t*>(smem);
    uint32_t* sp = reinterpret_cast<uint32_t*>(sk + lds_places(kMaxBuckets * kOver));
    const int64_t len = r.e - r.b;
    for (int i = threadIdx.x; i < ns; i += kSampleWg) {
        const SortKey v = load_key(key, skey, spos, r.scattered, r.b + (int32_t)(i * len / ns));
        sk[lds_at(i)] = v.k;
        sp[lds_at(i)] = v.p;
    }
    __syncthreads();
    sort_lds<kSampleWg>(sk, sp, ns);
    for (int i = threadIdx.x; i < r.k; i += kSampleWg) {
        const int at = min((i + 1) * kOver, ns - 1);
        split_k[r.first + i] = sk[lds_at(at)];
        split_p[r.first + i] = sp[lds_at(at)];
        count[r.first + i] = 0;
    }
}

// Bucket of a key: the number of splitters (of the first k - 1) not above it.
__device__ __forceinline__ int bucket_of(const uint64_t* sk, const uint32_t* sp, int k,
                                         const SortKey& v) {
    int lo = 0, hi = k - 1;
    while (lo < hi) {
        const int m = (lo + hi) >> 1;
        if (key_less(v.k, v.p, sk[m], sp[m])) hi = m;
        else lo = m + 1;
    }
    return lo;
}

// Per piece: the bucket of every position, and the buckets' counts.
__global__ __launch_bounds__(256) void bl_bucket_kernel(
    const CutRange* __restrict__ ranges, const Piece* __restrict__ pieces,
    const double* __restrict__ key, const uint64_t* __restrict__ skey,
    const uint32_t* __restrict__ spos, const uint64_t* __restrict__ split_k,
    const uint32_t* __restrict__ split_p, uint16_t* __restrict__ bucket,
    int32_t* __restrict__ count) {
    __shared__ uint64_t sk[kMaxBuckets];
    __shared__ uint32_t sp[kMaxBuckets];
    __shared__ int32_t cnt[kMaxBuckets];
    const Piece pc = pieces[blockIdx.x];
    const CutRange r = ranges[pc.seg];
    for (int i = threadIdx.x; i < r.k; i += 256) {
        sk[i] = split_k[r.first + i];
        sp[i] = split_p[r.first + i];
        cnt[i] = 0;
    }
    __syncthreads();
    for (int i = pc.b + (int)threadIdx.x; i < pc.e; i += 256) {
        const SortKey v = load_key(key, skey, spos, r.scattered, i);
        const int g = bucket_of(sk, sp, r.k, v);
        bucket[i] = (uint16_t)g;
        atomicAdd(&cnt[g], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < r.k; i += 256)
        if (cnt[i]) atomicAdd(&count[r.first + i], cnt[i]);
}

// Exclusive sums of each range's counts: the buckets' first positions, twice
// (kept, and as the scatter's cursors).
__global__ __launch_bounds__(kMaxBuckets) void bl_offset_kernel(
    const CutRange* __restrict__ ranges, const int32_t* __restrict__ count,
    int32_t* __restrict__ start, int32_t* __restrict__ cursor) {
    __shared__ int32_t s[kMaxBuckets];
    const CutRange r = ranges[blockIdx.x];
    const int i = threadIdx.x;
    const int own = i < r.k ? count[r.first + i] : 0;
    s[i] = own;
    __syncthreads();
    for (int off = 1; off < kMaxBuckets; off <<= 1) {
        const int v = i >= off ? s[i - off] : 0;
        __syncthreads();
        s[i] += v;
        __syncthreads();
    }
    if (i < r.k) {
        start[r.first + i] = r.b + s[i] - own;
        cursor[r.first + i] = r.b + s[i] - own;
    }
}

// Every (key, position) of a piece to its bucket, one reservation per piece
// and bucket.
__global__ __launch_bounds__(256) void bl_scatter_kernel(
    const CutRange* __restrict__ ranges, const Piece* __restrict__ pieces,
    const double* __restrict__ key, const uint64_t* __restrict__ skey,
    const uint32_t* __restrict__ spos, const uint16_t* __restrict__ bucket,
    int32_t* __restrict__ cursor, uint64_t* __restrict__ okey, uint32_t* __restrict__ opos) {
    __shared__ int32_t cnt[kMaxBuckets];
    const Piece pc = pieces[blockIdx.x];
    const CutRange r = ranges[pc.seg];
    for (int i = threadIdx.x; i < r.k; i += 256) cnt[i] = 0;
    __syncthreads();
    for (int i = pc.b + (int)threadIdx.x; i < pc.e; i += 256) atomicAdd(&cnt[bucket[i]], 1);
    __syncthreads();
    for (int i = threadIdx.x; i < r.k; i += 256)
        if (cnt[i]) cnt[i] = atomicAdd(&cursor[r.first + i], cnt[i]);
    __syncthreads();
    for (int i = pc.b + (int)threadIdx.x; i < pc.e; i += 256) {
        const SortKey v = load_key(key, skey, spos, r.scattered, i);
        const int32_t at = atomicAdd(&cnt[bucket[i]], 1);
        okey[at] = v.k;
        opos[at] = v.p;
    }
}

// One range per workgroup: sorted keys, and the ids at the sorted positions
// (unless perm is null).
__global__ __launch_bounds__(kSortWg) void bl_sort_kernel(
    const SortRange* __restrict__ ranges, const double* __restrict__ key,
    const uint64_t* __restrict__ skey, const uint32_t* __restrict__ spos,
    const int32_t* __restrict__ perm, double* __restrict__ key_out,
    int32_t* __restrict__ perm_out) {
    __shared__ uint64_t sk[lds_places(kSortCap)];
    __shared__ uint32_t sp[lds_places(kSortCap)];
    const SortRange r = ranges[blockIdx.x];
    const int n = r.e - r.b;
    for (int i = threadIdx.x; i < n; i += kSortWg) {
        const SortKey v = load_key(key, skey, spos, r.scattered, r.b + i);
        sk[lds_at(i)] = v.k;
        sp[lds_at(i)] = v.p;
    }
    __syncthreads();
    sort_lds<kSortWg>(sk, sp, n);
    for (int i = threadIdx.x; i < n; i += kSortWg) {
        key_out[r.b + i] = from_ordered_bits(sk[lds_at(i)]);
        if (perm) perm_out[r.b + i] = perm[sp[lds_at(i)]];
    }
}

// The sorted ids back into the leaf order, positions of the pieces only.
__global__ __launch_bounds__(256) void bl_copy_kernel(const Piece* __restrict__ pieces,
                                                       const int32_t* __restrict__ src,
                                                       int32_t* __restrict__ perm) {
    const Piece pc = pieces[blockIdx.x];
    for (int i = pc.b + (int)threadIdx.x; i < pc.e; i += 256) perm[i] = src[i];
}

// The cut of every node (one wave each): after j whole leaves, j within the
// middle 60 % of its leaves, at the widest gap of the sorted keys (the
// smallest such j); the middle leaf when no cut position qualifies.
__global__ __launch_bounds__(256) void bl_cut_kernel(const int32_t* __restrict__ seg_b,
                                                      const int32_t* __restrict__ seg_e, int m,
                                                      int leaf, const double* __restrict__ key,
                                                      int32_t* __restrict__ mid) {
    const int s = (int)(((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6);
    const int lane = threadIdx.x & 63;
    if (s >= m) return;
    const int b = seg_b[s], cnt = seg_e[s] - b;
    const int nleaves = (cnt + leaf - 1) / leaf;
    int jlo = max(1, (nleaves * 2) / 10);
    int jhi = min(nleaves - 1, nleaves - (nleaves * 2) / 10);
    if (jhi < jlo) jlo = jhi = nleaves / 2;
    double gap = -1.0;
    int best = 0x7fffffff;
    for (int j = jlo + lane; j <= jhi; j += 64) {
        const int64_t p = (int64_t)j * leaf;
        if (p <= 0 || p >= cnt) continue;
        const double g = key[b + p] - key[b + p - 1];
        if (g > gap) { gap = g; best = j; }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const double og = __shfl_xor(gap, off);
        const int ob = __shfl_xor(best, off);
        if (og > gap || (og == gap && ob < best)) { gap = og; best = ob; }
    }
    if (lane == 0) mid[s] = b + (gap < 0.0 ? nleaves / 2 : best) * leaf;
}

__device__ __forceinline__ double dist64(const float* p, const float* c) {
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < MP; ++j) {
        const double t = (double)p[j] - (double)c[j];
        acc = fma(t, t, acc);
    }
    return sqrt(acc);
}

// Mean of every node (sums / count, from bl_reduce_kernel) rounded to FP32.
__global__ void bl_centre_kernel(const double* __restrict__ mean, int64_t count,
                                 float* __restrict__ cf) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) cf[t] = (float)mean[t];
}

// The reduction of v over the wave by f (its order does not matter): rotations
// within each row of 16 lanes, then the other rows.
template <class F>
__device__ __forceinline__ double wave_of(double v, F f) {
    v = f(v, lane_ahead<8>(v));
    v = f(v, lane_ahead<4>(v));
    v = f(v, lane_ahead<2>(v));
    v = f(v, lane_ahead<1>(v));
    v = f(v, __shfl_xor(v, 16));
    return f(v, __shfl_xor(v, 32));
}

// Per piece: the largest FP64 distance of its points to their node's FP32
// centre, and for every pivot the smallest and largest distance to it
// (width 1 + 2 s per piece; min and max do not depend on the order).
__global__ __launch_bounds__(256, 4) void bl_ring_kernel(const float* __restrict__ proj,
                                                       const int32_t* __restrict__ perm,
                                                       const Piece* __restrict__ pieces,
                                                       const float* __restrict__ cf,
                                                       const float* __restrict__ piv, int s,
                                                       double* __restrict__ part) {
    const Piece pc = pieces[blockIdx.x];
    __shared__ float c[MP];
    __shared__ float pv[PMLSH_MAX_PIVOTS][MP];
    __shared__ double red[4][1 + 2 * PMLSH_MAX_PIVOTS];
    if (threadIdx.x < MP) c[threadIdx.x] = cf[(int64_t)pc.seg * MP + threadIdx.x];
    if (threadIdx.x < s * MP) pv[threadIdx.x / MP][threadIdx.x % MP] = piv[threadIdx.x];
    __syncthreads();
    double rad = 0.0, lo[PMLSH_MAX_PIVOTS], hi[PMLSH_MAX_PIVOTS];
#pragma unroll
    for (int t = 0; t < PMLSH_MAX_PIVOTS; ++t) {
        lo[t] = __longlong_as_double(0x7ff0000000000000ll);
        hi[t] = 0.0;
    }
    for (int i = pc.b + (int)threadIdx.x; i < pc.e; i += 256) {
        float p[MP];
        const float4* src = reinterpret_cast<const float4*>(proj + (int64_t)perm[i] * MP);
#pragma unroll
        for (int q = 0; q < MP / 4; ++q) {
            const float4 v = src[q];
            p[4 * q] = v.x;
            p[4 * q + 1] = v.y;
            p[4 * q + 2] = v.z;
            p[4 * q + 3] = v.w;
        }
        rad = fmax(rad, dist64(p, c));
#pragma unroll
        for (int t = 0; t < PMLSH_MAX_PIVOTS; ++t) {
            // the pivots are read again for every point: kept in registers
            // over the loop they leave room for one wave per SIMD
            asm volatile("" ::: "memory");
            if (t < s) {
                const double dd = dist64(p, pv[t]);
                lo[t] = fmin(lo[t], dd);
                hi[t] = fmax(hi[t], dd);
            }
        }
    }
    // (a wave without points holds the neutral values already)
    const int w = threadIdx.x >> 6;
    if (pc.b + 64 * w < pc.e) {
        rad = wave_of(rad, [](double a, double b) { return fmax(a, b); });
#pragma unroll
        for (int t = 0; t < PMLSH_MAX_PIVOTS; ++t) {
            if (t < s) {
                lo[t] = wave_of(lo[t], [](double a, double b) { return fmin(a, b); });
                hi[t] = wave_of(hi[t], [](double a, double b) { return fmax(a, b); });
            }
        }
    }
    if ((threadIdx.x & 63) == 0) {
        red[w][0] = rad;
        for (int t = 0; t < s; ++t) {
            red[w][1 + 2 * t] = lo[t];
            red[w][2 + 2 * t] = hi[t];
        }
    }
    __syncthreads();
    const int width = 1 + 2 * s;
    if (threadIdx.x < width) {
        const int e = threadIdx.x;
        const bool is_min = e >= 1 && (e & 1);
        double v = red[0][e];
        for (int k = 1; k < 4; ++k) v = is_min ? fmin(v, red[k][e]) : fmax(v, red[k][e]);
        part[(int64_t)blockIdx.x * width + e] = v;
    }
}

// Per node and entry, the max (entry 0 and the even ones) or min (odd ones)
// over its pieces.
__global__ void bl_reduce_ring_kernel(const double* __restrict__ part, int width,
                                      const int32_t* __restrict__ piece_begin, int m,
                                      double* __restrict__ out) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)m * width) return;
    const int sg = (int)(t / width), e = (int)(t % width);
    const bool is_min = e >= 1 && (e & 1);
    double v = part[(int64_t)piece_begin[sg] * width + e];
    for (int p = piece_begin[sg] + 1; p < piece_begin[sg + 1]; ++p) {
        const double x = part[(int64_t)p * width + e];
        v = is_min ? fmin(v, x) : fmax(v, x);
    }
    out[t] = v;
}

// Farthest-point step over the ids [0, n): the distance of every point to
// ref (an FP32 row), folded into mind[i] = min(mind[i], distance) when mind
// is given; per workgroup the largest value and its smallest id.
__global__ __launch_bounds__(256) void bl_far_kernel(const float* __restrict__ proj, int64_t n,
                                                      const float* __restrict__ ref,
                                                      double* mind, double* __restrict__ bval,
                                                      int64_t* __restrict__ bidx) {
    __shared__ float r[MP];
    __shared__ double sv[4];
    __shared__ int64_t si[4];
    if (threadIdx.x < MP) r[threadIdx.x] = ref[threadIdx.x];
    __syncthreads();
    double best = -1.0;
    int64_t bi = 0x7fffffffffffffffll;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        double v = dist64(proj + i * MP, r);
        if (mind) {
            v = fmin(mind[i], v);
            mind[i] = v;
        }
        if (v > best) { best = v; bi = i; }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const double ov = __shfl_xor(best, off);
        const int64_t oi = __shfl_xor(bi, off);
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
    }
    if ((threadIdx.x & 63) == 0) {
        sv[threadIdx.x >> 6] = best;
        si[threadIdx.x >> 6] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w)
            if (sv[w] > best || (sv[w] == best && si[w] < bi)) { best = sv[w]; bi = si[w]; }
        bval[blockIdx.x] = best;
        bidx[blockIdx.x] = bi;
    }
}

// The largest value over the workgroups of bl_far_kernel (smallest id on
// ties); its point is copied to dst (an FP32 row) and its value to *val.
__global__ __launch_bounds__(256) void bl_pick_kernel(const float* __restrict__ proj,
                                                       const double* __restrict__ bval,
                                                       const int64_t* __restrict__ bidx, int nb,
                                                       float* __restrict__ dst,
                                                       double* __restrict__ val) {
    __shared__ double sv[4];
    __shared__ int64_t si[4];
    __shared__ int64_t pick;
    double best = -1.0;
    int64_t bi = 0x7fffffffffffffffll;
    for (int b = threadIdx.x; b < nb; b += 256)
        if (bval[b] > best || (bval[b] == best && bidx[b] < bi)) { best = bval[b]; bi = bidx[b]; }
    for (int off = 32; off > 0; off >>= 1) {
        const double ov = __shfl_xor(best, off);
        const int64_t oi = __shfl_xor(bi, off);
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
    }
    if ((threadIdx.x & 63) == 0) {
        sv[threadIdx.x >> 6] = best;
        si[threadIdx.x >> 6] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w)
            if (sv[w] > best || (sv[w] == best && si[w] < bi)) { best = sv[w]; bi = si[w]; }
        sv[0] = best;
        pick = bi;
    }
    __syncthreads();
    if (threadIdx.x < MP && dst) dst[threadIdx.x] = proj[pick * MP + threadIdx.x];
    if (threadIdx.x == 0 && val) *val = sv[0];
}

// Any non-finite value among count floats sets *flag (a plain store).
__global__ void bl_finite_kernel(const float* __restrict__ x, int64_t count,
                                 int32_t* __restrict__ flag) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        if (!isfinite(x[i])) *flag = 1;
}

__global__ void bl_fill_kernel(double* __restrict__ x, int64_t count, double v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        x[i] = v;
}

// perm[i] = i.
__global__ void bl_iota_kernel(int32_t* __restrict__ perm, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        perm[i] = (int32_t)i;
}

// inv[perm[i]] = i.
__global__ void bl_invert_kernel(const int32_t* __restrict__ perm, int64_t n,
                                 int32_t* __restrict__ inv) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        inv[perm[i]] = (int32_t)i;
}

dim3 grid_of(int64_t n) {
    return dim3((unsigned)std::min<int64_t>(4096, std::max<int64_t>(1, (n + 255) / 256)));
}

// Device buffer that grows to at least twice its size, so that the levels of a
// build, each a little larger than the one before, do not free and allocate in
// turn. Its memory is the build's scratch while that has room.
template <class T>
struct DevVec {
    T* p = nullptr;
    size_t cap = 0;
    ~DevVec() { release(); }
    void release() {
        if (p && !BuildScratch::give_back(p)) (void)hipFree(p);
        p = nullptr;
        cap = 0;
    }
    T* get(size_t count) {
        if (count > cap || !p) {
            const size_t want = std::max<size_t>(count, std::max<size_t>(2 * cap, 1));
            release();
            p = static_cast<T*>(BuildScratch::take_piece(want * sizeof(T)));
            if (!p) p = static_cast<T*>(device_malloc(want * sizeof(T)));
            cap = want;
        }
        return p;
    }
};

// Device buffers of the level sorts, and their host lists.
struct LevelSort {
    DevVec<uint64_t> skey[2], split_k;
    DevVec<uint32_t> spos[2], split_p;
    DevVec<uint16_t> bucket;
    DevVec<int32_t> count;           // counts, starts and cursors of the buckets
    DevVec<CutRange> d_cut;
    DevVec<SortRange> d_sort;
    DevVec<Piece> d_pieces;
    std::vector<CutRange> cut, next;
    std::vector<SortRange> ready;
    std::vector<Piece> pieces;
    std::vector<int32_t> start;

    // Sorts [sb[s], se[s]) for every s < m by (key, position); ids and keys of
    // the sorted ranges go to perm_out and key_out.
    void run(const double* key, const int32_t* perm, int64_t n, const int32_t* sb,
             const int32_t* se, int m, double* key_out, int32_t* perm_out, hipStream_t st) {
        cut.clear();
        ready.clear();
        auto place = [&](int32_t b, int32_t e, int32_t scattered, std::vector<CutRange>& to) {
            if (e - b <= kSortCap) {
                if (e > b) ready.push_back({b, e, scattered});
            } else {
                to.push_back({b, e, scattered, std::min(kMaxBuckets, (e - b + kBucket - 1) / kBucket), 0});
            }
        };
        for (int s = 0; s < m; ++s) place(sb[s], se[s], 0, cut);
        int from = 1;   // the scattered copies read by this round are side `from`
        while (!cut.empty()) {
            sort_ready(key, perm, key_out, perm_out, from, st);
            const int to = from ^ 1;
            int32_t total = 0;
            pieces.clear();
            for (size_t s = 0; s < cut.size(); ++s) {
                cut[s].first = total;
                total += cut[s].k;
                for (int32_t x = cut[s].b; x < cut[s].e; x += kPiece)
                    pieces.push_back({(int32_t)s, x, std::min(cut[s].e, x + kPiece)});
            }
            uint64_t* ik = skey[from].get((size_t)n);
            uint32_t* ip = spos[from].get((size_t)n);
            uint64_t* ok = skey[to].get((size_t)n);
            uint32_t* op = spos[to].get((size_t)n);
            uint64_t* pk = split_k.get((size_t)total);
            uint32_t* pp = split_p.get((size_t)total);
            uint16_t* bk = bucket.get((size_t)n);
            int32_t* cn = count.get((size_t)total * 3);
            CutRange* dc = d_cut.get(cut.size());
            Piece* dp = d_pieces.get(pieces.size());
            PMLSH_HIP(hipMemcpyAsync(dc, cut.data(), cut.size() * sizeof(CutRange),
                                     hipMemcpyHostToDevice, st));
            PMLSH_HIP(hipMemcpyAsync(dp, pieces.data(), pieces.size() * sizeof(Piece),
                                     hipMemcpyHostToDevice, st));
            constexpr int lds = lds_places(kMaxBuckets * kOver) *
                                (int)(sizeof(uint64_t) + sizeof(uint32_t));
            PMLSH_HIP(hipFuncSetAttribute((const void*)bl_sample_kernel,
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            const dim3 gr((unsigned)cut.size()), gp((unsigned)pieces.size());
            hipLaunchKernelGGL(bl_sample_kernel, gr, dim3(kSampleWg), lds, st, dc, key, ik, ip, pk,
                               pp, cn);
            hipLaunchKernelGGL(bl_bucket_kernel, gp, dim3(256), 0, st, dc, dp, key, ik, ip, pk, pp,
                               bk, cn);
            hipLaunchKernelGGL(bl_offset_kernel, gr, dim3(kMaxBuckets), 0, st, dc, cn, cn + total,
                               cn + 2 * total);
            hipLaunchKernelGGL(bl_scatter_kernel, gp, dim3(256), 0, st, dc, dp, key, ik, ip, bk,
                               cn + 2 * total, ok, op);
            PMLSH_HIP(hipGetLastError());
            start.resize((size_t)total);
            PMLSH_HIP(hipMemcpyAsync(start.data(), cn + total, (size_t)total * sizeof(int32_t),
                                     hipMemcpyDeviceToHost, st));
            PMLSH_HIP(hipStreamSynchronize(st));
            next.clear();
            for (const CutRange& r : cut)
                for (int g = 0; g < r.k; ++g) {
                    const int32_t b = start[(size_t)(r.first + g)];
                    const int32_t e = g + 1 < r.k ? start[(size_t)(r.first + g + 1)] : r.e;
                    if (b < r.b || e < b || e > r.e)
                        fail(PMLSH_EDEVICE, "device sort produced an invalid bucket");
                    place(b, e, 1, next);
                }
            cut.swap(next);
            from = to;
        }
        sort_ready(key, perm, key_out, perm_out, from, st);
        PMLSH_HIP(hipGetLastError());
    }

private:
    void sort_ready(const double* key, const int32_t* perm, double* key_out, int32_t* perm_out,
                    int from, hipStream_t st) {
        if (ready.empty()) return;
        SortRange* dr = d_sort.get(ready.size());
        PMLSH_HIP(hipMemcpyAsync(dr, ready.data(), ready.size() * sizeof(SortRange),
                                 hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(bl_sort_kernel, dim3((unsigned)ready.size()), dim3(kSortWg), 0, st, dr,
                           key, skey[from].p, spos[from].p, perm, key_out, perm_out);
        ready.clear();
    }
};

}  // namespace

void device_split(const float* proj, int64_t n, int leaf, hipStream_t st,
                  int32_t* perm, std::vector<SplitNode>* nodes_out) {
    if (n <= 0 || n > 0x7fffffffLL - kPiece) fail(PMLSH_EUNSUPPORTED, "point count out of range");
    std::vector<SplitNode>& nodes = *nodes_out;
    nodes.clear();
    nodes.push_back({0, (n + leaf - 1) / leaf, -1, -1});
    std::vector<int32_t> cur;                          // nodes cut at this level
    std::vector<int32_t> nb{0}, ne{(int32_t)n};        // their point ranges
    if (n > leaf) cur.push_back(0);

    DevVec<int32_t> perm_alt, d_idx;
    DevVec<double> key, key_alt, part, mean, cov, dir;
    DevVec<Piece> d_pieces;
    LevelSort sorter;
    hipLaunchKernelGGL(bl_iota_kernel, grid_of(n), dim3(256), 0, st, perm, n);
    PMLSH_HIP(hipGetLastError());
    key.get((size_t)n);
    key_alt.get((size_t)n);
    perm_alt.get((size_t)n);

    std::vector<Piece> pieces;
    std::vector<int32_t> host_idx, mids;
    while (!cur.empty()) {
        const int m = (int)cur.size();
        // per node: begin, end, first piece (m + 1), point count
        pieces.clear();
        host_idx.assign((size_t)4 * m + 1, 0);
        int32_t* sb = host_idx.data();
        int32_t* se = sb + m;
        int32_t* pb = se + m;          // m + 1 entries
        int32_t* cnt = pb + m + 1;
        for (int s = 0; s < m; ++s) {
            const int32_t b = nb[(size_t)cur[(size_t)s]], e = ne[(size_t)cur[(size_t)s]];
            sb[s] = b;
            se[s] = e;
            cnt[s] = e - b;
            pb[s] = (int32_t)pieces.size();
            for (int32_t x = b; x < e; x += kPiece) pieces.push_back({s, x, std::min(e, x + kPiece)});
        }
        pb[m] = (int32_t)pieces.size();
        const int np = (int)pieces.size();
        int32_t* di = d_idx.get(host_idx.size());
        Piece* dp = d_pieces.get(pieces.size());
        PMLSH_HIP(hipMemcpyAsync(di, host_idx.data(), host_idx.size() * sizeof(int32_t),
                                 hipMemcpyHostToDevice, st));
        PMLSH_HIP(hipMemcpyAsync(dp, pieces.data(), pieces.size() * sizeof(Piece),
                                 hipMemcpyHostToDevice, st));
        const int32_t *dsb = di, *dse = di + m, *dpb = di + 2 * m, *dcnt = di + 3 * m + 1;

        // mean, covariance, direction
        double* dpart = part.get((size_t)np * kCov);
        double* dmean = mean.get((size_t)m * MP);
        double* dcov = cov.get((size_t)m * kCov);
        double* ddir = dir.get((size_t)m * MP);
        hipLaunchKernelGGL(bl_sum_kernel, dim3((unsigned)np), dim3(256), 0, st, proj, perm, dp,
                           dpart);
        hipLaunchKernelGGL(bl_reduce_kernel, dim3((unsigned)(((int64_t)m * MP + 255) / 256)),
                           dim3(256), 0, st, dpart, MP, dpb, m, dcnt, dmean);
        hipLaunchKernelGGL(bl_cov_kernel, dim3((unsigned)np), dim3(192), 0, st, proj, perm, dp,
                           dmean, dpart);
        hipLaunchKernelGGL(bl_reduce_kernel, dim3((unsigned)(((int64_t)m * kCov + 255) / 256)),
                           dim3(256), 0, st, dpart, kCov, dpb, m, nullptr, dcov);
        hipLaunchKernelGGL(bl_direction_kernel, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, st,
                           dcov, m, ddir);
        hipLaunchKernelGGL(bl_keys_kernel, dim3((unsigned)np), dim3(256), 0, st, proj, perm, dp,
                           ddir, key.p);
        PMLSH_HIP(hipGetLastError());

        sorter.run(key.p, perm, n, sb, se, m, key_alt.p, perm_alt.p, st);
        hipLaunchKernelGGL(bl_copy_kernel, dim3((unsigned)np), dim3(256), 0, st, dp, perm_alt.p,
                           perm);
        // the cuts, from the sorted keys
        int32_t* dmid = reinterpret_cast<int32_t*>(dcov);   // free after the directions
        hipLaunchKernelGGL(bl_cut_kernel, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, st, dsb,
                           dse, m, leaf, key_alt.p, dmid);
        PMLSH_HIP(hipGetLastError());
        mids.resize((size_t)m);
        PMLSH_HIP(hipMemcpyAsync(mids.data(), dmid, (size_t)m * sizeof(int32_t),
                                 hipMemcpyDeviceToHost, st));
        PMLSH_HIP(hipStreamSynchronize(st));

        std::vector<int32_t> next;
        for (int s = 0; s < m; ++s) {
            const int32_t id = cur[(size_t)s];
            const int32_t b = sb[s], e = se[s], md = mids[(size_t)s];
            if (md <= b || md >= e || (md - b) % leaf != 0)
                fail(PMLSH_EDEVICE, "device split produced an invalid cut");
            const int32_t l = (int32_t)nodes.size(), r = l + 1;
            nodes.push_back({b / leaf, (md + leaf - 1) / leaf, -1, -1});
            nodes.push_back({md / leaf, (e + leaf - 1) / leaf, -1, -1});
            nb.push_back(b);
            ne.push_back(md);
            nb.push_back(md);
            ne.push_back(e);
            nodes[(size_t)id].left = l;
            nodes[(size_t)id].right = r;
            if (md - b > leaf) next.push_back(l);
            if (e - md > leaf) next.push_back(r);
        }
        cur.swap(next);
    }
}

void device_invert(const int32_t* perm, int64_t n, int32_t* inv, hipStream_t st) {
    hipLaunchKernelGGL(bl_invert_kernel, grid_of(n), dim3(256), 0, st, perm, n, inv);
    PMLSH_HIP(hipGetLastError());
}

void device_sorted(const double* x, int64_t n, hipStream_t st, std::vector<double>* out) {
    LevelSort sorter;
    DevVec<double> sorted;
    const int32_t b = 0, e = (int32_t)n;
    out->resize((size_t)n);
    sorter.run(x, nullptr, n, &b, &e, 1, sorted.get((size_t)n), nullptr, st);
    PMLSH_HIP(hipMemcpyAsync(out->data(), sorted.p, (size_t)n * sizeof(double),
                             hipMemcpyDeviceToHost, st));
    PMLSH_HIP(hipStreamSynchronize(st));
}

namespace {

// Pieces of at most kPiece positions for every range [p0[s], p1[s]), and the
// first piece of every range (m + 1 entries).
void make_pieces(const std::vector<int64_t>& p0, const std::vector<int64_t>& p1,
                 std::vector<Piece>* pieces, std::vector<int32_t>* first) {
    pieces->clear();
    first->assign(p0.size() + 1, 0);
    for (size_t sg = 0; sg < p0.size(); ++sg) {
        if (p1[sg] > 0x7fffffffLL - kPiece) fail(PMLSH_EUNSUPPORTED, "point count out of range");
        (*first)[sg] = (int32_t)pieces->size();
        for (int64_t x = p0[sg]; x < p1[sg]; x += kPiece)
            pieces->push_back({(int32_t)sg, (int32_t)x, (int32_t)std::min(p1[sg], x + kPiece)});
    }
    (*first)[p0.size()] = (int32_t)pieces->size();
}

}  // namespace

bool device_all_finite(const float* x, int64_t count, hipStream_t st) {
    DevVec<int32_t> flag;
    int32_t* f = flag.get(1);
    PMLSH_HIP(hipMemsetAsync(f, 0, sizeof(int32_t), st));
    const int64_t blocks = std::min<int64_t>(4096, (count + 255) / 256);
    if (blocks > 0)
        hipLaunchKernelGGL(bl_finite_kernel, dim3((unsigned)blocks), dim3(256), 0, st, x, count, f);
    PMLSH_HIP(hipGetLastError());
    int32_t h = 0;
    PMLSH_HIP(hipMemcpyAsync(&h, f, sizeof(int32_t), hipMemcpyDeviceToHost, st));
    PMLSH_HIP(hipStreamSynchronize(st));
    return h == 0;
}

void device_pivots(const float* proj, int64_t n, int s, hipStream_t st, std::vector<float>* pivots,
                   double* max_norm) {
    constexpr int kFarBlocks = 1024;
    DevVec<double> bval, mind, part, mean, val;
    DevVec<int64_t> bidx;
    DevVec<float> rows;                 // centroid, zero row, then the s pivots
    DevVec<Piece> d_pieces;
    DevVec<int32_t> d_first;
    const int nb = (int)std::min<int64_t>(kFarBlocks, (n + 255) / 256);
    double* bv = bval.get((size_t)nb);
    int64_t* bi = bidx.get((size_t)nb);
    float* rw = rows.get((size_t)(2 + s) * MP);
    double* dv = val.get(1);
    PMLSH_HIP(hipMemsetAsync(rw, 0, (size_t)(2 + s) * MP * sizeof(float), st));
    // largest norm: the farthest point from the zero row
    hipLaunchKernelGGL(bl_far_kernel, dim3((unsigned)nb), dim3(256), 0, st, proj, n, rw + MP,
                       nullptr, bv, bi);
    hipLaunchKernelGGL(bl_pick_kernel, dim3(1), dim3(256), 0, st, proj, bv, bi, nb, nullptr, dv);
    PMLSH_HIP(hipGetLastError());
    PMLSH_HIP(hipMemcpyAsync(max_norm, dv, sizeof(double), hipMemcpyDeviceToHost, st));
    pivots->assign((size_t)s * MP, 0.f);
    if (s > 0) {
        // centroid: FP64 sums over pieces of the ids, reduced in order
        std::vector<Piece> pieces;
        std::vector<int32_t> first;
        make_pieces({0}, {n}, &pieces, &first);
        Piece* dp = d_pieces.get(pieces.size());
        int32_t* df = d_first.get(first.size());
        PMLSH_HIP(hipMemcpyAsync(dp, pieces.data(), pieces.size() * sizeof(Piece),
                                 hipMemcpyHostToDevice, st));
        PMLSH_HIP(hipMemcpyAsync(df, first.data(), first.size() * sizeof(int32_t),
                                 hipMemcpyHostToDevice, st));
        double* pt = part.get(pieces.size() * MP);
        double* mn = mean.get(MP);
        hipLaunchKernelGGL(bl_sum_kernel, dim3((unsigned)pieces.size()), dim3(256), 0, st, proj,
                           nullptr, dp, pt);
        hipLaunchKernelGGL(bl_reduce_kernel, dim3(1), dim3(256), 0, st, pt, MP, df, 1, nullptr, mn);
        PMLSH_HIP(hipGetLastError());
        // the reduce kernel sums; the mean divides by n in FP64 on the host
        double sums[MP];
        PMLSH_HIP(hipMemcpyAsync(sums, mn, sizeof(sums), hipMemcpyDeviceToHost, st));
        PMLSH_HIP(hipStreamSynchronize(st));
        float cf[MP];
        for (int j = 0; j < MP; ++j) cf[j] = (float)(sums[j] / (double)n);
        PMLSH_HIP(hipMemcpyAsync(rw, cf, sizeof(cf), hipMemcpyHostToDevice, st));
        // first pivot: the point farthest from the centroid; then each next
        // pivot is the point farthest from the pivots chosen so far
        double* md = mind.get((size_t)n);
        hipLaunchKernelGGL(bl_fill_kernel, dim3(1024), dim3(256), 0, st, md, n,
                           __builtin_huge_val());
        hipLaunchKernelGGL(bl_far_kernel, dim3((unsigned)nb), dim3(256), 0, st, proj, n, rw, nullptr,
                           bv, bi);
        hipLaunchKernelGGL(bl_pick_kernel, dim3(1), dim3(256), 0, st, proj, bv, bi, nb,
                           rw + 2 * MP, nullptr);
        for (int p = 1; p < s; ++p) {
            hipLaunchKernelGGL(bl_far_kernel, dim3((unsigned)nb), dim3(256), 0, st, proj, n,
                               rw + (size_t)(1 + p) * MP, md, bv, bi);
            hipLaunchKernelGGL(bl_pick_kernel, dim3(1), dim3(256), 0, st, proj, bv, bi, nb,
                               rw + (size_t)(2 + p) * MP, nullptr);
        }
        PMLSH_HIP(hipGetLastError());
        PMLSH_HIP(hipMemcpyAsync(pivots->data(), rw + 2 * MP, (size_t)s * MP * sizeof(float),
                                 hipMemcpyDeviceToHost, st));
    }
    PMLSH_HIP(hipStreamSynchronize(st));
}

void device_ball_summaries(const float* proj, const int32_t* perm, const std::vector<int64_t>& p0,
                           const std::vector<int64_t>& p1, const float* pivots, int s,
                           hipStream_t st, std::vector<float>* centre, std::vector<double>* radius,
                           std::vector<double>* ring) {
    const int64_t m = (int64_t)p0.size();
    const int width = 1 + 2 * s;
    centre->assign((size_t)m * MP, 0.f);
    radius->assign((size_t)m, 0.0);
    ring->assign((size_t)m * 2 * s, 0.0);
    if (m == 0) return;
    std::vector<Piece> pieces;
    std::vector<int32_t> first;
    make_pieces(p0, p1, &pieces, &first);
    std::vector<int32_t> cnt((size_t)m);
    for (int64_t i = 0; i < m; ++i) cnt[(size_t)i] = (int32_t)(p1[(size_t)i] - p0[(size_t)i]);
    DevVec<Piece> d_pieces;
    DevVec<int32_t> d_first, d_cnt;
    DevVec<double> part, mean, out;
    DevVec<float> cf, piv;
    Piece* dp = d_pieces.get(pieces.size());
    int32_t* df = d_first.get(first.size());
    int32_t* dc = d_cnt.get((size_t)m);
    PMLSH_HIP(hipMemcpyAsync(dp, pieces.data(), pieces.size() * sizeof(Piece),
                             hipMemcpyHostToDevice, st));
    PMLSH_HIP(hipMemcpyAsync(df, first.data(), first.size() * sizeof(int32_t),
                             hipMemcpyHostToDevice, st));
    PMLSH_HIP(hipMemcpyAsync(dc, cnt.data(), cnt.size() * sizeof(int32_t), hipMemcpyHostToDevice,
                             st));
    const int np = (int)pieces.size();
    double* pt = part.get((size_t)np * std::max(MP, width));
    double* mn = mean.get((size_t)m * MP);
    float* c = cf.get((size_t)m * MP);
    double* o = out.get((size_t)m * width);
    float* pv = piv.get((size_t)std::max(1, s) * MP);
    if (s > 0)
        PMLSH_HIP(hipMemcpyAsync(pv, pivots, (size_t)s * MP * sizeof(float), hipMemcpyHostToDevice,
                                 st));
    hipLaunchKernelGGL(bl_sum_kernel, dim3((unsigned)np), dim3(256), 0, st, proj, perm, dp, pt);
    hipLaunchKernelGGL(bl_reduce_kernel, dim3((unsigned)((m * MP + 255) / 256)), dim3(256), 0, st,
                       pt, MP, df, (int)m, dc, mn);
    hipLaunchKernelGGL(bl_centre_kernel, dim3((unsigned)((m * MP + 255) / 256)), dim3(256), 0, st,
                       mn, m * MP, c);
    hipLaunchKernelGGL(bl_ring_kernel, dim3((unsigned)np), dim3(256), 0, st, proj, perm, dp, c, pv,
                       s, pt);
    hipLaunchKernelGGL(bl_reduce_ring_kernel, dim3((unsigned)((m * width + 255) / 256)), dim3(256),
                       0, st, pt, width, df, (int)m, o);
    PMLSH_HIP(hipGetLastError());
    std::vector<double> h((size_t)m * width);
    PMLSH_HIP(hipMemcpyAsync(centre->data(), c, (size_t)m * MP * sizeof(float),
                             hipMemcpyDeviceToHost, st));
    PMLSH_HIP(hipMemcpyAsync(h.data(), o, h.size() * sizeof(double), hipMemcpyDeviceToHost, st));
    PMLSH_HIP(hipStreamSynchronize(st));
    for (int64_t i = 0; i < m; ++i) {
        (*radius)[(size_t)i] = h[(size_t)(i * width)];
        for (int t = 0; t < 2 * s; ++t) (*ring)[(size_t)(i * 2 * s + t)] = h[(size_t)(i * width + 1 + t)];
    }
}

}  // namespace pmlsh
