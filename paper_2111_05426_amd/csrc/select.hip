// select.hip -- feasibility filter and ordered top-k over the candidates.
//
// Selection of Sec. 5.2: drop candidates whose peak exceeds the per-device
// memory cap (or whose status is non-zero), rank the rest by predicted time
// (makespan ascending, ties to the lower index), keep the first k.
//
// Small sets are ranked by counting: with all keys in LDS, a key's place is
// the number of smaller ones, which takes one pass of broadcast reads and no
// rounds.  Calls of at most 512 keys (640 for k > 32, 1,024 at k = 1) are one
// block of that; beyond, the count costs more than a second launch (k = 4, us,
// one block against two passes: 400 keys 13.3 / 13.9, 512 16.6 / 13.9, 1,024
// 43 / 14).  Larger ones take two passes.  Pass 1: block b owns a contiguous
// chunk and writes its k smallest (makespan, index) keys in order; chunks have
// 256 keys while fewer than 256 blocks would run, and at most 1,024 blocks
// run, of 512 threads from chunks of 4,096 keys on (16 million keys, top-16,
// us: 512 blocks of 256 threads 1,352, 1,024 of 256 747, 1,024 of 512 429,
// with the loads of four keys in flight 291).  A chunk of 256 keys
// is ranked by counting for k > 8; else each wavefront takes its least
// remaining key round by round (in larger chunks the winning lane then looks
// for its next one) and the block's lists are merged by rank.  Pass 2:
// one block bounds the k-th smallest key -- by the lists' heads, or by their
// j-th keys where lists are few, and by the least of the lists' k-th keys --
// gathers the keys up to the bound and ranks them by counting.  The order is
// a total order on (makespan, index), so the result does not depend on the
// launch shape.
//
// Bound by the two launches and by the counts.  A call, us, k = 4, 16, 64:
// 3,000 keys 14, 18, 26; 65,536 14, 22, 34; a million 21, 52, 177; 16 million
// 96, 291, 1,093.  (Counting every head for small k as well: 100,000 keys,
// k = 4 26.2 against 12.9.)
#include "internal.h"

#include <math.h>

namespace dsim {
namespace {

constexpr int kSelBlock = 256;
constexpr int kWideBlock = 512;   // for chunks of kChunk keys and more
constexpr int kMergeBlock = 1024;
constexpr int kMergeWaves = kMergeBlock / 64;
constexpr int kMaxK = 64;
constexpr int64_t kChunk = 4096;
constexpr int64_t kMinChunk = 256;
constexpr int kMaxBlocks = 1024;
constexpr int kLeastBlocks = 512;  // at most so many where the workspace holds no more lists
constexpr int kRowK = 16;     // 16 lists stand as one in the merge up to this k: 16 k^2 <= kMaxK^2 keys
constexpr int kRoundK = 8;    // chunks of one key a thread take rounds up to this k
constexpr int kFillBlocks = 256;   // one chunk per CU at least, while chunks stay >= kMinChunk
// Keys of a call without a second pass: any number the block has threads for
// at k = 1; else up to where counting costs what the second pass does
constexpr int64_t one_block(int k) { return k == 1 ? kMergeBlock : (k <= 32 ? 512 : 640); }

struct Key {
    double mk;
    int64_t idx;
};

constexpr int64_t kNone = INT64_MAX;

__device__ __forceinline__ bool key_less(double am, int64_t ai, double bm, int64_t bi)
{
    return am < bm || (am == bm && ai < bi);
}

template <int CTRL, int ROWS> __device__ __forceinline__ double min_dpp(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    // (lanes without a source keep their own value)
    const int lo = __builtin_amdgcn_update_dpp((int)b, (int)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(b >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return fmin(v, __hiloint2double(hi, lo));
}

// The least key of the wavefront: its lane (keys are not NaN; lanes without a
// key hold (+inf, kNone)).
__device__ __forceinline__ int wave_least(double m, int64_t i)
{
    double v = m;
    v = min_dpp<0x111, 0xf>(v);
    v = min_dpp<0x112, 0xf>(v);
    v = min_dpp<0x114, 0xf>(v);
    v = min_dpp<0x118, 0xf>(v);
    v = min_dpp<0x142, 0xa>(v);
    v = min_dpp<0x143, 0xc>(v);
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63), hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    const double least = __hiloint2double(hi, lo);
    uint64_t at = __builtin_amdgcn_ballot_w64(m == least);
    if ((at & (at - 1)) != 0) {   // equal makespans: the lowest index
        int64_t b = m == least ? i : kNone;
        for (int o = 32; o > 0; o >>= 1) {
            const int64_t x = __shfl_xor(b, o, 64);
            b = x < b ? x : b;
        }
        at = __builtin_amdgcn_ballot_w64(m == least && i == b);
    }
    return __builtin_ctzll(at);
}

__device__ __forceinline__ double from_lane(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ __forceinline__ int64_t from_lane(int64_t v, int l)
{
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane((int)v, l));
}

// Merge of W ascending lists of k keys by rank: thread t's key and its place
// among all of them (-1: no key).  n: keys there are in all.
template <int W> __device__ __forceinline__ int rank_of(const double (&m)[W][kMaxK], const int64_t (&i)[W][kMaxK], int k,
                                                        int t, Key &key, int &n)
{
    n = 0;
    int place = -1;
    const int a = t / k, r = t % k;
    const bool has = t < W * k && i[a < W ? a : 0][r] != kNone;
    if (has) {
        key = Key{m[a][r], i[a][r]};
        place = r;
    }
    for (int b = 0; b < W; ++b) {
        // keys of list b below this one, and in all
        int lo = 0, hi = k, all = 0, end = k;
        while (lo < hi || all < end) {
            if (lo < hi) {
                const int mid = (lo + hi) / 2;
                if (has && key_less(m[b][mid], i[b][mid], key.mk, key.idx)) lo = mid + 1;
                else hi = mid;
            }
            if (all < end) {
                const int mid = (all + end) / 2;
                if (i[b][mid] != kNone) all = mid + 1;
                else end = mid;
            }
        }
        if (has && b != a) place += lo;
        n += all;
    }
    return place;
}

// The feasible makespan of entry i, NaN for an infeasible one (NaN compares
// false with everything, so it is never counted).
__device__ __forceinline__ double feasible(const double *mk, const uint64_t *pk, const int32_t *st, uint64_t cap,
                                           int64_t i)
{
    // (the loads do not wait for one another)
    const double m = mk[i];
    const uint64_t p = cap != 0 ? pk[i] : 0;
    return st[i] == 0 && p <= cap ? m : __longlong_as_double(-1);
}

// how many of the n keys (m[j], j) are less than (v, t)
__device__ __forceinline__ int count_less(const double *m, int n, double v, int t)
{
    int less = 0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) less += (m[j] < v) | ((m[j] == v) & (j < t)) ? 1 : 0;
    return less;
}

// The least (m, i) of a block of W wavefronts, in its thread 0's return value.
template <int W> __device__ __forceinline__ Key block_least(double m, int64_t i, double *s_m, int64_t *s_i)
{
    const int t = threadIdx.x;
    const int l = wave_least(m, i);
    const double wm = from_lane(m, l);
    const int64_t wi = from_lane(i, l);
    if ((t & 63) == 0) {
        s_m[t / 64] = wm;
        s_i[t / 64] = wi;
    }
    __syncthreads();
    Key k{s_m[0], s_i[0]};
    for (int v = 1; v < W; ++v)
        if (key_less(s_m[v], s_i[v], k.mk, k.idx)) k = Key{s_m[v], s_i[v]};
    return k;
}

// at most 1,024 keys
__global__ __launch_bounds__(kMergeBlock) void k_select_one(const double *mk, const uint64_t *pk, const int32_t *st,
                                                            int n, uint64_t cap, int k, int64_t *out_idx,
                                                            double *out_mk, int32_t *out_found)
{
    __shared__ double s_m[kMergeBlock];
    __shared__ int64_t s_i[kMergeWaves];
    __shared__ int s_n;
    const int t = threadIdx.x;
    const double v = t < n ? feasible(mk, pk, st, cap, t) : __longlong_as_double(-1);
    const bool has = v == v;
    if (k == 1) {
        const Key b = block_least<kMergeWaves>(has ? v : HUGE_VAL, has ? t : kNone, s_m, s_i);
        if (t == 0) {
            out_idx[0] = b.idx == kNone ? -1 : b.idx;
            out_mk[0] = b.mk;
            *out_found = b.idx == kNone ? 0 : 1;
        }
        return;
    }
    if (t == 0) s_n = 0;
    s_m[t] = v;
    __syncthreads();
    if (has) {
        const int r = count_less(s_m, n, v, t);
        if (r < k) {
            out_idx[r] = t;
            out_mk[r] = v;
        }
    }
    const int mine = __popcll(__builtin_amdgcn_ballot_w64(has));
    if ((t & 63) == 0) atomicAdd(&s_n, mine);
    __syncthreads();
    const int found = s_n < k ? s_n : k;
    if (t >= found && t < k) {
        out_idx[t] = -1;
        out_mk[t] = HUGE_VAL;
    }
    if (t == 0) *out_found = found;
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_select_chunks(const double *mk, const uint64_t *pk, const int32_t *st,
                                                         int64_t n, uint64_t cap, int k, int64_t chunk, Key *ws)
{
    constexpr int kWaves = BLOCK / 64;
    __shared__ double s_m[kWaves][kMaxK];
    __shared__ int64_t s_i[kWaves][kMaxK];
    const int t = threadIdx.x, wave = t / 64, lane = t % 64;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    Key *list = ws + (int64_t)blockIdx.x * k;
    // this thread's least key above (pm, pi)
    auto next = [&](double pm, int64_t pi, double &bm, int64_t &bi) {
        bm = HUGE_VAL;
        bi = kNone;
#pragma unroll 4
        for (int64_t i = lo + t; i < hi; i += BLOCK) {
            const double m = feasible(mk, pk, st, cap, i);
            if (key_less(pm, pi, m, i) && key_less(m, i, bm, bi)) {
                bm = m;
                bi = i;
            }
        }
    };
    double bm;
    int64_t bi;
    if (k == 1) {
        next(-HUGE_VAL, -1, bm, bi);
        const Key b = block_least<kWaves>(bm, bi, &s_m[0][0], &s_i[0][0]);
        if (t == 0) list[0] = Key{b.mk, b.idx == kNone ? -1 : b.idx};
        return;
    }
    // one key a thread: counting takes one pass over 256 keys, the rounds
    // below (without a second look at the chunk) a pass over 64 lanes each
    if (chunk == BLOCK && k > kRoundK) {
        static_assert(kWaves * kMaxK == BLOCK, "a place for every thread's key");
        double *all = &s_m[0][0];
        const double v = lo + t < hi ? feasible(mk, pk, st, cap, lo + t) : __longlong_as_double(-1);
        const bool has = v == v;
        all[t] = v;
        if (t < kWaves) s_i[0][t] = 0;
        __syncthreads();
        if (has) {
            const int r = count_less(all, BLOCK, v, t);
            if (r < k) list[r] = Key{v, lo + t};
        }
        const int mine = __popcll(__builtin_amdgcn_ballot_w64(has));
        if (lane == 0) s_i[0][wave] = mine;
        __syncthreads();
        int have = 0;
        for (int w = 0; w < kWaves; ++w) have += (int)s_i[0][w];
        if (t >= have && t < k) list[t] = Key{HUGE_VAL, -1};
        return;
    }
    next(-HUGE_VAL, -1, bm, bi);
    for (int r = 0; r < k; ++r) {
        const int l = wave_least(bm, bi);
        const double wm = from_lane(bm, l);
        const int64_t wi = from_lane(bi, l);
        if (lane == 0) {
            s_m[wave][r] = wm;
            s_i[wave][r] = wi;
        }
        if (wi == kNone) {
            for (int q = r + 1 + lane; q < k; q += 64) {
                s_m[wave][q] = HUGE_VAL;
                s_i[wave][q] = kNone;
            }
            break;
        }
        if (lane == l && r + 1 < k) {
            if (chunk == BLOCK) {
                bm = HUGE_VAL;
                bi = kNone;
            } else {
                next(wm, wi, bm, bi);
            }
        }
    }
    __syncthreads();
    Key key{HUGE_VAL, -1};
    int have;
    const int place = rank_of(s_m, s_i, k, t, key, have);
    if (place >= 0 && place < k) list[place] = key;
    if (t >= have && t < k) list[t] = Key{HUGE_VAL, -1};
}

__global__ __launch_bounds__(kMergeBlock) void k_select_merge(const Key *ws, int64_t nl, int k,
                                                            int64_t *out_idx, double *out_mk,
                                                            int32_t *out_found)
{
    static_assert(16 * kRowK * kRowK <= kMaxK * kMaxK && kMaxBlocks <= kMergeBlock, "room for the gathered keys, a thread for every list");
    __shared__ double s_m[kMaxK * kMaxK];
    __shared__ int64_t s_i[kMaxK * kMaxK];
    __shared__ double s_wm[kMergeWaves];
    __shared__ int64_t s_wi[kMergeWaves];
    __shared__ Key s_bound;
    __shared__ int s_n;
    const int t = threadIdx.x;
    const Key none{HUGE_VAL, kNone};
    Key head = t < nl ? ws[(int64_t)t * k] : none;
    if (head.idx < 0) head = none;
    if (k == 1) {
        const Key b = block_least<kMergeWaves>(head.mk, head.idx, s_wm, s_wi);
        if (t == 0) {
            out_idx[0] = b.idx == kNone ? -1 : b.idx;
            out_mk[0] = b.mk;
            *out_found = b.idx == kNone ? 0 : 1;
        }
        return;
    }
    Key tail = t < nl ? ws[(int64_t)t * k + k - 1] : none;
    if (tail.idx < 0) tail = none;
    // Every list's j-th key: where p = ceil(k / j) of them lie at or below a
    // key, so do k keys.  Few lists: a j that leaves about half the lists
    // above the bound.
    const int j = nl >= 2 * k ? 1 : (int)((2 * k + nl - 1) / nl);
    const int p = (k + j - 1) / j;
    Key mark = head;
    if (j > 1) {
        mark = t < nl && j <= k ? ws[(int64_t)t * k + j - 1] : none;
        if (mark.idx < 0) mark = none;
    }
    const bool has = mark.idx != kNone;
    // Many lists for few keys: the least of 16 lists stands for them (the
    // gathered keys then come from 16 k lists at most, 16 k^2 keys), and a
    // sixteenth of the keys is counted.
    const bool rows = k <= kRowK && nl >= 16 * k;
    bool lead = has;
    if (rows) {
        double v = mark.mk;
        v = min_dpp<0x111, 0xf>(v);
        v = min_dpp<0x112, 0xf>(v);
        v = min_dpp<0x114, 0xf>(v);
        v = min_dpp<0x118, 0xf>(v);
        v = __shfl(v, (t & 63) | 15, 64);
        const uint32_t at = (uint32_t)(__builtin_amdgcn_ballot_w64(has && mark.mk == v) >> (t & 48)) & 0xffffu;
        lead = at != 0 && (t & 15) == __builtin_ctz(at);
        if (lead || (at == 0 && (t & 15) == 0)) s_m[t / 16] = lead ? mark.mk : __longlong_as_double(-1);
    } else if (t < nl) {
        s_m[t] = has ? mark.mk : __longlong_as_double(-1);
    }
    if (t == 0) {
        s_bound = none;
        s_n = 0;
    }
    const Key last = block_least<kMergeWaves>(tail.mk, tail.idx, s_wm, s_wi);   // (its barrier covers the stores above)
    // lists hold ascending indices, so equal keys rank by their list
    const int place = rows ? t / 16 : t;
    if (lead && count_less(s_m, rows ? (int)((nl + 15) / 16) : (int)nl, mark.mk, place) == p - 1) s_bound = mark;
    __syncthreads();
    Key bound = s_bound;
    if (key_less(last.mk, last.idx, bound.mk, bound.idx)) bound = last;
    // the keys up to the bound: of p lists (16 k at most) all k at most, of
    // the others fewer than j
    for (int64_t q = t; q < nl * k; q += kMergeBlock) {
        const Key x = ws[q];
        if (x.idx >= 0 && !key_less(bound.mk, bound.idx, x.mk, x.idx)) {
            const int at = atomicAdd(&s_n, 1);
            s_m[at] = x.mk;
            s_i[at] = x.idx;
        }
    }
    __syncthreads();
    const int n = s_n;
    for (int q = t; q < n; q += kMergeBlock) {
        const double m = s_m[q];
        const int64_t i = s_i[q];
        int r = 0;
#pragma unroll 4
        for (int j = 0; j < n; ++j) r += key_less(s_m[j], s_i[j], m, i) ? 1 : 0;
        if (r < k) {
            out_idx[r] = i;
            out_mk[r] = m;
        }
    }
    const int found = n < k ? n : k;
    if (t >= found && t < k) {
        out_idx[t] = -1;
        out_mk[t] = HUGE_VAL;
    }
    if (t == 0) *out_found = found;
}

int64_t n_chunks(int64_t n, int64_t most, int64_t *chunk)
{
    int64_t c = kChunk;
    while ((n + c - 1) / c > most) c *= 2;
    while (c > kMinChunk && (n + c - 1) / c < kFillBlocks) c /= 2;
    *chunk = c;
    const int64_t b = (n + c - 1) / c;
    return b > 0 ? b : 1;
}

}  // namespace

size_t argmin_workspace(int64_t n, int32_t k)
{
    int64_t chunk;
    return (size_t)n_chunks(n, kMaxBlocks, &chunk) * (size_t)k * sizeof(Key);
}

size_t argmin_workspace_least(int64_t n, int32_t k)
{
    int64_t chunk;
    return (size_t)n_chunks(n, kLeastBlocks, &chunk) * (size_t)k * sizeof(Key);
}

dsim_status launch_argmin(const double *mk, const uint64_t *pk, const int32_t *st, int64_t n,
                          uint64_t cap, int32_t k, void *ws, size_t ws_bytes, int64_t *out_idx, double *out_mk,
                          int32_t *out_found, hipStream_t s)
{
    if (n <= one_block(k)) {
        hipLaunchKernelGGL(k_select_one, dim3(1), dim3(kMergeBlock), 0, s, mk, pk, st, (int)n, cap, k, out_idx, out_mk,
                           out_found);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? DSIM_OK : hip_fail(e, "select launch");
    }
    int64_t chunk;
    const int64_t blocks = n_chunks(n, ws_bytes >= argmin_workspace(n, k) ? kMaxBlocks : kLeastBlocks, &chunk);
    Key *w = static_cast<Key *>(ws);
    if (chunk >= kChunk)
        hipLaunchKernelGGL(k_select_chunks<kWideBlock>, dim3((unsigned)blocks), dim3(kWideBlock), 0, s, mk, pk, st, n,
                           cap, k, chunk, w);
    else
        hipLaunchKernelGGL(k_select_chunks<kSelBlock>, dim3((unsigned)blocks), dim3(kSelBlock), 0, s, mk, pk, st, n,
                           cap, k, chunk, w);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "select_chunks launch");
    hipLaunchKernelGGL(k_select_merge, dim3(1), dim3(kMergeBlock), 0, s, w, blocks, k, out_idx, out_mk, out_found);
    e = hipGetLastError();
    return e == hipSuccess ? DSIM_OK : hip_fail(e, "select_merge launch");
}

}  // namespace dsim
