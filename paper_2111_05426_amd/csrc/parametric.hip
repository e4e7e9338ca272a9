// parametric.hip -- the D/H/P/K transform's kernel for segments of 16 lanes and
// more, the pre-pass that groups the candidates, and the launches.
#include <mutex>

#include "parametric.h"

namespace dsim {
namespace {

constexpr int kScanBlock = 256;

// (three wavefronts per SIMD for the ZeRO kernels, at the price of 19
// registers spilled in their set-up, whose per-block maxima over the replicas
// otherwise take 187 and leave two: GPT-3-shaped ZeRO grid 1.83 -> 1.41 ms)
template <bool TF, bool RC, bool ZR, bool OV>
__global__ __launch_bounds__(kLanes) __attribute__((amdgpu_waves_per_eu(ZR ? 3 : 1))) void k_parametric(const ParArgs g)
{
    parametric_body<TF, false, RC, ZR, OV>(g, 0);
}

// the kernel of a launch, by family and model options
template <bool RC, bool ZR, bool OV>
void launch_variant(bool tf, dim3 grid, hipStream_t s, const ParArgs &g)
{
    if (tf) hipLaunchKernelGGL((k_parametric<true, RC, ZR, OV>), grid, dim3(kLanes), 0, s, g);
    else hipLaunchKernelGGL((k_parametric<false, RC, ZR, OV>), grid, dim3(kLanes), 0, s, g);
}

// (ZeRO and overlap exclude one another)
void launch_kernel(bool rc, bool zr, bool ov, bool tf, dim3 grid, hipStream_t s, const ParArgs &g)
{
    if (rc) {
        if (zr) launch_variant<true, true, false>(tf, grid, s, g);
        else if (ov) launch_variant<true, false, true>(tf, grid, s, g);
        else launch_variant<true, false, false>(tf, grid, s, g);
    } else {
        if (zr) launch_variant<false, true, false>(tf, grid, s, g);
        else if (ov) launch_variant<false, false, true>(tf, grid, s, g);
        else launch_variant<false, false, false>(tf, grid, s, g);
    }
}

// ---------------------------------------------------------------------------
// Pre-pass: stable counting sort of the candidates by segment class, and the
// order in which the wavefronts of 16 lanes and more a candidate start
// ---------------------------------------------------------------------------
// A slot's fixed work (schedule, Sends, memory updates) counts as this many
// layers of a stage.
constexpr uint32_t kSlotLayers = 8;

// Relative length of the wavefront that simulates a candidate: slots (the
// stage's blocks plus the pipeline's fill and drain) times the work of a
// slot (a fixed part and the stage's share of the layers), in half layers.
// Only orders the wavefronts.  (An estimate of the slots left after whole
// periods are skipped, weighted by the class, ran the two-stream and ZeRO
// grids 1 to 10% slower and GPipe 4% faster.)
__device__ __forceinline__ uint32_t wave_length(const dsim_strategy &st, int n_layers, bool train)
{
    const uint32_t P = (uint32_t)(st.P < 1 ? 1 : (st.P > kMaxStages ? kMaxStages : st.P));
    const uint32_t K = (uint32_t)(st.K < 1 ? 1 : (st.K > kMaxK ? kMaxK : st.K));
    const uint32_t L = (uint32_t)(n_layers < 1 ? 1 : (n_layers > 65536 ? 65536 : n_layers));
    const uint32_t slots = (train ? 2u : 1u) * K + 2u * P;      // <= 32,894
    const uint32_t work = 2u * kSlotLayers + (2u * L + P - 1) / P;   // <= 131,088
    const uint64_t len = (uint64_t)slots * work;
    return len > 0xffffffffu ? 0xffffffffu : (uint32_t)len;
}

// The narrow launch's rule: how many strategies of few stages, at most K
// microbatches each, a call must have for it.  Its wavefronts hold many
// candidates, so there are few of them and its time is the longest one's;
// wider: others run in a launch of their own after it, and the two add up.
// us, 16 lanes a candidate against the narrow launch, strategies of up to four
// stages:
//   10,000 of K <= 4: MLP 72 / 59, transformer 87 / 63;
//   10,000 and 30,000 of K <= 64: MLP 189 / 202 and 235 / 158, transformer
//   165 / 265 and 277 / 211; of K <= 256: 224 / 255 and 340 / 229, 205 / 344
//   and 347 / 303;
// with a quarter of eight stages beside them, K <= 4: 10,000 MLP 72 / 115,
// 30,000 146 / 121; K <= 64, transformer: 30,000 294 / 373, 100,000 790 / 612;
// K <= 256: 395 / 536 and 902 / 892.
constexpr uint32_t kNarrowAll = 24576, kEightMin = 12288;
__device__ __forceinline__ uint32_t narrow_min(uint32_t K, bool wider)
{
    if (K <= (uint32_t)kShortK) return wider ? 16384 : 0;
    if (K <= 64) return wider ? 40960 : 20480;
    return wider ? 65536 : kNarrowAll;
}

// meta as in ParArgs, from the classes' totals ([kClasses]: the largest K of
// the narrow ones)
__device__ void class_table(const uint32_t *total, bool tf, bool train, uint32_t *meta)
{
    bool wider = false;
    for (int i = kNarrow; i < kClasses; ++i) wider = wider || total[i] != 0;
    uint32_t few = 0;
    for (int i = 0; i < kNarrow - 1; ++i) few += total[i];
    // segments of 8 lanes: beside wider ones, in small calls and in large ones
    // of a transformer's training they are better off with those
    const uint32_t all = few + total[kNarrow - 1];
    const bool eight = !wider && all >= kEightMin && (!tf || !train || all < 65536);
    wider = wider || (!eight && total[kNarrow - 1] != 0);
    const bool on = (eight ? all : few) >= narrow_min(total[kClasses], wider);
    const int n_mine = !on ? 0 : (eight ? kNarrow : kNarrow - 1);   // narrow classes of the narrow launch
    uint32_t rank = 0, wave = 0, narrow = 0;
    for (int i = 0; i < kClasses; ++i) {
        uint32_t n = total[i];
        const uint32_t per = (uint32_t)kLanes >> i;   // candidates per wavefront
        meta[8 + i] = rank;
        meta[16 + i] = wave;
        rank += n;
        if (i < kNarrow) {
            // the others join class kMinClass
            meta[24 + i] = narrow;
            meta[i] = i < n_mine ? n : 0;
            if (i < n_mine) narrow += (n + per - 1) / per;
            continue;
        }
        if (i == kMinClass) {
            meta[29] = meta[8 + i];
            meta[8 + i] = meta[8 + n_mine];
            n = rank - meta[8 + n_mine];
        }
        meta[i] = n;
        wave += (n + per - 1) / per;
    }
    meta[24 + kNarrow] = narrow;
    meta[kClasses] = 0;
    meta[8 + kClasses] = rank;
    meta[16 + kClasses] = wave;
}

// (wave_len: n + 8 words cleared for k_class_scatter)
__global__ __launch_bounds__(kScanBlock) void k_class_count(const dsim_strategy *cand, int64_t n, int p_bound, bool narrow,
                                                           uint32_t *counts, uint32_t *wave_len)
{
    __shared__ uint32_t s_cnt[8];
    if (threadIdx.x < 8) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
    if (c < n) wave_len[c] = 0;
    if (c < 8) wave_len[n + c] = 0;
    if (c < n) {
        const dsim_strategy st = cand[c];
        const int j = seg_class(st, p_bound, narrow);
        atomicAdd(&s_cnt[j], 1u);
        if (j < kNarrow && st.P >= 1 && st.K <= kMaxK) atomicMax((int *)&s_cnt[kClasses], st.K);
    }
    __syncthreads();
    if (threadIdx.x < 8) counts[(size_t)blockIdx.x * 8 + threadIdx.x] = s_cnt[threadIdx.x];
}

// counts[b][j] -> exclusive prefix over blocks b, per class j; meta as in
// ParArgs.  One block; a wavefront per class, one for the largest K.
__global__ __launch_bounds__(kLanes * (kClasses + 1)) void k_class_scan(uint32_t *counts, int64_t nb, uint32_t *meta, bool tf,
                                                                         bool train)
{
    __shared__ uint32_t s_total[kClasses + 1];
    const int j = threadIdx.x / kLanes, lane = threadIdx.x % kLanes;
    uint32_t carry = 0;
    if (j == kClasses) {
        for (int64_t b = lane; b < nb; b += kLanes) carry = max(carry, counts[(size_t)b * 8 + j]);
        for (int o = 32; o > 0; o >>= 1) carry = max(carry, (uint32_t)__shfl_xor((int)carry, o, kLanes));
    } else {
        for (int64_t b0 = 0; b0 < nb; b0 += kLanes) {
            const int64_t b = b0 + lane;
            const uint32_t v = b < nb ? counts[(size_t)b * 8 + j] : 0;
            uint32_t sum = v;
            for (int o = 1; o < kLanes; o <<= 1) {
                const uint32_t up = (uint32_t)__shfl_up((int)sum, o, kLanes);
                sum += lane >= o ? up : 0;
            }
            if (b < nb) counts[(size_t)b * 8 + j] = carry + sum - v;
            carry += (uint32_t)__shfl((int)sum, kLanes - 1, kLanes);
        }
    }
    if (lane == 0) s_total[j] = carry;
    __syncthreads();
    if (threadIdx.x == 0) class_table(s_total, tf, train, meta);
}

// wave_length quantized: 16 steps per doubling
constexpr int kLenBuckets = 512;
constexpr int kOrderBlock = 1024;
__device__ __forceinline__ int len_bucket(uint32_t len)
{
    if (len == 0) return 0;
    const int e = 31 - __clz(len);
    const uint32_t f = e >= 4 ? (len >> (e - 4)) & 15u : (len << (4 - e)) & 15u;
    return e * 16 + (int)f;
}

// The wavefronts longest first: a counting sort of
// wave_len (each wavefront's longest candidate, from k_class_scatter) over
// len_bucket, wavefronts of one bucket in any order.  One block.
__global__ __launch_bounds__(kOrderBlock) void k_wave_order(const uint32_t *meta, const uint32_t *wave_len,
                                                           uint32_t *order)
{
    __shared__ uint32_t s_cnt[kLenBuckets], s_part[kLenBuckets / kLanes];
    const int t = threadIdx.x;
    const uint32_t n_w = meta[16 + kClasses];
    for (int i = t; i < kLenBuckets; i += kOrderBlock) s_cnt[i] = 0;
    __syncthreads();
    // (neighbouring wavefronts have nearly the same length, and a wavefront's
    // atomics on one bucket run one by one; a contiguous part of the list per
    // thread took 13 instead of 20 us here, but mixed the wavefronts of a
    // bucket and cost the simulation 20)
    for (uint32_t i = t; i < n_w; i += kOrderBlock) atomicAdd(&s_cnt[len_bucket(wave_len[i])], 1u);
    __syncthreads();
    // bucket starts, longest bucket first: a prefix sum from the last bucket
    const int b = kLenBuckets - 1 - t;
    uint32_t sum = t < kLenBuckets ? s_cnt[b] : 0;
    const uint32_t own = sum;
    for (int o = 1; o < kLanes; o <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)sum, o, kLanes);
        sum += t % kLanes >= o ? up : 0;
    }
    if (t < kLenBuckets && t % kLanes == kLanes - 1) s_part[t / kLanes] = sum;
    __syncthreads();
    if (t < kLenBuckets) {
        for (int w = 0; w < t / kLanes; ++w) sum += s_part[w];
        s_cnt[b] = sum - own;
    }
    __syncthreads();
    for (uint32_t i = t; i < n_w; i += kOrderBlock) order[atomicAdd(&s_cnt[len_bucket(wave_len[i])], 1u)] = i;
}

// (wave_len: each wavefront's longest wave_length)
__global__ __launch_bounds__(kScanBlock) void k_class_scatter(const dsim_strategy *cand, int64_t n, int p_bound,
                                                             bool narrow, const uint32_t *offsets, const uint32_t *meta,
                                                             uint32_t *perm, int n_layers, bool train,
                                                             uint32_t *wave_len)
{
    constexpr int kWaves = kScanBlock / kLanes;
    __shared__ uint32_t s_wcnt[kWaves][8];
    const int t = threadIdx.x, wv = t / kLanes, lane = t % kLanes;
    const int64_t c = (int64_t)blockIdx.x * kScanBlock + t;
    const int j = c < n ? seg_class(cand[c], p_bound, narrow) : kClasses;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint32_t rank = 0;
    for (int jj = 0; jj < kClasses; ++jj) {
        const uint64_t b = __ballot(j == jj);
        if (lane == 0) s_wcnt[wv][jj] = (uint32_t)__popcll(b);
        if (j == jj) rank = (uint32_t)__popcll(b & below);
    }
    __syncthreads();
    if (j < kClasses) {
        for (int v = 0; v < wv; ++v) rank += s_wcnt[v][j];
        const uint32_t slot = offsets[(size_t)blockIdx.x * 8 + j] + rank;
        const uint32_t at = meta[j == kMinClass ? 29 : 8 + j] + slot;
        perm[at] = (uint32_t)c;
        if (j >= kNarrow || meta[j] == 0) {   // (narrow classes with a total are in the narrow launch)
            const int w = max(j, kMinClass);
            atomicMax(&wave_len[meta[16 + w] + ((at - meta[8 + w]) >> (6 - w))], wave_length(cand[c], n_layers, train));
        }
    }
}

}  // namespace

// Scratch of dsim_simulate_parametric_static: the grouping workspace of at
// most kStaticMaxCand candidates, one copy per GPU for the whole process.
// Host code never uses this name as an address; it takes the device address
// once per GPU (static_scratch).
constexpr int64_t kStaticMaxCand = (int64_t)1 << 20;
constexpr int64_t kStaticWords = (kStaticMaxCand / kScanBlock) * 8 + 32 + 3 * kStaticMaxCand + 16;
static __device__ __align__(256) uint32_t scratch[kStaticWords];

dsim_status static_scratch(void **out)
{
    static std::mutex mu;
    static void *addr[kMaxGpus] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "parametric (static): current device");
    if (dev < 0 || dev >= kMaxGpus) return fail(DSIM_ERANGE, "parametric (static): device %d beyond %d", dev, kMaxGpus);
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e, "parametric (static): scratch address");
        addr[dev] = p;
    }
    *out = addr[dev];
    return DSIM_OK;
}

int64_t static_max_cand() { return kStaticMaxCand; }

size_t parametric_workspace(int64_t n_cand)
{
    const int64_t nb = (n_cand + kScanBlock - 1) / kScanBlock;
    // per-block class counts, the class table (32 words), the permutation,
    // the wavefronts' order and lengths (at most n_cand +
    // kClasses wavefronts each)
    return (size_t)(nb * 8 + 32 + 3 * n_cand + 16) * sizeof(uint32_t);
}

// Up to this many strategies get a wavefront each: the chip holds 4,096 of
// them at once (4 per SIMD; the transformer's ZeRO kernels, whose registers
// leave 3, run the last quarter after the others), no pre-pass is needed, and
// a wavefront's rare events are its one candidate's own.  4,096 of these
// against 4,097 that share, us, up to four stages and 64 microbatches: MLP 157
// / 187, transformer 131 / 173, with ZeRO 200 / 202; eight stages with ZeRO 213 /
// 198; up to 4 microbatches 50 / 68 and 68 / 86.
constexpr int64_t kAloneCand = 4096;
constexpr int64_t kNarrowBlocks = 2048;   // of the narrow launch at most: eight for every CU
// Calls that may have a narrow launch: of strategies of at most four stages
// (eight, where segments of 8 lanes may take part), and large ones.  An empty
// one costs 4 us, 2 to 4% of a call of 4,097 to 20,000 strategies of four
// stages and many microbatches, whose number the host does not see.
constexpr int kNarrowStages = 8;
constexpr int64_t kNarrowCall = 40960;

dsim_status launch_parametric(const dsim_model &m, const dsim_strategy *cand, int64_t n_cand, const CostConsts &c,
                              const dsim_results &r, void *ws, hipStream_t s, hipStream_t)   // (no second stream needed)
{
    if (n_cand > (int64_t)0x7fffffff)
        return fail(DSIM_ERANGE, "parametric: at most 2^31 - 1 candidates per call");
    ParArgs g;
    g.m = m;
    g.cand = cand;
    g.row_width = r.row_width;
    int pb = r.row_width > 0 ? r.row_width : kMaxStages;
    if (pb > kMaxStages) pb = kMaxStages;
    if (pb > m.n_layers) pb = m.n_layers;
    g.p_bound = pb;
    int wmax = 1;
    while (wmax < pb) wmax <<= 1;
    // the call's limit: the lanes of n_cand widest segments stay within a
    // dispatch's 32-bit count (the launch below, of at least 16 lanes a
    // candidate, is cut into several where it is larger)
    if ((n_cand * wmax + kLanes - 1) / kLanes + kClasses > (int64_t)(0xffffffffu / kLanes))
        return fail(DSIM_ERANGE, "parametric: n_cand * %d lanes (the widest segment for row_width %d) exceed one "
                                 "dispatch; split the call", wmax, pb);
    g.makespan = r.makespan;
    g.finish = r.finish;
    g.peak = r.peak;
    g.cand_peak = r.cand_peak;
    g.n_ops = r.n_ops;
    g.walked = r.walked_ops;
    g.status = r.status;
    g.c = ParConsts{c.inv_f, c.inv_b, c.inv_l, c.lat, c.launch, c.cap, c.mm, c.mm_c0, c.mm_c1, c.mm_c2,
                    c.mm_c3, c.mm_floor, c.node, c.net_lat, c.net_inv_l, c.streams, c.st_lat, c.st_inv_l};

    const bool rc = m.mode != DSIM_INFER && m.recompute != 0;
    const bool zr = m.mode != DSIM_INFER && m.zero != 0;
    const bool ov = m.mode != DSIM_INFER && m.overlap != 0;
    const bool tf = m.family == DSIM_TRANSFORMER;
    g.perm = g.meta = g.order = nullptr;
    g.wave0 = 0;
    hipError_t e = hipSuccess;
    if (n_cand <= kAloneCand) {
        launch_kernel(rc, zr, ov, tf, dim3((unsigned)n_cand), s, g);
        e = hipGetLastError();
        return e == hipSuccess ? DSIM_OK : hip_fail(e, "parametric launch");
    }

    // workspace: per-block class counts, class table, permutation, the
    // wavefronts' order and lengths (every word is written before it is read:
    // the caller clears nothing)
    const bool narrow = pb <= kNarrowStages / 2 || n_cand >= kNarrowCall || (pb <= kNarrowStages && n_cand >= kEightMin);
    const int64_t nb = (n_cand + kScanBlock - 1) / kScanBlock;
    uint32_t *counts = static_cast<uint32_t *>(ws);
    uint32_t *meta = counts + (size_t)nb * 8;
    uint32_t *perm = meta + 32;
    uint32_t *order = perm + n_cand;
    uint32_t *wave_len = order + n_cand + 8;
    g.perm = perm;
    g.order = order;
    g.meta = meta;
    const bool train = m.mode != DSIM_INFER;
    const bool all_narrow = pb <= kNarrowStages / 2 && n_cand >= kNarrowAll;
    hipLaunchKernelGGL(k_class_count, dim3((unsigned)nb), dim3(kScanBlock), 0, s, cand, n_cand, pb, narrow, counts, wave_len);
    hipLaunchKernelGGL(k_class_scan, dim3(1), dim3(kLanes * (kClasses + 1)), 0, s, counts, nb, meta, tf, train);
    hipLaunchKernelGGL(k_class_scatter, dim3((unsigned)nb), dim3(kScanBlock), 0, s, cand, n_cand, pb, narrow,
                       (const uint32_t *)counts, (const uint32_t *)meta, perm, m.n_layers, train, wave_len);
    if (!all_narrow)
        hipLaunchKernelGGL(k_wave_order, dim3(1), dim3(kOrderBlock), 0, s, (const uint32_t *)meta,
                           (const uint32_t *)wave_len, order);
    if (narrow) {
        const int64_t waves = ((n_cand << (kNarrow - 1)) + kLanes - 1) / kLanes + kNarrow;
        launch_narrow(rc, zr, ov, tf, (unsigned)(waves < kNarrowBlocks ? waves : kNarrowBlocks), s, g);
        e = hipGetLastError();
        if (e != hipSuccess || all_narrow) return e == hipSuccess ? DSIM_OK : hip_fail(e, "parametric launch");
    }
    // every class rounds up to whole wavefronts: at most one partial
    // wavefront per class beyond n * wmax lanes; one dispatch holds fewer
    // than 2^32 lanes
    if (wmax < (1 << kMinClass)) wmax = 1 << kMinClass;
    const int64_t waves = (n_cand * wmax + kLanes - 1) / kLanes + kClasses;
    constexpr int64_t kMaxWaves = (int64_t)1 << 25;
    for (int64_t w0 = 0; w0 < waves && e == hipSuccess; w0 += kMaxWaves) {
        g.wave0 = (uint32_t)w0;
        launch_kernel(rc, zr, ov, tf, dim3((unsigned)(waves - w0 < kMaxWaves ? waves - w0 : kMaxWaves)), s, g);
        e = hipGetLastError();
    }
    return e == hipSuccess ? DSIM_OK : hip_fail(e, "parametric launch");
}

}  // namespace dsim
