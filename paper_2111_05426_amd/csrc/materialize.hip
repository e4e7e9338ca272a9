// materialize.hip -- write the whole distributed program of a strategy as an
// explicit op table.
//
// One wavefront per candidate, or eight lanes of one in large calls of short
// programs, expands the transform of Sec. 4 for every device
// (device p*(D*H) + d*H + h runs stage p of data replica d, tensor rank h)
// in a program order whose per-device projections are those of the
// transform (Sec. 2.1 semantics depend on nothing else): the splits, then
// slot by slot every ready stage's block (each compute op once per replica
// device, each tensor-parallel all-reduce once per data replica over its H
// ranks) followed by the slot's Sends in ascending source order (one per
// replica), then every stage's weight update (each gradient all-reduce once
// per tensor rank over the D replicas, each optimizer op once per device).
// With ZeRO (Fig. 9) a weight read is preceded by a broadcast record from
// its owner per tensor rank, the reading op also frees the copy on the other
// replicas, and each gradient all-reduce becomes a reduce record onto the
// owner followed by the owner's optimizer op.  With overlap every GPU g is
// two devices, 2g computing and 2g + 1 communicating: the last backward
// block hands each finished gradient over (a Send of zero alloc and free
// per replica, then an all-reduce over the communication streams per tensor
// rank), and the weight update hands each one back before its optimizer op.
// The records go to the op-major, candidate-fastest table layout that
// dsim_simulate_tables reads.
//
// A block's records depend on its stage, direction and microbatch alone, and
// their number on even less, so the wavefront first walks the schedule (a
// lane per stage) to find where each block and Send starts, and then its
// lanes write 64 of them at a time, one each.  What bounds it is one block's
// chain of records in a lane: the 30 strategies of the tiny MLP, up to 440
// records each, took 444 us with a lane writing a whole program, 40 now; 888
// MLP strategies of up to 25,552 records 11.8 -> 0.75 ms.
#include "model.h"

namespace dsim {
namespace {

constexpr int kLanes = 64;
struct MatArgs {
    dsim_model m;
    const dsim_strategy *cand;
    int64_t n_cand;
    int32_t max_ops;
    int32_t n_dev;
    uint32_t *code;
    float *flops;
    float *bytes;
    uint32_t *alloc;
    uint32_t *freeb;
    uint32_t *mm_k;     // may be NULL
    uint32_t *n_ops;
    uint64_t *init_live;
    int32_t *status;
    int64_t c0;         // the launch's first candidate
};

// How many records a stage's ops make.
struct RecordCount {
    const Ctx &x;
    int64_t n;

    __device__ __forceinline__ void local(uint64_t, uint64_t, uint64_t, uint64_t) { n += x.D * x.H; }
    __device__ __forceinline__ void mm(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t) { n += x.D * x.H; }
    __device__ __forceinline__ void ar_tp(uint64_t) { n += x.H > 1 ? x.D : 0; }
    __device__ __forceinline__ void ar_dp(uint64_t) { n += x.D > 1 ? x.H : 0; }
    __device__ __forceinline__ void bcast(uint64_t, int) { n += x.zero ? x.H : 0; }
    __device__ __forceinline__ void reduce(uint64_t, int) { n += x.H; }
    __device__ __forceinline__ void owner_local(uint64_t, uint64_t, uint64_t, uint64_t, int) { n += x.H; }
    __device__ __forceinline__ void handover(uint64_t) { n += x.D * x.H + x.H; }
    __device__ __forceinline__ void handback(uint64_t) { n += x.D * x.H; }
};

// Appends records for one stage's ops on every replica device.
struct Emit {
    const Ctx &x;
    const MatArgs &g;
    int64_t c;
    int64_t j;          // records emitted so far (may pass max_ops: counted, not written)
    bool inexact;       // a value does not fit the record format exactly
    int base;           // first GPU of the stage
    uint64_t pend;      // ZeRO: bytes of the broadcast copy the next op frees on non-owners
    int pend_owner;     // ZeRO: the replica that owns it
    int S;              // devices per GPU: 1, or 2 with overlap

    // the computation device of GPU gpu (its communication stream is the next one)
    __device__ __forceinline__ uint32_t dv(int gpu) const { return (uint32_t)(S * gpu); }

    __device__ __forceinline__ void put(uint32_t code, uint64_t fl, uint64_t by, uint64_t al, uint64_t fr,
                                        uint64_t k = 0)
    {
        // flops and bytes must be exact in fp32, alloc, free and the
        // reduction length in u32
        const float ff = (float)fl, fb = (float)by;
        inexact |= fl >= (1ull << 62) || by >= (1ull << 62) || (uint64_t)ff != fl || (uint64_t)fb != by ||
                   al > 0xffffffffull || fr > 0xffffffffull || k > 0xffffffffull;
        if (j < (int64_t)g.max_ops) {
            const size_t o = (size_t)j * (size_t)g.n_cand + (size_t)c;
            g.code[o] = code;
            g.flops[o] = ff;
            g.bytes[o] = fb;
            g.alloc[o] = (uint32_t)al;
            g.freeb[o] = (uint32_t)fr;
            if (g.mm_k) g.mm_k[o] = (uint32_t)k;
        }
        ++j;
    }
    __device__ __forceinline__ void compute(uint32_t cls, uint64_t fl, uint64_t by, uint64_t al, uint64_t fr, uint64_t k)
    {
        for (int r = 0; r < x.D * x.H; ++r) {
            const uint64_t copy = (pend != 0 && r / x.H != pend_owner) ? pend : 0;
            put((dv(base + r) << 8) | (cls << 24), fl, by, al, fr + copy, k);
        }
        pend = 0;
    }
    __device__ __forceinline__ void local(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr) { compute(0u, fl, by, al, fr, 0); }
    // a matrix multiplication of reduction length k: cost class 1 of the
    // table format
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr, uint64_t k)
    {
        compute(1u, fl, by, al, fr, k);
    }
    // ZeRO: the owner's broadcast over the D replicas of each tensor rank
    // (kind 3, root = the owner: the others allocate their copy)
    __device__ __forceinline__ void bcast(uint64_t by, int grp)
    {
        if (!x.zero) return;
        const int o = grp % x.D;
        for (int h = 0; h < x.H; ++h)
            put(3u | (dv(base + o * x.H + h) << 8) | (dp_mask(h) << 16), 0, by, by, 0);
        pend = by;
        pend_owner = o;
    }
    // ZeRO: reduce onto the owner (kind 4: the owner allocates the reduced
    // gradient, every member frees its own)
    __device__ __forceinline__ void reduce(uint64_t by, int grp)
    {
        const int o = grp % x.D;
        for (int h = 0; h < x.H; ++h)
            put(4u | (dv(base + o * x.H + h) << 8) | (dp_mask(h) << 16), 0, by, by, by);
    }
    __device__ __forceinline__ void owner_local(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr, int grp)
    {
        const int o = grp % x.D;
        for (int h = 0; h < x.H; ++h) put(dv(base + o * x.H + h) << 8, fl, by, al, fr);
    }
    // the D replicas of tensor rank h on this stage (stream 0: computation,
    // 1: communication)
    __device__ __forceinline__ uint32_t dp_mask(int h, int stream = 0) const
    {
        uint32_t mask = 0;
        for (int d = 0; d < x.D; ++d) mask |= 1u << (dv(base + d * x.H + h) + (uint32_t)stream);
        return mask;
    }
    __device__ __forceinline__ void ar_tp(uint64_t by)
    {
        if (x.H <= 1) return;
        for (int d = 0; d < x.D; ++d) {
            uint32_t mask = 0;
            for (int h = 0; h < x.H; ++h) mask |= 1u << dv(base + d * x.H + h);
            put(2u | (mask << 16), 0, by, 0, 0);
        }
    }
    __device__ __forceinline__ void ar_dp(uint64_t by)
    {
        if (x.D <= 1) return;
        for (int h = 0; h < x.H; ++h) put(2u | (dp_mask(h) << 16), 0, by, 0, 0);
    }
    __device__ __forceinline__ void send(int t, uint64_t sz, uint64_t fre)
    {
        const int tbase = t * x.D * x.H;
        for (int r = 0; r < x.D * x.H; ++r)
            put(1u | (dv(base + r) << 8) | (dv(tbase + r) << 16), 0, sz, sz, fre);
    }
    // overlap: each replica hands the finished gradient to its communication
    // stream (nothing allocated or freed), whose D replicas all-reduce it
    __device__ __forceinline__ void handover(uint64_t by)
    {
        for (int r = 0; r < x.D * x.H; ++r) put(1u | (dv(base + r) << 8) | ((dv(base + r) + 1u) << 16), 0, by, 0, 0);
        for (int h = 0; h < x.H; ++h) put(2u | (dp_mask(h, 1) << 16), 0, by, 0, 0);
    }
    // overlap: the reduced gradient comes back to the computation stream
    __device__ __forceinline__ void handback(uint64_t by)
    {
        for (int r = 0; r < x.D * x.H; ++r) put(1u | ((dv(base + r) + 1u) << 8) | (dv(base + r) << 16), 0, by, 0, 0);
    }
};

// A block or Send of the schedule and its first record.
struct Item {
    int64_t at;
    int32_t k;
    uint16_t s;
    uint8_t bwd, send;
};

// G lanes per candidate; kLanes / G neighbouring candidates share a wavefront.
template <int G> __global__ __launch_bounds__(kLanes) void k_materialize(const MatArgs g)
{
    static_assert(G >= kMaxTableDev && kLanes % G == 0, "a lane for every stage");
    constexpr int kPer = kLanes / G;
    constexpr int kItems = G + 2 * kMaxTableDev;        // a slot adds at most two per stage
    __shared__ Item s_item[kPer][kItems];
    const int lane = threadIdx.x % G, sub = G == kLanes ? 0 : threadIdx.x / G;
    // Workgroups go round the XCDs in turn: 32 neighbouring candidates, whose
    // records share cache lines, on one XCD, so that its L2 puts their words
    // together (64,000 MLP strategies of 465 records on average: 3.7 -> 1.8 ms)
    constexpr uint32_t kNear = 32 / kPer, kTurn = 8 * kNear;
    uint32_t b = blockIdx.x;
    if (b < gridDim.x / kTurn * kTurn) b = b / kTurn * kTurn + b % 8 * kNear + b / 8 % kNear;
    const int64_t c = g.c0 + (int64_t)b * kPer + sub;
    dsim_strategy st = {1, 1, 1, 1};
    if (c < g.n_cand) st = g.cand[c];
    const int S = g.m.overlap ? 2 : 1;
    const bool ok = c < g.n_cand && strategy_ok(g.m, st.D, st.H, st.P, st.K) && st.K <= kMaxK &&
                    (int64_t)S * st.D * st.H * st.P <= (int64_t)g.n_dev;
    if (c < g.n_cand && !ok) {
        if (lane < g.n_dev) g.init_live[c * g.n_dev + lane] = 0;
        if (lane == 0) {
            g.n_ops[c] = 0;
            g.status[c] = DSIM_ST_BAD_STRATEGY;
        }
    }
    if (!ok) {
        if (G == kLanes) return;
        st = dsim_strategy{1, 1, 1, 1};   // (takes part in the wavefront's loops with no stage)
    }
    CostConsts none = {};
    Ctx x = {};
    make_ctx(g.m, none, st, x);
    const int DH = x.D * x.H;
    if (ok && lane < g.n_dev) {
        // a communication stream, and a device beyond the program's, holds nothing
        const int gpu = lane / S, s = gpu / DH;
        uint64_t r0 = 0;
        if (lane % S == 0 && s < x.P) {
            if (x.zero) {
                // each data replica holds the groups it owns
                ZStage zs;
                z_stage(x, s, zs);
                r0 = resident_inputs(x, s) + z_owned(x, zs, (gpu % DH) / x.H);
            } else {
                r0 = resident(x, s);
            }
        }
        g.init_live[c * g.n_dev + lane] = r0;
    }

    // records of this lane's stage: a forward block, the backward blocks of
    // microbatch 0, of the last one and of the others, the weight update
    const int s = lane;
    const bool stage = ok && s < x.P;
    int64_t n_f = 0, n_b0 = 0, n_b1 = 0, n_bl = 0, n_wu = 0;
    if (stage) {
        RecordCount f{x, 0}, b0{x, 0}, b1{x, 0}, bl{x, 0}, w{x, 0};
        block_fwd(x, f, s, 0);
        n_f = f.n;
        if (x.train) {
            block_bwd(x, b0, s, 0);
            if (x.K > 1) block_bwd(x, bl, s, x.K - 1);
            if (x.K > 2) block_bwd(x, b1, s, 1);
            weight_update(x, w, s);
            n_b0 = b0.n;
            n_b1 = b1.n;
            n_bl = bl.n;
            n_wu = w.n;
        }
    }
    // exclusive prefix sum over the stages' lanes, and their total
    auto before = [&](int64_t v, int64_t &total) {
        int64_t sum = v;
        for (int o = 1; o < kMaxTableDev; o <<= 1) {
            const int64_t up = __shfl_up(sum, o, G);
            sum += lane >= o ? up : 0;
        }
        total = __shfl(sum, kMaxTableDev - 1, G);
        return sum - v;
    };
    // whether any candidate of the wavefront is in p (the same for all lanes
    // of one), and the candidate's lanes for which p holds
    auto any = [](bool p) { return G == kLanes ? p : __ballot(p) != 0; };
    auto lanes = [&](bool p) { return (uint64_t)__ballot(p) >> (sub * G) & (~0ull >> (64 - G)); };

    Emit e{x, g, c, 0, false, 0, 0, 0, S};
    // microbatch splits before the pipeline: one lane each
    int64_t at = 0;
    if (ok && x.K > 1) {
        if (lane == 0) {
            split(x, e);
        } else if (lane == 1 && x.train) {
            e.j = DH;
            e.base = (x.P - 1) * DH;
            split(x, e);
        }
        at = x.train ? 2 * DH : DH;
    }

    const int len = stage ? (x.train ? 2 * x.K : x.K) : 0;
    // forwards before the first backward (synchronous 1F1B; all otherwise)
    const int warm = (x.train && x.schedule != DSIM_SCHED_GPIPE && x.P - 1 - s < x.K) ? x.P - 1 - s : x.K;
    int nf = 0, nb = 0, n = 0;
    bool stuck = false, more = ok;
    // (the loops' conditions are the wavefront's: a candidate that has ended
    // takes part with no stage ready and nothing to write)
    while (any(more)) {
        // one slot of the schedule
        const bool bwd = nf == x.K || nf - nb > warm;
        const int k = bwd ? nb : nf;
        const int left = __shfl_up(nf, 1, G), right = __shfl_down(nb, 1, G);
        const int avail = bwd ? (s == x.P - 1 ? nf : right) : (s == 0 ? INT32_MAX : left);
        const bool ready = nf + nb < len && avail > k;
        const uint64_t run = lanes(ready);
        const bool sends = ready && (bwd ? s > 0 : s < x.P - 1);
        const uint64_t out = lanes(sends), below = (1ull << lane) - 1ull;
        int64_t total;
        const int64_t mine = !ready ? 0 : (!bwd ? n_f : (k == 0 ? n_b0 : (k == x.K - 1 ? n_bl : n_b1)));
        const int64_t ahead = before(mine, total);
        if (ready) s_item[sub][n + __popcll(run & below)] = Item{at + ahead, k, (uint16_t)s, (uint8_t)bwd, 0};
        n += __popcll(run);
        at += total;
        if (sends) {
            const int p = __popcll(out & below);
            s_item[sub][n + p] = Item{at + (int64_t)p * DH, k, (uint16_t)s, (uint8_t)bwd, 1};
        }
        n += __popcll(out);
        at += (int64_t)__popcll(out) * DH;
        if (ready) {
            if (bwd) ++nb;
            else ++nf;
        }
        const bool rest_of_it = more && lanes(nf + nb < len) != 0;
        stuck = stuck || (rest_of_it && run == 0);   // no stage can proceed: impossible for these schedules
        more = rest_of_it && !stuck;
        // write up to G of each candidate's, once one has so many or has ended
        while (any(n >= G || (!more && n > 0))) {
            __syncthreads();
            const int now = n < G ? n : G;
            if (lane < now) {
                const Item it = s_item[sub][lane];
                if (it.at < (int64_t)g.max_ops) {   // (beyond, the program does not fit anyway)
                    e.j = it.at;
                    e.base = it.s * DH;
                    e.pend = 0;
                    if (it.send) {
                        uint64_t sz, fre;
                        send_size(x, it.s, mb_rows(x, it.k), it.bwd != 0, sz, fre);
                        e.send(it.bwd ? it.s - 1 : it.s + 1, sz, fre);
                    } else if (it.bwd) {
                        block_bwd(x, e, it.s, it.k);
                    } else {
                        block_fwd(x, e, it.s, it.k);
                    }
                }
            }
            __syncthreads();
            // (what is left moves to the front, up to G at a time)
            for (int m0 = 0; m0 < kItems - G; m0 += G) {
                const int m = m0 + lane;
                Item rest;
                const bool moves = m < n - now;
                if (moves) rest = s_item[sub][now + m];
                __syncthreads();
                if (moves) s_item[sub][m] = rest;
            }
            n -= now;
        }
    }
    int64_t total;
    const int64_t ahead = before(n_wu, total);
    if (stage && x.train) {
        e.j = at + ahead;
        e.base = s * DH;
        e.pend = 0;
        weight_update(x, e, s);
    }
    at += total;
    const bool inexact = lanes(e.inexact) != 0;
    if (ok && lane == 0) {
        const bool fits = at <= (int64_t)g.max_ops && !inexact;
        g.n_ops[c] = fits && !stuck ? (uint32_t)at : 0u;
        g.status[c] = stuck ? DSIM_ST_BAD_STRATEGY : (fits ? 0 : DSIM_ST_NOT_TABLE);
    }
}

// Tables of at most kGroupOps rows for more than kGroupCand candidates take
// eight lanes each: the lanes of a wavefront of its own would mostly idle,
// there are more than enough wavefronts, and eight neighbours' words of a
// record are written together.  Programs of 146 records on average (440 rows),
// us, 64 lanes against eight: 4,000 candidates 95 / 107, 8,000 149 / 108,
// 16,000 253 / 185, 64,000 920 / 700; 64,000 equal ones of 60 records 739 /
// 122.  With longer ones an eight-lane chain is too long, and the candidates
// of a wavefront wait for each other: 290 on average (1,160 rows), 16,000
// candidates 258 / 330, 64,000 897 / 1,250.
constexpr int kGroup = 8;
constexpr int32_t kGroupOps = 512;
constexpr int64_t kGroupCand = 8192;

}  // namespace

dsim_status launch_materialize(const dsim_model &m, const dsim_strategy *cand, int64_t n_cand, int32_t max_ops,
                               int32_t n_dev, uint32_t *code, float *flops, float *bytes, uint32_t *alloc,
                               uint32_t *freeb, uint32_t *mm_k, uint32_t *n_ops, uint64_t *init_live,
                               int32_t *status, hipStream_t s)
{
    MatArgs g;
    g.m = m;
    g.cand = cand;
    g.n_cand = n_cand;
    g.max_ops = max_ops;
    g.n_dev = n_dev;
    g.code = code;
    g.flops = flops;
    g.bytes = bytes;
    g.alloc = alloc;
    g.freeb = freeb;
    g.mm_k = mm_k;
    g.n_ops = n_ops;
    g.init_live = init_live;
    g.status = status;
    const bool group = max_ops <= kGroupOps && n_cand > kGroupCand;
    const int64_t per = group ? kLanes / kGroup : 1;
    // (one dispatch holds fewer than 2^32 lanes)
    constexpr int64_t kMaxBlocks = (int64_t)1 << 25;
    hipError_t e = hipSuccess;
    for (g.c0 = 0; g.c0 < n_cand && e == hipSuccess; g.c0 += kMaxBlocks * per) {
        const int64_t want = (n_cand - g.c0 + per - 1) / per;
        const dim3 blocks((unsigned)(want < kMaxBlocks ? want : kMaxBlocks));
        if (group) hipLaunchKernelGGL(k_materialize<kGroup>, blocks, dim3(kLanes), 0, s, g);
        else hipLaunchKernelGGL(k_materialize<kLanes>, blocks, dim3(kLanes), 0, s, g);
        e = hipGetLastError();
    }
    return e == hipSuccess ? DSIM_OK : hip_fail(e, "materialize launch");
}

}  // namespace dsim
