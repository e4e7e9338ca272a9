// materialize.hip -- write the whole distributed program of a strategy as an
// explicit op table.
//
// One wavefront per candidate expands the transform of Sec. 4 for every device
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
constexpr int kItems = kLanes + 2 * kMaxTableDev;   // a slot adds at most two per stage

__global__ __launch_bounds__(kLanes) void k_materialize(const MatArgs g)
{
    __shared__ Item s_item[kItems];
    const int lane = threadIdx.x;
    const int64_t c = g.c0 + (int64_t)blockIdx.x;
    const dsim_strategy st = g.cand[c];
    const int S = g.m.overlap ? 2 : 1;
    const bool ok = strategy_ok(g.m, st.D, st.H, st.P, st.K) && st.K <= kMaxK &&
                    (int64_t)S * st.D * st.H * st.P <= (int64_t)g.n_dev;
    if (!ok) {
        if (lane < g.n_dev) g.init_live[c * g.n_dev + lane] = 0;
        if (lane == 0) {
            g.n_ops[c] = 0;
            g.status[c] = DSIM_ST_BAD_STRATEGY;
        }
        return;
    }
    CostConsts none = {};
    Ctx x = {};
    make_ctx(g.m, none, st, x);
    const int DH = x.D * x.H;
    if (lane < g.n_dev) {
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
    const bool stage = s < x.P;
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
            const int64_t up = __shfl_up(sum, o, kLanes);
            sum += lane >= o ? up : 0;
        }
        total = __shfl(sum, kMaxTableDev - 1, kLanes);
        return sum - v;
    };

    Emit e{x, g, c, 0, false, 0, 0, 0, S};
    // microbatch splits before the pipeline: one lane each
    int64_t at = 0;
    if (x.K > 1) {
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
    bool stuck = false;
    for (bool more = true; more;) {
        // one slot of the schedule
        const bool bwd = nf == x.K || nf - nb > warm;
        const int k = bwd ? nb : nf;
        const int left = __shfl_up(nf, 1, kLanes), right = __shfl_down(nb, 1, kLanes);
        const int avail = bwd ? (s == x.P - 1 ? nf : right) : (s == 0 ? INT32_MAX : left);
        const bool ready = nf + nb < len && avail > k;
        const uint64_t run = __ballot(ready);
        const bool sends = ready && (bwd ? s > 0 : s < x.P - 1);
        const uint64_t out = __ballot(sends), below = (1ull << lane) - 1ull;
        int64_t total;
        const int64_t mine = !ready ? 0 : (!bwd ? n_f : (k == 0 ? n_b0 : (k == x.K - 1 ? n_bl : n_b1)));
        const int64_t ahead = before(mine, total);
        if (ready) s_item[n + __popcll(run & below)] = Item{at + ahead, k, (uint16_t)s, (uint8_t)bwd, 0};
        n += __popcll(run);
        at += total;
        if (sends) {
            const int p = __popcll(out & below);
            s_item[n + p] = Item{at + (int64_t)p * DH, k, (uint16_t)s, (uint8_t)bwd, 1};
        }
        n += __popcll(out);
        at += (int64_t)__popcll(out) * DH;
        if (ready) {
            if (bwd) ++nb;
            else ++nf;
        }
        more = __ballot(nf + nb < len) != 0;
        stuck = more && run == 0;   // no stage can proceed: impossible for these schedules
        more = more && !stuck;
        if (n < kLanes && more) continue;
        // write up to 64 of them
        do {
            __syncthreads();
            const int now = n < kLanes ? n : kLanes;
            if (lane < now) {
                const Item it = s_item[lane];
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
            Item rest;
            const bool moves = lane < n - now;
            if (moves) rest = s_item[now + lane];
            __syncthreads();
            if (moves) s_item[lane] = rest;
            n -= now;
        } while (!more && n > 0);
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
    const bool inexact = __ballot(e.inexact) != 0;
    if (lane == 0) {
        const bool fits = at <= (int64_t)g.max_ops && !inexact;
        g.n_ops[c] = fits && !stuck ? (uint32_t)at : 0u;
        g.status[c] = stuck ? DSIM_ST_BAD_STRATEGY : (fits ? 0 : DSIM_ST_NOT_TABLE);
    }
}

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
    // (one dispatch holds fewer than 2^32 lanes)
    constexpr int64_t kMaxBlocks = (int64_t)1 << 25;
    hipError_t e = hipSuccess;
    for (g.c0 = 0; g.c0 < n_cand && e == hipSuccess; g.c0 += kMaxBlocks) {
        const int64_t blocks = n_cand - g.c0 < kMaxBlocks ? n_cand - g.c0 : kMaxBlocks;
        hipLaunchKernelGGL(k_materialize, dim3((unsigned)blocks), dim3(kLanes), 0, s, g);
        e = hipGetLastError();
    }
    return e == hipSuccess ? DSIM_OK : hip_fail(e, "materialize launch");
}

}  // namespace dsim
