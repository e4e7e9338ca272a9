// parametric.h -- simulate the D/H/P/K transform without building op lists: the
// body of the kernels in parametric.hip and parametric_narrow.hip.
//
// Each candidate gets a segment of W = 16, 32 or 64 lanes of a wavefront (the
// least that holds its P stages), one lane per pipeline stage; segments of
// equal width share wavefronts (64 / W candidates each), in a small call
// every candidate has a wavefront of its own, and in a large one candidates
// of few stages take the narrow kernel, W = 1, 2, 4 or 8.  A lane expands, on
// the fly and in program order,
// the ops of its stage of the distributed program the transform of Sec. 4
// produces (ops in model.h) and simulates them with the semantics of Sec. 2.1
// and the cost model of Sec. 3.3:
//   * synchronous 1F1B or GPipe (training), forward-only (inference) per
//     stage;
//   * the global order is slot by slot: every stage runs its next block if
//     the block's input was produced in an earlier slot (the stages of a slot
//     touch disjoint devices, so they run in parallel lanes); then the slot's
//     Sends run in ascending order of source stage, a serial chain of
//     max-plus steps across neighbouring lanes (DPP wave shifts); the weight
//     update follows the last slot;
//   * every replica (d, h) of a stage runs the same ops at the same times, so
//     one replica per stage is walked: a collective over the H ranks or the
//     D replicas starts at the stage's own clock and costs the ring
//     all-reduce of its full group; a Send synchronises two stage clocks.
//   * with ZeRO (Fig. 9) the replicas still run the same ops at the same
//     times, except that only a parameter's owner runs its optimizer op; the
//     next gradient reduce waits for it, so the stage's latest device finishes
//     at the lane's clock.  Their memory differs: each holds only the groups
//     it owns and a copy of every other weight while an op reads it.  The
//     lane tracks the live bytes that do not depend on ownership plus the
//     largest owned resident, and each block kind's highest point is taken
//     as the maximum over the replicas in closed form (see zero_top).
//
// The layers of a stage repeat one op sequence (for the MLP with H > 1, one
// column/row layer pair) that does not depend on the stage, so the lanes of a
// segment record a candidate's programs once, together: the op costs of that
// unit and of the edges (embedding, LM head, loss, the MLP's first unit in
// backward) for every kind of block -- forward, backward without and with
// gradient accumulation, each for the two microbatch sizes -- and every
// block's memory (net bytes, highest point).  A block is then one addition:
// inside one binade of the clock, rounding to nearest adds each cost as a
// whole number of ulps, so the block adds a tabulated whole number (built by
// the wavefront when a candidate's clocks enter a binade).  A block that
// leaves the binade, and one whose costs include an exact half ulp, is walked
// cost by cost; adding the same costs in the same order gives the same
// rounding either way, and the memory is exact integer arithmetic.
//
// Recording a candidate's programs and tables takes a wavefront some
// thousand instructions however few stages there are, and more candidates in
// a wavefront do not share them: 100,000 MLP strategies of one stage and up to
// 64 microbatches took 582 us at 16 lanes each, 539 at 8, 839 at 4.  So in
// the narrow kernel every lane records its own block of each direction, again
// whenever its kind changes, and sums it binade-wise by itself: 84 us.
//
// A counting-sort pre-pass groups the candidates by segment width into a
// temporary permutation (stable, so the grid's own order keeps wavefronts
// uniform in K); a small grid needs none, each candidate has a wavefront.
#pragma once

#include <type_traits>

#include "model.h"

namespace dsim {

// the device-model constants the transform reads (the table format's
// per-group-size rows stay out of the kernel arguments)
struct ParConsts {
    double inv_f, inv_b, inv_l, lat, launch;
    uint64_t cap;
    int32_t mm;
    double mm_c0, mm_c1, mm_c2, mm_c3, mm_floor;
    int32_t node;
    double net_lat, net_inv_l;
    int32_t streams;
    double st_lat, st_inv_l;
};

struct ParArgs {
    dsim_model m;
    const dsim_strategy *cand;
    int32_t row_width;
    int32_t p_bound;
    const uint32_t *perm;   // candidates grouped by segment class; NULL: one candidate per wavefront, in order
    const uint32_t *meta;   // [0,8) class totals, [8,16) first perm index, [16,24) first wavefront,
                            // [24,29) first wavefront of the narrow launch, by class, and their number;
                            // [29] first perm index of class kMinClass without the narrow ones that join it
    const uint32_t *order;  // the wavefronts, longest first
    uint32_t wave0;         // the launch's first entry of order
    double *makespan;
    double *finish;
    uint64_t *peak;
    uint64_t *cand_peak;
    uint64_t *n_ops;
    uint64_t *walked;
    int32_t *status;
    ParConsts c;
};

// the narrow launch (parametric_narrow.hip)
void launch_narrow(bool rc, bool zr, bool ov, bool tf, unsigned blocks, hipStream_t s, const ParArgs &g);

namespace {

constexpr int kLanes = 64;
constexpr int kClasses = 7;       // segment widths 1, 2, 4, ..., 64

// Recorded block program of one lane and direction, in double2 entries:
// ops before the repeating units, one unit, ops after the units.  The
// regions are sized for the larger (backward) block; forward blocks use the
// F_* prefix of each region.
template <bool TF, bool Z> struct Shape;
template <> struct Shape<true, false> {
    static constexpr int PRE2 = 4;    // last stage backward: loss .. final LN grad (8 ops)
    static constexpr int U2 = 12;     // one layer backward: 17 compute + 4 accumulations + 2 all-reduces
    static constexpr int SUF2 = 1;    // stage 0 backward: embedding grad + accumulation
    static constexpr int F_PRE2 = 1;  // stage 0 forward: embedding + all-reduce
    static constexpr int F_U2 = 7;    // one layer forward: 12 compute + 2 all-reduces
    static constexpr int F_SUF2 = 1;  // last stage forward: final LN + LM head
};
template <> struct Shape<false, false> {
    static constexpr int PRE2 = 1;    // last stage backward: loss gradient
    static constexpr int U2 = 5;      // row layer (4 ops) + column layer (5) backward
    static constexpr int SUF2 = 5;    // the stage's first unit backward (frees the stage input)
    static constexpr int F_PRE2 = 0;
    static constexpr int F_U2 = 3;    // column layer (2 ops) + row layer (3) forward
    static constexpr int F_SUF2 = 3;  // the model's last unit in inference (dead output)
};
// ZeRO adds one broadcast before every op that reads a weight
template <> struct Shape<true, true> {
    static constexpr int PRE2 = 5;    // 8 ops + 1 broadcast
    static constexpr int U2 = 14;     // 22 ops + 4 broadcasts
    static constexpr int SUF2 = 2;    // the forward suffix is the larger one here
    static constexpr int F_PRE2 = 2;  // 2 ops + 1 broadcast
    static constexpr int F_U2 = 9;    // 14 ops + 4 broadcasts
    static constexpr int F_SUF2 = 2;  // 2 ops + 1 broadcast
};
template <> struct Shape<false, true> {
    static constexpr int PRE2 = 1;
    static constexpr int U2 = 6;      // 9 ops + 2 broadcasts
    static constexpr int SUF2 = 6;    // 9 ops + 2 broadcasts
    static constexpr int F_PRE2 = 0;
    static constexpr int F_U2 = 4;    // 5 ops + 2 broadcasts
    static constexpr int F_SUF2 = 3;  // inference only: no ZeRO
};
// a forward block's regions are prefixes of the backward block's
template <class Sh> constexpr bool shape_nested()
{
    return Sh::F_PRE2 <= Sh::PRE2 && Sh::F_U2 <= Sh::U2 && Sh::F_SUF2 <= Sh::SUF2;
}
static_assert(shape_nested<Shape<true, false>>() && shape_nested<Shape<false, false>>() &&
                  shape_nested<Shape<true, true>>() && shape_nested<Shape<false, true>>(),
              "forward regions must fit the backward ones");

// A grid shares wavefronts between segments of at least 16 lanes: what a
// candidate makes the whole wavefront do (tables for a binade its clocks
// enter, a phase that cannot skip) more of them would not share.  A million
// strategies of up to eight stages and 64 microbatches, ms, at least 4, 8 or 16
// lanes each: MLP 9.0 / 5.3 / 6.2, transformer 12.8 / 7.9 / 7.4; the
// GPT-3-shaped grid is bound by its deep pipelines.
constexpr int kMinClass = 4;
constexpr int kMaxSeg = kLanes >> kMinClass;
// Classes of the narrow launch: segments of 1, 2 and 4 lanes, and of 8 for at
// most kShortK microbatches.
constexpr int kNarrow = 4;
constexpr int kShortK = 8;
static_assert(kNarrow <= kMinClass, "the narrow launch's segments are narrower");

// narrow: the call may have a narrow launch (see narrow_min)
__device__ __forceinline__ int seg_class(const dsim_strategy &st, int p_bound, bool narrow)
{
    const int P = st.P;
    if (P < 1 || P > p_bound) return narrow ? 0 : kMinClass;
    int j = narrow ? 0 : kMinClass;
    while ((1 << j) < P) ++j;
    return j < kNarrow - 1 || (j < kNarrow && st.K <= kShortK) || j > kMinClass ? j : kMinClass;
}

// ---------------------------------------------------------------------------
// Sinks
// ---------------------------------------------------------------------------
// Records ops' costs into a region of LDS.
struct Record {
    const Ctx &x;
    double *base;
    int n;

    __device__ __forceinline__ void put(double c) { base[n++] = c; }
    __device__ __forceinline__ void pad(int entries)
    {
        while (n < entries) put(0.0);   // clock + 0.0 == clock
    }
    __device__ __forceinline__ void local(uint64_t fl, uint64_t by, uint64_t, uint64_t) { put(cost_local(x, fl, by)); }
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t, uint64_t, uint64_t k)
    {
        put(cost_mm(x, fl, by, k));
    }
    __device__ __forceinline__ void ar_tp(uint64_t by)
    {
        if (x.H <= 1) return;
        put(cost_ar_tp(x, by));
    }
    __device__ __forceinline__ void bcast(uint64_t by, int)
    {
        if (!x.zero) return;
        put(cost_chain_d(x, by));
    }
    // hand-overs are marked beside the program (Marks)
    __device__ __forceinline__ void handover(uint64_t) {}
};

// A hand-over in a recorded program: before entry `pos`, both streams meet
// and take `send`, then the communication stream's all-reduce takes `ar`.
struct Mark {
    int pos;
    double send, ar;
};
// Where the edges' programs of the last backward block hand gradients over.
struct Marks {
    const Ctx &x;
    Mark *at;
    int n;   // entries so far

    __device__ __forceinline__ void local(uint64_t, uint64_t, uint64_t, uint64_t) { ++n; }
    __device__ __forceinline__ void mm(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t) { ++n; }
    __device__ __forceinline__ void ar_tp(uint64_t)
    {
        if (x.H > 1) ++n;
    }
    __device__ __forceinline__ void bcast(uint64_t, int) {}   // no ZeRO under overlap
    __device__ __forceinline__ void handover(uint64_t by)
    {
        at->pos = n;
        at->send = cost_stream(x, by);
        at->ar = cost_ar_dp(x, by);
    }
};

// The repeating unit of an overlapped last backward block, padded with zero
// costs so that its hand-overs come before fixed entries whether or not it
// accumulates or all-reduces (the transformer's four weight gradients; the
// MLP layer's, or the row and the column layer's).
template <bool TF> struct OvUnit {
    static constexpr int kMarks = TF ? 4 : 2, kEntries = TF ? 22 : 9;
    static constexpr int pos(int i) { return TF ? (i == 0 ? 3 : (i == 1 ? 8 : (i == 2 ? 13 : 20))) : (i == 0 ? 3 : 7); }
    double cost[kEntries];
    double send[kMarks], ar[kMarks];   // send < 0: no such hand-over
};
template <bool TF> struct RecordOv {
    const Ctx &x;
    OvUnit<TF> &u;
    int n, k;   // entries and hand-overs so far

    __device__ __forceinline__ void put(double c) { u.cost[n++] = c; }
    __device__ __forceinline__ void local(uint64_t fl, uint64_t by, uint64_t, uint64_t) { put(cost_local(x, fl, by)); }
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t, uint64_t, uint64_t r)
    {
        put(cost_mm(x, fl, by, r));
    }
    __device__ __forceinline__ void ar_tp(uint64_t by) { put(x.H > 1 ? cost_ar_tp(x, by) : 0.0); }
    __device__ __forceinline__ void bcast(uint64_t, int) {}   // no ZeRO under overlap
    __device__ __forceinline__ void handover(uint64_t by)
    {
        while (n < OvUnit<TF>::pos(k)) put(0.0);
        u.send[k] = cost_stream(x, by);
        u.ar[k] = cost_ar_dp(x, by);
        ++k;
    }
    __device__ __forceinline__ void pad()
    {
        while (n < OvUnit<TF>::kEntries) put(0.0);
        for (; k < OvUnit<TF>::kMarks; ++k) u.send[k] = -1.0;
    }
};

// Memory summary only (net bytes, peak above the start), no costs.
struct Mem {
    const Ctx &x;
    int64_t cur, top;
    __device__ __forceinline__ void local(uint64_t, uint64_t, uint64_t al, uint64_t fr)
    {
        const int64_t a = cur + (int64_t)al;
        top = a > top ? a : top;
        cur = a - (int64_t)fr;
    }
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr, uint64_t)
    {
        local(fl, by, al, fr);
    }
    __device__ __forceinline__ void ar_tp(uint64_t) {}
    __device__ __forceinline__ void bcast(uint64_t, int) {}
    __device__ __forceinline__ void handover(uint64_t) {}   // allocates nothing
};

// ZeRO memory summary of ops that read the weights of one parameter group:
// net bytes and the highest point above the start, seen by a replica that
// does not own the group (tn: it holds each broadcast copy from the
// broadcast until the op that reads it) and by the owner (to: no copies).
// Copies die inside the summarised ops, so the net is the same for both.
struct MemZ {
    const Ctx &x;
    int64_t cur, tn, to, pend;
    __device__ __forceinline__ void local(uint64_t, uint64_t, uint64_t al, uint64_t fr)
    {
        const int64_t a = cur + (int64_t)al;
        tn = a + pend > tn ? a + pend : tn;
        to = a > to ? a : to;
        cur = a - (int64_t)fr;
        pend = 0;
    }
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr, uint64_t)
    {
        local(fl, by, al, fr);
    }
    __device__ __forceinline__ void ar_tp(uint64_t) {}
    __device__ __forceinline__ void bcast(uint64_t by, int)
    {
        if (!x.zero) return;
        tn = cur + (int64_t)by > tn ? cur + (int64_t)by : tn;
        to = cur > to ? cur : to;
        pend = (int64_t)by;
    }
    __device__ __forceinline__ void handover(uint64_t) {}   // allocates nothing
};

// Liveness of a forward unit.  kFwdBlock: as in a forward block (training
// keeps what the backward reads; inference and recomputation drop it);
// kFwdFirst: the first unit of a forward block under recomputation (its
// input is the checkpoint); kFwdReplay: the backward block's replay, which
// keeps what the backward reads.  Every variant has the same op costs.
enum FwdLive { kFwdBlock = 0, kFwdFirst = 1, kFwdReplay = 2 };

// The repeating unit of a block for microbatches of m rows: one transformer
// layer; one MLP layer (H = 1) or column/row pair (H > 1), in walk order.
// acc: with gradient accumulation (every backward microbatch but the first).
template <bool TF, class S>
__device__ void record_unit(const Ctx &x, bool bwd, uint64_t m, bool acc, S &r, int live = kFwdBlock, bool last = false)
{
    if (TF) {
        const TfSz z = tf_sizes(x, m);
        if (bwd) {
            tf_layer_bwd(x, r, z, acc, 0, last);
        } else {
            const bool save = live == kFwdReplay || (live == kFwdBlock && x.train && !x.rc);
            tf_layer_fwd(x, r, z, save, save || live == kFwdFirst, true, 0);
        }
    } else if (bwd) {
        if (x.H > 1) {
            mlp_layer_bwd(x, r, m, kRow, false, false, acc, 0, last);
            mlp_layer_bwd(x, r, m, kCol, false, false, acc, 0, last);
        } else {
            mlp_layer_bwd(x, r, m, kPlain, false, false, acc, 0, last);
        }
    } else {
        // free_in of the unit's first layer and of its second (pair) layer
        const bool fi_rest = live != kFwdReplay && (!x.train || x.rc);
        const bool fi_first = live == kFwdBlock && fi_rest;
        if (x.H > 1) {
            mlp_layer_fwd(x, r, m, kCol, fi_first, false, 0);
            mlp_layer_fwd(x, r, m, kRow, fi_rest, false, 0);
        } else {
            mlp_layer_fwd(x, r, m, kPlain, fi_first, false, 0);
        }
    }
}

// The replay's last, partial unit: a transformer layer up to its GeLU; the
// column layer of the MLP's last pair (H > 1); nothing for H = 1.  Its ops
// are the first ops of a forward unit, with the same costs.
template <bool TF, class S>
__device__ void record_partial(const Ctx &x, uint64_t m, S &r)
{
    if (TF) tf_layer_fwd(x, r, tf_sizes(x, m), true, true, false, 0);
    else if (x.H > 1) mlp_layer_fwd(x, r, m, kCol, false, false, 0);
}

// The ops of stage s's block before (pre) and after (suf) its repeating
// units: embedding, LM head, loss (transformer); loss, the last unit in
// inference and the stage's first unit in backward (MLP).
template <bool TF, class SP, class SS>
__device__ void record_edges(const Ctx &x, int s, bool bwd, uint64_t m, bool acc, SP &rp, SS &rs)
{
    if (TF) {
        const TfSz z = tf_sizes(x, m);
        if (!bwd) {
            if (s == 0) tf_fwd_first(x, rp, z);
            if (s == x.P - 1) tf_fwd_last(x, rs, z);
        } else {
            if (s == x.P - 1) tf_bwd_last(x, rp, z, acc);
            if (s == 0) tf_bwd_first(x, rs, z, acc);
        }
        return;
    }
    const int per = x.H > 1 ? 2 : 1, l0 = stage_l0(x, s), nl = stage_nl(x, s);
    if (!bwd) {
        if (!x.train && s == x.P - 1)
            for (int i = l0 + nl - per; i < l0 + nl; ++i)
                mlp_layer_fwd(x, rs, m, mlp_kind(x, i), true, i == x.L - 1, 0);
    } else {
        if (s == x.P - 1) mlp_loss(x, rp, m);
        for (int i = l0 + per - 1; i >= l0; --i) mlp_layer_bwd(x, rs, m, mlp_kind(x, i), i == l0, i == 0, acc, 0);
    }
}

// memory effect of pre, n units, suf: unit u starts at pre's net + u * ud;
// top >= 0 is enough (the running peak is never below the live bytes)
__device__ __forceinline__ void compose(int64_t pd, int64_t pt, int64_t ud, int64_t ut, int n, int64_t sd,
                                        int64_t st, int64_t &delta, int64_t &top)
{
    int64_t cur = pd, t = pt;
    if (n > 0) {
        const int64_t hi = cur + ut + (ud > 0 ? (int64_t)(n - 1) * ud : 0);
        t = hi > t ? hi : t;
        cur += (int64_t)n * ud;
    }
    t = cur + st > t ? cur + st : t;
    delta = cur + sd;
    top = t;
}

// appends a summary (d2, t2) to (delta, top)
__device__ __forceinline__ void chain(int64_t &delta, int64_t &top, int64_t d2, int64_t t2)
{
    const int64_t t = delta + t2;
    top = t > top ? t : top;
    delta += d2;
}

// pre, a first unit with its own summary, n - 1 units, suf (n >= 1)
__device__ __forceinline__ void compose_first(int64_t pd, int64_t pt, int64_t fd, int64_t ft, int64_t ud, int64_t ut,
                                              int n, int64_t sd, int64_t st, int64_t &delta, int64_t &top)
{
    int64_t d = pd, t = pt;
    chain(d, t, fd, ft);
    compose(d, t, ud, ut, n - 1, sd, st, delta, top);
}

// Units walked per block: every layer (transformer); every layer or layer
// pair (MLP) except the last unit in inference (last stage) and the
// stage's first unit in backward, which the block records separately.
__device__ __forceinline__ int block_units(const Ctx &x, int s, bool bwd, bool TF)
{
    const int nl = stage_nl(x, s);
    if (TF) return nl;
    const int per = x.H > 1 ? 2 : 1;
    if (bwd) return nl / per - 1;
    return nl / per - ((!x.train && s == x.P - 1) ? 1 : 0);
}

// Counts ops (walked and program ops) without simulating them.
struct Count {
    const Ctx &x;
    uint64_t walked, nops;
    __device__ __forceinline__ void local(uint64_t, uint64_t, uint64_t, uint64_t)
    {
        walked += 1;
        nops += x.mult_dev;
    }
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr, uint64_t)
    {
        local(fl, by, al, fr);
    }
    __device__ __forceinline__ void ar_tp(uint64_t)
    {
        if (x.H <= 1) return;
        walked += 1;
        nops += x.mult_tp;
    }
    // ZeRO collectives: one per tensor rank
    __device__ __forceinline__ void bcast(uint64_t, int)
    {
        if (!x.zero) return;
        walked += 1;
        nops += x.mult_dp;
    }
    __device__ __forceinline__ void handover(uint64_t) {}
    __device__ __forceinline__ void add(uint64_t n, const Count &c)
    {
        walked += n * c.walked;
        nops += n * c.nops;
    }
};

// Ops of stage s of one replica: splits, K forward blocks, in training K
// backward blocks (all but the first with gradient accumulation; the last
// one hands the gradients over under overlap), the Sends after them and the
// weight update.  Op counts do not depend on the microbatch size, and a
// block's layers all count alike.
template <bool TF>
__device__ __forceinline__ void count_stage(const Ctx &x, int s, uint64_t &walked, uint64_t &nops)
{
    const bool first = s == 0, last = s == x.P - 1;
    const int nl = stage_nl(x, s), per = (!TF && x.H > 1) ? 2 : 1;
    const uint64_t K = (uint64_t)x.K, units = (uint64_t)(nl / per);
    const TfSz z = {};
    Count uf{x, 0, 0}, all{x, 0, 0};
    record_unit<TF>(x, false, 1, false, uf);
    Count op{x, 1, x.mult_dev};   // a compute op or a Send
    if (x.K > 1) all.add((first ? 1 : 0) + (x.train && last ? 1 : 0), op);
    Count f{x, 0, 0};
    if (TF && first) tf_fwd_first(x, f, z);
    if (TF && last) tf_fwd_last(x, f, z);
    f.add(units, uf);
    if (!last) f.add(1, op);
    all.add(K, f);
    if (x.train) {
        const uint64_t params = TF ? 4 * (uint64_t)nl + (first ? 1 : 0) + (last ? 1 : 0) : (uint64_t)nl;
        for (int acc = 0; acc < 2; ++acc) {
            Count b{x, 0, 0}, u{x, 0, 0};
            if (last) {
                if (TF) tf_bwd_last(x, b, z, acc != 0);
                else mlp_loss(x, b, 1);
            }
            if (x.rc) {
                b.add(units - 1, uf);
                record_partial<TF>(x, 1, b);
            }
            record_unit<TF>(x, true, 1, acc != 0, u);
            b.add(units, u);
            if (TF && first) tf_bwd_first(x, b, z, acc != 0);
            if (!TF && first && x.H > 1) {   // layer 0's input gradient is not all-reduced
                b.walked -= 1;
                b.nops -= x.mult_tp;
            }
            if (!first) b.add(1, op);
            all.add(acc ? K - 1 : 1, b);
        }
        const Count dp{x, 1, x.mult_dp};   // a collective over the replicas, or an owner's op
        if (x.ov) {
            all.add(2 * params, op);       // hand-over and hand-back
            all.add(params, dp);
            all.add(params, op);
        } else {
            if (x.D > 1) all.add(params, dp);
            all.add(params, x.zero ? dp : op);
        }
    }
    walked = all.walked;
    nops = all.nops;
}

// ---------------------------------------------------------------------------
// ZeRO: one block kind's memory over the D replicas of a stage
// ---------------------------------------------------------------------------
// A run of n equal units (an edge is a run of one): net bytes d per unit,
// highest points tn (a replica that does not own the unit's group) and to
// (its owner) above the unit's start; unit u reads the weights of group
// gs + dir * u (gs < 0: no weight is read).
struct ZSeg {
    int n;
    int64_t d, tn, to;
    int gs, dir;
};

// highest point of a run above its start as replica d sees it (d < 0: a
// replica owning none of the groups).  Unit u starts at u * d; over the
// units a replica owns (u = r mod D) and those it does not, the highest
// start is the last one (d >= 0) or the first one (d < 0).
__device__ __forceinline__ int64_t run_top(const ZSeg &g, int d, int D)
{
    const int n = g.n;
    const int64_t ud = g.d;
    int r = -1;
    if (d >= 0 && g.gs >= 0) {
        r = (g.dir > 0 ? d - g.gs : g.gs - d) % D;
        if (r < 0) r += D;
    }
    int64_t best = INT64_MIN;
    if (ud >= 0) {
        if (r >= 0 && r <= n - 1) {
            const int64_t t = (int64_t)(r + ((n - 1 - r) / D) * D) * ud + g.to;
            best = t > best ? t : best;
        }
        const int un = (r >= 0 && (n - 1) % D == r) ? n - 2 : n - 1;   // D >= 2: n - 2 is not owned
        if (un >= 0) {
            const int64_t t = (int64_t)un * ud + g.tn;
            best = t > best ? t : best;
        }
    } else {
        if (r >= 0 && r <= n - 1) {
            const int64_t t = (int64_t)r * ud + g.to;
            best = t > best ? t : best;
        }
        const int un = r == 0 ? 1 : 0;
        if (un <= n - 1) {
            const int64_t t = (int64_t)un * ud + g.tn;
            best = t > best ? t : best;
        }
    }
    return best;
}

// Highest point of a block of stage s with ZeRO, relative to the live bytes
// at its start counted with the largest owned resident (z.rmax): the maximum
// over replicas d of owned(d) - rmax + the highest point of d's own walk
// through the block's segments (edge ops, replayed units and the partial
// unit under recomputation, units, edge ops).  n: units of the block; n_r:
// replayed units.  The block's net bytes do not depend on ownership.
//
// A replica's walk never rises above that of a replica owning none of the
// segments' groups (A), and reaches A unless it owns every unit at which A is
// reached.  Those units have one owner at most (consecutive groups belong to
// different replicas), so every other replica reaches A, the largest of them
// holding the largest owned resident besides that owner's, and only the
// owner's walk needs composing.
template <bool TF>
__device__ int64_t zero_top(const Ctx &x, int s, const ZStage &z, bool bwd, uint64_t m, bool acc, int n, int n_r)
{
    // five fixed slots (pre edge, first / replayed unit, the replay's partial
    // unit, the units, suf edge); absent ones hold no unit (n = 0).  Every
    // index below is a constant, so the list stays in registers.
    constexpr int kSeg = 5;
    ZSeg seg[kSeg];
#pragma unroll
    for (int i = 0; i < kSeg; ++i) seg[i] = ZSeg{0, 0, 0, 0, -1, 1};
    MemZ pre{x, 0, 0, 0, 0}, suf{x, 0, 0, 0, 0};
    record_edges<TF>(x, s, bwd, m, acc, pre, suf);
    int g_pre = -1, g_suf = -1;
    if (TF) {
        if (!bwd && s == 0) g_pre = 0;
        if (!bwd && s == x.P - 1) g_suf = z.g_head;
        if (bwd && s == x.P - 1) g_pre = z.g_head;
    } else if (bwd) {
        g_suf = z.gl_lo;   // the stage's first unit
    }
    seg[0] = ZSeg{1, pre.cur, pre.tn, pre.to, g_pre, 1};
    if (!bwd) {
        MemZ u{x, 0, 0, 0, 0};
        record_unit<TF>(x, false, m, false, u);
        if (x.rc && n >= 1) {
            MemZ f{x, 0, 0, 0, 0};
            record_unit<TF>(x, false, m, false, f, kFwdFirst);
            seg[1] = ZSeg{1, f.cur, f.tn, f.to, z.gl_lo, 1};
            seg[3] = ZSeg{n - 1, u.cur, u.tn, u.to, z.gl_lo + 1, 1};
        } else {
            seg[3] = ZSeg{n, u.cur, u.tn, u.to, z.gl_lo, 1};
        }
    } else {
        if (x.rc) {
            MemZ u{x, 0, 0, 0, 0}, q{x, 0, 0, 0, 0};
            record_unit<TF>(x, false, m, false, u, kFwdReplay);
            record_partial<TF>(x, m, q);
            seg[1] = ZSeg{n_r, u.cur, u.tn, u.to, z.gl_lo, 1};
            seg[2] = ZSeg{1, q.cur, q.tn, q.to, z.gl_hi - 1, 1};
        }
        MemZ u{x, 0, 0, 0, 0};
        record_unit<TF>(x, true, m, acc, u);
        seg[3] = ZSeg{n, u.cur, u.tn, u.to, z.gl_hi - 1, -1};
    }
    seg[4] = ZSeg{1, suf.cur, suf.tn, suf.to, g_suf, 1};
    const int D = x.D;
    // A, and the owner of the units at which it is reached
    int64_t a_none = INT64_MIN, at = 0;
#pragma unroll
    for (int i = 0; i < kSeg; ++i) {
        if (seg[i].n <= 0) continue;
        const int64_t v = at + run_top(seg[i], -1, D);
        a_none = v > a_none ? v : a_none;
        at += (int64_t)seg[i].n * seg[i].d;
    }
    int owner = -1;
    bool shared = false;   // reached where every replica reaches it
    at = 0;
#pragma unroll
    for (int i = 0; i < kSeg; ++i) {
        if (seg[i].n <= 0) continue;
        if (at + run_top(seg[i], -1, D) == a_none) {
            if (seg[i].gs < 0 || (seg[i].d == 0 && seg[i].n >= 2)) {
                shared = true;
            } else {
                int o = (seg[i].gs + seg[i].dir * (seg[i].d > 0 ? seg[i].n - 1 : 0)) % D;
                if (o < 0) o += D;
                shared = shared || (owner >= 0 && owner != o);
                owner = o;
            }
        }
        at += (int64_t)seg[i].n * seg[i].d;
    }
    if (shared || owner < 0) return a_none;
    int64_t t_o = INT64_MIN;
    at = 0;
#pragma unroll
    for (int i = 0; i < kSeg; ++i) {
        if (seg[i].n <= 0) continue;
        const int64_t v = at + run_top(seg[i], owner, D);
        t_o = v > t_o ? v : t_o;
        at += (int64_t)seg[i].n * seg[i].d;
    }
    const int64_t rmax = (int64_t)z.rmax;
    const int64_t others = (int64_t)(owner == z.arg ? z.rsec : z.rmax) - rmax + a_none;
    const int64_t own = (int64_t)z_owned(x, z, owner) - rmax + t_o;
    return others > own ? others : own;
}

// n repetitions of a unit of costs r: the same value as n * 2 * U2n
// sequential fp64 additions, with far fewer dependent steps.
//
// While the clock t stays in one binade [2^e, 2^(e+1)), it is a multiple
// of ulp = 2^(e-52), and rounding t + c to nearest lands on t plus c rounded
// to a multiple of ulp, whatever t is, unless c sits exactly half way
// between two multiples (then ties-to-even depends on t's last bit).  So
// each unit adds the same whole number I of ulps, and q units add q * I
// exactly, as long as t + q * I ulps stays below 2^(e+1).  The unit that
// crosses into the next binade, tiny clocks and the units of a binade in
// which some cost is a half-way case are added op by op.
template <int U2n>
__device__ __forceinline__ double units_seq(const double2 (&r)[U2n], double clk)
{
#pragma unroll
    for (int j = 0; j < U2n; ++j) {
        clk = clk + r[j].x;
        clk = clk + r[j].y;
    }
    return clk;
}

template <int U2n>
__device__ __forceinline__ double units_exact(const double2 (&r)[U2n], double clk, int n)
{
    while (n > 0) {
        // (an overflowed clock, +inf, stays +inf: op by op, n units)
        if (clk >= 0x1p-500 && clk <= 0x1.fffffffffffffp+1023) {
            const int e = ilogb(clk);
            const double sc = ldexp(1.0, 52 - e);
            const double k = clk * sc;                 // integer in [2^52, 2^53)
            const double room = 0x1p53 - k;            // ulps left in the binade
            double part[U2n];
            bool tie = false;
#pragma unroll
            for (int j = 0; j < U2n; ++j) {
                const double tx = r[j].x * sc, ty = r[j].y * sc;
                const double rx = rint(tx), ry = rint(ty);
                tie = tie || fabs(tx - rx) == 0.5 || fabs(ty - ry) == 0.5;
                part[j] = rx + ry;
            }
            // whole numbers: exact while below 2^53 (larger sums cannot fit)
#pragma unroll
            for (int w = 1; w < U2n; w <<= 1)
#pragma unroll
                for (int j = 0; j + w < U2n; j += 2 * w) part[j] = part[j] + part[j + w];
            const double I = part[0];
            if (tie) {
                // op by op until the clock leaves this binade (ties become
                // half as likely with every binade)
                const double top = ldexp(1.0, e + 1);
                for (; n > 0 && clk < top; --n) clk = units_seq(r, clk);
                continue;
            }
            if (I == 0.0) return clk;
            if ((double)n * I <= room - 1.0) return ldexp(k + (double)n * I, e - 52);
            double q = floor((room - 1.0) / I);
            const double rem = fma(-q, I, room - 1.0);   // exact: |rem| < 2^53
            if (rem < 0.0) q -= 1.0;
            else if (rem >= I) q += 1.0;
            if (q > 0.0) {
                clk = ldexp(k + q * I, e - 52);
                n -= (int)q;
            }
        }
        clk = units_seq(r, clk);   // crosses into the next binade (or a tiny clock)
        --n;
    }
    return clk;
}

// ---------------------------------------------------------------------------
// Cross-lane helpers
// ---------------------------------------------------------------------------
// lane i receives lane i-1's value (0 at lane 0) / lane i+1's (0 at lane 63)
__device__ __forceinline__ int shr1(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int shl1(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ double shr1(double v)
{
    return __hiloint2double(shr1(__double2hiint(v)), shr1(__double2loint(v)));
}
__device__ __forceinline__ double shl1(double v)
{
    return __hiloint2double(shl1(__double2hiint(v)), shl1(__double2loint(v)));
}
__device__ __forceinline__ uint64_t shr1(uint64_t v)
{
    return ((uint64_t)(uint32_t)shr1((int)(v >> 32)) << 32) | (uint32_t)shr1((int)(uint32_t)v);
}
__device__ __forceinline__ uint64_t shl1(uint64_t v)
{
    return ((uint64_t)(uint32_t)shl1((int)(v >> 32)) << 32) | (uint32_t)shl1((int)(uint32_t)v);
}

__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

// DPP moves within the wavefront: row_shr:n (0x110 + n, lane i of a row of
// 16 receives lane i - n of the same row), row_bcast:15 (0x142, lane 15 of
// each row into the next row; rows 1 and 3 written) and row_bcast:31 (0x143,
// lane 31 into rows 2 and 3).  Rows outside ROWS, and lanes whose source
// lies outside the row, receive 0.
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, true);
}
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp(double v)
{
    return __hiloint2double(dpp<CTRL, ROWS>(__double2hiint(v)), dpp<CTRL, ROWS>(__double2loint(v)));
}

// max of two clocks, which are never NaN or -0.0: the bare instruction
// (fmax would canonicalize both operands first, two more dependent steps)
__device__ __forceinline__ double max_nn(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Inclusive maximum over the segments of the wavefront (values never NaN):
// each lane over its segment from the segment's first lane (spos = 0 there)
// up to itself.  Rows of 16 lanes scan first, treating a row's first lane as
// a segment start; then lanes whose segment began in an earlier row take the
// carries, lane 15 of rows 0 and 2 into rows 1 and 3, then lane 31 into rows
// 2 and 3 (cross, uniform: some segment spans a row boundary).
__device__ __forceinline__ double seg_max(double v, int spos, int lane, bool cross)
{
    const int rl = lane & 15;
    const int sr = spos < rl ? spos : rl;
    double up = max_nn(v, dpp<0x111, 0xf>(v));
    v = sr >= 1 ? up : v;
    up = max_nn(v, dpp<0x112, 0xf>(v));
    v = sr >= 2 ? up : v;
    up = max_nn(v, dpp<0x114, 0xf>(v));
    v = sr >= 4 ? up : v;
    up = max_nn(v, dpp<0x118, 0xf>(v));
    v = sr >= 8 ? up : v;
    if (cross) {
        up = max_nn(v, dpp<0x142, 0xa>(v));
        v = ((lane & 16) != 0 && spos > rl) ? up : v;
        up = max_nn(v, dpp<0x143, 0xc>(v));
        v = (lane >= 32 && spos >= lane - 31) ? up : v;
    }
    return v;
}

// max of two byte counts in [0, 2^62) as one fp64 max of their bit patterns
// (non-negative doubles below 2^62's pattern order like the integers)
__device__ __forceinline__ int64_t max_bytes(int64_t a, int64_t b)
{
    return __double_as_longlong(max_nn(__longlong_as_double(a), __longlong_as_double(b)));
}

// The Sends of one slot as prefix scans, exact.
//
// Along a run of linked Sends (positions r = 0, 1, ... in ascending source
// stage), each Send starts at the later of the clock the previous Send left
// on the shared stage and a clock no earlier Send of the run has touched,
// and every stage it joins ends at start + cost:
//   v_r = fl(max(v_{r-1}, z_r) + w_r),
// z_r being the larger of the Send's own two stage clocks before the slot's
// Sends (a stage without a Send that received one from its left carries
// v_{r-1} on; any other position starts the recurrence afresh).  While every
// v stays in one binade [2^E, 2^(E+1)), rounding to nearest adds each w_r as
// the whole number W_r of ulps 2^(E-52) nearest to it, whatever v is, unless
// w_r lies exactly half way between two (then ties to even depend on v).  In
// integer ulps K_r = z_r / ulp, with Q_r = W_0 + ... + W_r, the recurrence is
// then v_r = Q_r + max_{i <= r} (K_i - Q_{i-1}) over a segment (a position
// that starts afresh starts one): a sum scan -- over the whole wavefront,
// what earlier segments add to Q cancels -- and a max scan within each
// segment, in exact integer-valued fp64 (below 2^53).  E is the binade of
// the first value at the candidate's first involved stage.
// Returns false, changing nothing, if some lane leaves those conditions (a
// start in another binade, 0, not finite or below 2^-500; a cost that is
// not finite or a half-way case; a result past the binade); the caller then
// walks the Sends step by step.  src: lanes with a Send (sdir its direction,
// scost its cost), left / right: lanes that receive from their left / right.
__device__ __forceinline__ bool send_scan(double &clk, bool bwd, double scost, uint64_t src, uint64_t left,
                                          uint64_t right, int lane, int W, uint64_t segmask)
{
    auto in = [](uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); };
    const bool sends = in(src);
    const double cl = shr1(clk), cr = shl1(clk);
    double z = max_nn(clk, bwd ? cl : cr);
    z = sends ? z : clk;
    const uint64_t back = ballot(sends && bwd);
    const uint64_t carry = back | left;
    const uint64_t involved = src | left | right;
    const uint64_t upto = ~carry & (lane == 63 ? ~0ull : ((2ull << lane) - 1));
    const int spos = lane - (63 - __builtin_clzll(upto));
    // the first involved segment start (a run starts at one)
    const uint64_t begins = involved & ~carry;
    if (begins == 0) return false;
    const int hi = __double2hiint(z);
    int e;
    if (W == 64) {
        e = __builtin_amdgcn_readlane(hi, __builtin_ctzll(begins));
    } else {
        const uint64_t mine = begins & segmask;
        e = __shfl(hi, mine != 0 ? __builtin_ctzll(mine) : lane, kLanes);
    }
    e = (int)((uint32_t)e >> 20);
    const int sh = 1075 - e;
    // a start in another binade, or a cost whose whole ulps are unknown
    bool bad = in(begins) && ((int)((uint32_t)hi >> 20) != e || e < 1023 - 500 || e >= 0x7ff);
    const double t = ldexp(scost, sh);
    double w = rint(t);
    bad = bad || (sends && !(fabs(t - w) < 0.5));   // (false also for t not finite)
    w = sends ? w : 0.0;
    const double K = ldexp(z, sh);
    double q = w;   // (below 2^53 or the result below leaves the binade)
    q += dpp<0x111, 0xf>(q);
    q += dpp<0x112, 0xf>(q);
    q += dpp<0x114, 0xf>(q);
    q += dpp<0x118, 0xf>(q);
    q += dpp<0x142, 0xa>(q);
    q += dpp<0x143, 0xc>(q);
    bad = bad || !(q < 0x1p53);
    const bool cross = ballot(spos > (lane & 15)) != 0;
    const double y = seg_max(K - (q - w), spos, lane, cross);
    const double v = q + y;
    bad = bad || (in(involved) && !(v < 0x1p53));
    if (ballot(bad) != 0) return false;
    const double vd = ldexp(v, -sh);
    const double vr = shl1(vd);
    clk = in(right) ? vr : (in(src | left) ? vd : clk);
    return true;
}

template <class T, class Op>
__device__ __forceinline__ T seg_reduce(T v, int W, Op op)
{
    for (int o = 1; o < W; o <<= 1) v = op(v, __shfl_xor(v, o, kLanes));
    return v;
}

// How many periods of two slots a stage can run on like its last one, by its
// own schedule: the blocks of the last period (and of the `back` periods
// before it) and of all periods counted have the same directions, the same
// microbatch size class (the first mr are one row longer) and the same
// accumulation; the last backward block is left out under overlap (it hands
// the gradients over).  nf, nb: the blocks run so far; pair: the last two
// were a forward and a backward one (1F1B), else both were bwd.
__device__ __forceinline__ int repeats(bool pair, bool bwd, int nf, int nb, int K, int mr, int back, bool ov)
{
    const int step = pair ? 1 : 2;
    int n = INT_MAX;
    if (pair || !bwd) {
        const int k0 = nf - step * (1 + back);
        n = K - nf;
        if (k0 < mr && mr - nf < n) n = mr - nf;
    }
    if (pair || bwd) {
        const int k0 = nb - step * (1 + back);
        if (k0 < 1) return 0;   // microbatch 0 does not accumulate
        const int e = (ov ? K - 1 : K) - nb;
        if (e < n) n = e;
        if (k0 < mr && mr - nb < n) n = mr - nb;
    }
    return n / step;
}

// ---------------------------------------------------------------------------
// The simulation kernel
// ---------------------------------------------------------------------------
// a stage with at least this many layers sums its weight update binade-wise
// (units_exact), else layer by layer: below it the dependent adds cost less
// than the binade arithmetic
constexpr int kFastUnits = 12;
// kinds of blocks: forward of a short and of a long microbatch; backward of
// microbatch 0 (no accumulation), of a short and of a long other one
constexpr int kKeys = 5;
__device__ __forceinline__ bool key_bwd(int key) { return key >= 2; }
__device__ __forceinline__ bool key_acc(int key) { return key >= 3; }
// the long microbatches (one row more) come first: microbatch 0 is one if
// there is any
__device__ __forceinline__ int key_long(int key, bool any) { return key == 2 ? (any ? 1 : 0) : (key >= 3 ? key - 3 : key); }
constexpr int kRoles = 4;   // stage 0; a middle stage of q + 1 or of q layers; the last stage (P > 1)
// binade tables are built for clocks of at least this biased exponent (below,
// a cost over the ulp could overflow) and below that of infinity
constexpr int kMinExp = 1023 - 500, kInfExp = 0x7ff;
// whole ulps of a block that has to be walked: added to a finite clock they
// leave its binade
constexpr int64_t kWalk = (int64_t)1 << 61;

// rounds of eight lanes over n entries
template <int N> using Rounds = std::integral_constant<int, (N + 7) / 8>;

// clk plus the NB (backward) or NF (forward) entry pairs at a, in order
template <int NF, int NB> __device__ __forceinline__ double walk(const double *a, bool bwd, double clk)
{
    const double2 *v = reinterpret_cast<const double2 *>(a);
    double2 r[NF < NB ? NB : NF];
#pragma unroll
    for (int j = 0; j < (NF < NB ? NB : NF); ++j) {
        const bool has = j < (bwd ? NB : NF);
        r[j] = v[has ? j : 0];
        if (!has) r[j] = make_double2(0.0, 0.0);   // clock + 0.0 == clock
    }
#pragma unroll
    for (int j = 0; j < (NF < NB ? NB : NF); ++j) {
        clk = clk + r[j].x;
        clk = clk + r[j].y;
    }
    return clk;
}

// The narrow launch's programs: a lane's own, an array per direction, entry j
// of lane l at [j][l], with the block's net bytes and its highest point.
template <class Sh> struct LaneProg {
    static constexpr int F = Sh::F_PRE2 + Sh::F_U2 + Sh::F_SUF2, B = Sh::PRE2 + Sh::U2 + Sh::SUF2;
    double2 f[F][kLanes], b[B][kLanes];
    int64_t sum[2][2][kLanes];   // [backward][net bytes, highest point]
};

// Records ops' costs into a lane's program and summarises their memory.
struct LaneRecord {
    const Ctx &x;
    double2 *base;
    int n;
    int64_t cur, top;

    __device__ __forceinline__ void put(double c)
    {
        reinterpret_cast<double *>(base + (n >> 1) * kLanes)[n & 1] = c;
        ++n;
    }
    __device__ __forceinline__ void pad(int pairs)
    {
        while (n < 2 * pairs) put(0.0);   // clock + 0.0 == clock
    }
    __device__ __forceinline__ void op(double c, uint64_t al, uint64_t fr)
    {
        put(c);
        const int64_t a = cur + (int64_t)al;
        top = a > top ? a : top;
        cur = a - (int64_t)fr;
    }
    __device__ __forceinline__ void local(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr)
    {
        op(cost_local(x, fl, by), al, fr);
    }
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t al, uint64_t fr, uint64_t k)
    {
        op(cost_mm(x, fl, by, k), al, fr);
    }
    __device__ __forceinline__ void ar_tp(uint64_t by)
    {
        if (x.H > 1) put(cost_ar_tp(x, by));
    }
    __device__ __forceinline__ void bcast(uint64_t by, int)
    {
        if (x.zero) put(cost_chain_d(x, by));
    }
    __device__ __forceinline__ void handover(uint64_t) {}   // (that block is walked, see HandWalk)
};

// Records stage s's block of one direction (pre, unit, suf at pp) and its
// memory: n units; under recomputation the forward block's first unit keeps
// its input and the backward block replays n_r forward units and the partial
// unit after its pre ops.
template <bool TF, bool RC, class Sh>
__device__ void record_lane(const Ctx &x, int s, bool bwd, uint64_t m, bool acc, int n, int n_r, double2 *pp,
                            int64_t &delta, int64_t &top)
{
    const int n_pre = bwd ? Sh::PRE2 : Sh::F_PRE2, n_unit = bwd ? Sh::U2 : Sh::F_U2, n_suf = bwd ? Sh::SUF2 : Sh::F_SUF2;
    LaneRecord p{x, pp, 0, 0, 0}, u{x, pp + n_pre * kLanes, 0, 0, 0}, f{x, pp + (n_pre + n_unit) * kLanes, 0, 0, 0};
    record_edges<TF>(x, s, bwd, m, acc, p, f);
    record_unit<TF>(x, bwd, m, acc, u);
    p.pad(n_pre);
    u.pad(n_unit);
    f.pad(n_suf);
    int64_t d = 0, t = 0;
    if (!RC || (!bwd && n < 1)) {
        compose(p.cur, p.top, u.cur, u.top, n, f.cur, f.top, d, t);
    } else if (!bwd) {
        Mem q{x, 0, 0};
        record_unit<TF>(x, false, m, false, q, kFwdFirst);
        compose_first(p.cur, p.top, q.cur, q.top, u.cur, u.top, n, f.cur, f.top, d, t);
    } else {
        Mem v{x, 0, 0}, q{x, 0, 0};
        record_unit<TF>(x, false, m, false, v, kFwdReplay);
        record_partial<TF>(x, m, q);
        compose(p.cur, p.top, v.cur, v.top, n_r, q.cur, q.top, d, t);
        int64_t d2, t2;
        compose(0, 0, u.cur, u.top, n, f.cur, f.top, d2, t2);
        chain(d, t, d2, t2);
    }
    delta = d;
    top = t;
}

// clk plus the NB (backward) or NF (forward) entry pairs of a lane's program
// at v, n times over; fast: binade-wise
template <int NF, int NB>
__device__ __forceinline__ double lane_units(const double2 *v, bool bwd, double clk, int n, bool fast)
{
    static_assert(NF <= NB, "a forward region is the shorter one");
    if constexpr (NB > 0) {
        double2 r[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const bool has = j < (bwd ? NB : NF);
            r[j] = v[(has ? j : 0) * kLanes];
            if (!has) r[j] = make_double2(0.0, 0.0);
        }
        if (fast) return units_exact(r, clk, n);
        for (int i = 0; i < n; ++i) clk = units_seq(r, clk);
    }
    return clk;
}

// The last backward block under overlap, op by op on both streams' clocks.
struct HandWalk {
    const Ctx &x;
    double clk, tm;
    __device__ __forceinline__ void local(uint64_t fl, uint64_t by, uint64_t, uint64_t) { clk = clk + cost_local(x, fl, by); }
    __device__ __forceinline__ void mm(uint64_t fl, uint64_t by, uint64_t, uint64_t, uint64_t k)
    {
        clk = clk + cost_mm(x, fl, by, k);
    }
    __device__ __forceinline__ void ar_tp(uint64_t by)
    {
        if (x.H > 1) clk = clk + cost_ar_tp(x, by);
    }
    __device__ __forceinline__ void bcast(uint64_t, int) {}   // no ZeRO under overlap
    __device__ __forceinline__ void handover(uint64_t by)
    {
        clk = max_nn(clk, tm) + cost_stream(x, by);
        tm = clk + cost_ar_dp(x, by);
    }
};

// (collective or hand-back, optimizer) of a parameter of N elements in the
// weight update
__device__ __forceinline__ double2 update_cost(const Ctx &x, uint64_t N)
{
    uint64_t fl, by;
    opt_cost(x, N, fl, by);
    const double coll = x.zero ? cost_chain_d(x, x.e * N)
                               : (x.ov ? cost_stream(x, x.e * N) : (x.D > 1 ? cost_ar_dp(x, x.e * N) : 0.0));
    return make_double2(coll, cost_local(x, fl, by));
}
// of a layer's parameters
template <bool TF> __device__ __forceinline__ void update_costs(const Ctx &x, double2 *r)
{
    if (TF) {
        r[0] = update_cost(x, x.d * 3 * x.dH);
        r[1] = update_cost(x, x.dH * x.d);
        r[2] = update_cost(x, x.d * x.FH);
        r[3] = update_cost(x, x.FH * x.d);
    } else {
        r[0] = update_cost(x, x.d * x.dH);
    }
}

// One candidate's programs, recorded once by all lanes of its segment.  A
// block of a stage is pre, its repeating units, suf; every stage has the same
// unit, stage 0 and the last stage have edges: the transformer's embedding,
// head and loss; the MLP's loss (pre) and, on stage 0, the first unit's
// backward (suf), whose input gradient is not all-reduced (every other MLP
// stage's first unit costs what its others do).
template <bool TF, bool ZR, bool OV> struct Prog {
    using Sh = Shape<TF, ZR>;
    double2 uf[2][Sh::F_U2], ub[3][Sh::U2];
    double2 pf[2][Sh::F_PRE2 > 0 ? Sh::F_PRE2 : 1], pb[3][Sh::PRE2];
    double2 sf[2][Sh::F_SUF2], sb[3][Sh::SUF2];
    double2 wu[5];                        // weight update: a layer's parameters, [4] the embedding / head
    int64_t mem[kKeys][kRoles][2];        // a block's net bytes, highest point above its start
    int64_t blk[2][kKeys][kRoles];        // a block's whole ulps in the binade held for each exponent parity, or kWalk
    double2 unit_ulps[2][kKeys];          // one unit's, and their reciprocal; negative: walk it
    int nu[2][kRoles], nrep[kRoles];      // units walked [backward], replayed
    int npart, single, any_long;          // entries of the replay's partial unit; P == 1; uneven microbatches
    typename std::conditional<OV, OvUnit<TF>, int>::type ov;   // the last backward block's unit
    Mark mark[OV ? 2 : 1];                // and its hand-overs in pre and suf (transformer)

    __device__ __forceinline__ const double *unit(int key) const { return key < 2 ? &uf[key][0].x : &ub[key - 2][0].x; }
    __device__ __forceinline__ const double *pre(int key) const { return key < 2 ? &pf[key][0].x : &pb[key - 2][0].x; }
    __device__ __forceinline__ const double *suf(int key) const { return key < 2 ? &sf[key][0].x : &sb[key - 2][0].x; }
    // entries of each
    static __device__ __forceinline__ int n_unit(bool bwd) { return bwd ? 2 * Sh::U2 : 2 * Sh::F_U2; }
    static __device__ __forceinline__ int n_pre(bool bwd) { return bwd ? 2 * Sh::PRE2 : 2 * Sh::F_PRE2; }
    static __device__ __forceinline__ int n_suf(bool bwd) { return bwd ? 2 * Sh::SUF2 : 2 * Sh::F_SUF2; }
    // whether a stage of these places has them
    static __device__ __forceinline__ bool has_pre(bool bwd, bool first, bool last) { return bwd ? last : (TF && first); }
    static __device__ __forceinline__ bool has_suf(bool bwd, bool first, bool last) { return bwd ? first : (TF && last); }
};

// a stage of the given role (-1: the strategy has none)
__device__ __forceinline__ int role_stage(const Ctx &x, int role)
{
    if (role == 0) return 0;
    if (role == 3) return x.P > 1 ? x.P - 1 : -1;
    if (x.P < 3) return -1;
    if (role == 1) return x.r > 1 ? 1 : -1;
    return x.P - 2 >= x.r ? x.P - 2 : -1;
}

// The memory of stage s's block of one kind: net bytes and highest point
// above its start; under recomputation the forward block's first unit keeps
// its input and the backward block replays units and the partial unit after
// its pre ops.
template <bool TF, bool RC>
__device__ void block_mem(const Ctx &x, int s, bool bwd, uint64_t m, bool acc, int64_t &d, int64_t &t)
{
    Mem p{x, 0, 0}, f{x, 0, 0}, u{x, 0, 0};
    record_edges<TF>(x, s, bwd, m, acc, p, f);
    record_unit<TF>(x, bwd, m, acc, u);
    const int n = block_units(x, s, bwd, TF);
    if (!RC || (!bwd && n < 1)) {
        compose(p.cur, p.top, u.cur, u.top, n, f.cur, f.top, d, t);
    } else if (!bwd) {
        Mem q{x, 0, 0};
        record_unit<TF>(x, false, m, false, q, kFwdFirst);
        compose_first(p.cur, p.top, q.cur, q.top, u.cur, u.top, n, f.cur, f.top, d, t);
    } else {
        Mem v{x, 0, 0}, q{x, 0, 0};
        record_unit<TF>(x, false, m, false, v, kFwdReplay);
        record_partial<TF>(x, m, q);
        const int nl = stage_nl(x, s);
        compose(p.cur, p.top, v.cur, v.top, TF ? nl - 1 : nl / (x.H > 1 ? 2 : 1) - 1, q.cur, q.top, d, t);
        int64_t d2, t2;
        compose(0, 0, u.cur, u.top, n, f.cur, f.top, d2, t2);
        chain(d, t, d2, t2);
    }
}

// Records one of a candidate's programs: jobs 0-4 a unit, 5-9 a kind's
// edges, 10 the weight update's parameters, 11 an overlapped last backward
// block.
constexpr int kJobs = 2 * kKeys + 2;
template <bool TF, bool ZR, bool OV>
__device__ __forceinline__ void record_job(const Ctx &x, Prog<TF, ZR, OV> &q, int job)
{
    using Pr = Prog<TF, ZR, OV>;
    const int key = job < kKeys ? job : job - kKeys;
    const bool bwd = key_bwd(key), acc = key_acc(key);
    const uint64_t m = x.mq + (uint64_t)key_long(key, x.mr > 0);
    if (job < kKeys) {
        Record r{x, const_cast<double *>(q.unit(key)), 0};
        record_unit<TF>(x, bwd, m, acc, r);
        r.pad(Pr::n_unit(bwd));
    } else if (job < 2 * kKeys) {
        Record p{x, const_cast<double *>(q.pre(key)), 0}, f{x, const_cast<double *>(q.suf(key)), 0};
        if (TF) {
            const TfSz z = tf_sizes(x, m);
            if (bwd) {
                tf_bwd_last(x, p, z, acc);
                tf_bwd_first(x, f, z, acc);
            } else {
                tf_fwd_first(x, p, z);
                tf_fwd_last(x, f, z);
            }
        } else if (bwd) {
            mlp_loss(x, p, m);
            for (int i = x.H > 1 ? 1 : 0; i >= 0; --i) mlp_layer_bwd(x, f, m, mlp_kind(x, i), false, i == 0, acc, 0);
        }
        p.pad(Pr::n_pre(bwd));
        f.pad(Pr::n_suf(bwd));
    } else if (job == 2 * kKeys) {
        update_costs<TF>(x, q.wu);
        if (TF) q.wu[4] = update_cost(x, x.Vh * x.d);
    } else if constexpr (OV) {
        const bool a = x.K > 1;
        RecordOv<TF> u{x, q.ov, 0, 0};
        record_unit<TF>(x, true, x.mq, a, u, kFwdBlock, true);
        u.pad();
        if (TF) {
            Marks p{x, &q.mark[0], 0}, f{x, &q.mark[1], 0};
            const TfSz z = tf_sizes(x, x.mq);
            tf_bwd_last(x, p, z, a, true);
            tf_bwd_first(x, f, z, a, true);
        }
    }
}

// ZeRO's weight update: the highest point above the live bytes at its start.
// At each parameter's reduce the owner holds the reduced gradient beside
// every replica's own, then every gradient dies; the owner's optimizer op
// frees the reduced one again.  The live bytes only fall, so of the groups
// of one owner the stage's first is enough.
template <bool TF>
__device__ __forceinline__ int64_t update_top(const Ctx &x, int s, const ZStage &z)
{
    int64_t live = 0, top = 0;
    uint64_t own = 0, other = 0;
    auto owner = [&](int grp) {
        const int o = grp % x.D;
        own = z_owned(x, z, o);
        other = o == z.arg ? z.rsec : z.rmax;
    };
    auto reduce = [&](uint64_t N) {
        const int64_t by = (int64_t)(x.e * N);
        const int64_t mine = (int64_t)own + by, rest = (int64_t)other;
        const int64_t hi = live - (int64_t)z.rmax + (mine > rest ? mine : rest);
        top = hi > top ? hi : top;
        live -= by;
    };
    const int l0 = stage_l0(x, s), nl = stage_nl(x, s);
    if (!TF) {
        const int per = x.H > 1 ? 2 : 1;
        for (int i = 0; i < nl && i / per < x.D; ++i) {
            owner(mlp_group(x, l0 + i));
            reduce(x.d * x.dH);
        }
        return top;
    }
    if (s == 0) {
        owner(0);
        reduce(x.Vh * x.d);
    }
    const int64_t before = live;
    for (int i = 0; i < nl && i < x.D; ++i) {
        owner(tf_group_layer(l0 + i));
        reduce(x.d * 3 * x.dH);
        reduce(x.dH * x.d);
        reduce(x.d * x.FH);
        reduce(x.FH * x.d);
    }
    if (s == x.P - 1) {
        live = before - (int64_t)(x.e * (uint64_t)nl * (4 * x.d * x.dH + 2 * x.d * x.FH));
        owner(tf_group_head(x));
        reduce(x.Vh * x.d);
    }
    return top;
}

// RC: training with activation recomputation; ZR: training with ZeRO; OV:
// training with the gradient all-reduce on the communication streams
// (separate instantiations keep the replay, the broadcasts and the two-stream
// walk out of the other kernels).
//
// The kernel's time is the slots' instructions and their latency (a slot is
// a serial chain, and a wavefront's slots follow one another), so a slot
// does as little as it can: which blocks and Sends run is held in wave-wide
// masks, the blocks' memory and, in the clocks' binade, the whole ulps a
// block adds are tabulated per candidate, and whole periods are skipped.
// Against two launches (1-8 and 16-64 lanes) that walked every block's costs
// and re-recorded a program whenever a lane's block kind changed: 39,965
// GPT-3-shaped strategies 2.03 -> 1.06 ms, with ZeRO 3.10 -> 1.37, two-stream
// 3.59 -> 1.31, 2,240 MLP ones 350 -> 149 us, 398 GPT-2-small-shaped training
// ones 195 -> 105 us (selection and pre-pass included); vector instructions
// per GPT-3-shaped call 929M (before either change) -> 531M, which keep the
// SIMDs issuing 83% of the kernel's cycles.
//
// NARROW: the body of the narrow launch, for segments of 1 to 8 lanes; w: its
// wavefront.
template <bool TF, bool NARROW, bool RC, bool ZR, bool OV>
__device__ __forceinline__ void parametric_body(const ParArgs &g, uint32_t w)
{
    using Pr = Prog<TF, ZR, OV>;
    using Sh = Shape<TF, ZR>;
    __shared__ typename std::conditional<NARROW, LaneProg<Sh>, Pr>::type L[NARROW ? 1 : kMaxSeg];
    // ZeRO: the highest point of every block kind over the stage's replicas
    __shared__ int64_t s_ztop[ZR ? kKeys : 1][kLanes];

    const int lane = threadIdx.x;
    int cls = kClasses - 1;
    int64_t c = (int64_t)blockIdx.x;
    if (NARROW || g.perm) {
        // wavefronts start longest first (the pre-pass's order), so that
        // short ones fill the tail; the grid is sized for the worst case
        if (!NARROW) {
            const uint32_t b = g.wave0 + blockIdx.x;
            if (b >= g.meta[16 + kClasses]) return;
            w = g.order[b];
        }
        constexpr int kFirst = NARROW ? 24 : 16;
        cls = NARROW ? 0 : kMinClass;
        while (cls + 1 < (NARROW ? kNarrow : kClasses) && w >= g.meta[kFirst + cls + 1]) ++cls;
        const uint32_t slot = ((w - g.meta[kFirst + cls]) << (6 - cls)) + (uint32_t)(lane >> cls);
        c = slot < g.meta[cls] ? (int64_t)g.perm[g.meta[8 + cls] + slot] : -1;
    }
    const int W = 1 << cls;
    const int seg = lane >> cls;
    const int s = lane & (W - 1);   // stage of this lane
    const uint64_t segmask = W == 64 ? ~0ull : (((1ull << W) - 1) << (lane & ~(W - 1)));

    const dsim_model &M = g.m;
    dsim_strategy st = {1, 1, 1, 1};
    bool ok = false;
    if (c >= 0) {
        st = g.cand[c];
        ok = strategy_ok(M, st.D, st.H, st.P, st.K) && st.P <= g.p_bound && st.P <= W && st.K <= kMaxK &&
             placement_ok(g.c.node, st.D, st.H);
    }
    const int P = ok ? st.P : 0, K = st.K;
    const bool train = M.mode != DSIM_INFER;
    const bool live_stage = s < P;
    int32_t status = (c >= 0 && !ok) ? DSIM_ST_BAD_STRATEGY : 0;
    const bool first = s == 0, last = s == P - 1;
    const bool ov_c = OV && M.overlap != 0 && st.D > 1;
    const bool zero_c = ZR && M.zero != 0 && st.D > 1;
    const bool f1b = train && M.schedule != DSIM_SCHED_GPIPE;

    double clk = 0.0;
    double clkm = 0.0;   // overlap: the communication stream's clock
    int64_t live = 0, peak = 0, wu_top = 0;
    uint64_t walked = 0, nops = 0;
    int nf = 0, nb = 0, len = 0, mr = 0, wu = 0, role = 0, nl = 0;
    double cl0 = 0.0, cl1 = 0.0, cr0 = 0.0, cr1 = 0.0;   // Send costs over the left / right link, by size class
    int64_t sz0 = 0, sz1 = 0;                            // and bytes
    // narrow: rows of a short microbatch, units of a forward, a backward
    // block and the replay, entries of its partial unit, the kinds recorded
    uint64_t mq = 0;
    int n_f = 0, n_b = 0, n_r = 0, n_part = 0, key_f = -1, key_b = -1;
    if (ok) {
        Ctx x = {};
        make_ctx(M, g.c, st, x);
        x.mlp = !TF;   // the family is uniform per launch: compiles out the other
        if constexpr (NARROW) {
            if (live_stage) {
                mq = x.mq;
                n_f = block_units(x, s, false, TF);
                n_b = block_units(x, s, true, TF);
                if (RC) {
                    n_r = TF ? stage_nl(x, s) - 1 : stage_nl(x, s) / (x.H > 1 ? 2 : 1) - 1;
                    Count n{x, 0, 0};
                    record_partial<TF>(x, 1, n);
                    n_part = (int)n.walked;
                }
            }
        } else {
            Pr &q = L[seg];
            for (int job = s; job < (OV ? kJobs : kJobs - 1); job += W) record_job<TF, ZR, OV>(x, q, job);
            for (int job = s; job < kKeys * kRoles; job += W) {
                const int key = job / kRoles, ss = role_stage(x, job % kRoles);
                int64_t d = 0, t = 0;
                if (ss >= 0)
                    block_mem<TF, RC>(x, ss, key_bwd(key), x.mq + (uint64_t)key_long(key, x.mr > 0), key_acc(key), d, t);
                q.mem[key][job % kRoles][0] = d;
                q.mem[key][job % kRoles][1] = t;
            }
            if (s < kRoles) {
                const int ss = role_stage(x, s), per = (!TF && x.H > 1) ? 2 : 1;
                const int units = ss >= 0 ? stage_nl(x, ss) / per : 0;
                q.nu[0][s] = units;
                q.nu[1][s] = units - ((!TF && s == 0) ? 1 : 0);
                q.nrep[s] = units - 1;
                if (s == 0) {
                    Count n{x, 0, 0};
                    if (RC) record_partial<TF>(x, 1, n);
                    q.npart = (int)n.walked;
                    q.single = P == 1;
                    q.any_long = x.mr > 0;
                }
            }
        }
        if (live_stage) {
            uint64_t res0;
            if (ZR && x.zero) {
                ZStage zs;
                z_stage(x, s, zs);
                res0 = resident_inputs(x, s) + zs.rmax;
#pragma unroll 1
                for (int key = 0; key < kKeys; ++key) {
                    const bool bwd = key_bwd(key);
                    s_ztop[key][lane] = zero_top<TF>(x, s, zs, bwd, x.mq + (uint64_t)key_long(key, x.mr > 0), key_acc(key),
                                                     block_units(x, s, bwd, TF),
                                                     TF ? stage_nl(x, s) - 1 : stage_nl(x, s) / (x.H > 1 ? 2 : 1) - 1);
                }
                wu_top = update_top<TF>(x, s, zs);
            } else {
                res0 = resident(x, s);
            }
            live = peak = (int64_t)res0;
            // microbatch splits before the pipeline: the replica's whole
            // input (stage 0) and target (last stage, training)
            const int splits = x.K > 1 ? (first ? 1 : 0) + (train && last ? 1 : 0) : 0;
            if (splits > 0) {
                const uint64_t whole = input_row(x) * x.rows;
                const double cs = cost_local(x, 0, 2 * whole);
                peak = live + (int64_t)whole;
                for (int i = 0; i < splits; ++i) clk = clk + cs;
            }
            len = train ? 2 * K : K;
            wu = f1b ? ((P - 1 - s) < K ? P - 1 - s : K) : K;   // forwards before the first backward
            mr = (int)x.mr;
            nl = stage_nl(x, s);
            role = first ? 0 : (last ? 3 : (s < x.r ? 1 : 2));
            // a stage's activations and gradients have the same size
            uint64_t rb, fre;
            send_size(x, s, 1, false, rb, fre);
            sz0 = (int64_t)(x.mq * rb);
            sz1 = (int64_t)((x.mq + 1) * rb);
            const bool nl_ = send_spans(g.c.node, st.D, st.H, s, s - 1), nr_ = send_spans(g.c.node, st.D, st.H, s, s + 1);
            cl0 = (nl_ ? g.c.net_lat : g.c.lat) + (double)(uint64_t)sz0 * (nl_ ? g.c.net_inv_l : g.c.inv_l);
            cl1 = (nl_ ? g.c.net_lat : g.c.lat) + (double)(uint64_t)sz1 * (nl_ ? g.c.net_inv_l : g.c.inv_l);
            cr0 = (nr_ ? g.c.net_lat : g.c.lat) + (double)(uint64_t)sz0 * (nr_ ? g.c.net_inv_l : g.c.inv_l);
            cr1 = (nr_ ? g.c.net_lat : g.c.lat) + (double)(uint64_t)sz1 * (nr_ ? g.c.net_inv_l : g.c.inv_l);
            count_stage<TF>(x, s, walked, nops);
        }
    }
    // op counts (they depend on the strategy alone)
    walked = seg_reduce(walked, W, [](uint64_t a, uint64_t b) { return a + b; });
    nops = seg_reduce(nops, W, [](uint64_t a, uint64_t b) { return a + b; });
    if (c >= 0 && first) {
        if (g.n_ops) g.n_ops[c] = nops;
        if (g.walked) g.walked[c] = walked;
    }
    __syncthreads();
    const auto &prog = L[NARROW ? 0 : seg];

    // The whole ulps of candidate sg's blocks and units while the clock has
    // the biased exponent e: inside one binade, rounding to nearest adds each
    // cost as the whole number of ulps nearest to it, whatever the clock is,
    // unless the cost lies exactly half way between two.
    // Eight lanes per block kind.
    int tag0 = -1, tag1 = -1;   // exponents held for this lane's segment, by parity
    auto build = [&](auto &progs, int sg, int e) {
        auto &q = progs[sg];
        const double sc = ldexp(1.0, 1075 - e);   // 1 / ulp
        const int key = lane >> 3, part = lane & 7;
        const bool bwd = key_bwd(key);
        double u = 0.0, p = 0.0, f = 0.0, up = 0.0;
        bool tie = false;
        // entry j = part, part + 8, ... of n (at most 8 * MAX); *head: the
        // sum over the first nh
        auto add = [&](auto max, const double *a, int n, double &sum, double *head, int nh) {
            double t[max.value];
#pragma unroll
            for (int i = 0; i < max.value; ++i) t[i] = part + 8 * i < n ? a[part + 8 * i] * sc : 0.0;
#pragma unroll
            for (int i = 0; i < max.value; ++i) {
                const double r = rint(t[i]);
                tie = tie || fabs(t[i] - r) == 0.5;
                sum += r;
                if (RC && head) *head += part + 8 * i < nh ? r : 0.0;
            }
        };
        if (key < kKeys) {
            add(Rounds<2 * Pr::Sh::U2>(), q.unit(key), Pr::n_unit(bwd), u, &up, q.npart);
            add(Rounds<2 * Pr::Sh::PRE2>(), q.pre(key), Pr::n_pre(bwd), p, nullptr, 0);
            add(Rounds<2 * Pr::Sh::SUF2>(), q.suf(key), Pr::n_suf(bwd), f, nullptr, 0);
        }
        // lanes 1, 2 apart, then the other half of the eight
        auto sum8 = [](double v) {
            v += dpp<0xb1, 0xf>(v);
            v += dpp<0x4e, 0xf>(v);
            v += dpp<0x141, 0xf>(v);
            return v;
        };
        u = sum8(u);
        p = sum8(p);
        f = sum8(f);
        const uint64_t ties = ballot(tie);
        bool bad = ((ties >> (lane & 56)) & 0xff) != 0;
        double rep = 0.0, repp = 0.0;
        if (RC) {
            // backward blocks replay the forward units of their row class
            up = sum8(up);
            const int fwd = 8 * (key_long(key, q.any_long != 0) & 1);   // (lanes past the keys: any lane)
            rep = __shfl(u, fwd, kLanes);
            repp = __shfl(up, fwd, kLanes);
            bad = bad || (bwd && ((ties >> fwd) & 0xff) != 0);
        }
        // (whole numbers: exact below 2^53; a block of 2^52 ulps or more
        // leaves the binade anyway)
        if (key < kKeys && part < kRoles) {
            const bool fr = part == 0, ls = part == 3 || (part == 0 && q.single);
            double t = (double)q.nu[bwd][part] * u;
            if (Pr::has_pre(bwd, fr, ls)) t += p;
            if (Pr::has_suf(bwd, fr, ls)) t += f;
            if (RC && bwd) t += (double)q.nrep[part] * rep + repp;
            q.blk[e & 1][key][part] = (!bad && t < 0x1p52) ? (int64_t)t : kWalk;
        }
        if (key < kKeys && part == 4) q.unit_ulps[e & 1][key] = (!bad && u < 0x1p52) ? make_double2(u, 1.0 / u) : make_double2(-1.0, 0.0);
        __syncthreads();
        if (seg == sg) {
            if (e & 1) tag1 = e;
            else tag0 = e;
        }
    };
    // builds the tables that the lanes of `want` miss, one exponent per segment
    auto build_for = [&](auto &progs, uint64_t want, int ex) {
        while (want != 0) {
            const int l0 = __builtin_ctzll(want);
            build(progs, l0 >> cls, __builtin_amdgcn_readlane(ex, l0));
            want &= ~(W == 64 ? ~0ull : (((1ull << W) - 1) << (l0 & ~(W - 1))));
        }
    };
    auto exponent = [](double v) { return (int)((uint32_t)__double2hiint(v) >> 20); };
    auto held = [&](int ex) { return (ex & 1) ? tag1 : tag0; };
    // n units of kind `key` on the lanes that are `on`: as many at once as
    // stay in the clock's binade, the one that leaves it op by op
    auto advance = [&](auto &progs, bool on, int key, int n) {
        const auto &q = progs[seg];
        int left = on ? n : 0;
        while (ballot(left > 0) != 0) {
            const int ex = exponent(clk);
            const uint64_t want = ballot(left > 1 && held(ex) != ex && ex >= kMinExp && ex < kInfExp);
            if (want != 0) build_for(progs, want, ex);
            if (left > 1) {
                if (ex == kInfExp) {
                    left = 0;   // an overflowed clock stays +inf
                } else if (held(ex) == ex) {
                    const double2 u = q.unit_ulps[ex & 1][key];
                    if (u.x >= 0.0) {
                        // the clock and its room in ulps, whole and below
                        // 2^53; room / u may come out a little off
                        const double at = ldexp(clk, 1075 - ex), room = (0x1p53 - 1.0) - at;
                        double k = floor(fmin(room * u.y, (double)left));   // u = 0: +inf
                        k = k * u.x > room ? k - 1.0 : k;
                        clk = ldexp(at + k * u.x, ex - 1075);
                        left -= (int)k;
                    }
                }
            }
            if (left > 0) {
                // (the forward unit is the shorter one: the rest only where
                // some lane's unit is a backward one)
                const double *a = q.unit(key);
                clk = walk<Pr::Sh::F_U2, Pr::Sh::F_U2>(a, false, clk);
                if (key_bwd(key)) {
                    constexpr int kRest = Pr::Sh::U2 - Pr::Sh::F_U2;
                    clk = walk<kRest, kRest>(a + 2 * Pr::Sh::F_U2, false, clk);
                }
                --left;
            }
        }
    };
    // under overlap: a hand-over on both clocks, and the last backward
    // block's programs (an edge with its one hand-over; a unit, the MLP's on
    // stage 0 without the last entry, its input gradient's all-reduce)
    auto hand = [&](double send, double ar) {
        clk = max_nn(clk, clkm) + send;
        clkm = clk + ar;
    };
    auto marked = [&](const double *a, int n, const Mark &mk) {
        for (int j = 0; j < n; ++j) {
            if (j == mk.pos) hand(mk.send, mk.ar);
            clk = clk + a[j];
        }
        if (mk.pos >= n) hand(mk.send, mk.ar);
    };
    auto ov_unit = [&](const auto &q, bool whole) {
        if constexpr (OV) {
            using U = OvUnit<TF>;
#pragma unroll
            for (int j = 0; j < U::kEntries; ++j) {
#pragma unroll
                for (int i = 0; i < U::kMarks; ++i)
                    if (j == U::pos(i) && (TF || q.ov.send[i] >= 0.0)) hand(q.ov.send[i], q.ov.ar[i]);
                clk = clk + ((TF || whole || j + 1 < U::kEntries) ? q.ov.cost[j] : 0.0);
            }
        }
    };

    // Repeated periods.  In the steady phase of a schedule every stage runs
    // the same blocks again every two slots (1F1B: a forward and a backward
    // one; otherwise two of one direction), so K microbatches repeat one
    // period.  All of a period's operations are maxima and rounded sums of
    // clocks; if every stage's clock moved by the same whole number d of ulps
    // and all of them stayed in one binade, the same period started from the
    // moved clocks does the same, moved by d: maxima commute with the shift,
    // and so does rounding to nearest inside a binade -- with ties to even
    // only for an even d, so an odd d must have come twice and periods are
    // then taken two at a time.  The remaining periods up to the next
    // binade, size class or phase are added at once: the doubles that walking
    // them gives.  Memory moves by the period's net bytes (whole numbers).
    const uint64_t stage_mask = ballot(live_stage);
    const uint64_t next_mask = ballot(live_stage && !first);   // lanes compared with the stage before
    const uint64_t last_mask = ballot(live_stage && last);
    uint64_t rdy_prev = 0, bwd_prev = 0;
    int64_t c0 = 0, live0 = 0, peak0 = 0;   // clock bits and bytes at the period's start
    int64_t d_prev = -1;                    // the last period's shift, -1: none
    bool odd = false;

    for (;;) {
        // forward-only, GPipe or synchronous 1F1B: the next block's direction
        // (its microbatch is the count of blocks of that direction), ready
        // once its input was produced in an earlier slot
        const bool bwd = nf == K || nf - nb > wu;
        const int nf_left = shr1(nf), nb_right = shl1(nb);   // slot-start counters
        const int k = bwd ? nb : nf;
        const int avail = bwd ? (last ? nf : nb_right) : (first ? INT_MAX : nf_left);
        const bool ready = nf + nb < len && avail > k;
        const uint64_t rdy_mask = ballot(ready);
        if (rdy_mask == 0) break;
        const uint64_t bwd_mask = ballot(ready && bwd);
        const bool mc = k < mr;
        const uint64_t mc_mask = ballot(mc);
        const int key = bwd ? (nb > 0 ? (mc ? 4 : 3) : 2) : (mc ? 1 : 0);

        // ---- the blocks
        const bool hov = OV && ov_c && bwd && nb == K - 1;   // hands its gradients over
        if constexpr (NARROW) {
            if (ready) {
                auto &q = L[0];
                const bool other = RC && bwd && key_f != (mc ? 1 : 0);   // the replay walks the forward unit
                if ((bwd ? key_b : key_f) != key || other) {
                    Ctx x = {};
                    make_ctx(M, g.c, st, x);
                    x.mlp = !TF;
                    const uint64_t m = mq + (mc ? 1u : 0u);
                    if ((bwd ? key_b : key_f) != key) {
                        record_lane<TF, RC, Sh>(x, s, bwd, m, bwd && nb > 0, bwd ? n_b : n_f, n_r,
                                                bwd ? &q.b[0][lane] : &q.f[0][lane], q.sum[bwd][0][lane],
                                                q.sum[bwd][1][lane]);
                        if (bwd) key_b = key;
                        else key_f = key;
                    }
                    if (other) {
                        record_lane<TF, RC, Sh>(x, s, false, m, false, n_f, n_r, &q.f[0][lane], q.sum[0][0][lane],
                                                q.sum[0][1][lane]);
                        key_f = mc ? 1 : 0;
                    }
                }
            }
            const bool walks = ready && !hov;
            const int n = bwd ? n_b : n_f;
            const bool fast = ballot(walks && n >= kFastUnits) != 0;
            const bool replay = RC && ballot(walks && bwd) != 0;
            const bool fast_r = replay && ballot(walks && bwd && n_r >= kFastUnits) != 0;
            if (walks) {
                const double2 *pre = bwd ? &prog.b[0][lane] : &prog.f[0][lane];
                const double2 *unit = pre + (bwd ? Sh::PRE2 : Sh::F_PRE2) * kLanes;
                const double2 *suf = unit + (bwd ? Sh::U2 : Sh::F_U2) * kLanes;
                if (bwd_mask == 0) {
                    clk = lane_units<Sh::F_PRE2, Sh::F_PRE2>(pre, false, clk, 1, false);
                    clk = lane_units<Sh::F_U2, Sh::F_U2>(unit, false, clk, n, fast);
                    clk = lane_units<Sh::F_SUF2, Sh::F_SUF2>(suf, false, clk, 1, false);
                } else {
                    clk = lane_units<Sh::F_PRE2, Sh::PRE2>(pre, bwd, clk, 1, false);
                    if (replay) {
                        const double2 *fu = &prog.f[Sh::F_PRE2][lane];
                        clk = lane_units<Sh::F_U2, Sh::F_U2>(fu, false, clk, bwd ? n_r : 0, fast_r);
                        for (int j = 0; j < (bwd ? n_part : 0); ++j) {
                            const double2 v = fu[(j >> 1) * kLanes];
                            clk = clk + ((j & 1) ? v.y : v.x);
                        }
                    }
                    clk = lane_units<Sh::F_U2, Sh::U2>(unit, bwd, clk, n, fast);
                    clk = lane_units<Sh::F_SUF2, Sh::SUF2>(suf, bwd, clk, 1, false);
                }
            }
            if (OV && ready && hov) {
                Ctx x = {};
                make_ctx(M, g.c, st, x);
                x.mlp = !TF;
                HandWalk h{x, clk, clkm};
                block_bwd(x, h, s, K - 1);
                clk = h.clk;
                clkm = h.tm;
            }
        } else {
            const int ex = exponent(clk);
            if (ballot(ready && held(ex) != ex) != 0) {
                const uint64_t miss = ballot(ready && held(ex) != ex && ex >= kMinExp && ex < kInfExp);
                if (miss != 0) build_for(L, miss, ex);
            }
            const double next = __longlong_as_double(__double_as_longlong(clk) + prog.blk[ex & 1][key][role]);
            bool fits = held(ex) == ex && exponent(next) == ex;
            if (OV) fits = fits && !hov;
            const uint64_t slow = ballot(ready && !fits);
            if (ready && fits) clk = next;
            if (slow != 0) {
                const bool on = __builtin_amdgcn_inverse_ballot_w64(slow);
                if (on && Pr::has_pre(bwd, first, last)) {
                    const double *a = prog.pre(key);
                    if (OV && TF && hov) marked(a, Pr::n_pre(true), prog.mark[0]);
                    else clk = walk<Pr::Sh::F_PRE2, Pr::Sh::PRE2>(a, bwd, clk);
                }
                if (RC) {
                    advance(L, on && bwd, mc ? 1 : 0, prog.nrep[role]);
                    if (on && bwd) {
                        const double *a = prog.unit(mc ? 1 : 0);
                        for (int j = 0; j < prog.npart; ++j) clk = clk + a[j];
                    }
                }
                if (OV && hov && on)
                    for (int i = 0; i < prog.nu[1][role]; ++i) ov_unit(prog, true);
                advance(L, on && !hov, key, prog.nu[bwd ? 1 : 0][role]);
                if (on && Pr::has_suf(bwd, first, last)) {
                    const double *a = prog.suf(key);
                    if (OV && TF && hov) marked(a, Pr::n_suf(true), prog.mark[1]);
                    else if (OV && hov) ov_unit(prog, false);
                    else clk = walk<Pr::Sh::F_SUF2, Pr::Sh::SUF2>(a, bwd, clk);
                }
            }
        }
        if (ready) {
            int64_t delta, top;
            if constexpr (NARROW) {
                delta = prog.sum[bwd][0][lane];
                top = prog.sum[bwd][1][lane];
            } else {
                delta = prog.mem[key][role][0];
                top = prog.mem[key][role][1];
            }
            // with ZeRO the net bytes do not depend on ownership; the highest point does
            if (ZR && zero_c) top = s_ztop[key][lane];
            peak = max_bytes(live + top, peak);
            live += delta;
            if (bwd) ++nb;
            else ++nf;
        }

        // ---- the slot's Sends, ascending by source stage.  Send s depends on
        // Send s-1 only if that went forward (it moved clock s) or this one
        // goes backward (it reads clock s-1); elsewhere the chain splits into
        // runs that touch disjoint clocks and proceed in parallel.
        const uint64_t fs = rdy_mask & ~bwd_mask & ~last_mask, bs = bwd_mask & next_mask;   // sources
        const uint64_t fl = fs << 1, fr = bs >> 1;                                          // receivers
        if ((fs | bs) != 0) {
            const uint64_t linked = fl | bs;
            const bool l_mc = __builtin_amdgcn_inverse_ballot_w64(mc_mask << 1);
            const bool r_mc = __builtin_amdgcn_inverse_ballot_w64(mc_mask >> 1);
            const double own = bwd ? (mc ? cl1 : cl0) : (mc ? cr1 : cr0);
            const double c_left = l_mc ? cl1 : cl0, c_right = r_mc ? cr1 : cr0;
            const bool from_left = __builtin_amdgcn_inverse_ballot_w64(fl);
            const bool from_right = __builtin_amdgcn_inverse_ballot_w64(fr);
            const bool sends = __builtin_amdgcn_inverse_ballot_w64(fs | bs);
            // runs of 12 and more Sends after the first (pipeline fill and
            // drain) take the scans, shorter ones the steps: from there on
            // the scans never lost
            uint64_t run = linked & (linked << 1);
            run &= run << 2;
            run &= run << 4;
            run &= run << 4;
            if (NARROW || run == 0 || !send_scan(clk, bwd, own, fs | bs, fl, fr, lane, W, segmask)) {
                for (uint64_t at = ~linked; at != 0; at = (at << 1) & linked) {
                    const uint64_t af = at & fs, ab = at & bs;
                    if ((af | ab) == 0) continue;
                    // a Send's two stages both end at the later clock plus
                    // its cost (clocks are never NaN or -0.0)
                    const bool src = __builtin_amdgcn_inverse_ballot_w64(af | ab);
                    const bool left = __builtin_amdgcn_inverse_ballot_w64((af << 1) | ab);   // partner on the left
                    const double lc = shr1(clk), rc_ = shl1(clk);
                    const double e = max_nn(left ? lc : rc_, clk) + (src ? own : (left ? c_left : c_right));
                    clk = __builtin_amdgcn_inverse_ballot_w64(af | ab | (af << 1) | (ab >> 1)) ? e : clk;
                }
            }
            if (from_left) {
                live += l_mc ? sz1 : sz0;
                peak = max_bytes(live, peak);
            }
            // (an MLP's training stage keeps the activation it sends)
            if (sends && (TF || bwd || !train)) live -= mc ? sz1 : sz0;
            if (from_right) {
                live += r_mc ? sz1 : sz0;
                peak = max_bytes(live, peak);
            }
        }

        // ---- every second slot: whole periods ahead (see above)
        if (odd) {
            const uint64_t both = rdy_prev & rdy_mask, pairs = bwd_prev ^ bwd_mask;
            // a stage that did not run twice, not the pattern of its
            // schedule, or another direction than the stage before
            const uint64_t off = ((~both | (f1b ? ~pairs : pairs)) & stage_mask) |
                                 (f1b ? 0 : (bwd_mask ^ (bwd_mask << 1)) & next_mask);
            const int64_t now = __double_as_longlong(clk);
            // some segment's stages all ran (narrow: some stage did)
            bool whole = NARROW ? (off & stage_mask) != stage_mask : off == 0;
            for (int i = 0; !NARROW && !whole && i < kLanes; i += W) {
                const uint64_t sm = W == 64 ? ~0ull : ((1ull << W) - 1) << i;
                whole = (off & sm) == 0 && (stage_mask & sm) != 0;
            }
            const int64_t d = now - c0;
            if (whole) {
                const int64_t dl = live - live0;
                const int ec = (int)(now >> 52);
                const int back = (int)(d & 1);
                const int64_t dn = (int64_t)shr1((uint64_t)d);
                const int en = shr1(ec);
                const bool bad = live_stage &&
                                 (__builtin_amdgcn_inverse_ballot_w64(off) || ec == 0 || ec == kInfExp ||
                                  ec != (int)(c0 >> 52) || (dl > 0 && peak <= peak0) ||
                                  (!first && (d != dn || ec != en)));
                const bool seg_ok = live_stage && (ballot(bad) & segmask) == 0;
                if (ballot(seg_ok) != 0) {
                    int q = INT_MAX;
                    if (seg_ok) {
                        q = repeats(f1b, bwd, nf, nb, K, mr, back, ov_c);
                        if (back && d_prev != d) q = 0;
                        if (q > 0 && d > 0) {
                            const int64_t room = (((int64_t)ec + 1) << 52) - 1 - now;
                            const double est = (double)room / (double)d;
                            if (est < (double)q) {
                                q = (int)est;
                                if (q > 0 && (int64_t)q * d > room) --q;
                            }
                        }
                    }
                    q = seg_reduce(q, W, [](int a, int b) { return a < b ? a : b; });
                    if (back) q &= ~1;
                    if (seg_ok && q > 0) {
                        clk = __longlong_as_double(now + (int64_t)q * d);
                        live += (int64_t)q * dl;
                        if (dl > 0) peak += (int64_t)q * dl;
                        nf += f1b ? q : (bwd ? 0 : 2 * q);
                        nb += f1b ? q : (bwd ? 2 * q : 0);
                    }
                }
                d_prev = seg_ok ? d : -1;
            } else {
                d_prev = -1;
            }
            c0 = __double_as_longlong(clk);
            live0 = live;
            peak0 = peak;
        }
        odd = !odd;
        rdy_prev = rdy_mask;
        bwd_prev = bwd_mask;
    }
    // (blocks left over that no stage can run: impossible for these schedules)
    if (nf + nb < len) status |= DSIM_ST_BAD_STRATEGY;
    if (live_stage && train) {
        // the weight update: each parameter's collective, then its optimizer
        // op (no memory above what the blocks reached, but ZeRO's reduced
        // gradients).  Under overlap the reduced gradients come back from the
        // communication stream, which is behind after the first hand-back.
        if (OV && ov_c) clk = max_nn(clk, clkm);
        auto param = [&](const double2 v) {
            clk = clk + v.x;
            clk = clk + v.y;
        };
        auto edge = [&]() {
            if constexpr (NARROW) {
                Ctx x = {};
                make_ctx(M, g.c, st, x);
                return update_cost(x, x.Vh * x.d);
            } else {
                return prog.wu[4];
            }
        };
        if (TF && first) param(edge());
        constexpr int kPar = TF ? 4 : 1;
        double2 r[kPar];
        if constexpr (NARROW) {
            Ctx x = {};
            make_ctx(M, g.c, st, x);
            update_costs<TF>(x, r);
        } else {
#pragma unroll
            for (int j = 0; j < kPar; ++j) r[j] = prog.wu[j];
        }
        if (nl >= kFastUnits) {
            clk = units_exact(r, clk, nl);
        } else {
            for (int i = 0; i < nl; ++i) clk = units_seq(r, clk);
        }
        if (TF && last) param(edge());
        if (ZR && zero_c) {
            const int64_t hi = live + wu_top;
            peak = hi > peak ? hi : peak;
        }
    }

    // per-candidate results: reductions over the segment
    status = seg_reduce(status, W, [](int32_t a, int32_t b) { return a | b; });
    const bool valid = status == 0;
    const bool mine = valid && live_stage;
    const double mk = seg_reduce(mine ? clk : 0.0, W, [](double a, double b) { return a > b ? a : b; });
    const uint64_t cp = seg_reduce(mine ? (uint64_t)peak : 0ull, W, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
    if (c < 0) return;
    if (first) {
        int32_t stt = status;
        if (valid && g.c.cap != 0 && cp > g.c.cap) stt |= DSIM_ST_OVER_CAP;
        g.makespan[c] = mk;
        g.cand_peak[c] = cp;
        g.status[c] = stt;
        if (!valid) {
            if (g.n_ops) g.n_ops[c] = 0;
            if (g.walked) g.walked[c] = 0;
        }
    }
    if (g.finish) {
        double *row = g.finish + (size_t)c * g.row_width;
        for (int j = s; j < g.row_width; j += W) row[j] = (mine && j == s) ? clk : 0.0;
    }
    if (g.peak) {
        uint64_t *row = g.peak + (size_t)c * g.row_width;
        for (int j = s; j < g.row_width; j += W) row[j] = (mine && j == s) ? (uint64_t)peak : 0;
    }
}

}  // namespace
}  // namespace dsim
