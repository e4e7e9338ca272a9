// sim_tables.hip -- batched simulation of explicit op tables on CDNA4.
//
// One lane per candidate walks the candidate's ops in program order (DistIR
// semantics, Sec. 2.1: an op starts when all its devices are free, all of
// them finish together; Sec. 3.3: clock advance by the op's cost, live-memory
// tracking with the peak sampled after allocation and before the free).
//
// Layout: the tables are op-major and candidate-fastest, so at every step the
// 64 lanes of a wavefront read 64 consecutive records of each field (five
// coalesced 256-byte loads per op).  The record stream is read once with
// non-temporal raw buffer loads: one descriptor per field and group of ops,
// based at the workgroup's first record, so the per-lane address is a 32-bit
// byte offset and no lane does 64-bit address arithmetic.  Two register sets
// of kUnroll ops alternate: one is processed while the other is in flight.
//
// Per-lane state: the device clocks live in VGPRs (n_dev <= 8 fp64) and take
// the op's device mask as their sign bits (set outside the op) while the
// start is taken, so an op touching any subset of devices runs the same
// branch-free sequence; the per-device (live,
// peak) byte counters are indexed by a per-lane device id and live in LDS as
// 16-byte pairs laid out [device][lane], so the 64 lanes of a wavefront
// always hit 64 distinct pairs.  An op's cost is base + coef * x with
// x = max(flops * g, bytes * w): (base, coef) and (w, g) come from small LDS
// tables indexed by the op class (compute: launch, 1, 1/B, 1/F; send:
// latency, 1, 1/L, 0; all-reduce over n devices: the ring terms for n, 1/L,
// 0), so every lane runs one straight sequence.  The tables hold one copy per
// lane of a 16-lane group, so that lanes reading different classes spread
// over the banks (a 64-lane b128 read still takes several LDS cycles).
//
// The kernel runs close to the rate at which HBM returns its op records
// (a million 2,048-op programs 7.0 ms, 5.9 TB/s; about 84 vector
// instructions per op keep the vector units partly busy beside that); it has a fast path for the ops every lane of a wavefront
// has, which assumes valid compute, send and all-reduce ops of cost class 0
// (indices clamped, so even an invalid op stays in bounds) and only tests
// whether each op is one.  A lane that meets an op it cannot vouch for (a
// free that would underflow, a broadcast or reduce record, a matrix
// multiplication record), every lane's ops past the wavefront's common count,
// and every op when the device model has a MatMul regression, nodes or
// streams take the general path below it: pipelined loads too, each op
// decoded in full.  (One op at a time with its loads in turn, that path took
// 1.1 us per op; now 0.65.  40,001 programs of 150 to 600 ops: 960 -> 308 us.)
//
// A call of few candidates cannot fill the chip with a lane each, and one
// lane's chain through an op (LDS counters, an eight-device maximum, the
// decoding) is long: there k_sim_tables_group gives each candidate eight
// lanes, one per device, with clocks and counters in registers.  The eight
// decode eight ops at a time, one each, and take them in turn.  (640 programs
// of 256 ops 73 -> 36 us; 400 lowered GPT-2-shaped programs of up to 271
// records, MatMul regression and nodes, 300 -> 39 us.)
#include <limits.h>

#include <type_traits>

#include "internal.h"

namespace dsim {
namespace {

constexpr int kBlock = 256;       // 4 wavefronts; 32 KB of LDS counters
constexpr int kWavesPerSimd = 4;
constexpr int kUnroll = 4;   // ops per register set; two sets in flight
constexpr int kCopies = 16;  // copies of the per-class cost rows (one per lane of an LDS phase)

struct TabArgs {
    const uint32_t *code;
    const float *flops;
    const float *bytes;
    const uint32_t *alloc;
    const uint32_t *freeb;
    const uint32_t *n_ops;
    const uint64_t *init_live;
    const uint32_t *mm_k;   // reduction lengths of class-1 records (NULL: 0)
    int64_t n_cand;
    int32_t max_ops;
    int32_t row_width;
    double *makespan;
    double *finish;
    uint64_t *peak;
    uint64_t *cand_peak;
    uint64_t *n_ops_out;
    uint64_t *walked;
    int32_t *status;
    // device d's GPU and node, four bits each (nodes or streams)
    uint32_t gpu_of, node_of;
    CostConsts c;
};

// Cost rows of the general path: compute, then per tier (links, network,
// streams of one GPU) send, all-reduce over n devices and chain over n
// devices.  An op costs base + coef * max(flops * g, bytes * w).
struct CostRow {
    double base, coef, w, g;
};
constexpr int kTierRows = 1 + 2 * (kMaxTableDev + 1);
constexpr int kCostRows = 1 + 3 * kTierRows;
__device__ __forceinline__ CostRow cost_row(const CostConsts &c, int i)
{
    if (i == 0) return CostRow{c.launch, 1.0, c.inv_b, c.inv_f};
    const int tier = (i - 1) / kTierRows, k = (i - 1) % kTierRows;
    const double lat = tier == 2 ? c.st_lat : (tier == 1 ? c.net_lat : c.lat);
    const double w = tier == 2 ? c.st_inv_l : (tier == 1 ? c.net_inv_l : c.inv_l);
    if (k == 0) return CostRow{lat, 1.0, w, 0.0};
    const int n = (k - 1) % (kMaxTableDev + 1);
    // over one device a collective costs nothing, whatever its bytes
    if (n <= 1) return CostRow{0.0, 1.0, 0.0, 0.0};
    if (k > kMaxTableDev + 1) return CostRow{(double)(n - 1) * lat, 1.0, w, 0.0};
    return CostRow{tier == 2 ? c.ar_lat_st[n] : (tier == 1 ? c.ar_lat_net[n] : c.ar_lat[n]), c.ar_coef[n], w, 0.0};
}

// Buffer resource covering one workgroup's 64 consecutive 4-byte records of
// one op row (raw buffer, gfx9 descriptor word 3); the base is wave-uniform,
// so the per-lane address is just a 32-bit byte offset.
constexpr int kRsrcWord3 = 0x00020000;
constexpr int kNonTemporal = 2;   // streamed once: do not keep in the caches
// the fast path's loads reach kUnroll op rows (kUnroll * n_cand * 4 bytes)
// from one descriptor with 32-bit offsets
constexpr int64_t kMaxFastCand = (int64_t)(0xffffffffu / (4u * kUnroll));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t group_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, kRsrcWord3);
}

// max of two doubles that are never NaN.  The compiler's fmax first
// canonicalizes an operand it cannot prove canonical (a loop-carried clock),
// one extra instruction per device and op; the bare instruction gives the
// same value (of +0.0 and -0.0 it may return either).
__device__ __forceinline__ double max_nn(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// max(|a|, b), the absolute value taken by the instruction's input modifier
__device__ __forceinline__ double max_abs(double a, double b)
{
    double r;
    asm("v_max_f64 %0, |%1|, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// x with its sign bit replaced by bit 31 of s (one bit-field insert on the
// high word; the low word is untouched)
__device__ __forceinline__ double with_sign(double x, uint32_t s)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t hi = (s & 0x80000000u) | ((uint32_t)(b >> 32) & 0x7fffffffu);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | (b & 0xffffffffull)));
}

// max of two byte counts below 2^63 as one fp64 max of their bit patterns:
// those are non-negative doubles (denormal below 2^52; fp64 denormals are
// preserved in this kernel's float mode), which order like the integers
__device__ __forceinline__ uint64_t max_bits(uint64_t a, uint64_t b)
{
    return (uint64_t)__double_as_longlong(max_nn(__longlong_as_double((long long)a), __longlong_as_double((long long)b)));
}

__device__ __forceinline__ double bits_double(uint32_t lo, uint32_t hi)
{
    return __hiloint2double((int)hi, (int)lo);
}

// One op decoded in full: the devices it synchronises, those that allocate
// and those that free (bit masks; 0 for an op that is skipped), its cost and
// its status bits, exactly as the table format defines validity.  on: the
// candidate has the op.  The lanes' op kinds differ, so everything is bit
// arithmetic on all-ones / all-zeros words, without branches.
struct TabOp {
    double cost;
    uint32_t m, am, fm, flag;
};
__device__ __forceinline__ uint32_t ones(bool b) { return b ? ~0u : 0u; }

template <int ND>
__device__ __forceinline__ TabOp decode(const TabArgs &a, const CostRow *rows, uint32_t code, uint32_t fl, uint32_t by,
                                        uint32_t k, bool on)
{
    TabOp o;
    const uint32_t kind = code & 0xffu, ia = (code >> 8) & 0xffu, ib = (code >> 16) & 0xffu;
    const uint32_t ma = 1u << (ia & 31u), mb = 1u << (ib & 31u);
    const uint32_t k0 = ones(kind == 0u), k1 = ones(kind == 1u), k2 = ones(kind == 2u), k3 = ones(kind == 3u),
                   k4 = ones(kind == 4u);
    // kind, cost class (1 only on compute records), and flops/bytes finite
    // and >= 0 (bit patterns below +inf)
    const uint32_t bad_op = ~(k0 | k1 | k2 | k3 | k4) | ones((code >> 24) > (k0 & 1u)) | ones(max(fl, by) >= 0x7f800000u);
    // devices below ND, a mask within them and not empty; the root of a
    // broadcast or reduce is a member
    const uint32_t a_out = ones(ia >= (uint32_t)ND), b_out = ones(ib >= (uint32_t)ND), mask_out = ones((ib >> ND) != 0u);
    const uint32_t bad_dev = (~k2 & a_out) | (k1 & b_out) | (k2 & (mask_out | ones(ib == 0u))) |
                             ((k3 | k4) & (mask_out | ones((ib & ma) == 0u)));
    const uint32_t self = k1 & ones(ia == ib);
    const uint32_t live = ones(on);
    o.flag = live & ((bad_op & DSIM_ST_BAD_OP) | (~bad_op & ((bad_dev & DSIM_ST_BAD_DEVICE) | (~bad_dev & self & DSIM_ST_SELF_SEND))));
    const uint32_t ok = live & ~(bad_op | bad_dev | self);   // an invalid op is skipped: no time, no memory
    const uint32_t m = ok & (((k0 | k1) & ma) | (k1 & mb) | (~(k0 | k1) & ib));
    o.m = m;
    // compute allocates and frees on a; send allocates on b and frees on a;
    // broadcast allocates on the members but a and frees on a; reduce
    // allocates on a and frees on every member
    o.am = ok & (((k0 | k4) & ma) | (k1 & mb) | (k3 & ib & ~ma));
    o.fm = ok & (((k0 | k1 | k3) & ma) | (k4 & ib));
    // the tier a communication op crosses: the streams of one GPU when all
    // its devices lie on one GPU (GPUs hold consecutive devices, so its
    // lowest and highest device decide), the network when its GPUs lie in
    // more than one node, the node's links otherwise
    uint32_t tier = 0;
    if (a.c.node || a.c.streams) {
        const int lo = 4 * ((__ffs(m) - 1) & 7), hi = 4 * ((31 - __clz(m)) & 7);
        const uint32_t one_gpu = ones(((a.gpu_of >> lo) & 15u) == ((a.gpu_of >> hi) & 15u)) & ones(a.c.streams != 0);
        const uint32_t nodes = ones(((a.node_of >> lo) & 15u) != ((a.node_of >> hi) & 15u)) & ones(a.c.node != 0);
        tier = (one_gpu & 2u) | (~one_gpu & nodes & 1u);
    }
    const uint32_t n = (uint32_t)__popc(m);
    const uint32_t r = ok & ~k0 & (1u + tier * (uint32_t)kTierRows + (k2 & (1u + n)) +
                                   ((k3 | k4) & ((uint32_t)kMaxTableDev + 2u + n)));
    const CostRow c = rows[r];
    const double f = (double)__uint_as_float(fl), b = (double)__uint_as_float(by);
    o.cost = c.base + c.coef * max_nn(f * c.g, b * c.w);
    if (a.c.mm) {
        // a matrix multiplication: the empirical regression of Sec. 4, with
        // its reduction-length term and floor
        const double lin = ((a.c.mm_c0 + a.c.mm_c1 * f) + a.c.mm_c2 * b) + a.c.mm_c3 * (double)k;
        const double mm = a.c.mm_floor > lin ? a.c.mm_floor : lin;
        o.cost = (code & 0xff0000ffu) == 1u << 24 ? mm : o.cost;
    }
    return o;
}

template <int ND>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kWavesPerSimd))) void k_sim_tables(
    const TabArgs a)
{
    __shared__ ulonglong2 s_mem[ND][kBlock];   // (live, peak) bytes
    // per op class -- all-reduce over n = 0..ND devices, then compute, then
    // send -- the cost terms (base, coef) and (1/bandwidth, 1/flop rate or 0)
    // (one array: the second pair sits at a fixed offset from the first, so
    // one address serves both loads)
    __shared__ double2 s_ct[2][ND + 3][kCopies];
    __shared__ CostRow s_row[kCostRows];   // the general path's costs

    const int tid = threadIdx.x;
    for (int i = tid; i < (ND + 3) * kCopies; i += kBlock) {
        const int e = i / kCopies, k = i % kCopies;
        const bool cmp = e == ND + 1;
        s_ct[0][e][k] = make_double2(e <= ND ? a.c.ar_lat[e] : (cmp ? a.c.launch : a.c.lat), e <= ND ? a.c.ar_coef[e] : 1.0);
        // an all-reduce over one device costs nothing, whatever its bytes
        // (zero weights keep an overflowing byte term out: 0 * inf is NaN)
        s_ct[1][e][k] = make_double2(e <= 1 ? 0.0 : (cmp ? a.c.inv_b : a.c.inv_l), cmp ? a.c.inv_f : 0.0);
    }

    const int64_t c = (int64_t)blockIdx.x * kBlock + tid;
    const bool active = c < a.n_cand;
    // the fast path compares live bytes as fp64 bit patterns, which order
    // like the integers below 2^63 - 2^52: a lane starting at 2^62 or more
    // live bytes on a device (its ops add less than 2^43) takes the general path
    bool big_init = false;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        const uint64_t init = (active && a.init_live) ? a.init_live[c * ND + d] : 0;
        big_init |= init >= (1ull << 62);
        s_mem[d][tid] = make_ulonglong2(init, init);
    }
    __syncthreads();

    uint32_t nops = active ? (a.n_ops ? a.n_ops[c] : (uint32_t)a.max_ops) : 0xffffffffu;
    // a lane whose op count exceeds max_ops is flagged and simulates max_ops
    // ops; the flag survives the general path's restart (st0)
    const int32_t st0 = (active && nops > (uint32_t)a.max_ops) ? DSIM_ST_BAD_OP : 0;
    int32_t st = st0;
    if (st0) nops = (uint32_t)a.max_ops;
    // ops every lane of the wavefront has (inactive lanes do not constrain it)
    uint32_t wave_min = nops;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wave_min = min(wave_min, (uint32_t)__shfl_xor((int)wave_min, off));
    if (!active) return;
    double clk[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) clk[d] = 0.0;

    const size_t N = (size_t)a.n_cand;

    // ---- fast path: the ops every lane of the wavefront has ------------------
    // Ops are assumed valid; a cheap test marks any lane that meets an op it
    // cannot vouch for, and that lane is re-simulated by the general path below.
    // Indices are clamped so that even an invalid op stays inside the arrays.
    // (with nodes or streams, communication costs depend on which devices an
    // op spans, and a MatMul regression makes two costs of compute ops: every
    // op takes the general path; so do tables of more than kMaxFastCand
    // candidates, whose op rows are too far apart for the 32-bit offsets of
    // the fast path's loads)
    const int32_t fast_end = (a.c.mm || a.c.node || a.c.streams || a.n_cand > kMaxFastCand)
                                 ? 0
                                 : (int32_t)(__builtin_amdgcn_readfirstlane(wave_min) / kUnroll) * kUnroll;

    const size_t blk = (size_t)blockIdx.x * kBlock;
    const uint32_t lane_b = (uint32_t)tid * 4u;
    bool suspect = big_init;
    uint32_t fb_max = 0;   // largest flops or bytes bit pattern met on the fast path

    // two register sets of kUnroll op records: one is processed while the
    // other is in flight
    uint32_t cdA[kUnroll], flA[kUnroll], byA[kUnroll], alA[kUnroll], frA[kUnroll];
    uint32_t cdB[kUnroll], flB[kUnroll], byB[kUnroll], alB[kUnroll], frB[kUnroll];
    // One buffer descriptor per field and group of kUnroll op rows (based at
    // this workgroup's first record); op u of the group is u*N records
    // further, a scalar offset.
    const uint32_t row_bytes = (uint32_t)(N * 4u);
    const uint32_t grp_bytes = (uint32_t)min((size_t)0xffffffffu, (size_t)kUnroll * N * 4u);
    auto load_group = [&](int32_t j0, uint32_t(&cd)[kUnroll], uint32_t(&fl)[kUnroll], uint32_t(&by)[kUnroll],
                          uint32_t(&al)[kUnroll], uint32_t(&fr)[kUnroll]) {
        const size_t base = (size_t)j0 * N + blk;
        const __amdgpu_buffer_rsrc_t rc = group_rsrc(a.code + base, grp_bytes);
        const __amdgpu_buffer_rsrc_t rf = group_rsrc(a.flops + base, grp_bytes);
        const __amdgpu_buffer_rsrc_t rb = group_rsrc(a.bytes + base, grp_bytes);
        const __amdgpu_buffer_rsrc_t ra = group_rsrc(a.alloc + base, grp_bytes);
        const __amdgpu_buffer_rsrc_t rr = group_rsrc(a.freeb + base, grp_bytes);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int so = (int)(u * row_bytes);
            cd[u] = __builtin_amdgcn_raw_buffer_load_b32(rc, (int)lane_b, so, kNonTemporal);
            fl[u] = __builtin_amdgcn_raw_buffer_load_b32(rf, (int)lane_b, so, kNonTemporal);
            by[u] = __builtin_amdgcn_raw_buffer_load_b32(rb, (int)lane_b, so, kNonTemporal);
            al[u] = __builtin_amdgcn_raw_buffer_load_b32(ra, (int)lane_b, so, kNonTemporal);
            fr[u] = __builtin_amdgcn_raw_buffer_load_b32(rr, (int)lane_b, so, kNonTemporal);
        }
    };
    auto run_group = [&](const uint32_t(&cd)[kUnroll], const uint32_t(&fl)[kUnroll],
                         const uint32_t(&by)[kUnroll], const uint32_t(&al)[kUnroll],
                         const uint32_t(&fr)[kUnroll]) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            // Everything below is computed for every lane and combined with
            // selects, so the wavefront runs one straight sequence whatever
            // the op kinds of its lanes.
            const uint32_t code = cd[u];
            const uint32_t ia = (code >> 8) & 0xffu, ib = (code >> 16) & 0xffu;
            bool is_c, is_s, is_a;
            if constexpr ((ND & (ND - 1)) == 0) {
                // one masked compare per kind tests the reserved byte, the
                // kind and the device fields that must be < ND at once; an
                // op that passes none is invalid, and the selects below
                // treat it as an all-reduce over its (clamped) fields
                constexpr uint32_t hi = ~(uint32_t)(ND - 1) & 0xffu;
                constexpr uint32_t m0 = 0xff0000ffu | (hi << 8), m1 = m0 | (hi << 16), m2 = 0xff0000ffu;
                is_c = (code & m0) == 0u;
                is_s = (code & m1) == 1u;
                is_a = (code & m2) == 2u;
                const uint32_t ma = ib & ((1u << ND) - 1u);
                suspect |= !(is_c | (is_s & (ia != ib)) | (is_a & (ma != 0u) & (ib == ma)));
            } else {
                const uint32_t kind = code & 0xffu;
                is_c = kind == 0u;
                is_s = kind == 1u;
                is_a = kind == 2u;
                suspect |= (code >= (1u << 24)) | (kind > 2u) | ((ia >= (uint32_t)ND) & !is_a) |
                           (is_s & ((ib >= (uint32_t)ND) | (ia == ib))) | (is_a & ((ib == 0u) | (ib >= (1u << ND))));
            }
            // flops and bytes must be finite and >= 0: as integers, below
            // the bits of +inf (negative values have the sign bit set)
            fb_max = max(fb_max, max(fl[u], by[u]));
            const uint32_t ias = min(ia, (uint32_t)ND - 1u), ibs = min(ib, (uint32_t)ND - 1u);
            const uint32_t mc = 1u << ias, ms = mc | (1u << ibs), ma = ib & ((1u << ND) - 1u);
            const uint32_t m = is_c ? mc : (is_s ? ms : ma);

            // op cost (Sec. 3.3 / Sec. 4 cost functions) as base + coef * x:
            // compute (launch, 1, max(flops/F, bytes/B)), send (lat, 1,
            // bytes/L), all-reduce over n devices (ar_lat[n], ar_coef[n],
            // bytes/L); multiplying by 1.0 is exact
            const uint32_t idx = is_c ? (uint32_t)ND + 1u : (is_s ? (uint32_t)ND + 2u : (uint32_t)__popc(m));
            const double2 bc = s_ct[0][idx][tid & (kCopies - 1)], rw = s_ct[1][idx][tid & (kCopies - 1)];
            // a non-compute class carries 0 as its flop reciprocal: a valid
            // op's flops are finite, so that term is +0 and the max is the
            // bandwidth term, as in the per-kind formulas
            const double f = (double)__uint_as_float(fl[u]), b = (double)__uint_as_float(by[u]);
            const double cost = bc.x + bc.y * max_nn(f * rw.y, b * rw.x);

            // synchronous start on the device set, common end.  Bit 31 of
            // xs[d] is set for a device outside the op; the clocks take it
            // as their sign, so the max over all of them is the max over the
            // participants (clocks are >= 0: outside clocks become <= -0.0,
            // below every participant's).  The update takes max(|clk|, e)
            // with e = end for a participant and -end outside: participants
            // (clk <= start <= end) get end, the others keep their clock,
            // bit-exact.  A clock may come out as -0.0 (max of +0.0 and
            // -0.0), which compares equal to 0.0; the epilogue adds +0.0
            // to every stored clock.
            const uint32_t nm = ~m;
            uint32_t xs[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) xs[d] = nm << (31 - d);
#pragma unroll
            for (int d = 0; d < ND; ++d) clk[d] = with_sign(clk[d], xs[d]);
            // pairwise max tree (max is exact, so the order does not matter)
            double v[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) v[d] = clk[d];
#pragma unroll
            for (int w = 1; w < ND; w *= 2)
#pragma unroll
                for (int d = 0; d + w < ND; d += 2 * w) v[d] = max_nn(v[d], v[d + w]);
            const double end = v[0] + cost;
#pragma unroll
            for (int d = 0; d < ND; ++d) clk[d] = max_abs(clk[d], with_sign(end, xs[d]));

            // live memory: allocate on the target, sample, free on the
            // source (an all-reduce moves no memory).  A free that would
            // underflow marks the lane for the exact path.
            const uint32_t alloc = is_a ? 0u : al[u];
            const uint32_t fre = is_a ? 0u : fr[u];
            const uint32_t tdev = is_s ? ibs : ias;
            const uint32_t fdev = ias;
            const ulonglong2 tm = s_mem[tdev][tid];
            const uint64_t lt = tm.x + (uint64_t)alloc;
            s_mem[tdev][tid] = make_ulonglong2(lt, max_bits(lt, tm.y));
            // read after that write: a compute op frees on the device it
            // allocated on, and sees its own allocation
            const uint64_t lf = s_mem[fdev][tid].x;
            suspect |= (uint64_t)fre > lf;
            s_mem[fdev][tid].x = lf - (uint64_t)fre;
        }
    };
    if (fast_end > 0) load_group(0, cdA, flA, byA, alA, frA);
    for (int32_t j0 = 0; j0 < fast_end; j0 += 2 * kUnroll) {
        if (j0 + kUnroll < fast_end) load_group(j0 + kUnroll, cdB, flB, byB, alB, frB);
        run_group(cdA, flA, byA, alA, frA);
        if (j0 + kUnroll >= fast_end) break;
        if (j0 + 2 * kUnroll < fast_end) load_group(j0 + 2 * kUnroll, cdA, flA, byA, alA, frA);
        run_group(cdB, flB, byB, alB, frB);
    }

    suspect |= fb_max >= 0x7f800000u;

    // ---- general path: this lane's remaining ops, or all of them again if
    // the fast path met an op it could not vouch for ---------------------------
    int32_t from = fast_end;
    if (suspect) {
        from = 0;
        st = st0;
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            clk[d] = 0.0;
            // read again rather than kept in registers across the fast path
            const uint64_t init = a.init_live ? a.init_live[c * ND + d] : 0;
            s_mem[d][tid] = make_ulonglong2(init, init);
        }
    }
    // the wavefront's range: from its earliest lane to its longest program
    int32_t lo = 0, end = 0;
    if (__ballot(from < (int32_t)nops) != 0) {
        lo = from < (int32_t)nops ? from : INT_MAX;
        end = from < (int32_t)nops ? (int32_t)nops : 0;
        const uint64_t here = __ballot(true);   // (lanes past n_cand have left)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const int32_t l2 = __shfl_xor(lo, off), e2 = __shfl_xor(end, off);
            const bool there = ((here >> ((tid & 63) ^ off)) & 1) != 0;
            lo = there && l2 < lo ? l2 : lo;
            end = there && e2 > end ? e2 : end;
        }
        lo = __builtin_amdgcn_readfirstlane(lo);
        end = __builtin_amdgcn_readfirstlane(end);
        // every wavefront that comes here writes the same rows
        const int rank = __popcll(here & ((1ull << (tid & 63)) - 1ull)), lanes = __popcll(here);
        for (int i = rank; i < kCostRows; i += lanes) s_row[i] = cost_row(a.c, i);
        __builtin_amdgcn_wave_barrier();
    }
    const bool with_k = a.c.mm && a.mm_k;
    const uint32_t *k_arr = with_k ? a.mm_k : a.code;   // (its values go unused then)
    auto load_any = [&](int32_t j0, uint32_t(&cd)[kUnroll], uint32_t(&fl)[kUnroll], uint32_t(&by)[kUnroll],
                        uint32_t(&al)[kUnroll], uint32_t(&fr)[kUnroll], uint32_t(&mk)[kUnroll]) {
        // (rows past the tables' last one read it again, so that no load is
        // conditional; scalar row bases, any n_cand)
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const size_t base = (size_t)min(j0 + u, a.max_ops - 1) * N + blk;
            cd[u] = __builtin_nontemporal_load(a.code + base + tid);
            fl[u] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(a.flops) + base + tid);
            by[u] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(a.bytes) + base + tid);
            al[u] = __builtin_nontemporal_load(a.alloc + base + tid);
            fr[u] = __builtin_nontemporal_load(a.freeb + base + tid);
            mk[u] = __builtin_nontemporal_load(k_arr + base + tid);
        }
    };
    auto run_any = [&](int32_t j0, const uint32_t(&cd)[kUnroll], const uint32_t(&fl)[kUnroll],
                       const uint32_t(&by)[kUnroll], const uint32_t(&al)[kUnroll], const uint32_t(&fr)[kUnroll],
                       const uint32_t(&mk)[kUnroll]) {
        // all ops decoded first (they do not depend on one another), then
        // the clocks, then the counters
        TabOp o[kUnroll];
        bool many = false;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int32_t j = j0 + u;
            o[u] = decode<ND>(a, s_row, cd[u], fl[u], by[u], with_k ? mk[u] : 0u, (j >= from) & (j < (int32_t)nops));
            st |= (int32_t)o[u].flag;
            many |= ((o[u].am & (o[u].am - 1u)) | (o[u].fm & (o[u].fm - 1u))) != 0u;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            // the fast path's update (an op that is skipped has no members:
            // every clock stays)
            const uint32_t nm = ~o[u].m;
            uint32_t xs[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) xs[d] = nm << (31 - d);
            double v[ND];
#pragma unroll
            for (int d = 0; d < ND; ++d) v[d] = clk[d] = with_sign(clk[d], xs[d]);
#pragma unroll
            for (int w = 1; w < ND; w *= 2)
#pragma unroll
                for (int d = 0; d + w < ND; d += 2 * w) v[d] = max_nn(v[d], v[d + w]);
            const double e = v[0] + o[u].cost;
#pragma unroll
            for (int d = 0; d < ND; ++d) clk[d] = max_abs(clk[d], with_sign(e, xs[d]));
        }
        // every allocation is sampled (a member that allocates nothing is at
        // or below its peak already), then the frees
        auto alloc_on = [&](int d, uint64_t by) {
            ulonglong2 t = s_mem[d][tid];
            t.x += by;
            t.y = t.x > t.y ? t.x : t.y;
            s_mem[d][tid] = t;
        };
        auto free_on = [&](int d, uint64_t by) {
            const uint64_t lf = s_mem[d][tid].x;
            st |= by > lf ? DSIM_ST_MEM_UNDERFLOW : 0;
            s_mem[d][tid].x = by > lf ? 0 : lf - by;
        };
        if (__ballot(many) == 0) {
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                alloc_on(o[u].am ? __ffs(o[u].am) - 1 : 0, o[u].am ? al[u] : 0u);
                free_on(o[u].fm ? __ffs(o[u].fm) - 1 : 0, o[u].fm ? fr[u] : 0u);
            }
        } else {   // a broadcast or reduce record among the lanes
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                for (uint32_t q = o[u].am; q != 0u; q &= q - 1u) alloc_on(__ffs(q) - 1, al[u]);
                for (uint32_t q = o[u].fm; q != 0u; q &= q - 1u) free_on(__ffs(q) - 1, fr[u]);
            }
        }
    };
    if (lo < end) {
        uint32_t cd0[kUnroll], fl0[kUnroll], by0[kUnroll], al0[kUnroll], fr0[kUnroll], mk0[kUnroll];
        uint32_t cd1[kUnroll], fl1[kUnroll], by1[kUnroll], al1[kUnroll], fr1[kUnroll], mk1[kUnroll];
        load_any(lo, cd0, fl0, by0, al0, fr0, mk0);
        for (int32_t j0 = lo; j0 < end; j0 += 2 * kUnroll) {
            load_any(j0 + kUnroll, cd1, fl1, by1, al1, fr1, mk1);
            run_any(j0, cd0, fl0, by0, al0, fr0, mk0);
            if (j0 + kUnroll >= end) break;
            load_any(j0 + 2 * kUnroll, cd0, fl0, by0, al0, fr0, mk0);
            run_any(j0 + kUnroll, cd1, fl1, by1, al1, fr1, mk1);
        }
    }

    double mk = 0.0;
    uint64_t cp = 0;
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        mk = clk[d] > mk ? clk[d] : mk;
        const uint64_t p = s_mem[d][tid].y;
        cp = p > cp ? p : cp;
    }
    if (a.c.cap != 0 && cp > a.c.cap) st |= DSIM_ST_OVER_CAP;
    a.makespan[c] = mk;
    a.cand_peak[c] = cp;
    a.status[c] = st;
    if (a.n_ops_out) a.n_ops_out[c] = nops;
    if (a.walked) a.walked[c] = nops;
    if (a.finish) {
        double *row = a.finish + (size_t)c * a.row_width;
#pragma unroll
        for (int d = 0; d < ND; ++d) row[d] = clk[d] + 0.0;   // -0.0 -> +0.0
        for (int d = ND; d < a.row_width; ++d) row[d] = 0.0;
    }
    if (a.peak) {
        uint64_t *row = a.peak + (size_t)c * a.row_width;
#pragma unroll
        for (int d = 0; d < ND; ++d) row[d] = s_mem[d][tid].y;
        for (int d = ND; d < a.row_width; ++d) row[d] = 0;
    }
}

// max / or over the eight lanes of a candidate, in every one of them: lanes 1
// and 2 apart, then the other half of the eight (mirrored)
template <int CTRL> __device__ __forceinline__ uint32_t dpp8(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ uint64_t dpp8(uint64_t v)
{
    return ((uint64_t)dpp8<CTRL>((uint32_t)(v >> 32)) << 32) | dpp8<CTRL>((uint32_t)v);
}
template <int CTRL> __device__ __forceinline__ double dpp8(double v)
{
    return __longlong_as_double((long long)dpp8<CTRL>((uint64_t)__double_as_longlong(v)));
}
template <class T, class Op> __device__ __forceinline__ T over8(T v, Op op)
{
    v = op(v, dpp8<0xb1>(v));
    v = op(v, dpp8<0x4e>(v));
    return op(v, dpp8<0x141>(v));
}
// lane U's value of each eight: broadcast within each four lanes, then the
// other four take it mirrored (vector moves; ds_swizzle does it in one, but
// through the LDS pipe)
template <int U> __device__ __forceinline__ uint32_t from8(uint32_t v)
{
    constexpr int q = U & 3;
    const int t = __builtin_amdgcn_update_dpp(0, (int)v, q | (q << 2) | (q << 4) | (q << 6), 0xf, 0xf, true);
    return (uint32_t)__builtin_amdgcn_update_dpp(t, t, 0x141, 0xf, U < 4 ? 0xa : 0x5, false);
}

constexpr int kGroup = 8;

// One candidate per eight lanes, lane d its device d.  Each round the eight
// lanes load and decode one op each (two rounds ahead in flight) and then
// take the eight ops in order: the op's masks, cost and sizes from the lane
// that decoded it, the start as a maximum over the lanes, clock and counters
// in registers.
template <int ND> __global__ __launch_bounds__(64) void k_sim_tables_group(const TabArgs a)
{
    __shared__ CostRow s_row[kCostRows];
    const int lane = threadIdx.x, d = lane & (kGroup - 1);
    if (lane < kCostRows) s_row[lane] = cost_row(a.c, lane);
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * (64 / kGroup) + lane / kGroup;
    const bool active = c < a.n_cand;
    const size_t N = (size_t)a.n_cand;
    uint32_t nops = active ? (a.n_ops ? a.n_ops[c] : (uint32_t)a.max_ops) : 0u;
    uint32_t st = 0;
    if (nops > (uint32_t)a.max_ops) {   // flagged, and max_ops ops are simulated
        st = DSIM_ST_BAD_OP;
        nops = (uint32_t)a.max_ops;
    }
    uint32_t end = nops;
#pragma unroll
    for (int off = 32; off >= kGroup; off >>= 1) end = max(end, (uint32_t)__shfl_xor((int)end, off));
    end = (uint32_t)__builtin_amdgcn_readfirstlane((int)end);
    const bool with_k = a.c.mm && a.mm_k;

    double clk = 0.0;
    uint64_t live = (active && d < ND && a.init_live) ? a.init_live[c * ND + d] : 0;
    uint64_t peak = live;

    struct Rec {
        uint32_t cd, fl, by, al, fr, mk;
    };
    // (loads are unconditional: past the end they read the last row or
    // candidate again, and decode ignores them)
    const uint32_t *k_arr = with_k ? a.mm_k : a.code;
    const size_t cl = active ? (size_t)c : N - 1;
    auto load = [&](uint32_t j) {
        const size_t o = (size_t)min(j, (uint32_t)a.max_ops - 1u) * N + cl;
        return Rec{a.code[o], __float_as_uint(a.flops[o]), __float_as_uint(a.bytes[o]), a.alloc[o], a.freeb[o], k_arr[o]};
    };
    auto run = [&](uint32_t j0, const Rec &r) {
        const TabOp o = decode<ND>(a, s_row, r.cd, r.fl, r.by, with_k ? r.mk : 0u, j0 + d < nops);
        st |= o.flag;
        const uint32_t masks = o.m | (o.am << 8) | (o.fm << 16);
        const uint64_t cb = (uint64_t)__double_as_longlong(o.cost);
        auto take = [&](auto u) {
            constexpr int U = decltype(u)::value;
            const uint32_t mm = from8<U>(masks);
            const double cost = bits_double(from8<U>((uint32_t)cb), from8<U>((uint32_t)(cb >> 32)));
            const uint32_t al = from8<U>(r.al), fr = from8<U>(r.fr);
            const uint32_t me = mm >> d;
            const bool in = (me & 1u) != 0u;
            const double start = over8(in ? clk : 0.0, [](double x, double y) { return max_nn(x, y); });
            const double e = start + cost;
            clk = in ? e : clk;
            live += (uint64_t)((me & 0x100u) ? al : 0u);
            peak = live > peak ? live : peak;
            const uint64_t f = (uint64_t)((me & 0x10000u) ? fr : 0u);
            const bool under = f > live;
            st |= under ? (uint32_t)DSIM_ST_MEM_UNDERFLOW : 0u;
            live = under ? 0 : live - f;
        };
        take(std::integral_constant<int, 0>());
        take(std::integral_constant<int, 1>());
        take(std::integral_constant<int, 2>());
        take(std::integral_constant<int, 3>());
        take(std::integral_constant<int, 4>());
        take(std::integral_constant<int, 5>());
        take(std::integral_constant<int, 6>());
        take(std::integral_constant<int, 7>());
    };
    // (each set is loaded again right after its use: copying a set whose
    // loads are in flight would wait for them)
    if (end > 0) {
        Rec r0 = load(d), r1 = load(kGroup + d);
        for (uint32_t j0 = 0; j0 < end; j0 += 2 * kGroup) {
            run(j0, r0);
            r0 = load(j0 + 2 * kGroup + d);
            run(j0 + kGroup, r1);
            r1 = load(j0 + 3 * kGroup + d);
        }
    }

    const double mk = over8(clk, [](double x, double y) { return max_nn(x, y); });
    const uint64_t cp = over8(peak, [](uint64_t x, uint64_t y) { return x > y ? x : y; });
    st = over8(st, [](uint32_t x, uint32_t y) { return x | y; });
    if (!active) return;
    if (d == 0) {
        if (a.c.cap != 0 && cp > a.c.cap) st |= DSIM_ST_OVER_CAP;
        a.makespan[c] = mk;
        a.cand_peak[c] = cp;
        a.status[c] = (int32_t)st;
        if (a.n_ops_out) a.n_ops_out[c] = nops;
        if (a.walked) a.walked[c] = nops;
    }
    if (a.finish)
        for (int i = d; i < a.row_width; i += kGroup) a.finish[(size_t)c * a.row_width + i] = i < ND ? clk : 0.0;
    if (a.peak)
        for (int i = d; i < a.row_width; i += kGroup) a.peak[(size_t)c * a.row_width + i] = i < ND ? peak : 0;
}

// Calls of at most this many candidates take eight lanes each.  256 random
// ops over 8 devices, eight lanes against one: 36 / 76 us at 640 candidates,
// 37 / 86 at 8,192 (one wavefront per SIMD), 59 / 88 at 16,384, 124 / 89 at
// 32,768; where every op takes the general path 39 / 175, 39 / 172, 62 / 173,
// 121 / 173, and 224 / 176 at 65,536.
constexpr int64_t kGroupCand = 20480, kGroupCandGeneral = 45056;

template <int ND>
hipError_t launch_nd(const TabArgs &a, hipStream_t s)
{
    const bool general = a.c.mm || a.c.node || a.c.streams;
    if (a.n_cand <= (general ? kGroupCandGeneral : kGroupCand)) {
        const int64_t blocks = (a.n_cand * kGroup + 63) / 64;
        hipLaunchKernelGGL(k_sim_tables_group<ND>, dim3((unsigned)blocks), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    const int64_t blocks = (a.n_cand + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_sim_tables<ND>, dim3((unsigned)blocks), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

}  // namespace

dsim_status launch_sim_tables(const dsim_tables &t, int64_t n_cand, const CostConsts &c,
                              const dsim_results &r, hipStream_t s)
{
    if (n_cand == 0) return DSIM_OK;
    TabArgs a;
    a.code = t.code;
    a.flops = t.flops;
    a.bytes = t.bytes;
    a.alloc = t.alloc_bytes;
    a.freeb = t.free_bytes;
    a.n_ops = t.n_ops;
    a.init_live = t.init_live;
    a.mm_k = t.mm_k;
    a.n_cand = n_cand;
    a.max_ops = t.max_ops;
    a.row_width = r.row_width;
    a.makespan = r.makespan;
    a.finish = r.finish;
    a.peak = r.peak;
    a.cand_peak = r.cand_peak;
    a.n_ops_out = r.n_ops;
    a.walked = r.walked_ops;
    a.status = r.status;
    a.c = c;
    a.gpu_of = a.node_of = 0;
    for (int d = 0; d < kMaxTableDev; ++d) {
        const uint32_t gpu = (uint32_t)(c.streams ? d / c.streams : d);
        a.gpu_of |= gpu << (4 * d);
        a.node_of |= (c.node ? gpu / (uint32_t)c.node : 0u) << (4 * d);
    }
    hipError_t e;
    switch (t.n_dev) {
    case 1: e = launch_nd<1>(a, s); break;
    case 2: e = launch_nd<2>(a, s); break;
    case 3: e = launch_nd<3>(a, s); break;
    case 4: e = launch_nd<4>(a, s); break;
    case 5: e = launch_nd<5>(a, s); break;
    case 6: e = launch_nd<6>(a, s); break;
    case 7: e = launch_nd<7>(a, s); break;
    default: e = launch_nd<8>(a, s); break;
    }
    return e == hipSuccess ? DSIM_OK : hip_fail(e, "sim_tables launch");
}

}  // namespace dsim
