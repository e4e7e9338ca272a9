// gen_tables.hip -- the random-program workload, generated on the GPU.
//
// One lane per candidate writes its op records in program order, straight
// into the op-major / candidate-fastest table layout (coalesced stores).
//
// Every random decision is a pure function of (seed, candidate, op, field):
// draw f of op j of candidate c is output number c*2^32 + j*32 + f + 1 of
// SplitMix64 (Steele, Lea & Flood, OOPSLA 2014) seeded with `seed`, i.e.
// mix(seed + n * 0x9E3779B97F4A7C15).  Fields:
//   0 op kind: floor(hi32 * 10 / 2^32): 0..6 compute, 7..8 send, 9 all-reduce
//   1 device a: uniform in [0, n_dev)
//   2 send: destination a + 1 + uniform[0, n_dev - 1) mod n_dev;
//     all-reduce: index into the ascending list of masks with >= 2 bits
//   3 compute FLOPs, log-uniform in [1e6, 1e12]
//   4 compute / all-reduce bytes, log-uniform in [1e3, 1e9]
//   5 compute / send: free one of device a's live buffers (top bit = coin,
//     low 32 bits pick the buffer uniformly; the last buffer moves into the
//     hole)
//   6 compute: allocate a new buffer on a (top bit = coin, if a has < 16)
//   7 size of the new buffer (compute) or of the message (send), log-uniform
//     in [1e3, 1e9] bytes; a send's message becomes a live buffer of the
//     destination when the destination has < 16
// Log-uniform in [lo, hi]: 2^t rounded once to fp32, t = log2(lo) + u
// (log2(hi) - log2(lo)) with u the top 53 bits of the draw over 2^53 and
// the logarithms taken as the nearest doubles; 2^t = 2^floor(t) e^(y),
// y = (t - floor(t)) ln 2, e^y summed as its Taylor series up to y^13
// (Horner form, fp64, no contraction: the oracle computes the same bits).
#include "internal.h"

namespace dsim {
namespace {

constexpr int kGenBlock = 64;
constexpr int kSlots = 16;
// Unused slots that make a block's share of the LDS 40 KB: a CU then holds
// four wavefronts, one per SIMD.  With 32 KB it holds five, one SIMD runs two
// of them at half speed and the others wait for it (1.48 against 1.95 ms at
// 250,000 x 512 records; 16-bit buffers, the size drawn again when one is
// freed, and two wavefronts per SIMD: 1% less, but for 65,536 ops at most).
constexpr int kPad = 4;

struct GenArgs {
    uint64_t seed;
    int64_t n_cand;
    int32_t n_ops, n_dev;
    uint32_t *code;
    float *flops;
    float *bytes;
    uint32_t *alloc;
    uint32_t *freeb;
    uint32_t *n_ops_out;
};

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
// SplitMix64's output for the state z
__device__ __forceinline__ uint64_t mix(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint32_t pick(uint64_t r, uint32_t n)
{
    return (uint32_t)(((r >> 32) * (uint64_t)n) >> 32);
}

// base-2 logarithms of the bounds (nearest doubles)
constexpr double kLog2_1e3 = 0x1.3ee7b471b3a95p+3, kLog2_1e6 = 0x1.3ee7b471b3a95p+4;
constexpr double kLog2_1e9 = 0x1.de5b8eaa8d7e0p+4, kLog2_1e12 = 0x1.3ee7b471b3a95p+5;

__device__ __forceinline__ float log_uniform(uint64_t r, double log2_lo, double log2_hi)
{
    // 1 / k! for k = 13 down to 0
    constexpr double c[14] = {0x1.6124613a86d09p-33, 0x1.1eed8eff8d898p-29, 0x1.ae64567f544e4p-26,
                              0x1.27e4fb7789f5cp-22, 0x1.71de3a556c734p-19, 0x1.a01a01a01a01ap-16,
                              0x1.a01a01a01a01ap-13, 0x1.6c16c16c16c17p-10, 0x1.1111111111111p-7,
                              0x1.5555555555555p-5, 0x1.5555555555555p-3, 0.5, 1.0, 1.0};
    const double u = (double)(r >> 11) * 0x1p-53;
    const double t = log2_lo + u * (log2_hi - log2_lo);
    const double n = floor(t);
    const double y = (t - n) * 0x1.62e42fefa39efp-1;
    double e = c[0];
#pragma unroll
    for (int k = 1; k < 14; ++k) e = e * y + c[k];
    return (float)ldexp(e, (int)n);
}

// The k-th number (k = 0, 1, ...) with two bits set or more: m is number
// m - 2 - floor(log2 m) of them, so m = k + 2 + floor(log2 m), and the
// logarithm of k + 2 is that of m or one less.
__device__ __forceinline__ uint32_t nth_mask(uint32_t k)
{
    const uint32_t m = k + 33u - (uint32_t)__clz((int)(k + 2u));
    return k + 33u - (uint32_t)__clz((int)m);
}

// Bound by vector issue: the draws' 64-bit products and the three powers of
// two per op are about 1,700 cycles of a SIMD for 64 records.  So every op
// kind shares one straight sequence -- the draws that only one kind needs
// take each other's places (flops / destination / mask; bytes / message), a
// draw's state is the op's plus a constant -- where three divergent branches
// ran eleven draws and five powers; the buffer counts are bytes of one
// register pair.  250,000 x 512 records over 8 devices: 2.29 -> 1.48 ms
// (2.6 GB of records: a fill of that size takes 0.37 ms).
__global__ __launch_bounds__(kGenBlock) void k_gen_tables(const GenArgs g)
{
    __shared__ uint32_t s_buf[8][kSlots + kPad][kGenBlock];
    const int tid = threadIdx.x;
    const int64_t cand = (int64_t)blockIdx.x * kGenBlock + tid;
    if (cand >= g.n_cand) return;

    const uint32_t nd = (uint32_t)g.n_dev;
    const uint32_t n_masks = (1u << nd) - 1u - nd;   // masks of two devices or more
    const size_t N = (size_t)g.n_cand;
    // the state of draw 0 of op j is that of op 0 plus 32 j kGamma
    uint64_t z = g.seed + (((uint64_t)cand << 32) + 1u) * kGamma;
    uint64_t counts = 0;   // live buffers, a byte per device

    // an op's draws: everything that does not depend on the live buffers
    struct Op {
        uint32_t code, a, b, size, which;
        float fl, by;
        bool frees, allocs, is_s;
    };
    auto draw = [&](uint64_t zj) {
        Op o;
        const uint32_t kd = pick(mix(zj), 10u);
        const bool is_c = kd < 7u;
        o.is_s = kd == 7u || kd == 8u;
        const uint32_t a = pick(mix(zj + kGamma), nd);
        const uint64_t r_a = mix(zj + (is_c ? 3u * kGamma : 2u * kGamma));     // flops; destination; mask
        const uint64_t r_b = mix(zj + (o.is_s ? 7u * kGamma : 4u * kGamma));   // bytes; message
        const uint64_t r5 = mix(zj + 5u * kGamma), r6 = mix(zj + 6u * kGamma), r7 = mix(zj + 7u * kGamma);
        const float fl = log_uniform(r_a, kLog2_1e6, kLog2_1e12);
        const float v = log_uniform(r_b, kLog2_1e3, kLog2_1e9);
        const float size = log_uniform(r7, kLog2_1e3, kLog2_1e9);
        const uint32_t msg = (uint32_t)v;
        uint32_t b = a + 1u + pick(r_a, nd - 1u);
        b = b >= nd ? b - nd : b;
        const uint32_t mask = nth_mask(pick(r_a, n_masks));
        o.code = is_c ? a << 8 : (o.is_s ? 1u | (a << 8) | (b << 16) : 2u | (mask << 16));
        o.fl = is_c ? fl : 0.f;
        o.by = o.is_s ? (float)msg : v;
        o.a = a;
        o.b = o.is_s ? b : a;   // the device that allocates
        o.size = o.is_s ? msg : (uint32_t)size;
        o.frees = (is_c || o.is_s) && (r5 >> 63) != 0;
        o.which = (uint32_t)r5;
        o.allocs = o.is_s || (is_c && (r6 >> 63) != 0);
        return o;
    };
    // free a live buffer of a, then allocate one on a (compute) or b (send)
    auto apply = [&](const Op &p, int32_t j) {
        uint32_t fr = 0, al = 0;
        const uint32_t na = (uint32_t)(counts >> (8u * p.a)) & 0xffu;
        if (p.frees && na > 0u) {
            const uint32_t i = (uint32_t)(((uint64_t)p.which * (uint64_t)na) >> 32);
            fr = s_buf[p.a][i][tid];
            s_buf[p.a][i][tid] = s_buf[p.a][na - 1u][tid];
            counts -= 1ull << (8u * p.a);
        }
        const uint32_t nt = (uint32_t)(counts >> (8u * p.b)) & 0xffu;
        if (p.allocs && nt < (uint32_t)kSlots) {
            al = p.size;
            s_buf[p.b][nt][tid] = al;
            counts += 1ull << (8u * p.b);
        }
        const size_t o = (size_t)j * N + (size_t)cand;
        __builtin_nontemporal_store(p.code, g.code + o);
        __builtin_nontemporal_store(p.fl, g.flops + o);
        __builtin_nontemporal_store(p.by, g.bytes + o);
        __builtin_nontemporal_store(al, g.alloc + o);
        __builtin_nontemporal_store(fr, g.freeb + o);
    };
    // (two ops' draws together: about one wavefront runs per SIMD, and their
    // products and polynomials fill one another's latencies)
    int32_t j = 0;
    for (; j + 1 < g.n_ops; j += 2, z += 64u * kGamma) {
        const Op p0 = draw(z), p1 = draw(z + 32u * kGamma);
        apply(p0, j);
        apply(p1, j + 1);
    }
    if (j < g.n_ops) apply(draw(z), j);
    if (g.n_ops_out) g.n_ops_out[cand] = (uint32_t)g.n_ops;
}

}  // namespace

dsim_status launch_gen_tables(uint64_t seed, int64_t n_cand, int32_t n_ops, int32_t n_dev,
                              uint32_t *code, float *flops, float *bytes, uint32_t *alloc,
                              uint32_t *freeb, uint32_t *n_ops_out, hipStream_t s)
{
    if (n_cand == 0) return DSIM_OK;
    GenArgs g{seed, n_cand, n_ops, n_dev, code, flops, bytes, alloc, freeb, n_ops_out};
    const int64_t blocks = (n_cand + kGenBlock - 1) / kGenBlock;
    hipLaunchKernelGGL(k_gen_tables, dim3((unsigned)blocks), dim3(kGenBlock), 0, s, g);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? DSIM_OK : hip_fail(e, "gen_tables launch");
}

}  // namespace dsim
