// Down-sampled gradient entropy on gfx950 (GDS, Sec. IV-B; Definition 1 / Eq. (1)
// estimated with an equal-width histogram).
//
// Two streaming kernels over the sampled chunks plus nothing else:
//   k_minmax  range of the finite sample per block: per-lane min/max, wavefront DPP
//             reduction, LDS across the block's waves
//   k_hist    the blocks' ranges folded, bin index in fp32 (separately rounded subtract /
//             multiply, the scale comes from one correctly rounded division), LDS histogram
//             with lane-interleaved replicas so equal bins in one wavefront hit
//             different banks, flush to global counters, and the last block reduces
//             the counters to the Shannon entropy in fp64
// or, where one block holds the sample in one round, k_estimate_one alone; where every block of a grid takes one round
// (1 % of a transformer block), k_minmax_small and k_hist_small.
// What bounds them at a 1 % sample (0.01 to 0.5 M items): latency.  Both kernels, one after the other, for 2 M fp32
// elements of four buffers on 4096 bins: 15.8 us (22.8 before they had kernels of their own, 20.3 with a release per block and the
// library's logarithms); clock stamps in the second: 1.4 us until the items are requested, 1.0 range, 1.4 bins, 2.3 until the
// counters are added, 1.6 ticket, 2.2 the counters and their logarithms, 1.1 the block's sum and the result.
// The chunk-strided sample is read with 16-byte loads whenever chunks are a
// multiple of the vector width, so a wavefront touches whole cache lines.
// Both kernels take a list of buffers (EntGroup): the estimate is over the union
// of the buffers' samples (one entropy for a pipeline stage whose gradients are
// separate tensors); a single buffer is a list of one.  The result goes straight
// into the caller's pinned host memory when it is device-accessible.
#include "edgc_internal.h"

#include <algorithm>
#include <math.h>
#include <type_traits>

namespace edgc {

struct RangeParams {
    float lo, hi, w, scale;
};

constexpr int kMMBlock   = 256;
constexpr int kMMBlockFat = 1024;                 // large samples: one block per CU
constexpr uint64_t kBigSampleItems = 8ull << 20;  // items (16 bytes each) from which a sample counts as large
constexpr int kHistBlock = 512;
constexpr int kOneBlock = 1024;       // k_estimate_one
// k_minmax_small, k_hist_small: blocks of 512 threads, of four items each; of two up to 64 Ki items, where there are so few
// blocks that more of them do not queue up at the ticket.  Per pass, two / four items: two hidden-768 blocks (18 K items) 88.4 /
// 90.2 us, three odd matrices (35 K) 134.3 / 135.5, hidden-2048 block (126 K) 229.8 / 229.1, four buffers of 0.5 M items 23.4 /
// 20.9; 1024 threads of four items (22.4, and 94.8 on the hidden-768 blocks), 256 of four (26.6) and 512 of eight (22.5) are slower.
constexpr int kSmallBlock = 512;
constexpr uint64_t kSmallTwo = 64 << 10;
constexpr int kHistBlockFat = 1024;   // when the LDS histogram leaves room for one block per CU

// ---------------------------------------------------------------------------
// wavefront reductions with DPP row shifts / row broadcasts (64 lanes)
// ---------------------------------------------------------------------------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_move(float identity, float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(identity), __float_as_int(v),
                                                      CTRL, ROW_MASK, 0xf, false));
}

// Result is valid in lane 63 and returned to every lane through a read-lane.
template <bool IS_MIN>
__device__ __forceinline__ float wave_reduce_minmax(float v)
{
    const float id = IS_MIN ? INFINITY : -INFINITY;
#define EDGC_OP(a, b) (IS_MIN ? fminf((a), (b)) : fmaxf((a), (b)))
    v = EDGC_OP(v, (dpp_move<0x111, 0xf>(id, v)));   // row_shr:1
    v = EDGC_OP(v, (dpp_move<0x112, 0xf>(id, v)));   // row_shr:2
    v = EDGC_OP(v, (dpp_move<0x114, 0xf>(id, v)));   // row_shr:4
    v = EDGC_OP(v, (dpp_move<0x118, 0xf>(id, v)));   // row_shr:8  -> lane 15 of each row
    v = EDGC_OP(v, (dpp_move<0x142, 0xa>(id, v)));   // row_bcast:15 into rows 1 and 3
    v = EDGC_OP(v, (dpp_move<0x143, 0xc>(id, v)));   // row_bcast:31 into rows 2 and 3
#undef EDGC_OP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double v)          // v + (v of the lane that CTRL names; 0 where there is none)
{
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(b), CTRL, ROW_MASK, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(b >> 32), CTRL, ROW_MASK, 0xf, false);
    return v + __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}
__device__ __forceinline__ double wave_sum_f64(double v)
{
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    v = dpp_add<0x143, 0xc>(v);
    return v;   // lane 63
}

// ---------------------------------------------------------------------------
// sample addressing
// ---------------------------------------------------------------------------
template <typename T> struct ElemTraits;
template <> struct ElemTraits<float> {
    static __device__ __forceinline__ float widen(float x) { return x; }
};
template <> struct ElemTraits<uint16_t> {   // raw bf16 bits
    static __device__ __forceinline__ float widen(uint16_t h)
    {
        return __uint_as_float(static_cast<uint32_t>(h) << 16);
    }
};

// The VEC elements of a whole item from its 16 raw bytes.
template <typename T, int VEC>
__device__ __forceinline__ void unpack_item(const uint4& q, float (&v)[VEC])
{
    static_assert(VEC * sizeof(T) == 16, "a vector item is 16 bytes");
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int p = 0; p < 4; ++p) v[p] = __uint_as_float(w[p]);
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            v[2 * p]     = __uint_as_float(w[p] << 16);
            v[2 * p + 1] = __uint_as_float(w[p] & 0xffff0000u);
        }
    }
}

// Element index of the e-th item of the k-th sampled chunk
template <typename Sampler>      // SampleGeom or EntGroup
__device__ __forceinline__ uint64_t item_elem(const Sampler& g, uint64_t k, uint32_t e, int vec)
{
    return (g.slot + k * g.stride) * g.chunk + static_cast<uint64_t>(e) * vec;
}

// The item of one thread: item -> (k-th sampled chunk, e-th item in it), and from there in steps of a constant number of items
// without a division or a product: the element index grows by the same amount every step, and by what the sampler leaves
// out where the step ends in a later chunk.
struct ItemCursor {
    uint64_t at;            // element index
    uint64_t dat, jump;
    uint32_t e, de;
    // item `base` (the same for the whole block) + `off`; advances by `step` items
    template <typename Sampler>
    __device__ __forceinline__ void init(const Sampler& g, uint64_t base, uint32_t off, uint32_t step, int vec)
    {
        const uint32_t ipc = g.ipc;
        const uint64_t q = (base >> 32) ? base / ipc : static_cast<uint32_t>(base) / ipc;
        const uint32_t s = static_cast<uint32_t>(base - q * ipc) + off;
        const uint32_t sq = s / ipc;
        e = s - sq * ipc;
        at = item_elem(g, q + sq, e, vec);
        const uint32_t dk = step / ipc;
        de = step - dk * ipc;
        dat = dk * (g.stride * g.chunk) + static_cast<uint64_t>(de) * vec;
        jump = (g.stride - 1u) * g.chunk;
    }
    __device__ __forceinline__ void advance(uint32_t ipc)
    {
        at += dat;
        e += de;
        if (e >= ipc) { e -= ipc; at += jump; }
    }
};
// any item
template <typename Sampler>
__device__ __forceinline__ uint64_t elem_of_item(const Sampler& g, uint64_t item, int vec)
{
    const uint64_t k = (item >> 32) ? item / g.ipc : static_cast<uint32_t>(item) / g.ipc;
    return item_elem(g, k, static_cast<uint32_t>(item - k * g.ipc), vec);
}

// Memory at an address that went through integer registers: without the address space the compiler takes it for flat memory,
// whose loads count as LDS accesses too (k_wide_hist 69 against 62 us).
template <typename T> using GlobalPtr = const __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ GlobalPtr<T> global_ptr(uint64_t address) { return reinterpret_cast<GlobalPtr<T>>(address); }

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ uint4 load_item(GlobalPtr<T> p)
{
    const u32x4_t v = *reinterpret_cast<GlobalPtr<u32x4_t>>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// The first `left` < VEC elements of an item, requested together.
template <typename T, int VEC, typename Elem>
__device__ __forceinline__ void partial_item(GlobalPtr<T> at, uint64_t left, Elem&& elem)
{
    T x[VEC - 1];
#pragma unroll
    for (int p = 0; p < VEC - 1; ++p) x[p] = p < static_cast<int>(left) ? at[p] : T(0);
#pragma unroll
    for (int p = 0; p < VEC - 1; ++p)
        if (p < static_cast<int>(left)) elem(x[p]);
}

// What a wave needs to know of a group's buffers, lane l holding buffer l's (lanes past the last: an empty one at the end of
// the union): one round of loads whose addresses depend on nothing, where a walk over the argument's fields is a chain of
// them, each of a line that no cache holds yet.
__device__ __forceinline__ uint64_t readlane64(uint64_t v, uint32_t lane)
{
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(v), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(v >> 32), lane);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
struct BufferTable {
    uint64_t first, next, base, n;
    __device__ __forceinline__ void load(const EntGroup& grp)
    {
        const uint32_t lane = threadIdx.x & 63u;
        constexpr uint32_t kLast = kMaxEntGroup;
        first = grp.first[min(lane, kLast)];
        next = grp.first[min(lane + 1u, kLast)];
        base = reinterpret_cast<uint64_t>(grp.base[min(lane, kLast - 1u)]);
        n = grp.n[min(lane, kLast - 1u)];
    }
    // buffer of item `pos`, and the number of buffers that begin before item `end`
    __device__ __forceinline__ uint32_t at(uint64_t pos) const { return static_cast<uint32_t>(__popcll(__ballot(next <= pos))); }
    __device__ __forceinline__ uint32_t before(uint64_t end) const { return static_cast<uint32_t>(__popcll(__ballot(first < end))); }
};

// Up to U items per thread of a block, items [pos, end) of the union whatever buffers they are in, all requested at once.
template <typename T, int VEC, int BLOCK, int U>
struct ItemRound {
    uint4 raw[U];
    T one[U];
    GlobalPtr<T> at[U];
    uint64_t left[U];                                  // elements from the item's first on; 0: no item
    __device__ __forceinline__ void request(const EntGroup& grp, const BufferTable& tab, uint64_t pos, uint64_t end)
    {
        const uint32_t ti = tab.at(pos), t_end = tab.before(end);
        uint64_t f[U], base[U], n[U];
        if (t_end - ti <= 1) {
            const uint64_t f0 = readlane64(tab.first, ti), b0 = readlane64(tab.base, ti), n0 = readlane64(tab.n, ti);
#pragma unroll
            for (int u = 0; u < U; ++u) { f[u] = f0; base[u] = b0; n[u] = n0; }
        } else {
            uint32_t t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) t[u] = ti;
            for (uint32_t b = ti + 1; b < t_end; ++b) {
                const uint64_t fb = readlane64(tab.first, b);
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] += (pos + u * BLOCK + threadIdx.x >= fb) ? 1u : 0u;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                f[u] = __shfl(tab.first, t[u], 64);
                base[u] = __shfl(tab.base, t[u], 64);
                n[u] = __shfl(tab.n, t[u], 64);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            raw[u] = make_uint4(0u, 0u, 0u, 0u);
            one[u] = T(0);
            const uint64_t i = pos + u * BLOCK + threadIdx.x;
            const uint64_t e0 = elem_of_item(grp, i - f[u], VEC);
            at[u] = global_ptr<T>(base[u]) + e0;
            left[u] = (i < end && e0 < n[u]) ? n[u] - e0 : 0;
            if constexpr (VEC > 1) {
                if (left[u] >= VEC) raw[u] = load_item(at[u]);
            } else {
                if (left[u]) one[u] = *at[u];
            }
        }
    }
    template <typename Item, typename Elem>
    __device__ __forceinline__ void visit(Item&& item, Elem&& elem) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (VEC > 1) {
                if (left[u] >= VEC) item(raw[u]);
                else if (left[u]) partial_item<T, VEC>(at[u], left[u], elem);
            } else {
                if (left[u]) elem(one[u]);
            }
        }
    }
};

// Visits the items [begin, end) of the union of the buffers' samples (buffer i holds the items first[i] ..
// first[i + 1]), by one block: `item(raw)` gets the 16 bytes of every whole item, `elem(x)` every element of a
// partial one (the end of a buffer) and, where VEC is 1, every element; `round()` is called by the whole block after
// every round of at most U items per thread.  A round's loads are issued together.  With `ahead`, the next round's
// loads are issued before the current round is used; they need no condition, since every item before a buffer's last
// sampled chunk is whole (the chunk size is a multiple of VEC).
// Blocks share the union, not every buffer: a block's range touches one or two of the buffers of a transformer
// stage (24 buffers, 143 K elements sampled: with every buffer split among all blocks each block walked all 24, 105 us
// for the two kernels).
// A round that would touch more than two buffers (norm weights and biases) is one round over all of them, in which every
// thread finds its item's buffer; only such a round: with 31 short buffers beside one of 134 M fp32 elements the block that
// holds them takes the large one's part as every other block does (387 -> 210 us for the estimate).
template <typename T, int VEC, int BLOCK, typename Item, typename Elem, typename Round>
__device__ __forceinline__ void walk_items(const EntGroup& grp, uint64_t begin, uint64_t end, bool ahead, Item&& item,
                                           Elem&& elem, Round&& round)
{
    constexpr int U = 4;
    constexpr uint32_t STEP = U * BLOCK;
    BufferTable tab;
    tab.load(grp);
    for (uint64_t pos = begin; pos < end;) {
        const uint64_t round_end = min(end, pos + STEP);
        const uint32_t ti = tab.at(pos);
        if (tab.before(round_end) - ti > 2) {
            ItemRound<T, VEC, BLOCK, U> r;
            r.request(grp, tab, pos, round_end);
            r.visit(item, elem);
            round();
            pos = round_end;
            continue;
        }
        // else: buffer `ti` from here to its end, or the range's
        const GlobalPtr<T> g = global_ptr<T>(readlane64(tab.base, ti));
        const uint64_t n = readlane64(tab.n, ti), f0 = readlane64(tab.first, ti), next = readlane64(tab.next, ti);
        const uint64_t lb = pos - f0, le = min(end, next) - f0, items = next - f0;
        pos = f0 + le;
        const uint32_t ipc = grp.ipc;
        ItemCursor cur;
        cur.init(grp, lb, threadIdx.x, BLOCK, VEC);
        uint64_t rb = lb;                              // first item of the round
        if constexpr (VEC > 1) {
            const uint64_t fast_end = (items >= ipc) ? min(le, items - ipc) : 0;
            auto fetch = [&](uint4 (&raw)[U]) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    raw[u] = load_item(g + cur.at);
                    cur.advance(ipc);
                }
            };
            auto use = [&](const uint4 (&raw)[U]) {
#pragma unroll
                for (int u = 0; u < U; ++u) item(raw[u]);
                round();
            };
            if (ahead && rb + STEP <= fast_end) {
                // No array is left undefined on any path: with exits between the two halves of the loop body the compiler
                // reused registers of loads that one of the paths had yet to use (words 1 to 3 of three loads in four lost).
                uint4 ra[U];
                fetch(ra);
                for (; rb + 3 * STEP <= fast_end; rb += 2 * STEP) {
                    uint4 rc[U];
                    fetch(rc);
                    use(ra);
                    fetch(ra);
                    use(rc);
                }
                if (rb + 2 * STEP <= fast_end) {
                    uint4 rc[U];
                    fetch(rc);
                    use(ra);
#pragma unroll
                    for (int u = 0; u < U; ++u) ra[u] = rc[u];
                    rb += STEP;
                }
                use(ra);
                rb += STEP;
            }
            for (; rb < le; rb += STEP) {
                uint4 raw[U];
                uint64_t at[U];
                uint32_t whole = 0, partial = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    raw[u] = make_uint4(0u, 0u, 0u, 0u);
                    at[u] = cur.at;
                    if (rb + u * BLOCK + threadIdx.x < le) {
                        if (at[u] + VEC <= n) {
                            raw[u] = load_item(g + at[u]);
                            whole |= 1u << u;
                        } else if (at[u] < n) {
                            partial |= 1u << u;
                        }
                    }
                    cur.advance(ipc);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if ((whole >> u) & 1u) item(raw[u]);
                if (partial) {
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if ((partial >> u) & 1u) partial_item<T, VEC>(g + at[u], n - at[u], elem);
                }
                round();
            }
        } else {
            for (; rb < le; rb += STEP) {
                T x[U];
                uint32_t have = 0;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    x[u] = T(0);
                    const uint64_t at = cur.at;
                    if (rb + u * BLOCK + threadIdx.x < le && at < n) {
                        x[u] = g[at];
                        have |= 1u << u;
                    }
                    cur.advance(ipc);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if ((have >> u) & 1u) elem(x[u]);
                round();
            }
        }
    }
}

// The range of the union that one block of a grid visits.
__device__ __forceinline__ void block_range(const EntGroup& grp, uint64_t& begin, uint64_t& end)
{
    const uint64_t per = (grp.n_items + gridDim.x - 1) / gridDim.x;
    begin = min(static_cast<uint64_t>(blockIdx.x) * per, grp.n_items);
    end = min(begin + per, grp.n_items);
}

__device__ __forceinline__ bool finite_f32(float x)
{
    return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u;
}

// The logarithms that do not depend on the bins: of the sample's size (less e0, see entropy_base), and of a bin's width (what the
// differential entropy adds).  Formed by a wave that would otherwise wait.
struct EstimateLogs {
    double log2_n, log_w;
};
// All logarithms of an estimate are taken less this integer, the binary exponent of the sample's size:
// H = (log2 n - e0) - (1/n) sum c (log2 c - e0), without the cancellation of log2 n.
__device__ __forceinline__ int entropy_base(unsigned long long n_sampled) { return __builtin_amdgcn_frexp_exp(static_cast<double>(n_sampled)); }
// log2 of a positive integer (some finite value for 0) less the integer e0, in fp64: x = 2^e m with m in [sqrt 1/2, sqrt 2), log2 m
// from the series of artanh at s = (m - 1) / (m + 1), s^2 < 0.0295, to s^19 (what is left out is below 2^-55 of it).  Some 25 dependent
// operations and short code, which the last block of a grid runs alone and from a cold cache: the library's function, one bin after
// the other, was 3 to 4 of the 17 us that the histogram kernel of a 1 % sample took on 4096 bins.
__device__ __forceinline__ double log2_count(double x, int e0)
{
    double m = __builtin_amdgcn_frexp_mant(x);                       // [1/2, 1)
    int e = __builtin_amdgcn_frexp_exp(x);
    if (m < 0.70710678118654752440) { m += m; e -= 1; }
    const double f = m - 1.0, a = m + 1.0;
    double y = __builtin_amdgcn_rcp(a);                              // an estimate; two Newton steps, and one on the quotient
    y = fma(fma(-a, y, 1.0), y, y);
    y = fma(fma(-a, y, 1.0), y, y);
    double q = f * y;
    q = fma(fma(-a, q, f), y, q);
    const double z = q * q;
    double p = 1.0 / 19.0;
    p = fma(p, z, 1.0 / 17.0);
    p = fma(p, z, 1.0 / 15.0);
    p = fma(p, z, 1.0 / 13.0);
    p = fma(p, z, 1.0 / 11.0);
    p = fma(p, z, 1.0 / 9.0);
    p = fma(p, z, 1.0 / 7.0);
    p = fma(p, z, 1.0 / 5.0);
    p = fma(p, z, 1.0 / 3.0);
    return fma(fma(q * z, p, q), 2.88539008177792681472, static_cast<double>(e - e0));       // 2 / ln 2
}
__device__ __forceinline__ EstimateLogs estimate_logs(const RangeParams& rp, uint32_t bins, unsigned long long n_sampled)
{
    const double w = static_cast<double>(rp.w);
    return {log2_count(static_cast<double>(n_sampled), entropy_base(n_sampled)), w > 0.0 ? log(w / static_cast<double>(bins)) : 0.0};
}

// The estimate from sum c (log2 c - e0) (`acc`) and sum c (`tot`) over the bins, by one thread, in fp64, and the result record.
// `res` may be the caller's pinned host memory: the end of the kernel makes it visible.
__device__ __forceinline__ void emit_result(double acc, double tot, const EstimateLogs& logs, const RangeParams& rp,
                                            unsigned long long n_sampled, edgc_entropy_result* res)
{
    edgc_entropy_result r;
    r.lo = rp.lo; r.hi = rp.hi;
    r.n_sampled = n_sampled;
    // every finite element of the sample was counted in exactly one bin (values outside a caller's
    // range in the edge bins), so what the bins do not hold is the non-finite part; the counts are
    // integers below 2^53, their sum in fp64 is exact
    r.n_nonfinite = n_sampled - static_cast<unsigned long long>(tot);
    r._pad = 0;
    if (tot > 0.0) {
        // (the product is rounded as a bin's is: with one bin only the difference is zero)
        double H = (tot * (r.n_nonfinite == 0 ? logs.log2_n : log2_count(tot, entropy_base(n_sampled))) - acc) / tot;
        if (H < 0.0) H = 0.0;
        r.H_bits = H;
        r.h_diff_nats = (rp.w > 0.0f) ? H * 0.69314718055994530942 + logs.log_w : -INFINITY;
        r.status = EDGC_OK;
    } else {
        r.H_bits = NAN; r.h_diff_nats = NAN;
        r.status = EDGC_ENONFINITE;
    }
    *res = r;
}

__device__ __forceinline__ void entropy_term(unsigned long long c, int e0, double& acc, double& tot)
{
    if (c) {
        const double d = static_cast<double>(c);
        acc = fma(d, log2_count(d, e0), acc);
        tot += d;
    }
}
// four bins at a time, their logarithms side by side; a wave passes over bins that hold nothing
__device__ __forceinline__ void entropy_terms(const unsigned long long (&c)[4], int e0, double& acc, double& tot)
{
    if (c[0] | c[1] | c[2] | c[3]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double d = static_cast<double>(c[e]);
            acc = fma(d, log2_count(d, e0), acc);
            tot += d;
        }
    }
}

// Sums the threads' (acc, tot) over the block; thread BLOCK - 1 returns the totals.
template <int BLOCK>
__device__ __forceinline__ void block_sum_pair(double& acc, double& tot)
{
    constexpr uint32_t W = BLOCK / 64;
    static_assert(W <= 16, "one row of lanes sums the waves'");
    __shared__ double s_a[16], s_b[16];
    acc = wave_sum_f64(acc);
    tot = wave_sum_f64(tot);
    __syncthreads();              // the arrays may still be read from an earlier call
    if ((threadIdx.x & 63u) == 63u) { s_a[threadIdx.x >> 6] = acc; s_b[threadIdx.x >> 6] = tot; }
    __syncthreads();
    if (threadIdx.x >= BLOCK - 64) {
        const uint32_t l = threadIdx.x & 63u;
        acc = wave_sum_f64(l < W ? s_a[l] : 0.0);
        tot = wave_sum_f64(l < W ? s_b[l] : 0.0);
    }
}

// ---------------------------------------------------------------------------
// kernel 1: range of the finite sample
// ---------------------------------------------------------------------------
// What folds the items and elements that a walk or a round hands out into (lo, hi), per thread
template <typename T, int VEC>
struct RangeFold {
    float &lo, &hi;
    __device__ __forceinline__ void value(float x)
    {
        // no branch: a non-finite value stands in as the bound itself
        const bool fin = finite_f32(x);
        lo = fminf(lo, fin ? x : lo);
        hi = fmaxf(hi, fin ? x : hi);
    }
    __device__ __forceinline__ void operator()(const uint4& raw)
    {
        if constexpr (VEC > 1) {
            float v[VEC];
            unpack_item<T, VEC>(raw, v);
#pragma unroll
            for (int p = 0; p < VEC; ++p) value(v[p]);
        }
    }
    __device__ __forceinline__ void operator()(T x) { value(ElemTraits<T>::widen(x)); }
};
// (lo, hi) of the finite elements of the block's range, of its one round, per thread
template <typename T, int VEC, int BLOCK>
__device__ __forceinline__ void range_of_items(const EntGroup& grp, uint64_t begin, uint64_t end, float& lo, float& hi)
{
    RangeFold<T, VEC> fold{lo, hi};
    walk_items<T, VEC, BLOCK>(grp, begin, end, true, fold, fold, [] {});
}
template <typename T, int VEC, int BLOCK, int U>
__device__ __forceinline__ void range_of_round(const ItemRound<T, VEC, BLOCK, U>& items, float& lo, float& hi)
{
    RangeFold<T, VEC> fold{lo, hi};
    items.visit(fold, fold);
}

__device__ __forceinline__ RangeParams make_range(float lo, float hi, float fbins)
{
    RangeParams r;
    if (lo <= hi) {
        r.lo = lo; r.hi = hi;
        r.w = __fsub_rn(hi, lo);
        r.scale = (r.w > 0.0f) ? __fdiv_rn(fbins, r.w) : 0.0f;
    } else {   // no finite sample at all
        r.lo = NAN; r.hi = NAN; r.w = 0.0f; r.scale = 0.0f;
    }
    return r;
}

// Folds (lo, hi) over the block; every thread returns the block's values.
template <int BLOCK>
__device__ __forceinline__ void block_range_minmax(float& lo, float& hi)
{
    __shared__ float s_lo[BLOCK / 64], s_hi[BLOCK / 64];
    lo = wave_reduce_minmax<true>(lo);
    hi = wave_reduce_minmax<false>(hi);
    if ((threadIdx.x & 63) == 0) { s_lo[threadIdx.x >> 6] = lo; s_hi[threadIdx.x >> 6] = hi; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) { lo = fminf(lo, s_lo[w]); hi = fmaxf(hi, s_hi[w]); }
}

// The blocks' (lo, hi) go to `part` as they stand: every block of the histogram kernel folds them itself (a ticket and
// a last block here cost some 4 us more than those 2 KB of loads there).  Zeroes the `zero_words` 32-bit words at
// `zero`, the counters that kernel accumulates into.
template <typename T, int VEC, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_minmax(const EntGroup grp, float2* __restrict__ part,
                                                  uint32_t* __restrict__ zero, uint32_t zero_words)
{
    for (uint32_t i = blockIdx.x * BLOCK + threadIdx.x; i < zero_words; i += gridDim.x * BLOCK) zero[i] = 0u;
    float lo = INFINITY, hi = -INFINITY;
    uint64_t begin, end;
    block_range(grp, begin, end);
    range_of_items<T, VEC, BLOCK>(grp, begin, end, lo, hi);
    block_range_minmax<BLOCK>(lo, hi);
    if (threadIdx.x == 0) part[blockIdx.x] = make_float2(lo, hi);
}

// Caller-supplied range: stands in as the one block's (lo, hi); zeroes the counters.
__global__ void k_set_range(float2* part, float lo, float hi, uint32_t* __restrict__ zero, uint32_t zero_words)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < zero_words; i += gridDim.x * blockDim.x) zero[i] = 0u;
    if (threadIdx.x == 0 && blockIdx.x == 0) part[0] = make_float2(lo, hi);
}

// ---------------------------------------------------------------------------
// kernel 2: histogram + entropy
// ---------------------------------------------------------------------------
// What bins the items and elements that a walk or a round hands out into the LDS counters h[bin - bin_base][replica], bins
// [bin_base, bin_base + local_n).
// bin = trunc((x - lo) * scale), each operation rounded on its own, clamped to [0, bins - 1].
template <typename T, int VEC, bool WHOLE>           // WHOLE: one slice holds every bin
struct Binner {
    float lo, scale, top;                            // top: largest float below the bin count; truncating a value clamped to
    uint32_t bin_base, local_n, rep_shift;           // [0, top] gives 0 .. bins - 1
    uint32_t* h_rep;                                 // this lane's replica
    __device__ __forceinline__ Binner(float lo_, float scale_, uint32_t bins, uint32_t bin_base_, uint32_t local_n_,
                                      uint32_t rep_shift_, uint32_t* h)
        : lo(lo_), scale(scale_), top(__uint_as_float(__float_as_uint(static_cast<float>(bins)) - 1u)), bin_base(bin_base_),
          local_n(local_n_), rep_shift(rep_shift_), h_rep(h + (threadIdx.x & ((1u << rep_shift_) - 1u))) {}
    // No branch per element: the bin of a non-finite value is some valid bin (the clamp maps NaN to 0) and it adds 0.
    __device__ __forceinline__ void value(float x)
    {
        const float f = __builtin_amdgcn_fmed3f(__fmul_rn(__fsub_rn(x, lo), scale), 0.0f, top);
        const uint32_t b = static_cast<uint32_t>(f), one = finite_f32(x) ? 1u : 0u;
        if (WHOLE) atomicAdd(&h_rep[b << rep_shift], one);
        else if (b - bin_base < local_n) atomicAdd(&h_rep[(b - bin_base) << rep_shift], one);
    }
    __device__ __forceinline__ void operator()(const uint4& raw)
    {
        if constexpr (VEC > 1) {
            float v[VEC];
            unpack_item<T, VEC>(raw, v);
#pragma unroll
            for (int p = 0; p < VEC; ++p) value(v[p]);
        }
    }
    __device__ __forceinline__ void operator()(T x) { value(ElemTraits<T>::widen(x)); }
};
template <typename T, int VEC, int BLOCK>
__device__ __forceinline__ void bin_items(const EntGroup& grp, uint64_t begin, uint64_t end, float lo, float scale,
                                          uint32_t bins, uint32_t bin_base, uint32_t local_n, uint32_t rep_shift,
                                          bool ahead, uint32_t* h)
{
    if (local_n == bins) {
        Binner<T, VEC, true> bin(lo, scale, bins, bin_base, local_n, rep_shift, h);
        walk_items<T, VEC, BLOCK>(grp, begin, end, ahead, bin, bin, [] {});
    } else {
        Binner<T, VEC, false> bin(lo, scale, bins, bin_base, local_n, rep_shift, h);
        walk_items<T, VEC, BLOCK>(grp, begin, end, ahead, bin, bin, [] {});
    }
}
template <typename T, int VEC, int BLOCK, int U>
__device__ __forceinline__ void bin_round(const ItemRound<T, VEC, BLOCK, U>& items, float lo, float scale, uint32_t bins,
                                          uint32_t rep_shift, uint32_t* h)
{
    Binner<T, VEC, true> bin(lo, scale, bins, 0, bins, rep_shift, h);
    items.visit(bin, bin);
}

// (lo, hi) of the sample from the blocks' partials, by one block
template <int BLOCK>
__device__ __forceinline__ RangeParams fold_range(const float2* __restrict__ part, uint32_t nparts, float fbins)
{
    float lo = INFINITY, hi = -INFINITY;
    for (uint32_t i = threadIdx.x; i < nparts; i += BLOCK) {
        const float2 v = part[i];
        lo = fminf(lo, v.x);
        hi = fmaxf(hi, v.y);
    }
    block_range_minmax<BLOCK>(lo, hi);
    return make_range(lo, hi, fbins);
}

// True in every thread of the block that finishes last of the grid (the ticket is zero before and after); the block's last
// wave does `meanwhile` while the ticket is on its way.
// What the blocks hand to the last one they have written by device-scope atomics, which take effect where every XCD sees them:
// every wave waits for its own, and no release is needed.  (A release writes the XCD's L2 back, some 0.1 us that the blocks of an
// XCD queue up for: one per wave, the histogram kernel of a 1 % sample took 59 us on 384 blocks; one per block, the ticket
// of 246 blocks came back 3.5 us after the last of them had asked, without 1.6.)
template <int BLOCK, typename F>
__device__ __forceinline__ bool last_block(unsigned int* ticket, F&& meanwhile)
{
    __shared__ bool s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool last = atomicAdd(ticket, 1u) == gridDim.x * gridDim.y - 1u;
        if (last) *ticket = 0u;
        s_last = last;
    }
    if (threadIdx.x >= BLOCK - 64) meanwhile();
    __syncthreads();
    const bool last = s_last;
    if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return last;
}

__host__ __device__ constexpr uint32_t copy_stride(uint32_t bins) { return (bins + 3u) & ~3u; }   // words per set

// The last block's part: the histogram from the sets of 32-bit counters (S of them; 0: from the 64-bit counters themselves),
// and H = log2 n - (1/n) sum c log2 c (== -sum p log2 p).  A thread has the counters of 4 U bins in flight: four
// neighbours a load from a set, which is padded to a multiple of four counters that stay zero, and bins BLOCK apart where they are
// 64-bit words at any address.
template <int BLOCK, int S, int U>
__device__ __forceinline__ void sum_bins(const uint32_t* copies, unsigned long long* counts, uint32_t bins, int e0, double& acc, double& tot)
{
    if constexpr (S > 0) {
        for (uint32_t i0 = threadIdx.x * 4u; i0 < bins; i0 += BLOCK * 4u * U) {
            uint4 x[U][S];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < S; ++k)
                    x[u][k] = *reinterpret_cast<const uint4*>(copies + static_cast<size_t>(k) * copy_stride(bins) +
                                                              min(i0 + BLOCK * 4u * u, copy_stride(bins) - 4u));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = i0 + BLOCK * 4u * u;
                if (i >= bins) break;
                unsigned long long c[4] = {0, 0, 0, 0};
#pragma unroll
                for (int k = 0; k < S; ++k) { c[0] += x[u][k].x; c[1] += x[u][k].y; c[2] += x[u][k].z; c[3] += x[u][k].w; }
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e)
                    if (i + e < bins) counts[i + e] = c[e];
                entropy_terms(c, e0, acc, tot);
            }
        }
    } else {
        for (uint32_t i0 = threadIdx.x; i0 < bins; i0 += BLOCK * 4u * U) {
            unsigned long long c[U][4];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e) c[u][e] = counts[min(i0 + BLOCK * (4u * u + e), bins - 1u)];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
#pragma unroll
                for (uint32_t e = 0; e < 4; ++e)
                    if (i0 + BLOCK * (4u * u + e) >= bins) c[u][e] = 0ull;
                entropy_terms(c[u], e0, acc, tot);
            }
        }
    }
}
template <int BLOCK>
__device__ __forceinline__ void finish(double acc, double tot, const EstimateLogs& logs, const RangeParams& rp,
                                       unsigned long long n_sampled, edgc_entropy_result* res)
{
    block_sum_pair<BLOCK>(acc, tot);
    if (threadIdx.x == BLOCK - 1) emit_result(acc, tot, logs, rp, n_sampled, res);
}

// `sets` = 8: the blocks of equal id modulo 8, which the dispatcher places on one XCD, share a set of 32-bit counters at
// `copies`, and the last block adds the sets up: a counter line that all XCDs add to moves between their caches
// (192 blocks 19.3 us, with eight sets 17.3; 384 blocks 24.5 and 20.2).  1: one set for all blocks.  0 (samples of 2^32
// elements or more, or more bins than the sets hold): `counts` itself.
template <typename T, int VEC, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_hist(
    const EntGroup grp, const float2* __restrict__ part, uint32_t nparts, uint32_t bins,
    uint32_t bins_local, uint32_t rep_shift, uint32_t* copies, uint32_t sets, unsigned long long* counts,
    unsigned int* ticket, edgc_entropy_result* res)
{
    extern __shared__ uint32_t h[];   // [bins_local << rep_shift], replica = lane & (R-1)
    const uint32_t bin_base = blockIdx.y * bins_local;
    const uint32_t local_n = min(bins_local, bins - bin_base);
    const uint32_t words = local_n << rep_shift;
    for (uint32_t i = threadIdx.x; i < words; i += BLOCK) h[i] = 0u;
    const RangeParams rp = fold_range<BLOCK>(part, nparts, static_cast<float>(bins));
    __syncthreads();

    uint64_t begin, end;
    block_range(grp, begin, end);
    // (loads one round ahead, measured on a 1e9-element buffer: with every element sampled 0.86 instead of 0.91 ms on
    // fp32 and 0.51 instead of 0.63 ms on bf16; on the 10 % sample, 256-byte runs 2.5 KB apart, 0.19 instead of
    // 0.15 ms, so strided samples go without)
    bin_items<T, VEC, BLOCK>(grp, begin, end, rp.lo, rp.scale, bins, bin_base, local_n, rep_shift,
                             gridDim.y == 1 && grp.stride == 1, h);
    __syncthreads();

    // fold the replicas and flush non-empty bins
    uint32_t* const copy = sets ? copies + static_cast<size_t>(blockIdx.x & (sets - 1u)) * copy_stride(bins) : nullptr;
    for (uint32_t i = threadIdx.x; i < local_n; i += BLOCK) {
        uint32_t s = 0;
        for (uint32_t r = 0; r < (1u << rep_shift); ++r) s += h[(i << rep_shift) | r];
        if (!s) continue;
        if (copy) atomicAdd(&copy[i], s);
        else atomicAdd(&counts[bin_base + i], static_cast<unsigned long long>(s));
    }
    EstimateLogs logs{};
    if (!last_block<BLOCK>(ticket, [&] { logs = estimate_logs(rp, bins, grp.n_sampled); })) return;
    double acc = 0.0, tot = 0.0;
    if (sets == 8) sum_bins<BLOCK, 8, 1>(copies, counts, bins, entropy_base(grp.n_sampled), acc, tot);
    else if (sets) sum_bins<BLOCK, 1, 2>(copies, counts, bins, entropy_base(grp.n_sampled), acc, tot);
    else sum_bins<BLOCK, 0, 2>(copies, counts, bins, entropy_base(grp.n_sampled), acc, tot);
    finish<BLOCK>(acc, tot, logs, rp, grp.n_sampled, res);
}

// The same for a sample of which every block takes one round of loads: 1 % of a transformer block and less.  What bounds it
// is a chain of latencies, and the kernels of one round are cut for that: the items are requested before the range that they
// are binned with is folded, nothing is divided that the host can divide, and the code is short, since every
// instruction of it is fetched once, by one wave, from a cold cache.
template <typename T, int VEC, int BLOCK, int U>
__global__ __launch_bounds__(BLOCK) void k_minmax_small(const EntGroup grp, float2* __restrict__ part,
                                                        uint32_t* __restrict__ zero, uint32_t zero_words)
{
    BufferTable tab;
    tab.load(grp);
    const uint64_t begin = static_cast<uint64_t>(blockIdx.x) * (BLOCK * U);
    ItemRound<T, VEC, BLOCK, U> items;
    items.request(grp, tab, begin, min(begin + BLOCK * U, grp.n_items));
    for (uint32_t i = blockIdx.x * BLOCK + threadIdx.x; i < zero_words; i += gridDim.x * BLOCK) zero[i] = 0u;
    float lo = INFINITY, hi = -INFINITY;
    range_of_round(items, lo, hi);
    block_range_minmax<BLOCK>(lo, hi);
    if (threadIdx.x == 0) part[blockIdx.x] = make_float2(lo, hi);
}

template <typename T, int VEC, int BLOCK, int U>
__global__ __launch_bounds__(BLOCK) void k_hist_small(const EntGroup grp, const float2* __restrict__ part, uint32_t nparts,
                                                      uint32_t bins, uint32_t rep_shift, uint32_t* copies, uint32_t sets,
                                                      unsigned long long* counts, unsigned int* ticket,
                                                      edgc_entropy_result* res)
{
    extern __shared__ uint32_t h[];   // [bins << rep_shift]
    BufferTable tab;
    tab.load(grp);
    const uint64_t begin = static_cast<uint64_t>(blockIdx.x) * (BLOCK * U);
    ItemRound<T, VEC, BLOCK, U> items;
    items.request(grp, tab, begin, min(begin + BLOCK * U, grp.n_items));
    for (uint32_t i = threadIdx.x; i < (bins << rep_shift); i += BLOCK) h[i] = 0u;
    const RangeParams rp = fold_range<BLOCK>(part, nparts, static_cast<float>(bins));
    __syncthreads();
    bin_round(items, rp.lo, rp.scale, bins, rep_shift, h);
    __syncthreads();
    uint32_t* const copy = copies + static_cast<size_t>(blockIdx.x & (sets - 1u)) * copy_stride(bins);
    for (uint32_t i = threadIdx.x; i < bins; i += BLOCK) {
        uint32_t s = 0;
        for (uint32_t r = 0; r < (1u << rep_shift); ++r) s += h[(i << rep_shift) | r];
        if (s) atomicAdd(&copy[i], s);
    }
    EstimateLogs logs{};
    if (!last_block<BLOCK>(ticket, [&] { logs = estimate_logs(rp, bins, grp.n_sampled); })) return;
    double acc = 0.0, tot = 0.0;
    if (sets == 2) sum_bins<BLOCK, 2, 2>(copies, counts, bins, entropy_base(grp.n_sampled), acc, tot);
    else sum_bins<BLOCK, 1, 2>(copies, counts, bins, entropy_base(grp.n_sampled), acc, tot);
    finish<BLOCK>(acc, tot, logs, rp, grp.n_sampled, res);
}

// The whole estimate of a small sample by one block: range, histogram and entropy without a second launch, global
// counters or a ticket.  Its latency chain is that of one block of k_hist_small without the device-wide part; the items stay in
// registers between the range and the bins.
template <typename T, int VEC>
__global__ __launch_bounds__(kOneBlock) void k_estimate_one(const EntGroup grp, int has_range, float range_lo,
                                                            float range_hi, uint32_t bins, uint32_t rep_shift,
                                                            unsigned long long* __restrict__ counts,
                                                            edgc_entropy_result* res)
{
    extern __shared__ uint32_t h[];   // [bins << rep_shift]
    for (uint32_t i = threadIdx.x; i < (bins << rep_shift); i += kOneBlock) h[i] = 0u;
    BufferTable tab;
    tab.load(grp);
    ItemRound<T, VEC, kOneBlock, 4> items;
    items.request(grp, tab, 0, grp.n_items);
    float lo = INFINITY, hi = -INFINITY;
    if (has_range) {
        lo = range_lo; hi = range_hi;
        __syncthreads();
    } else {
        range_of_round(items, lo, hi);
        block_range_minmax<kOneBlock>(lo, hi);
    }
    const RangeParams rp = make_range(lo, hi, static_cast<float>(bins));
    bin_round(items, rp.lo, rp.scale, bins, rep_shift, h);
    __syncthreads();
    double acc = 0.0, tot = 0.0;
    for (uint32_t i = threadIdx.x; i < bins; i += kOneBlock) {
        uint32_t s = 0;
        for (uint32_t r = 0; r < (1u << rep_shift); ++r) s += h[(i << rep_shift) | r];
        counts[i] = s;
        entropy_term(s, entropy_base(grp.n_sampled), acc, tot);
    }
    EstimateLogs logs{};
    if (threadIdx.x >= kOneBlock - 64) logs = estimate_logs(rp, bins, grp.n_sampled);
    finish<kOneBlock>(acc, tot, logs, rp, grp.n_sampled, res);
}

// ---------------------------------------------------------------------------
// 65536 counters per block in LDS, as 16-bit fields (two per 32-bit word, 128 KiB, one block of
// 1024 threads per CU).  Two uses:
//  * fp32 samples on more than 16384 bins: the key of an element is its bin, and the sample is
//    binned in ONE read (32-bit counters cover 32768 bins per read);
//  * bf16 samples, whatever the number of bins: the key is the raw bit pattern.  A bf16 value is
//    one of 65536 patterns, and range, bin and finiteness are functions of the pattern alone, so
//    the sample is read ONCE, with no range pass before it, and the rest (range of the finite
//    sample, bin of every pattern by the same fp32 operations the binning kernel applies to
//    every element, entropy) is derived from the 65536 pattern counts.
// A round of the block adds at most 32768 elements (1024 threads, four items of eight; with items of four or of one element
// two or eight rounds do), so a field that is below 0x8000 when it begins cannot carry into its neighbour; after it each
// thread looks through its own 32 words and moves fields that have reached 0x8000 off to the key's 64-bit global counter
// (`wide`), 32768 at a time.  (A sweep after every round of single elements: 134 M bf16 elements at an odd address 417 us
// against 344.)
// (Adds that return the old value and move the field off at once need no such sweep, but every one of them waits for
// the LDS: 134 M bf16 elements 90 us against 61, 4.4 TB/s.)
// At its end a block stores its fields as they stand to its own 128 KiB of `part16` (plain
// 16-byte stores: no atomics on global memory, of which 256 blocks x some thousand keys would be
// the larger part of a small estimate), and k_wide_reduce sums them.  Only the runs of 256 fields that hold anything are
// stored, and marked in `occupied`: the values of a gradient touch some thirty of the 256 runs of bf16 patterns, and the
// middle and a few outliers of 65536 bins.
// ---------------------------------------------------------------------------
constexpr int kWideBlock = 1024;
constexpr uint32_t kFoldedRange = kMaxReduceBlocks - 1;                   // where k_wide_hist leaves the range for k_wide_reduce (bins as keys)
constexpr uint32_t kWideKeys = 65536;
constexpr uint32_t kReduceKeys = 256;                                     // keys that one block of k_wide_reduce sums
constexpr uint32_t kOccupiedWords = kWideKeys / kReduceKeys / 32;         // 32-bit words of a block's marks
static_assert(kReduceKeys / 8 == 32 && kWideKeys / 8 == kOccupiedWords * kWideBlock && kWideBlock / 32 == 32,
              "k_wide_hist: half a wave stores the fields of one block of k_wide_reduce, each of 32 half waves one of each word");

__device__ __forceinline__ void note_pattern(uint32_t key, float& lo, float& hi)     // key: of a bf16 value that occurs
{
    const float x = __uint_as_float(key << 16);
    if (finite_f32(x)) { lo = fminf(lo, x); hi = fmaxf(hi, x); }
}

template <typename T, int VEC, bool PATTERN>
__global__ __launch_bounds__(kWideBlock) void k_wide_hist(
    const EntGroup grp, float2* __restrict__ part, uint32_t nparts, uint32_t bins, uint16_t* __restrict__ part16,
    uint32_t* __restrict__ occupied, unsigned long long* __restrict__ wide, unsigned long long* __restrict__ counts)
{
    static_assert(!PATTERN || sizeof(T) == 2, "the raw pattern is the key of 16-bit elements only");
    constexpr uint32_t kRounds = 32768 / (kWideBlock * 4 * VEC);   // rounds that together add at most 32768 to a field
    static_assert(kRounds >= 1, "what a round can add to one field");
    extern __shared__ __align__(256) uint32_t h[];   // [kWideKeys / 2]
    __shared__ uint32_t s_occupied[kOccupiedWords];
    uint4* const h4 = reinterpret_cast<uint4*>(h);
    // PATTERN: range of the finite patterns whose fields were moved off (they may be zero at the end), in the order of their
    // values.  In LDS, so that the loop over the sample carries no registers for what happens to few fields.
    __shared__ uint32_t s_moved_lo, s_moved_hi;
    auto note_moved = [&](uint32_t key) {
        if (!PATTERN || (key & 0x7f80u) == 0x7f80u) return;
        const uint32_t order = key & 0x8000u ? 0xffffu - key : key | 0x8000u;
        atomicMin(&s_moved_lo, order);
        atomicMax(&s_moved_hi, order);
    };
    if (threadIdx.x < kOccupiedWords) s_occupied[threadIdx.x] = 0u;
    if (threadIdx.x == 0) { s_moved_lo = 0xffffu; s_moved_hi = 0u; }
    for (uint32_t i = threadIdx.x; i < kWideKeys / 8; i += kWideBlock) h4[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();

    float lo = 0.0f, scale = 0.0f, top = 0.0f;
    if constexpr (PATTERN) {
        for (uint32_t i = blockIdx.x * kWideBlock + threadIdx.x; i < bins; i += gridDim.x * kWideBlock) counts[i] = 0ull;
    } else {
        const float fbins = static_cast<float>(bins);
        const RangeParams rp = fold_range<kWideBlock>(part, nparts, fbins);
        lo = rp.lo; scale = rp.scale;
        top = __uint_as_float(__float_as_uint(fbins) - 1u);     // largest float below the bin count
        if (blockIdx.x == 0 && threadIdx.x == 0) part[kFoldedRange] = make_float2(rp.lo, rp.hi);
    }
    auto add = [&](uint32_t key, uint32_t k) { atomicAdd(&h[key >> 1], k << ((key & 1u) << 4)); };
    // bin = trunc((x - lo) * scale), each operation rounded on its own, clamped to [0, bins - 1]
    auto add_bin = [&](float x) {
        const float t = __fsub_rn(x, lo);
        add(static_cast<uint32_t>(__builtin_amdgcn_fmed3f(__fmul_rn(t, scale), 0.0f, top)), finite_f32(x) ? 1u : 0u);
    };

    uint64_t begin, end;
    block_range(grp, begin, end);
    uint32_t since = 0;                                            // rounds since the last sweep, the same in every thread
    walk_items<T, VEC, kWideBlock>(grp, begin, end, true,
        [&](const uint4& raw) {
            if constexpr (PATTERN) {
                const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t a = w[q] & 0xffffu, b = w[q] >> 16;
                    add(a, a == b ? 2u : 1u);                  // runs of equal values (zeros) in one add
                    if (a != b) add(b, 1u);
                }
            } else if constexpr (VEC > 1) {
                float v[VEC];
                unpack_item<T, VEC>(raw, v);
#pragma unroll
                for (int q = 0; q < VEC; ++q) add_bin(v[q]);
            }
        },
        [&](T x) {
            if constexpr (PATTERN) add(x, 1u);
            else add_bin(ElemTraits<T>::widen(x));
        },
        [&] {
            if constexpr (kRounds > 1) {
                if (++since < kRounds) return;
                since = 0;
            }
            __syncthreads();
            uint32_t full = 0;                                     // which of this thread's 16-byte words hold such a field
#pragma unroll
            for (uint32_t j = 0; j < kOccupiedWords; ++j) {
                const uint4 v = h4[threadIdx.x + j * kWideBlock];
                full |= ((v.x | v.y | v.z | v.w) & 0x80008000u) ? 1u << j : 0u;
            }
            // rare, and compiled into every call of this function: short code, not fast code (written out, 8 x 8 fields per
            // call, the kernel was 150 KB and its few rounds ran from a cold instruction cache)
#pragma unroll 1
            for (; full; full &= full - 1u) {
                const uint32_t at = (threadIdx.x + (__ffs(full) - 1) * kWideBlock) * 4;
#pragma unroll 1
                for (uint32_t q = at; q < at + 4; ++q) {
                    const uint32_t w = h[q];
                    if (w & 0x8000u) { atomicAdd(&wide[2 * q], 32768ull); note_moved(2 * q); }
                    if (w & 0x80000000u) { atomicAdd(&wide[2 * q + 1], 32768ull); note_moved(2 * q + 1); }
                    h[q] = w & 0x7fff7fffu;
                }
            }
            __syncthreads();
        });
    __syncthreads();
    uint4* __restrict__ dst = reinterpret_cast<uint4*>(part16 + static_cast<size_t>(blockIdx.x) * kWideKeys);
    float key_lo = INFINITY, key_hi = -INFINITY;
    if constexpr (PATTERN) {
        if (threadIdx.x == 0 && s_moved_lo <= s_moved_hi) {
            const uint32_t a = s_moved_lo, b = s_moved_hi;
            note_pattern(a & 0x8000u ? a & 0x7fffu : 0xffffu - a, key_lo, key_hi);
            note_pattern(b & 0x8000u ? b & 0x7fffu : 0xffffu - b, key_lo, key_hi);
        }
    }
#pragma unroll
    for (uint32_t j = 0; j < kOccupiedWords; ++j) {
        const uint32_t i = threadIdx.x + j * kWideBlock;
        const uint4 v = h4[i];
        const uint64_t any = __ballot((v.x | v.y | v.z | v.w) != 0u);
        if (static_cast<uint32_t>(threadIdx.x & 32u ? any >> 32 : any) == 0u) continue;
        dst[i] = v;
        if constexpr (PATTERN) {
            // values of one sign rise or fall with the pattern: the first and the last that occurs of the eight
            const uint32_t m = ((v.x & 0xffffu) ? 1u : 0u) | ((v.x >> 16) ? 2u : 0u) | ((v.y & 0xffffu) ? 4u : 0u) |
                               ((v.y >> 16) ? 8u : 0u) | ((v.z & 0xffffu) ? 16u : 0u) | ((v.z >> 16) ? 32u : 0u) |
                               ((v.w & 0xffffu) ? 64u : 0u) | ((v.w >> 16) ? 128u : 0u);
            if (m) {
                note_pattern(i * 8 + __ffs(m) - 1, key_lo, key_hi);
                note_pattern(i * 8 + 31 - __clz(m), key_lo, key_hi);
            }
        }
        if ((threadIdx.x & 31u) == 0u) atomicOr(&s_occupied[j], 1u << (threadIdx.x >> 5));
    }
    if constexpr (PATTERN) {
        block_range_minmax<kWideBlock>(key_lo, key_hi);
        if (threadIdx.x == 0) part[blockIdx.x] = make_float2(key_lo, key_hi);
    }
    __syncthreads();
    if (threadIdx.x < kOccupiedWords) occupied[blockIdx.x * kOccupiedWords + threadIdx.x] = s_occupied[threadIdx.x];
}

// Sums the blocks' 16-bit fields and the 64-bit credits per key, 256 keys per block, and the last block to finish
// turns the histogram into the estimate.
//  fp32 (keys are bins): the totals are the histogram.
//  bf16 (keys are bit patterns): every block folds the range of the patterns that k_wide_hist's blocks saw and adds its
//  256 totals to the bins of their patterns.
// What bounds it: latency, of the marks, the marked blocks' fields (all of a thread's eight 16-byte loads in flight together),
// the ticket and the last block's loads of the bins.  134 M bf16 elements of a gradient, both kernels: all of
// 33 MB of fields read and the patterns binned by the last block alone 86.0 us, marked fields only 80.4, binned by every block
// and k_wide_hist's short sweep 73.8, without releases and with short logarithms 65.9; 10 M fp32 elements on 65536 bins (range
// kernel included) 43.7 us, marked fields only 35.5, and 30.6.
constexpr uint32_t kReduceGroups = kWideBlock / (kReduceKeys / 8);        // 32 groups of 32 threads
static_assert(kMaxPart16Blocks <= kWideBlock && kMaxPart16Blocks * 65535ull < (1ull << 32),
              "k_wide_reduce: a thread looks at one block's marks, and a key's fields are summed in 32 bits");
constexpr size_t kWideReduceLds = (kReduceGroups + 4) * kReduceKeys * sizeof(uint32_t);

template <bool PATTERN>
__global__ __launch_bounds__(kWideBlock) void k_wide_reduce(
    const uint16_t* __restrict__ part16, const uint32_t* __restrict__ occupied, uint32_t nblocks, unsigned long long* __restrict__ wide,
    uint32_t bins, int has_range, float range_lo, float range_hi, unsigned long long* counts,
    const float2* __restrict__ mm_part, double* part_d, unsigned int* ticket, unsigned long long n_sampled,
    edgc_entropy_result* res)
{
    extern __shared__ __align__(256) uint32_t red[];                  // the groups' sums: [kReduceGroups][kReduceKeys], then [4][kReduceKeys]
    const bool mine = threadIdx.x < kReduceKeys;      // one key per thread
    const uint32_t key = blockIdx.x * kReduceKeys + threadIdx.x;
    __shared__ uint32_t s_from[kWideBlock], s_nfrom;  // the blocks that counted any of this block's keys, in any order
    if (threadIdx.x == 0) s_nfrom = 0u;
    unsigned long long c = mine ? wide[key] : 0ull;
    const uint32_t marks = threadIdx.x < nblocks ? occupied[threadIdx.x * kOccupiedWords + (blockIdx.x >> 5)] : 0u;
    __syncthreads();
    if ((marks >> (blockIdx.x & 31u)) & 1u) s_from[atomicAdd(&s_nfrom, 1u)] = threadIdx.x;
    if (c) wide[key] = 0ull;                          // zero between estimates
    RangeParams rp{};
    if constexpr (!PATTERN) {
        const float2 v = mm_part[kFoldedRange];
        rp = make_range(v.x, v.y, static_cast<float>(bins));
    } else {
        float lo = INFINITY, hi = -INFINITY;
        if (threadIdx.x < nblocks) { lo = mm_part[threadIdx.x].x; hi = mm_part[threadIdx.x].y; }
        block_range_minmax<kWideBlock>(lo, hi);
        if (has_range) { lo = range_lo; hi = range_hi; }
        rp = make_range(lo, hi, static_cast<float>(bins));
    }
    __syncthreads();
    const uint32_t nfrom = s_nfrom;
    if (nfrom) {
        // The block's keys are 32 columns of eight 16-bit fields (one 16-byte load); each of its 32 groups of 32 threads
        // sums the fields of every 32nd listed block, and the groups' sums meet in LDS.
        const uint32_t col = threadIdx.x & 31u, grp = threadIdx.x >> 5;
        const uint4* __restrict__ src = reinterpret_cast<const uint4*>(part16 + blockIdx.x * kReduceKeys) + col;
        constexpr size_t kRow = kWideKeys / 8;                             // 16-byte items per block's fields
        uint32_t sm[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};                 // of at most 32 fields; 1024 per key: below 2^26
        for (uint32_t b = grp; b < nfrom; b += 8 * kReduceGroups) {
            uint4 v[8];
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u)
                v[u] = (b + kReduceGroups * u < nfrom) ? src[static_cast<size_t>(s_from[b + kReduceGroups * u]) * kRow]
                                                       : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                sm[0] += v[u].x & 0xffffu; sm[1] += v[u].x >> 16;
                sm[2] += v[u].y & 0xffffu; sm[3] += v[u].y >> 16;
                sm[4] += v[u].z & 0xffffu; sm[5] += v[u].z >> 16;
                sm[6] += v[u].w & 0xffffu; sm[7] += v[u].w >> 16;
            }
        }
        uint4* const dst = reinterpret_cast<uint4*>(red + grp * kReduceKeys + col * 8);
        dst[0] = make_uint4(sm[0], sm[1], sm[2], sm[3]);
        dst[1] = make_uint4(sm[4], sm[5], sm[6], sm[7]);
        __syncthreads();
        const uint32_t k = threadIdx.x & (kReduceKeys - 1u), quarter = threadIdx.x / kReduceKeys;
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t gI = 0; gI < kReduceGroups / 4; ++gI) sum += red[(quarter * (kReduceGroups / 4) + gI) * kReduceKeys + k];
        uint32_t* const red2 = red + kReduceGroups * kReduceKeys;
        red2[quarter * kReduceKeys + k] = sum;
        __syncthreads();
        if (mine) c += red2[k] + red2[kReduceKeys + k] + red2[2 * kReduceKeys + k] + red2[3 * kReduceKeys + k];
    }
    if constexpr (!PATTERN) {
        // the totals are the histogram; this block's share of the entropy sums goes with them
        double acc = 0.0, tot = 0.0;
        if (mine && key < bins) {
            counts[key] = c;
            entropy_term(c, entropy_base(n_sampled), acc, tot);
        }
        block_sum_pair<kWideBlock>(acc, tot);
        if (threadIdx.x == kWideBlock - 1) {
            __hip_atomic_store(&part_d[2 * blockIdx.x], acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&part_d[2 * blockIdx.x + 1], tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    } else if (threadIdx.x < kReduceKeys) {           // whole waves
        const float x = __uint_as_float(key << 16);
        if (!finite_f32(x)) c = 0ull;
        // bin = trunc((x - lo) * scale), each operation rounded on its own, clamped to [0, bins - 1]
        const float top = __uint_as_float(__float_as_uint(static_cast<float>(bins)) - 1u);   // largest float below the bin count
        const uint32_t bin = static_cast<uint32_t>(
            __builtin_amdgcn_fmed3f(__fmul_rn(__fsub_rn(x, rp.lo), rp.scale), 0.0f, top));
        // Patterns next to each other share a bin wherever values are small: one addition per run of equal bins in a wave,
        // of the difference of two running sums.
        const uint32_t lane = threadIdx.x & 63u;
        unsigned long long sum = c;
#pragma unroll
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const unsigned long long below = __shfl_up(sum, d, 64);
            if (lane >= d) sum += below;
        }
        const uint32_t bin_below = __shfl_up(bin, 1, 64);
        const uint64_t heads = __ballot(lane == 0 || bin != bin_below);
        const uint32_t head = 63u - __clzll(heads & (~0ull >> (63u - lane)));
        const unsigned long long before = __shfl(sum, static_cast<int>(head) - 1, 64);
        const bool tail = lane == 63u || ((heads >> lane >> 1) & 1u);
        const unsigned long long run = sum - (head ? before : 0ull);
        if (tail && run) atomicAdd(&counts[bin], run);
    }
    EstimateLogs logs{};
    if (!last_block<kWideBlock>(ticket, [&] { logs = estimate_logs(rp, bins, n_sampled); })) return;
    double acc = 0.0, tot = 0.0;
    if constexpr (PATTERN) {
        sum_bins<kWideBlock, 0, 1>(nullptr, counts, bins, entropy_base(n_sampled), acc, tot);
    } else if (threadIdx.x < gridDim.x) {
        acc = part_d[2 * threadIdx.x];
        tot = part_d[2 * threadIdx.x + 1];
    }
    finish<kWideBlock>(acc, tot, logs, rp, n_sampled, res);
}

// ---------------------------------------------------------------------------
// sampled indices (same cursor as the kernels above)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_sample_indices(SampleGeom geom, uint64_t* __restrict__ idx,
                                                        uint64_t cap)
{
    const uint64_t G = static_cast<uint64_t>(gridDim.x) * 256;
    const int vec = static_cast<int>(geom.vec);
    for (uint64_t item = static_cast<uint64_t>(blockIdx.x) * 256; item < geom.n_items; item += G) {
        const uint64_t it = item + threadIdx.x;
        if (it >= geom.n_items) break;
        const uint64_t i0 = elem_of_item(geom, it, vec);
        const uint64_t pos0 = it * vec;               // (a chunk is ipc items of vec elements)
        for (int p = 0; p < vec; ++p)
            if (i0 + p < geom.n && pos0 + p < cap) idx[pos0 + p] = i0 + p;
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
SampleGeom make_geom(const void* base, edgc_dtype dt, uint64_t n, uint64_t stride, uint32_t chunk,
                     uint64_t seed, uint64_t step, bool allow_vec)
{
    SampleGeom g{};
    const uint32_t elem = (dt == EDGC_F32) ? 4u : 2u;
    const uint32_t V = 16u / elem;
    const bool aligned = allow_vec && (reinterpret_cast<uintptr_t>(base) % 16u) == 0;
    g.n = n;
    g.stride = stride;
    g.slot = mix64(seed, step) % stride;
    g.chunk = chunk;
    if (stride == 1) {
        // every element is sampled whatever the chunk size: read it as long runs
        g.slot = 0;
        if (aligned) g.chunk = 4096;
    }
    const uint64_t total_chunks = (n + g.chunk - 1) / g.chunk;
    g.n_chunks = (g.slot < total_chunks) ? (total_chunks - g.slot + stride - 1) / stride : 0;
    g.n_sampled = 0;
    if (g.n_chunks) {
        const uint64_t last = g.slot + (g.n_chunks - 1) * stride;
        const uint64_t last_len = (n - last * g.chunk < g.chunk) ? n - last * g.chunk : g.chunk;
        g.n_sampled = (g.n_chunks - 1) * g.chunk + last_len;
    }
    g.vec = (aligned && g.chunk % V == 0) ? V : 1u;
    g.ipc = g.chunk / g.vec;
    g.n_items = g.n_chunks * g.ipc;
    return g;
}

static uint32_t grid_for(uint64_t n_items, int block, int per_thread, int max_blocks)
{
    uint64_t want = (n_items + static_cast<uint64_t>(block) * per_thread - 1) /
                    (static_cast<uint64_t>(block) * per_thread);
    if (want < 1) want = 1;
    if (want > static_cast<uint64_t>(max_blocks)) want = max_blocks;
    return static_cast<uint32_t>(want);
}

// The device memory an estimate works in beyond its inputs and outputs: the context's own
// allocations, or the file-scope array of the entry point that allocates nothing.
struct EntScratch {
    float2*             mm_part;       // [kMaxReduceBlocks] per-block (lo, hi)
    unsigned int*       ticket;        // [kTicketWords] last-block ticket; zero between calls
    uint32_t*           copies;        // [8][kCopyBins] histogram counters by XCD
    uint16_t*           part16;        // [part16_blocks][65536] 16-bit counters per block, or null: plain kernels only
    uint32_t            part16_blocks;
    uint32_t*           occupied;      // [part16_blocks][kOccupiedWords] which of a block's fields hold anything, a bit per 256 keys
    unsigned long long* wide;          // [65536] 64-bit credits per key, zero between calls
    unsigned long long* counts;        // histogram when the caller gives none
    void*               result_dev;    // edgc_entropy_result
};
template <typename T, int VEC>
static int run_entropy(edgc_ctx* ctx, const EntScratch& s, const EntGroup& g, uint32_t bins, const float* range,
                       uint64_t* counts_out, edgc_entropy_result* res, hipStream_t st)
{
    auto* counts = counts_out ? reinterpret_cast<unsigned long long*>(counts_out) : s.counts;

    const double sample_bytes = static_cast<double>(g.n_sampled) * sizeof(T);
    const bool small = g.n_items <= static_cast<uint64_t>(kHistBlock) * 4 * ctx->num_cu * 2;
    // One read into 16-bit counters per block (the kernels above), where the context has the memory
    // for the blocks' fields: every bf16 sample of some size (no range pass, any number of bins), and
    // fp32 samples on more bins than 32-bit counters hold in LDS at once.
    const bool wide_ok = s.part16 != nullptr && ctx->tune_pattern != 0;
    // The line for bf16 lies at 8 Mi elements, where two-pass samples leave the kernels of short blocks, and at half of that above 16384
    // bins.  It was drawn there when the sums over the bins took longer in the one read, and it is not where the two meet now: without a
    // caller's range that is at some 6 M elements up to 4096 bins, 3 to 4 M on 8192 and below 0.5 M from 12000 on (up to a fifth of the
    // estimate is left there); with one, which spares the two passes their first, beyond 8 Mi up to 4096 bins.  Per estimate in us, two passes
    // / one read, every element of a buffer (1 sampled in 3 and in 10: the same within 2; 12 and 24 buffers within 3):
    //                  256 bins      4096 bins      8192 bins    16384 bins    16385 bins    65536 bins
    //      1 M         13.0 / 17.4   15.5 / 18.4   19.9 / 20.0   28.1 / 22.8   25.4 / 22.9   45.3 / 35.5
    //      4 M         15.4 / 18.3   17.9 / 19.4   22.4 / 20.8   29.3 / 24.7   26.8 / 24.5   48.1 / 38.2
    //      6 M         18.4 / 19.2   21.6 / 20.5   25.2 / 21.8   31.2 / 25.6   28.5 / 25.7   49.9 / 39.6
    //      8.4 M       20.8 / 19.8   23.7 / 20.9   28.1 / 22.3   32.4 / 25.5   29.8 / 25.7   50.1 / 39.7
    //     12 M         25.7 / 22.1   28.1 / 23.1                 37.3 / 28.2   74.8 / 28.5   88.1 / 41.7
    //     24 M         36.2 / 28.0   38.5 / 28.8                 47.9 / 33.7   80.2 / 34.1   92.9 / 47.8
    //     64 M         58.8 / 40.8   63.8 / 42.0                 73.5 / 47.2   93.5 / 47.8  109.8 / 62.8
    //   a range given:
    //      4 M         13.4 / 18.4   14.6 / 19.6   21.9 / 20.8   26.0 / 24.5   23.3 / 24.7   50.6 / 45.6
    //      8.4 M       16.8 / 20.0   19.0 / 21.0   28.2 / 22.4   30.5 / 26.2   26.3 / 26.2   52.7 / 45.1
    //   buffers off 16-byte boundaries:
    //      1 M         16.4 / 17.7   18.0 / 18.8   24.3 / 20.5   38.0 / 23.4   34.5 / 23.5   64.6 / 35.9
    //      4 M         30.2 / 20.1   29.1 / 21.1   32.1 / 22.3   38.0 / 26.0   50.0 / 26.4   65.8 / 39.6
    const uint64_t pattern_min = static_cast<uint64_t>(ctx->tune_pattern_min);
    const bool by_pattern = sizeof(T) == 2 && wide_ok &&
                            (g.n_sampled >= pattern_min || (bins > 16384 && g.n_sampled >= pattern_min / 2));
    const bool by_wide_bins = sizeof(T) == 4 && wide_ok && bins > 16384 && bins <= kWideKeys;
    const uint32_t wide_blocks = grid_for(g.n_items, kWideBlock, 4, min(ctx->num_cu, static_cast<int>(s.part16_blocks)));
    // of k_wide_reduce, what is moved whatever the sample holds: marks, credits and bins (the host does not know which fields)
    const double reduce_bytes = 4.0 * kOccupiedWords * wide_blocks + 8.0 * kWideKeys + 8.0 * bins;
    uint32_t nparts = 0;                                   // blocks' (lo, hi) in s.mm_part
    double* const pair_part = reinterpret_cast<double*>(s.mm_part + kMaxReduceBlocks / 2);
    if constexpr (sizeof(T) == 2) {
        if (by_pattern) {
            EDGC_LAUNCH(ctx, st, KID_WIDE_HIST, sample_bytes, 0.0,
                        k_wide_hist<T, VEC, true><<<wide_blocks, kWideBlock, kWideKeys * 2, st>>>(
                            g, s.mm_part, nparts, bins, s.part16, s.occupied, s.wide, counts));
            EDGC_LAUNCH(ctx, st, KID_WIDE_REDUCE, reduce_bytes, 0.0,
                        k_wide_reduce<true><<<kWideKeys / kReduceKeys, kWideBlock, kWideReduceLds, st>>>(
                            s.part16, s.occupied, wide_blocks, s.wide, bins, range ? 1 : 0, range ? range[0] : 0.0f,
                            range ? range[1] : 0.0f, counts, s.mm_part, pair_part, s.ticket, g.n_sampled, res));
            EDGC_HIP_TRY(ctx, hipGetLastError());
            return EDGC_OK;
        }
    }
    // LDS plan: up to 64 KiB of 32-bit counters, replicated per lane where bins are few;
    // more than 16384 bins are covered in slices of 32768 (128 KiB), one slice per blockIdx.y
    // small samples get blocks of few items each, and then fewer replicas so that zeroing
    // and folding the LDS histogram does not outweigh the sampling itself
    const uint32_t word_cap = small ? 4096u : 16384u;
    uint32_t bins_local = bins, rep_shift = 0;
    if (bins <= 16384) {
        while (rep_shift < 5 && (static_cast<uint64_t>(bins) << (rep_shift + 1)) <= word_cap) ++rep_shift;
    } else if (bins > 32768) {
        bins_local = 32768;
    }
    const uint32_t ny = (bins + bins_local - 1) / bins_local;
    const size_t lds = static_cast<size_t>(bins_local << rep_shift) * sizeof(uint32_t);
    if (bins <= 16384 && !by_pattern && g.n_items <= 4u * kOneBlock) {
        EDGC_LAUNCH(ctx, st, KID_ESTIMATE_ONE, sample_bytes * (range ? 1.0 : 2.0), 0.0,
                    k_estimate_one<T, VEC><<<1, kOneBlock, lds, st>>>(g, range ? 1 : 0, range ? range[0] : 0.0f,
                                                                      range ? range[1] : 0.0f, bins, rep_shift, counts, res));
        EDGC_HIP_TRY(ctx, hipGetLastError());
        return EDGC_OK;
    }
    if constexpr (VEC > 1) {
        if (bins <= 4096 && small && ctx->tune_ept == 0) {
            auto launch = [&](auto u_tag) {
                constexpr int U = decltype(u_tag)::value;
                const uint32_t gx = static_cast<uint32_t>((g.n_items + kSmallBlock * U - 1) / (kSmallBlock * U));
                const uint32_t sets = gx > 16 ? 2u : 1u, zero_words = sets * copy_stride(bins);
                nparts = range ? 1u : gx;
                if (range)
                    EDGC_LAUNCH(ctx, st, KID_SET_RANGE, 4.0 * zero_words, 0.0,
                                k_set_range<<<(zero_words + 255) / 256, 256, 0, st>>>(s.mm_part, range[0], range[1], s.copies, zero_words));
                else
                    EDGC_LAUNCH(ctx, st, KID_MINMAX, sample_bytes, 0.0,
                                k_minmax_small<T, VEC, kSmallBlock, U><<<gx, kSmallBlock, 0, st>>>(g, s.mm_part, s.copies, zero_words));
                EDGC_LAUNCH(ctx, st, KID_HIST, sample_bytes, 0.0,
                            k_hist_small<T, VEC, kSmallBlock, U><<<gx, kSmallBlock, lds, st>>>(
                                g, s.mm_part, nparts, bins, rep_shift, s.copies, sets, counts, s.ticket, res));
            };
            if (g.n_items <= kSmallTwo) launch(std::integral_constant<int, 2>{});
            else launch(std::integral_constant<int, 4>{});
            EDGC_HIP_TRY(ctx, hipGetLastError());
            return EDGC_OK;
        }
    }
    // One block of 1024 threads per CU when a histogram of more than 64 KiB leaves room for one block only
    // (1e9 fp32 elements on 65536 bins: 1.6 instead of 3.6 ms) and for samples of 8 Mi items or more (1e8
    // fp32 elements on 4096 bins: 0.13 instead of 0.18 ms; 1e9: 0.83 instead of 0.86 ms); two blocks of
    // 512 per CU otherwise (1e7 bf16 elements: 0.040 against 0.044 ms; two blocks of 1024: slower throughout)
    const bool fat = lds > 65536 || g.n_items >= kBigSampleItems;
    // enough items per block that zeroing and flushing the LDS histogram stays small
    const int floor_items = small ? std::max(4, static_cast<int>((bins_local << rep_shift) / (kHistBlock * VEC / 2)))
                                  : ((bins_local << rep_shift) > 16384 ? 64 : 16);
    const int per_thread = ctx->tune_ept > 0 ? ctx->tune_ept : floor_items;
    // (EDGC_TUNE_EPT given: these kernels at every size)
    const uint32_t gx = fat ? grid_for(g.n_items, kHistBlockFat, per_thread, ctx->num_cu)
                            : grid_for(g.n_items, kHistBlock, per_thread, ctx->num_cu * 2);
    // the counters the histogram kernel accumulates into
    const uint32_t sets = (bins <= kCopyBins && g.n_sampled < (1ull << 32)) ? (gx > 16 ? 8u : 1u) : 0u;
    uint32_t* zero = sets ? s.copies : reinterpret_cast<uint32_t*>(counts);
    const uint32_t zero_words = by_wide_bins ? 0u : sets ? sets * copy_stride(bins) : 2u * bins;
    if (range) {
        nparts = 1;
        EDGC_LAUNCH(ctx, st, KID_SET_RANGE, 4.0 * zero_words, 0.0,
                    k_set_range<<<std::clamp((zero_words + 255) / 256, 1u, 1024u), 256, 0, st>>>(s.mm_part, range[0], range[1], zero,
                                                                                    zero_words));
    } else if (g.n_items >= kBigSampleItems) {
        // a large sample: one block of 1024 threads per CU (1e8 fp32 elements out of 1e9: 0.08 instead
        // of 0.12 ms, bf16 0.05 instead of 0.08; every element of 1e9: 0.70 instead of 0.71 ms)
        nparts = grid_for(g.n_items, kMMBlockFat, 16, ctx->num_cu);
        EDGC_LAUNCH(ctx, st, KID_MINMAX, sample_bytes, 0.0,
                    k_minmax<T, VEC, kMMBlockFat><<<nparts, kMMBlockFat, 0, st>>>(g, s.mm_part, zero, zero_words));
    } else {
        nparts = grid_for(g.n_items, kMMBlock, ctx->tune_ept > 0 ? 2 * ctx->tune_ept : 8, ctx->num_cu * 4);
        EDGC_LAUNCH(ctx, st, KID_MINMAX, sample_bytes, 0.0,
                    k_minmax<T, VEC, kMMBlock><<<nparts, kMMBlock, 0, st>>>(g, s.mm_part, zero, zero_words));
    }

    if constexpr (sizeof(T) == 4) {
        if (by_wide_bins) {
            EDGC_LAUNCH(ctx, st, KID_WIDE_HIST, sample_bytes, 0.0,
                        k_wide_hist<T, VEC, false><<<wide_blocks, kWideBlock, kWideKeys * 2, st>>>(
                            g, s.mm_part, nparts, bins, s.part16, s.occupied, s.wide, counts));
            EDGC_LAUNCH(ctx, st, KID_WIDE_REDUCE, reduce_bytes, 0.0,
                        k_wide_reduce<false><<<(bins + kReduceKeys - 1) / kReduceKeys, kWideBlock, kWideReduceLds, st>>>(
                            s.part16, s.occupied, wide_blocks, s.wide, bins, 0, 0.0f, 0.0f, counts, s.mm_part,
                            pair_part, s.ticket, g.n_sampled, res));
            EDGC_HIP_TRY(ctx, hipGetLastError());
            return EDGC_OK;
        }
    }

    if (fat) {
        EDGC_LAUNCH(ctx, st, KID_HIST, sample_bytes * ny, 0.0,
                    k_hist<T, VEC, kHistBlockFat><<<dim3(gx, ny), kHistBlockFat, lds, st>>>(
                        g, s.mm_part, nparts, bins, bins_local, rep_shift, s.copies, sets, counts, s.ticket, res));
    } else {
        EDGC_LAUNCH(ctx, st, KID_HIST, sample_bytes * ny, 0.0,
                    k_hist<T, VEC, kHistBlock><<<dim3(gx, ny), kHistBlock, lds, st>>>(
                        g, s.mm_part, nparts, bins, bins_local, rep_shift, s.copies, sets, counts, s.ticket, res));
    }
    EDGC_HIP_TRY(ctx, hipGetLastError());
    return EDGC_OK;
}

int prepare_entropy_kernels(edgc_ctx* ctx)
{
    constexpr int lds = 32768 * 4;     // one slice of 32768 bins
    constexpr int wide_lds = kWideKeys * 2;
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_wide_hist<uint16_t, 8, true>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_wide_hist<uint16_t, 1, true>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_wide_hist<float, 4, false>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_wide_hist<float, 1, false>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<float, 4, kHistBlock>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<float, 4, kHistBlockFat>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<float, 1, kHistBlock>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<float, 1, kHistBlockFat>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<uint16_t, 8, kHistBlock>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<uint16_t, 8, kHistBlockFat>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<uint16_t, 1, kHistBlock>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    EDGC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(&k_hist<uint16_t, 1, kHistBlockFat>),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, lds));
    return EDGC_OK;
}

static int launch_entropy_on(edgc_ctx* ctx, const EntScratch& s, const EntGroup& g, edgc_dtype dt, uint32_t bins,
                             const float* range, edgc_entropy_result* out, uint64_t* counts_out, hipStream_t st)
{
    // the kernels are compiled for one vector width: every buffer of the group was given the same
    const bool vec = g.vec > 1;
    // Pinned (device-accessible) host memory takes the result straight from the kernel; any
    // other host memory gets it through a copy on the stream.
    auto* res = static_cast<edgc_entropy_result*>(s.result_dev);
    bool direct = false;
    hipPointerAttribute_t attr;
    if (reinterpret_cast<uintptr_t>(out) % alignof(edgc_entropy_result) == 0 &&
        hipPointerGetAttributes(&attr, out) == hipSuccess && attr.type == hipMemoryTypeHost &&
        attr.devicePointer != nullptr) {
        res = static_cast<edgc_entropy_result*>(attr.devicePointer);
        direct = true;
    } else {
        (void)hipGetLastError();      // pageable memory is reported as an error: not one here
    }
    int rc;
    if (dt == EDGC_F32)
        rc = vec ? run_entropy<float, 4>(ctx, s, g, bins, range, counts_out, res, st)
                 : run_entropy<float, 1>(ctx, s, g, bins, range, counts_out, res, st);
    else
        rc = vec ? run_entropy<uint16_t, 8>(ctx, s, g, bins, range, counts_out, res, st)
                 : run_entropy<uint16_t, 1>(ctx, s, g, bins, range, counts_out, res, st);
    if (rc != EDGC_OK || direct) return rc;
    EDGC_HIP_TRY(ctx, hipMemcpyAsync(out, s.result_dev, sizeof(edgc_entropy_result),
                                     hipMemcpyDeviceToHost, st));
    return EDGC_OK;
}

int launch_entropy(edgc_ctx* ctx, const EntGroup& g, edgc_dtype dt, uint32_t bins,
                   const float* range, edgc_entropy_result* out, uint64_t* counts_out, hipStream_t st)
{
    const Scratch& c = ctx->s;
    const EntScratch s{reinterpret_cast<float2*>(c.mm_part), c.ticket, c.copies, c.part16, c.part16_blocks, c.occupied, c.wide,
                       c.counts, c.result_dev};
    return launch_entropy_on(ctx, s, g, dt, bins, range, out, counts_out, st);
}

// ---------------------------------------------------------------------------
// The estimate for callers that cannot allocate: its scratch is a file-scope device array, so
// nothing has to be allocated for it, by the library or by the caller.  Each GPU holds its own
// copy of the array at its own address; the address is looked up once per device, at the first
// edgc_create on that device (with that device current), and host code only ever uses that
// pointer, never the array's name.
// ---------------------------------------------------------------------------
constexpr size_t kStaticOffTicket = sizeof(float2) * kMaxReduceBlocks;
constexpr size_t kStaticOffResult  = kStaticOffTicket + sizeof(unsigned int) * kTicketWords;
constexpr size_t kStaticOffCopies  = kStaticOffResult + 256;
constexpr size_t kStaticOffCounts  = kStaticOffCopies + sizeof(uint32_t) * 8 * kCopyBins;
constexpr size_t kStaticBytes      = kStaticOffCounts + sizeof(unsigned long long) * kStaticMaxBins;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

constexpr int kMaxDevices = 64;
static unsigned char* g_static_scratch[kMaxDevices] = {};     // per device, set once

int resolve_static_scratch(edgc_ctx* ctx)
{
    const int dev = ctx->device;
    if (dev < 0 || dev >= kMaxDevices) return fail(ctx, EDGC_EINVAL, "device index beyond the static scratch table");
    if (g_static_scratch[dev]) return EDGC_OK;
    unsigned char* ptr = nullptr;
    EDGC_HIP_TRY(ctx, hipGetSymbolAddress(reinterpret_cast<void**>(&ptr), HIP_SYMBOL(scratch)));
    if (!ptr) return fail(ctx, EDGC_EHIP, "hipGetSymbolAddress returned a null address");
    // the ticket must start at zero; the array is zero-initialised when the code object is loaded
    // and every estimate leaves them at zero, but a process may have been interrupted mid-call
    EDGC_HIP_TRY(ctx, hipMemset(ptr + kStaticOffTicket, 0, sizeof(unsigned int) * kTicketWords));
    EDGC_HIP_TRY(ctx, hipDeviceSynchronize());
    g_static_scratch[dev] = ptr;
    return EDGC_OK;
}

int launch_entropy_static(edgc_ctx* ctx, const EntGroup& g, edgc_dtype dt, uint32_t bins, const float* range,
                          edgc_entropy_result* out, uint64_t* counts_out, hipStream_t st)
{
    unsigned char* base = (ctx->device >= 0 && ctx->device < kMaxDevices) ? g_static_scratch[ctx->device] : nullptr;
    if (!base) return fail(ctx, EDGC_EHIP, "the static scratch of this device was not set up");
    const EntScratch s{reinterpret_cast<float2*>(base),
                       reinterpret_cast<unsigned int*>(base + kStaticOffTicket),
                       reinterpret_cast<uint32_t*>(base + kStaticOffCopies),
                       nullptr, 0u, nullptr, nullptr,     // no room for the blocks' 16-bit counters: plain kernels
                       reinterpret_cast<unsigned long long*>(base + kStaticOffCounts), base + kStaticOffResult};
    return launch_entropy_on(ctx, s, g, dt, bins, range, out, counts_out, st);
}

int launch_sample_indices(edgc_ctx* ctx, const SampleGeom& g, uint64_t* idx, uint64_t cap,
                          hipStream_t st)
{
    if (g.n_items == 0) return EDGC_OK;
    const uint32_t gx = grid_for(g.n_items, 256, 4, 65535);
    EDGC_LAUNCH(ctx, st, KID_SAMPLE_IDX, 8.0 * g.n_sampled, 0.0,
                k_sample_indices<<<gx, 256, 0, st>>>(g, idx, cap));
    EDGC_HIP_TRY(ctx, hipGetLastError());
    return EDGC_OK;
}

}  // namespace edgc
