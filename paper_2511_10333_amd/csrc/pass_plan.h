// How the passes cut the tensors of a group into blocks.  Plain C++: the plans are checked on the CPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace edgc {

// Blocks of equal length: tensor i is `across[i]` blocks wide, and its `along[i]` stages are cut into runs of the returned
// number of stages, the smallest of at least `least` with which the launch has at most `target` blocks (`blocks`: how many
// it has).
inline uint32_t uniform_step(uint32_t count, const uint32_t* across, const uint32_t* along, uint32_t least, uint64_t target,
                             uint64_t& blocks)
{
    uint32_t lo = least, hi = least;
    for (uint32_t i = 0; i < count; ++i) hi = std::max(hi, along[i]);
    auto count_blocks = [&](uint32_t step) {
        uint64_t b = 0;
        for (uint32_t i = 0; i < count; ++i) b += static_cast<uint64_t>(across[i]) * ((along[i] + step - 1) / step);
        return b;
    };
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (count_blocks(mid) <= target) hi = mid; else lo = mid + 1;
    }
    blocks = count_blocks(lo);
    return lo;
}

// Stages (of 64 columns) per block of the P-pass.  `rp`: columns of a partial factor; `d_bytes`: the group's residual;
// `most`: how many splits the scratch of each tensor has room for (at least one): no plan with more is looked at, so that the
// launch is the plan that was weighed; `per_cu`: blocks per CU to aim at, 0 for the rule.
//
// Fewer column splits mean fewer partials to write and to sum, more blocks even out the load and keep more loads in flight.
// Measured per pass, against blocks in proportion to the tensors' size, four per CU (256-row blocks: two); fp32 and bf16,
// ranks 16, 64 and 128, stored and deferred:
//  * 256-row blocks (rank 128, whole tiles): two per CU.  Hidden-1024 to hidden-6144 blocks -9 to +1 %; three per CU +1 to
//    +15 %, four +3 to +15 % (hidden-1024: 175 us with three, 156 with two).
//  * 128-row blocks, residual up to 224 MB: two per CU, or three and four where that leaves CUs with one block while others
//    have two.  Hidden-1280 block -5 to -9 %, hidden-2048 (201 MB) -4 to +1, 832 x 11584 -4 to -9, 600 x 12818 -9 to -17;
//    four per CU 0 to +1.  What is left idle counts for more the longer the pass: at 3/4 of the places taken, 1381 x 9200
//    (51 MB) -3 to -7 %, hidden-1024 (50 MB) -6 to +2, four hidden-1024 blocks (201 MB) 0 to +8, 50257 x 768 (154 MB) -3 to +7.
//  * larger residuals: from four per CU on.  8192 x 8192 (268 MB) with two +4 to +7 %, 4000 x 16384 +2 to +6, hidden-3584
//    +4 to +13, hidden-4096 +4 to +7 and with four -5 to -1.  The line lies between 201 and 262 MB.  Four where
//    that fills nine tenths of the places, five and more otherwise: hidden-3072 (864 blocks) with four +1 to +5, with five
//    (1152) -4 to 0; 50257 x 4096 (786 blocks) 0, with five -5 to -10.
//  * more than four per CU only while the partials stay below a sixteenth of what a block reads and writes (8 rp bytes
//    against 16 per column): 662 x 13048 with five (one stage per block) +12 to +17 %, hidden-2304 at rank 128 stored +3.
inline uint32_t pass_p_step(uint32_t count, const uint32_t* across, const uint32_t* along, const uint64_t* most,
                            uint32_t rows_per_block, uint32_t rp, double d_bytes, uint32_t cu, uint32_t per_cu)
{
    constexpr double MB = 1024.0 * 1024.0;
    uint64_t blocks = 0;
    uint32_t least = 1;
    for (uint32_t i = 0; i < count; ++i) least = std::max(least, static_cast<uint32_t>((along[i] + most[i] - 1) / most[i]));
    if (per_cu == 0 && rows_per_block == 256) per_cu = 2;
    if (per_cu) return uniform_step(count, across, along, least, static_cast<uint64_t>(cu) * per_cu, blocks);
    const bool large = d_bytes > 224.0 * MB;
    const double enough = large ? 0.9 : d_bytes > 96.0 * MB ? 0.8 : 0.75;
    uint32_t step = least;
    double best = 0.0;
    for (uint32_t k = large ? 4 : 2; k <= 8 && best < enough; ++k) {
        const uint32_t s = uniform_step(count, across, along, least, static_cast<uint64_t>(cu) * k, blocks);
        if (k > 4 && 8u * s < rp) break;
        const uint64_t places = (blocks + cu - 1) / cu * cu;
        const double taken = static_cast<double>(blocks) / static_cast<double>(places);
        if (taken > best) { best = taken; step = s; }
    }
    return step;
}

// The Q-pass of waves by themselves (pass_q_direct.hip), up to rank 64, fp32 gradients.  Column groups per block, 0 where the other
// kernels stay: that is a D that the last-level cache cannot hold, where every form waits for HBM (per pass without an estimate, others /
// this: hidden-4096 block at rank 16 824 / 824 to 831 us, stored at rank 64 1157 / 1159 to 1168; stored hidden-2304 (255 MB) at rank
// 64 58 / 65, the Q-pass alone), while hidden-2048 (201 MB) takes 215 / 209.  Two groups where rows are not whole lines and strips of one
// group would share them: three odd matrices at rank 13 95.8 / 93.6 with one / 92.1 with two, 3002 x 5002 91.4 / 90.6 / 90.8;
// above rank 32 the sums of two weigh more: 8191 x 4097 at rank 64 261.0 / 261.5 / 263.9, 2047 x 2049 82.3 / 80.1 / 81.7.
inline uint32_t q_direct_groups(double d_bytes, uint32_t rp, bool lines)
{
    if (d_bytes > 224.0 * 1024 * 1024) return 0;
    return lines || rp > 32 ? 1 : 2;
}
// Blocks (of four waves) per CU aimed at.  Three are resident up to rank 32 (150 registers) and two above (190); a fourth, which begins
// as others end, is worth its row splits where a block would have few: two / three / four, two hidden-768 blocks at rank 16 77.3 / 76.9 /
// 75.2, 4096 x 4096 at rank 32 148.8 / 149.1 / 149.1, hidden-2048 block at rank 16 207.2 / 204.6 / 205.0; above rank 32 3072 x
// 3072 at rank 64 91.6 / 93.2 / 93.4; two groups: three odd matrices 92.8 / 93.2 / 95.8.
inline uint32_t q_direct_per_cu(uint32_t groups, uint32_t rp) { return groups == 1 && rp <= 32 ? 4 : 2; }
// ... but beyond 32 row splits no more than two per CU are worth their partials (tall matrices of few columns): 50257 x 1024 bf16 at
// rank 32 280.6 / 282.3 / 285.3, 50257 x 768 fp32 220.9 / 222.9 / 225.2, 100000 x 96 bf16 87.6 / 87.4 / 92.2, 16384 x 1024 92.3 / 92.4 / 93.9.
inline uint32_t q_direct_splits(uint32_t splits, uint32_t per_cu)
{
    return per_cu > 2 && splits > 32 ? std::max(32u, splits * 2 / per_cu) : splits;
}

// bf16: columns per wave of k_pass_q_ring, 0 where k_pass_q and k_pass_q_full stay.  It takes their row splits, which give one wave of 64
// columns per SIMD up to 80 MB of D: there strips of 32, twice the waves, are the fastest.  Between events, those / 64 / 32 at rank 32:
// 1024 x 1024 4.0 / 3.3 / 2.3 us, 2048 x 2048 7.3 / 6.5 / 5.8, 4096 x 4096 16.3 / 12.4 / 12.7, 16384 x 1024 12.9 / 13.1 / 10.8,
// hidden-1024 block 12.5 / 10.1 / 8.5, two hidden-768 blocks 12.6 / 11.8 / 9.7, 3002 x 5002 13.2 / 12.9 / 12.1.  With two waves per SIMD, above
// that, the passes of all forms are the same, and of ragged rows the ones here the slower (hidden-1500 block at rank 16 160 / 175 / 175,
// hidden-768 block and 50257 x 768 190 / 206 / 207).  Above rank 32 there are registers for 64 columns only, and groups of whole
// tiles of some size, which k_pass_q_full takes, gain nothing: 4096 x 4096 at rank 64 15.5 / 15.5, hidden-1024 block 12.0 / 13.0, but 2048 x 2048
// 11.9 / 9.4, 1024 x 1024 5.8 / 4.8, two hidden-768 blocks 15.7 / 13.9.
inline uint32_t q_ring_strip(double d_bytes, uint32_t rp, bool whole_tiles)
{
    constexpr double MB = 1024.0 * 1024;
    if (d_bytes > 80 * MB) return 0;
    if (rp > 32) return whole_tiles && d_bytes > 32 * MB ? 0 : 64;
    return 32;
}

// Stages (of 64 columns) per block of the decompress.  `splits`: into how many its share of the blocks aimed at would cut the
// tensor; `as_asked`: the whole-tile kernel, or a count of blocks per CU that was asked for.
// Otherwise at most eight stages: many rounds of short blocks keep every CU busy to the end.  Stored form, per pass: hidden-4096
// fp32 block at rank 64 with 24 stages per block 1276 us, 8: 1208, 6: 1215, 4: 1199 (the kernel 498 -> 425 us, 5.7 TB/s,
// what a plain copy reaches); at rank 16 1229 / 1168 (8) / 1148 (4); 8192 x 8192 at rank 64 with 8 stages 396, 4: 400,
// 1: 411; hidden-3072 at rank 128 with 14 stages 866, 7: 844, 5: 862.
inline uint32_t decompress_step(uint32_t stages, uint32_t splits, bool as_asked)
{
    const uint32_t step = (stages + splits - 1) / splits;
    return as_asked ? step : std::min(step, 8u);
}

// Whether a launch moves its tensors' gradients (reconstructions) past the caches: all of them, none, or each as its
// TensorArgs::past says.  Only mixed groups get the kernel that holds both forms: it has twice the code and some registers more.
// One form for a whole mixed group, that of the worst tensor, costs the other tensors.  Per pass, past for all / through for all /
// each its own: hidden-4096 fp32 block with a 2056 x 1028 matrix beside it, rank 64, deferred 975 / 1043 / 972 us, bf16 786 / 824 /
// 776; hidden-2048 with 2048 x 2054, rank 32, fp32 291 / 305 / 287, bf16 stored 307 / 303 / 293.
// Small groups through the caches take kernels without the loop whose loads can be counted: they are bound by latencies, and its second
// copy costs code, registers and, in the stored decompress, one of two waves per SIMD.  Per pass with / without it: 501 x 501 bf16 at
// rank 64 61.5 / 58.7 us, 2047 x 2049 (16 MB) 89.5 / 85.7 and stored 94.9 / 90.0, 3002 x 3002 (34 MB) 101.2 / 96.6, 3300 x 3302 (42 MB) 1.5 % less,
// hidden-1000 block (46 MB) 1 % more, hidden-1200 (66 MB) 5 % more, hidden-2056 fp32 5 % more; the stored decompress alone 2047 x 2049
// 18.8 / 14.0, 5000 x 1002 19.8 / 14.6, hidden-500 block 12.2 / 9.3.
enum class Caching { past, through, by_tensor, small };
constexpr double kSmallGroup = 40.0 * 1024 * 1024;                       // bytes of D
inline Caching group_caching(uint32_t n_past, uint32_t count, double d_bytes)
{
    if (n_past == count) return Caching::past;
    if (n_past) return Caching::by_tensor;
    return d_bytes <= kSmallGroup ? Caching::small : Caching::through;
}

// Whether the P-pass reads a gradient past the caches whose rows are not whole lines of them.  Through them, the two stages that
// share a line fetch it once; but a group's gradients beside its D (`d_bytes`) then push D out of the 256 MB last-level cache,
// where the Q-pass or the decompress would find it.  `pairs`: the kernels whose lanes read two columns (k_pass_p_deferred); k_pass_p's
// read four and share fewer lines.  Per pass without an estimate, past / through, in us, by the size of D:
//  * k_pass_p: 16 MB (2047 x 2049 fp32 at rank 13) 68.3 / 65.8, 19 MB (5000 x 1002, rank 64) 113.0 / 105.8, 29 MB (hidden-777 block)
//    91.8 / 87.8, 34 MB 90.1 / 84.8, 42 MB (3300 x 3302) 98.9 / 98.1 and at rank 64 129.9 / 130.2, 46 MB 135.2 / 137.2, 64 MB 161.0 /
//    165.9, 103 MB 231.9 / 239.4.
//  * pairs, stored, bf16: 46 MB 101.4 / 91.1, 64 MB (4097 x 4095) 121.1 / 111.9, 66 MB (hidden-1200) 117.9 / 121.1, 103 MB 203.8 / 216.7,
//    194 MB (hidden-2056) 289.3 / 300.2, 412 MB (hidden-3001) 785 / 778.
//  * pairs, deferred (D is not read again after the Q-pass), fp32: 46 MB 84.9 / 84.9, 66 MB at rank 64 151.7 / 156.7, 69 MB (3002 x
//    6002) 111.3 / 116.3, 103 MB 167.5 / 166.7, 128 MB (8191 x 4097) 210.4 / 204.2, 194 MB 278.8 / 274.1; bf16: 46 MB 82.9 / 76.4,
//    69 MB 105.0 / 121.9, 103 MB 170.6 / 183.0, 132 MB 172.8 / 179.1, 194 MB 244.9 / 235.4, 412 MB 546 / 529.
inline bool gradient_past(double d_bytes, uint32_t elem_bytes, bool pairs, bool defer)
{
    constexpr double MB = 1024.0 * 1024.0;
    const double both = d_bytes * (1.0 + elem_bytes / 4.0);             // D and G
    if (!pairs) return both > 80.0 * MB;
    return both > 96.0 * MB && (defer ? both : d_bytes) <= 256.0 * MB;
}

// rows that begin and end with a line of the caches
inline bool whole_lines(const void* p, uint64_t row_bytes)
{
    return row_bytes % 128 == 0 && reinterpret_cast<uintptr_t>(p) % 128 == 0;
}

}  // namespace edgc
