// Device helpers shared by the compressor's translation units: MFMA operand types, the
// conversion of fp32 values to bf16 operand planes, and the lookup of a block's tensor in a
// grouped launch.
//
// MFMA 32x32x16 operand layout (64 lanes): lane l supplies A[i = l%32][k = 8*(l/32) .. +8]
// and B[k = 8*(l/32) .. +8][j = l%32]; accumulator register v of lane l holds
// D[i = 8*(v/4) + 4*(l/32) + v%4][j = l%32].
#pragma once

#include "edgc_internal.h"

#include <cstddef>

namespace edgc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kLdsRow = 144;   // 128 B of operand data + 16 B pad: conflict-free 16-byte reads

__device__ __forceinline__ float bf16_bits_widen(uint32_t h) { return __uint_as_float(h << 16); }

// x -> planes: p[0] = bf16(x); with two planes p[1] = bf16(x - p[0])
template <int NP>
__device__ __forceinline__ void to_planes(float x, __bf16 (&p)[NP])
{
    p[0] = static_cast<__bf16>(x);
    if constexpr (NP == 2) p[1] = static_cast<__bf16>(x - static_cast<float>(p[0]));
}

// Two floats -> packed bf16 pairs, one 32-bit word per plane (v_cvt_pk_bf16_f32, RNE):
// w[0] = (bf16(x), bf16(y)); with two planes w[1] holds the rounded remainders.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <int NP>
__device__ __forceinline__ void pack_pair(float x, float y, uint32_t (&w)[NP])
{
    const f32x2 v = {x, y};
    const bf16x2 h = __builtin_convertvector(v, bf16x2);
    w[0] = __builtin_bit_cast(uint32_t, h);
    if constexpr (NP == 2) {
        const f32x2 hf = __builtin_convertvector(h, f32x2);
        const bf16x2 l = __builtin_convertvector(v - hf, bf16x2);
        w[1] = __builtin_bit_cast(uint32_t, l);
    }
}
// eight floats -> one MFMA fragment per plane
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int NP>
__device__ __forceinline__ void pack8(const float (&v)[8], bf16x8 (&f)[NP])
{
    uint32_t w[4][NP];
#pragma unroll
    for (int i = 0; i < 4; ++i) pack_pair<NP>(v[2 * i], v[2 * i + 1], w[i]);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const u32x4 q = {w[0][p], w[1][p], w[2][p], w[3][p]};
        f[p] = __builtin_bit_cast(bf16x8, q);
    }
}
template <int NP>
__device__ __forceinline__ void pack4(const float (&v)[4], bf16x4 (&f)[NP])
{
    uint32_t w[2][NP];
    pack_pair<NP>(v[0], v[1], w[0]);
    pack_pair<NP>(v[2], v[3], w[1]);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const u32x2 q = {w[0][p], w[1][p]};
        f[p] = __builtin_bit_cast(bf16x4, q);
    }
}

template <int NP>
__device__ __forceinline__ f32x16 mma(const bf16x8 (&a)[NP], const bf16x8 (&b)[NP], f32x16 acc)
{
    if constexpr (NP == 2) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc, 0, 0, 0);
    }
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc, 0, 0, 0);
}

// Where the bf16 operand copy of P^ holds eight rows of one factor column (one 16-byte unit): in the order of the Q-pass's
// B-fragments, 16 rows x 32 columns each, so that a wave's lanes (unit = lane: 8 (lane / 32) rows on, column lane % 32) store and
// load a fragment as 1 KB in a row, and the fragments of a 64-row stage are one contiguous tile.  Per pass, as
// [plane][column][row] (16-byte stores apart, LDS reads eight rows apart in k_apply) / in this order: hidden-5120 bf16 block at
// rank 128 1163 / 1145 us, two hidden-768 bf16 blocks at rank 16 87.7 / 86.0.
template <int NP, int RT>
__device__ __forceinline__ size_t pt_unit(uint32_t row16, uint32_t ct, uint32_t plane, uint32_t unit)
{
    return ((static_cast<size_t>(row16) * RT + ct) * NP + plane) * 64 + unit;
}

// Columns of a split partial: the padded rank, but 16 up to rank 16 (the accumulators hold 32 there, of which the upper half is
// zero): half the bytes to write and to sum.  Between events, 32 / 16: hidden-2048 fp32 block at rank 16, the Q-pass 33.4 to 35.5 /
// 30.5 us, the sums of P 3.0 / 2.3; three odd fp32 matrices at rank 13 3.8 / 3.0 and 2.5 / 2.1.  (Stores under a condition, not an
// early end of the lanes without: that one changed the registers of the kernels for small groups, 18.4 / 20.9 us.)
template <int RT>
__device__ __forceinline__ uint32_t part_width(uint32_t r)
{
    if constexpr (RT == 1) return r <= 16 ? 16u : 32u;
    return RT * 32u;
}

// Tensor of a grouped launch that owns block `bid` (tensors with no blocks are skipped).
// Blocks keep the order of the grid: consecutive blocks, which the dispatcher spreads
// round-robin over the 8 XCDs, walk along the rows of the matrix, so that neighbouring
// 256-byte pieces of a DRAM page are requested at about the same time (measured 5 to 20 %
// faster on small matrices than giving each XCD a contiguous range of tiles; the factor
// slices the blocks share are small enough to sit in every XCD's L2).
// The lines of the first tensor are asked for together with the list of first blocks, so that a group of one (every
// single-tensor call) does not wait for memory twice in a row at the head of every launch.  Without: 0.3 us per launch more,
// 256 x 256 fp32 at rank 64 through the single calls 52.7 us in eight launches.
__device__ __forceinline__ const TensorArgs& tensor_of(const Group& g, uint32_t bid)
{
    constexpr size_t at = offsetof(Group, t);
    static_assert(at / 64 == 1 && (at + offsetof(TensorArgs, gram)) / 64 == 2 && (at + offsetof(TensorArgs, m_pad)) / 64 == 3 &&
                  at + sizeof(TensorArgs) <= 256, "a word of each of the first tensor's lines");
    const uint64_t line1 = reinterpret_cast<uint64_t>(g.t[0].G), line2 = reinterpret_cast<uint64_t>(g.t[0].gram);
    const uint32_t line3 = g.t[0].m_pad;
    uint32_t t = 0;
#pragma unroll
    for (int i = 1; i < kMaxGroup; ++i) t += (bid >= g.first[i]) ? 1u : 0u;
    asm volatile("" :: "s"(line1), "s"(line2), "s"(line3));
    return g.t[t];
}

// element type of the gradient: one bf16 plane <=> bf16 gradients (raw bits), two planes <=> fp32
template <int NP> struct GradElem { using type = float; };
template <> struct GradElem<1> { using type = uint16_t; };

typedef float vf2 __attribute__((ext_vector_type(2)));

// Two or four neighbouring elements at whatever address the first one has: the hardware takes 4-, 8- and 16-byte accesses to
// global memory at any address (rows of an odd length begin at every one).  Same instructions as for aligned addresses; element by
// element, per pass: 8191 x 4097 fp32 at rank 13 deferred 245 us, with these 220; bf16 at rank 40 stored 390 and 322, hidden-3001
// bf16 block 813 and 548, hidden-500 fp32 block stored 80 and 67.
// Ordinary accesses are to structs of elements: an access to a vector type may alias anything and keeps the compiler from
// moving the next loads above it (k_pass_p on 3136 x 6528 at rank 60: 41.8 against 37.1 us).
struct Floats2 { float x, y; };
struct Floats4 { float x, y, z, w; };
struct __attribute__((packed, aligned(2))) Bf16Pair { uint32_t x; };       // raw bits
struct __attribute__((packed, aligned(2))) Bf16Quad { uint32_t x, y; };
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));   // for accesses past the caches
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t bf16x2_any __attribute__((aligned(2)));
typedef uint32_t bf16x4_any __attribute__((ext_vector_type(2), aligned(2)));

template <typename E>
__device__ __forceinline__ E at_any(const void* p) { return *static_cast<const E*>(p); }
template <typename E>
__device__ __forceinline__ void put_any(void* p, E v) { *static_cast<E*>(p) = v; }

// the next two elements of a gradient row; PAST: read once, past the caches
template <bool PAST>
__device__ __forceinline__ Floats2 load_pair(const float* p)
{
    if constexpr (!PAST) return at_any<Floats2>(p);
    const f32x2_any v = __builtin_nontemporal_load(reinterpret_cast<const f32x2_any*>(p));
    return {v.x, v.y};
}
template <bool PAST>
__device__ __forceinline__ uint32_t load_pair(const uint16_t* p)
{
    if constexpr (!PAST) return at_any<Bf16Pair>(p).x;
    return __builtin_nontemporal_load(reinterpret_cast<const bf16x2_any*>(p));
}

}  // namespace edgc
