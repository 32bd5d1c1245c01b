// Q-pass  Q_partial[s] = D[row range s, :]^T P^[row range s, :]  (Sec. II-B: the second product of the PowerSGD step)
// up to rank 64, any shape of at least two columns (checked on the host): every wave by itself.  A lane's loads of D are
// A-fragments as they stand, as in k_pass_q (compress.hip); the B-fragments of P^ come straight from memory, where
// k_apply has laid them out in the order of a wave's lanes (pt_unit): 1 KB loads that the XCD's L2 serves, no LDS tile
// and no barrier in the loop.
//   fp32 gradients, k_pass_q_direct: the waves of a block take the stages of its row range in turn (WR of them to a column group
// of 64, WC groups) and add their sums up in LDS at the end, in wave order, so that a block of four waves writes one
// partial where four blocks would write four.
//   bf16 gradients, k_pass_q_ring: a wave has a row range to itself, on the splits of k_pass_q and k_pass_q_full, and writes its partial: Q is
// theirs bit for bit.  (In another order of the sums a last bit of Q turns the bf16 rounding of operands and of the
// reconstruction: 2e-4 to 7e-4 of the result's norm.  In fp32 it stays a last bit.)
// What bounds them: the last-level cache for a D of some size (a read of it without arithmetic: 64 MB 13.6 us between events),
// launch, latency and the partials for a small one.  k_pass_q and k_pass_q_full keep one to two waves per SIMD in step by a barrier
// per stage.  Between events, those / these, D just written, fp32: 4096 x 4096 at rank 32 18.0 / 11.5 us, hidden-2048 block at
// rank 16 35 / 31; bf16 (pass_plan.h) two hidden-768 blocks at rank 16 12.6 / 9.5, where row ranges and partials of its own would save
// nothing, but 2048 x 2048 at rank 32 7.3 / 5.8 where they would save 3.5 more.
#include "compress_common.h"
#include "pass_plan.h"

namespace edgc {

template <int RT, bool STREAM, int WR, int WC>
__global__ __launch_bounds__(64 * WR * WC, 2) void k_pass_q_direct(const Group grp)
{
    constexpr int NP = 2;
    const TensorArgs& ta = tensor_of(grp, blockIdx.x);
    const float* __restrict__ D = ta.E;
    const bf16x8* __restrict__ pt = static_cast<const bf16x8*>(ta.pt);
    float* __restrict__ part = ta.part;
    const uint32_t m = ta.m, n = ta.n, sps = ta.d0, CB = ta.d1;
    __shared__ __attribute__((aligned(16))) float sums[WR * WC * 64 * 32];      // [column group][wave][column][factor column]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave % WR, wc = wave / WR;
    const int jl = lane & 31, g = lane >> 5;
    const uint32_t lid = blockIdx.x - ta.first;
    const uint32_t s = lid / CB, cb = lid % CB;
    const uint32_t jw0 = (cb * WC + wc) * 64u;                       // first column of this wave
    const uint32_t st_end = min((m + 63u) / 64u, (s + 1u) * sps);
    const uint32_t whole = min(st_end, m / 64u);                     // the stages before it have all their 64 rows
    // Columns jw0 + 2jl and + 1.  Past the last column a lane reads the last pair of the row again (n >= 2), and where the last
    // column is the first of a pair its value is the second of that one: what does not exist is not written below, and
    // a column's sums depend on that column alone.
    const uint32_t col = min(jw0 + 2u * jl, n - 2u);
    const bool odd_last = jw0 + 2u * jl == n - 1u;
    const uint32_t off = 8u * g * n + col;                           // element offset in a 16-row step (n < 2^28: fits 32 bits)

    f32x16 acc[RT][2];
#pragma unroll
    for (int ct = 0; ct < RT; ++ct)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ct][t][v] = 0.0f;
    float dv[4][8][2];

    // the 16-row steps U0 and U0 + 1 of stage ST: rows 8g + q of each step
#define EDGC_QDIRECT_FETCH_D(ST, U0)                                                                      \
    _Pragma("unroll") for (int uu = 0; uu < 2; ++uu) {                                                    \
        _Pragma("unroll") for (int q = 0; q < 8; ++q) {                                                   \
            const float* p_ = D + static_cast<uint64_t>((ST) * 64 + 16 * ((U0) + uu) + q) * n + off;       \
            const Floats2 x = load_pair<STREAM>(p_);                                                      \
            dv[(U0) + uu][q][0] = x.x; dv[(U0) + uu][q][1] = x.y;                                         \
        }                                                                                                 \
    }
    // half H of stage ST: to fragments; the same half of this wave's next stage is requested into the registers; multiplied
#define EDGC_QDIRECT_HALF(ST, MORE, H)                                                                    \
    {                                                                                                     \
        bf16x8 b[2][RT][NP];                                                                              \
        _Pragma("unroll") for (int uu = 0; uu < 2; ++uu)                                                  \
            _Pragma("unroll") for (int ct = 0; ct < RT; ++ct)                                             \
                _Pragma("unroll") for (int p = 0; p < NP; ++p)                                            \
                    b[uu][ct][p] = pt[pt_unit<NP, RT>((ST) * 4 + 2 * (H) + uu, ct, p, lane)];             \
        bf16x8 a[2][2][NP];                                                                               \
        _Pragma("unroll") for (int uu = 0; uu < 2; ++uu) {                                                \
            _Pragma("unroll") for (int t = 0; t < 2; ++t) {                                               \
                float col8[8];                                                                            \
                _Pragma("unroll") for (int q = 0; q < 8; ++q)                                             \
                    col8[q] = (t == 0 && odd_last) ? dv[2 * (H) + uu][q][1] : dv[2 * (H) + uu][q][t];     \
                pack8<NP>(col8, a[uu][t]);                                                                \
            }                                                                                             \
        }                                                                                                 \
        if constexpr (MORE) EDGC_QDIRECT_FETCH_D((ST) + WR, 2 * (H))                                      \
        _Pragma("unroll") for (int uu = 0; uu < 2; ++uu)                                                  \
            _Pragma("unroll") for (int ct = 0; ct < RT; ++ct)                                             \
                _Pragma("unroll") for (int t = 0; t < 2; ++t) acc[ct][t] = mma<NP>(a[uu][t], b[uu][ct], acc[ct][t]); \
    }

    uint32_t st = s * sps + wr;
    if (jw0 < n && st < st_end) {
        if (st < whole) {
            EDGC_QDIRECT_FETCH_D(st, 0)
            EDGC_QDIRECT_FETCH_D(st, 2)
            for (; st + WR < whole; st += WR) {
                EDGC_QDIRECT_HALF(st, true, 0)
                EDGC_QDIRECT_HALF(st, true, 1)
            }
            EDGC_QDIRECT_HALF(st, false, 0)
            EDGC_QDIRECT_HALF(st, false, 1)
            st += WR;
        }
        if (st < st_end) {                                           // the last rows; those past them as zeros
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const uint32_t row = st * 64u + 16u * u + 8u * g + q;
                    const Floats2 x = load_pair<STREAM>(D + static_cast<uint64_t>(min(row, m - 1u)) * n + col);
                    dv[u][q][0] = row < m ? x.x : 0.0f;
                    dv[u][q][1] = row < m ? x.y : 0.0f;
                }
            EDGC_QDIRECT_HALF(st, false, 0)
            EDGC_QDIRECT_HALF(st, false, 1)
        }
    }
#undef EDGC_QDIRECT_HALF
#undef EDGC_QDIRECT_FETCH_D

    // accumulator (ct, t, v) of lane l: column j = jw0 + 2 rho + t with rho = 8*(v/4) + 4*g + v%4, factor column
    // c = ct*32 + jl  ->  part[s][j][c], c < part_width, 32 factor columns at a time through LDS
    const uint32_t pw = part_width<RT>(grp.r);
    constexpr int ITEMS = WC * 64 * 8, NTH = 64 * WR * WC;           // of four factor columns
    float4* const s4 = reinterpret_cast<float4*>(sums);
#pragma unroll
    for (int ct = 0; ct < RT; ++ct) {
        if (ct) __syncthreads();                                     // the sums before are read
        float* mine = sums + (wc * WR + wr) * 64 * 32;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) mine[(2 * (8 * (v / 4) + 4 * g + v % 4) + t) * 32 + jl] = acc[ct][t][v];
        __syncthreads();
#pragma unroll
        for (int i0 = 0; i0 < ITEMS; i0 += NTH) {
            static_assert(ITEMS % NTH == 0, "the items divide evenly among the threads");
            const int i = i0 + tid, c = i / (64 * 8), e = i % (64 * 8);
            float4 x = s4[c * WR * 64 * 8 + e];
#pragma unroll
            for (int w = 1; w < WR; ++w) {
                const float4 y = s4[(c * WR + w) * 64 * 8 + e];
                x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w;
            }
            const uint32_t j = (cb * WC + c) * 64u + e / 8;
            if (j < n && (RT > 1 || e % 8 * 4u < pw))
                *reinterpret_cast<float4*>(part + (static_cast<size_t>(s) * n + j) * pw + ct * 32 + e % 8 * 4) = x;
        }
    }
}

template <int NT, bool STREAM>
__device__ __forceinline__ void load_columns(const float* p, float (&v)[NT])
{
    if constexpr (NT == 2) {
        const Floats2 x = load_pair<STREAM>(p);
        v[0] = x.x; v[1] = x.y;
    } else {
        v[0] = STREAM ? __builtin_nontemporal_load(p) : *p;
    }
}

// NT: columns per lane, 32 NT per wave.  Blocks go through the row ranges first, so that the blocks that read the same rows of P^
// and neighbouring columns of D are a multiple of the number of ranges apart, mostly on one XCD: the other way round 16384 x 1024
// at rank 32 15.8 / 10.8 us, hidden-1024 block 10.3 / 8.5, but 4096 x 4096 11.1 / 12.7.
template <int RT, int NT, bool STREAM>
__global__ __launch_bounds__(256, NT == 1 ? 4 : 2) void k_pass_q_ring(const Group grp)
{
    const TensorArgs& ta = tensor_of(grp, blockIdx.x);
    const float* __restrict__ D = ta.E;
    const bf16x8* __restrict__ pt = static_cast<const bf16x8*>(ta.pt);
    float* __restrict__ part = ta.part;
    const uint32_t m = ta.m, n = ta.n, sps = ta.d0, S = ta.sq;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int jl = lane & 31, g = lane >> 5;
    const uint32_t lid = blockIdx.x - ta.first;
    const uint32_t s = lid % S, cb = lid / S;
    const uint32_t jw0 = (cb * 4u + wave) * (32u * NT);              // first column of this wave
    if (jw0 >= n) return;
    const uint32_t st0 = s * sps;                                    // (below the number of stages: S = ceil(stages / sps))
    const uint32_t st_end = min((m + 63u) / 64u, st0 + sps);
    const uint32_t whole = min(st_end, m / 64u);                     // the stages before it have all their 64 rows
    // the lane's columns, past the last one and where that is the first of a pair: as in k_pass_q_direct
    const uint32_t col = min(jw0 + NT * jl, n - NT);
    const bool odd_last = NT == 2 && jw0 + NT * jl == n - 1u;
    const uint32_t off = 8u * g * n + col;                           // element offset in a 16-row step (n < 2^28: fits 32 bits)

    f32x16 acc[RT][NT];
#pragma unroll
    for (int ct = 0; ct < RT; ++ct)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[ct][t][v] = 0.0f;
    // Two places for the halves (32 rows) of a stage: what is requested of D, and the fragments of P^ for it.  Both are requested when the
    // half before the last has been consumed: loads complete in order, so that fragments requested just before their use would
    // wait for all of D requested before them (4096 x 4096 at rank 32, strips of 64, the fp32 operands: 22.2 us, so 16.3).
    // With three or four halves in flight the kernel is no faster.
    float dv[2][2][8][NT];
    bf16x8 b[2][2][RT][1];

#define EDGC_QRING_FETCH_D(HALF, H)                                                                       \
    _Pragma("unroll") for (int u = 0; u < 2; ++u) {                                                       \
        _Pragma("unroll") for (int q = 0; q < 8; ++q)                                                     \
            load_columns<NT, STREAM>(D + static_cast<uint64_t>((HALF) * 32u + 16 * u + q) * n + off, dv[H][u][q]); \
    }
#define EDGC_QRING_FETCH_P(HALF, H)                                                                       \
    _Pragma("unroll") for (int u = 0; u < 2; ++u) {                                                       \
        _Pragma("unroll") for (int ct = 0; ct < RT; ++ct)                                                 \
            b[H][u][ct][0] = pt[pt_unit<1, RT>((HALF) * 2u + u, ct, 0, lane)];                            \
    }
    // half HALF, in place H: to fragments; the half after the next is requested into the registers; multiplied
#define EDGC_QRING_HALF(HALF, MORE, H)                                                                    \
    {                                                                                                     \
        bf16x8 a[2][NT][1];                                                                               \
        _Pragma("unroll") for (int u = 0; u < 2; ++u) {                                                   \
            _Pragma("unroll") for (int t = 0; t < NT; ++t) {                                              \
                float col8[8];                                                                            \
                _Pragma("unroll") for (int q = 0; q < 8; ++q)                                             \
                    col8[q] = (t == 0 && odd_last) ? dv[H][u][q][NT - 1] : dv[H][u][q][t];                \
                pack8<1>(col8, a[u][t]);                                                                  \
            }                                                                                             \
        }                                                                                                 \
        if constexpr (MORE) EDGC_QRING_FETCH_D((HALF) + 2, H)                                             \
        _Pragma("unroll") for (int u = 0; u < 2; ++u)                                                     \
            _Pragma("unroll") for (int ct = 0; ct < RT; ++ct)                                             \
                _Pragma("unroll") for (int t = 0; t < NT; ++t) acc[ct][t] = mma<1>(a[u][t], b[H][u][ct], acc[ct][t]); \
        if constexpr (MORE) EDGC_QRING_FETCH_P((HALF) + 2, H)                                             \
    }

    uint32_t st = st0;
    if (st < whole) {
        EDGC_QRING_FETCH_D(2 * st, 0)
        EDGC_QRING_FETCH_P(2 * st, 0)
        EDGC_QRING_FETCH_D(2 * st + 1, 1)
        EDGC_QRING_FETCH_P(2 * st + 1, 1)
        for (; st + 1 < whole; ++st) {
            EDGC_QRING_HALF(2 * st, true, 0)
            EDGC_QRING_HALF(2 * st + 1, true, 1)
        }
        EDGC_QRING_HALF(2 * st, false, 0)
        EDGC_QRING_HALF(2 * st + 1, false, 1)
        ++st;
    }
    if (st < st_end) {                                               // the last rows; those past them as zeros
#pragma unroll 1
        for (uint32_t half = 2 * st; half < 2 * st + 2; ++half) {
            EDGC_QRING_FETCH_P(half, 0)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const uint32_t row = half * 32u + 16u * u + 8u * g + q;
                    load_columns<NT, STREAM>(D + static_cast<uint64_t>(min(row, m - 1u)) * n + col, dv[0][u][q]);
#pragma unroll
                    for (int t = 0; t < NT; ++t) dv[0][u][q][t] = row < m ? dv[0][u][q][t] : 0.0f;
                }
            EDGC_QRING_HALF(half, false, 0)
        }
    }
#undef EDGC_QRING_HALF
#undef EDGC_QRING_FETCH_P
#undef EDGC_QRING_FETCH_D

    // accumulator (ct, t, v) of lane l: column j = jw0 + NT*rho + t with rho = 8*(v/4) + 4*g + v%4,
    // factor column c = ct*32 + jl  ->  part[s][j][c], c < part_width
    const uint32_t pw = part_width<RT>(grp.r);
#pragma unroll
    for (int ct = 0; ct < RT; ++ct)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint32_t j = jw0 + NT * (8 * (v / 4) + 4 * g + v % 4) + t;
                if (j < n && (RT > 1 || static_cast<uint32_t>(jl) < pw))
                    part[(static_cast<size_t>(s) * n + j) * pw + ct * 32 + jl] = acc[ct][t][v];
            }
}

template <int RT, int WR, int WC>
static hipError_t launch_qdirect(const Group& g, uint32_t blocks, hipStream_t st)
{
    if (g.stream) k_pass_q_direct<RT, true, WR, WC><<<blocks, 64 * WR * WC, 0, st>>>(g);
    else k_pass_q_direct<RT, false, WR, WC><<<blocks, 64 * WR * WC, 0, st>>>(g);
    return hipGetLastError();
}

hipError_t launch_pass_q_direct(const Group& g, int rt, uint32_t blocks, uint32_t column_groups, hipStream_t st)
{
    if (column_groups == 1) return rt == 1 ? launch_qdirect<1, 4, 1>(g, blocks, st) : launch_qdirect<2, 4, 1>(g, blocks, st);
    return rt == 1 ? launch_qdirect<1, 2, 2>(g, blocks, st) : launch_qdirect<2, 2, 2>(g, blocks, st);
}

template <int RT, int NT>
static hipError_t launch_qring(const Group& g, uint32_t blocks, hipStream_t st)
{
    if (g.stream) k_pass_q_ring<RT, NT, true><<<blocks, 256, 0, st>>>(g);
    else k_pass_q_ring<RT, NT, false><<<blocks, 256, 0, st>>>(g);
    return hipGetLastError();
}

hipError_t launch_pass_q_ring(const Group& g, int rt, uint32_t blocks, uint32_t strip, hipStream_t st)
{
    if (rt == 2) return launch_qring<2, 2>(g, blocks, st);
    return strip == 32 ? launch_qring<1, 1>(g, blocks, st) : launch_qring<1, 2>(g, blocks, st);
}

}  // namespace edgc
