// How far the band of a tile reaches before the gate has erased it.
//
// The gate's decay grows along the band and soon outweighs what a score can add, which the norms bound: scale |q.k| <= scale |q| |k|.
// A key whose score then lies more than 127 binary orders (kErased: 126, the smallest normal fp32 number, and one for the roundings of scores
// and references) below the reference of a row has no part in it:
//   backward  p = exp2(x - L) is exactly zero: exp2 returns zero for every argument below -126 (measured over -120 .. -151), and then every
//             product it enters is zero.  No bit of a gradient changes.  (The split dK/dV kernels add up the column sums of a band's last block
//             rounded otherwise, so that a shorter band may move d(alpha) by such roundings, 5e-7 of its largest value, and deal the blocks that
//             are left of grouped heads out to their waves anew, another order of additions.)
//   forward   the row's reference is at least the score of its own key.  Where the whole band is measured against it (whole-tile kernels of bf16)
//             p is exactly zero again.  The split and the fp32 kernels form partial sums against references of their own first, in which far
//             keys weigh more, and scale them afterwards; so the line moves on by the doublings of the largest value row there, and
//             every product left out is below the smallest normal number by itself.
// Nothing less will do: a weight of 2^-50 is all that a row has where the values close by are zero or their loss is masked.
// (softplus(N(-2, 1)) decays by 190 over 1024 keys, unit-variance rows of d = 128 have |q| |k| / sqrt(d) of 11 to 15: the far 450 keys are
// left out.)
//
// So a pass over the rows in front of the kernels takes the largest norm of every block of them, and a workgroup shortens its band, in front
// of its first step, by the blocks at the far end that are erased for all rows of its tile.  The pass costs one reading of a
// matrix or two, the band of a step as many readings from the L2 as there are tiles in a window; workgroups that look at the rows of their
// band by themselves read as much as the steps they save (forward B4 H16 N8192 d128 w1024, gates as above: 288 us without, 284 so).
// Blocks whose gate decays too little read nothing (reach_pays).  A row that is not finite keeps its block, and a kept
// block all that lie in front of it: zero times infinity is NaN, here as in the kernels without this.
//
// The blocks' values travel in the rows of an output that is not written yet (O in front of the forward, dalpha in front of the
// backward), so that no call needs more memory for them.
//
// Measured, us, whole bands / shortened, the pass for the norms included; gates of softplus(N(mu, 1)), of which mu = -6 erases nothing:
//                                        mu        -6            -3           -2           -1
//   forward   B4 H16   N8192  d128 w1024       296 / 301     295 / 297    284 / 257    280 / 195
//             B1 H32   N16384 d128 w1024       308 / 311     307 / 312    300 / 267    293 / 201
//             B1 H32/8 N8192  d128 w4096       392 / 395     365 / 205    358 / 120    355 /  87
//             B4 H16   N4096  d64  causal      154 / 157     146 / 113    142 /  75    140 /  57
//             B1 H8    N5003  d128 w3000        52 /  55      52 /  56     52 /  46     53 /  39
//             B2 H16   N4096  d128 w1024 fp32  345 / 348     345 / 348    348 / 298    347 / 210
//   backward  B4 H16   N8192  d128 w1024       954 / 961     956 / 961    935 / 733    919 / 531
//             B1 H32   N16384 d128 w1024       971 / 981     974 / 978    942 / 749    931 / 548
//             B1 H32/8 N8192  d128 w4096      1320 / 1333   1268 / 590   1233 / 331   1230 / 229
//             B4 H16/4 N4096  d64  causal      576 / 579     560 / 336    545 / 189    542 / 128
//             B1 H8    N5003  d128 w3000       161 / 163     160 / 127    158 /  90    158 /  67
//             B2 H16   N4096  d128 w1024 fp32 1122 / 1135   1129 / 1126  1084 / 789   1055 / 521
#pragma once
#include <initializer_list>
#include <type_traits>

#include "gfwa_internal.h"
#include "tile_stage.h"

namespace gfwa {

constexpr float kErased = 127.f;
// Whether it can pay to read norms: `decay` over the `len` rows that see a block (that it sees).  Scores and values of unit-variance rows add about
// 22 to the 88 of kErased (in units of the gate); `few` rows fewer have to be worth the reading: of one matrix of three in front of the backward,
// of two in a launch of their own in front of the forward (key_reach.hip).  (Two products compared, so that two kernels which ask the same
// always agree: there is nothing the compiler could fuse in one of them.)
constexpr float kTypicalReach = 110.f;
constexpr int kFewBackward = 192;
__device__ __forceinline__ bool reach_pays(float decay, int len, int few) {
    return decay > kTypicalReach && decay * (float)(len - few) > kTypicalReach * (float)len;
}

// Integers in the order of the floats (its own inverse); NaN, which must not let anything be erased, as the lowest or the highest.
__device__ __forceinline__ int int_order(int bits) { return bits ^ ((bits >> 31) & 0x7fffffff); }
__device__ __forceinline__ int lowest_order(float x) { return x == x ? int_order(__float_as_int(x)) : (int)0x80000000; }
__device__ __forceinline__ int highest_order(float x) { return x == x ? int_order(__float_as_int(x)) : 0x7fffffff; }
__device__ __forceinline__ float from_order(int o) { return __int_as_float(int_order(o)); }
__device__ __forceinline__ bool finite(float x) { return fabsf(x) <= 3.402823466e38f; }

// op over LANES (32 or 64) lanes of a wave, result in all of them: within four, eight and sixteen lanes by moves, then between
// the rows of sixteen.
template <int LANES, typename Op>
__device__ __forceinline__ int over_lanes(int x, Op&& op) {
    x = op(x, __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true));   // quad_perm 1 0 3 2
    x = op(x, __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true));   // quad_perm 2 3 0 1
    x = op(x, __builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true));  // row_half_mirror
    x = op(x, __builtin_amdgcn_mov_dpp(x, 0x140, 0xF, 0xF, true));  // row_mirror
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = op((int)r[0], (int)r[1]);
    if (LANES == 64) {
        const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        x = op((int)q[0], (int)q[1]);
    }
    return x;
}
template <int LANES = 64>
__device__ __forceinline__ int lanes_max(int x) {
    return over_lanes<LANES>(x, [](int a, int b) { return max(a, b); });
}
template <int LANES = 64>
__device__ __forceinline__ int lanes_min(int x) {
    return over_lanes<LANES>(x, [](int a, int b) { return min(a, b); });
}
// Sum over the 4, 8 or 16 lanes of a row, in all of them.
template <int LANES>
__device__ __forceinline__ float row_sum(float x) {
    auto moved = [](float v, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    x += moved(x, std::integral_constant<int, 0xB1>{});
    x += moved(x, std::integral_constant<int, 0x4E>{});
    if (LANES >= 8) x += moved(x, std::integral_constant<int, 0x141>{});
    if (LANES == 16) x += moved(x, std::integral_constant<int, 0x140>{});
    return x;
}
// Sums of products of eight values; of squares as bits in the order of the floats (NaN above infinity).
__device__ __forceinline__ float dot8(const bf16x8& a, const bf16x8& b, float x) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) x = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{a[e], a[e + 1]}, bf16x2{b[e], b[e + 1]}, x, false);
    return x;
}
__device__ __forceinline__ int norm_bits(float n2) { return __float_as_int(n2) & 0x7fffffff; }

// What a wave (or workgroup) knows of its own rows: the largest squared norm, times (scale log2 e)^2 and a thousandth for the
// roundings of norms and products.
__device__ __forceinline__ float reach2_of(int norm, float sl) { return __int_as_float(norm) * (sl * sl * 1.004f); }
// room: what a score would have to exceed, in base-2 exponents, for a weight of 2^-kErased
__device__ __forceinline__ bool is_erased(float n2, float reach2, float room) { return room > 0.f && n2 * reach2 < room * room; }

// ---- keys in front of a query tile (forward).  A tile of queries from q0 finds in its own rows of O, as entry e, what there is to know of the
// block of `block` keys that is e + 1 blocks before the one that holds q0 (key_reach.hip): the largest squared norms of its key and of its
// value rows, each rounded up to bf16, and its highest gate.
struct KeyBlock {
    unsigned norms;  // value rows in the upper half
    float c;
    __device__ __forceinline__ float k2() const { return __uint_as_float(norms << 16); }
    __device__ __forceinline__ float v2() const { return __uint_as_float(norms & 0xffff0000u); }
};
constexpr int kInfBits = 0x7f800000;
__device__ __forceinline__ unsigned pack_norms(int k2, int v2) {  // (NaN becomes infinite)
    const unsigned k = (unsigned)min(k2, kInfBits) + 0xffffu, v = (unsigned)min(v2, kInfBits) + 0xffffu;
    return (k >> 16) | (v & 0xffff0000u);
}
// Entries that `rows` rows of O have room for, T the storage type.  (A last tile of one to three rows may lack some: its band stays whole.)
template <int D, typename T>
__host__ __device__ __forceinline__ constexpr int key_blocks_in(int rows) { return rows * (D * (int)sizeof(T) / (int)sizeof(KeyBlock)); }
// Entry `lane` of the tile whose first row of O is at `first`.
template <int D, typename T>
__device__ __forceinline__ KeyBlock key_block(const T* first, int rows, int lane) {
    const bool there = lane < key_blocks_in<D, T>(rows);
    const KeyBlock kb = reinterpret_cast<const KeyBlock*>(first)[there ? lane : 0];
    return {there ? kb.norms : pack_norms(kInfBits, kInfBits), kb.c};
}
// First key that the 32 queries of a wave need.  reach2 and `lowest` of the wave (lowest: the lowest exponent, relative to gate cbase,
// that a weight of a row is measured against, less kErased).
__device__ __forceinline__ int first_needed_key(const KeyBlock& kb, int q0, int k_lo, int block, float reach2, float lowest, float cbase, int lane) {
    const int hi = q0 / block - 1, n = hi - k_lo / block + 1;  // (n <= 64, reach_of sees to that)
    const float doublings = fmaxf(0.f, 0.5f * fast_log2(kb.v2()));
    const bool kept = lane < n && !is_erased(kb.k2(), reach2, lowest - (kb.c - cbase) * kLog2e - doublings);
    const unsigned long long mask = __builtin_amdgcn_ballot_w64(kept);
    const int farthest = mask ? 63 - __builtin_clzll(mask) : -1;
    return max(k_lo, (hi - farthest) * block);
}
// The lowest (highest) of the waves' values, in all of them; for uniform control flow, at[WAVES] of LDS.
template <int WAVES, bool LOWEST>
__device__ __forceinline__ int over_waves(int x, int* at, int wv, int lane) {
    if (lane == 0) at[wv] = x;
    wg_barrier();
    int r = at[0];
#pragma unroll
    for (int k = 1; k < WAVES; ++k) r = LOWEST ? min(r, at[k]) : max(r, at[k]);
    return __builtin_amdgcn_readfirstlane(r);
}

// The forward's side of a query tile of bf16 rows: first key that the workgroup needs.  q: the lane's fragments of row tc (halves of a
// wave: complementary columns), kd: the key of the same row.
template <int D, int WAVES>
__device__ __forceinline__ int forward_reach(const bf16x8 (&q)[D / 16], const bf16_t* kd, const KeyBlock& kb, float cq, int q0, int k_lo,
                                             int block, float cbase, float sl, int* at, int wv, int lane) {
    float q2 = 0.f, k2 = 0.f, own = 0.f;
#pragma unroll
    for (int kc = 0; kc < D / 16; ++kc) {
        const bf16x8 k = *reinterpret_cast<const bf16x8*>(kd + 16 * kc);
        q2 = dot8(q[kc], q[kc], q2);
        k2 = dot8(k, k, k2);
        own = dot8(q[kc], k, own);
    }
    q2 = xhalf_sum(q2);
    // the reference is at least the score of the query's own key, which its wave meets first
    const float edge = cq * kLog2e + sl * (xhalf_sum(own) - 1e-4f * sqrtf(q2 * xhalf_sum(k2)));
    const float reach2 = reach2_of(lanes_max<32>(norm_bits(q2)), sl), lowest = from_order(lanes_min<32>(lowest_order(edge))) - kErased;
    return over_waves<WAVES, true>(first_needed_key(kb, q0, k_lo, block, reach2, lowest, cbase, lane), at, wv, lane);
}

// ---- both sides of the backward.  Every 64-row block has values in its first rows of dalpha, which the row-dot kernels write:
constexpr int kReachRows = 64;
enum : int {
    kReachNorm,      // largest squared norm of its query rows (infinite: the block is kept), ..
    kReachEdge,      // .. lowest (c - c of the first row) + L;
    kReachKeyNorm,   // and, for passes that cannot look at their keys by themselves (split kernels, fp32), the largest squared norm of its
    kReachKeyHigh,   // .. key rows (infinite where a value row is not finite), their highest gate.
    kReachLast,      // From the whole-tile dK/dV kernel on, in the first block of its 128-key tiles: the last block of queries that needs a key.
    kReachValues
};
// Bands of up to this many keys, on average over the queries, are not looked at: of shorter ones only gates above 0.27 a key would erase enough, and a
// look in vain costs 1 to 2 % of the backward.  us, whole bands / looked at, mu -6, -2, -1: B4 H16/4 N4096 d64 w512 161 / 163, 160 / 162, 155 / 130;
// H16 d128 w512 300 / 302, 298 / 302, 297 / 260; H16 d64 w700 199 / 202, 196 / 196, 193 / 134 (that one is looked at).
constexpr double kShortestMean = 600;
// Row of dalpha from which on block i has its values: its first, or for a last block of too few rows the ninth of the one before.
__device__ __forceinline__ int reach_row(int i, int N) { return kReachRows * i + kReachValues <= N ? kReachRows * i : kReachRows * (i - 1) + 8; }

// dalpha, if the passes of a backward may leave rows out and may use it as scratch, else nullptr.
inline float* backward_reach(float* dalpha, const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* c, const float* L,
                             size_t size, int B, int H, int Hkv, int N, int d, int w, float scale) {
    const size_t rows = (size_t)B * H * N, gate = rows * sizeof(float), q = rows * d * size, kv = (size_t)B * Hkv * N * d * size;
    const double band = w < N ? w : N;
    bool free = scale > 0.f && band - band * band / (2.0 * N) > kShortestMean;
    for (const void* m : {Q, O, dO}) free = free && !overlap(dalpha, gate, m, q);
    for (const void* m : {K, V}) free = free && !overlap(dalpha, gate, m, kv);
    for (const float* v : {c, L}) free = free && !overlap(dalpha, gate, v, gate);
    return free ? dalpha : nullptr;
}

// What the own rows of a tile are: (scale log2 e |row|)^2 of the largest, and their edge relative to gate cbase in base-2 exponents (the lowest of
// queries, the highest of keys).
struct OwnRows {
    float reach2, edge;
};
// Blocks i0 and i1 (the same, or next to each other) of queries.
__device__ __forceinline__ OwnRows own_queries(const float* at, const float* ch, int i0, int i1, int N, float cbase, float sl) {
    const float *r0 = at + reach_row(i0, N), *r1 = at + reach_row(i1, N);
    const int norm = max(norm_bits(r0[kReachNorm]), norm_bits(r1[kReachNorm]));
    const int edge = min(lowest_order((ch[64 * i0] - cbase) + r0[kReachEdge]), lowest_order((ch[64 * i1] - cbase) + r1[kReachEdge]));
    return {reach2_of(norm, sl), from_order(edge) * kLog2e};
}
// Blocks i0 and i1 of keys.
__device__ __forceinline__ OwnRows own_keys(const float* at, int i0, int i1, int N, float cbase, float sl) {
    const float *r0 = at + reach_row(i0, N), *r1 = at + reach_row(i1, N);
    const int norm = max(norm_bits(r0[kReachKeyNorm]), norm_bits(r1[kReachKeyNorm]));
    const int edge = max(highest_order(r0[kReachKeyHigh] - cbase), highest_order(r1[kReachKeyHigh] - cbase));
    return {reach2_of(norm, sl), from_order(edge) * kLog2e};
}
// What block i of queries has to say to a key tile.
struct QueryBlock {
    float norm, edge, c;
};
__device__ __forceinline__ QueryBlock query_block(const float* at, const float* ch, int i, int N) {
    const float* r = at + reach_row(i, N);
    return {r[kReachNorm], r[kReachEdge], ch[64 * i]};
}
__device__ __forceinline__ bool needs_keys(const QueryBlock& b, const OwnRows& own, float cbase) {
    return !is_erased(b.norm, own.reach2, ((b.c - cbase) + b.edge) * kLog2e - own.edge - kErased);
}
// Last block of queries from i_hi down to i_min + 1 that needs one of the keys, else i_min.  at: of the head; first: block i_hi - lane, if
// there is one.
__device__ __forceinline__ int last_needing_block(const float* at, const float* ch, int i_min, int i_hi, int N, const OwnRows& own, float cbase, int lane,
                                                  QueryBlock first) {
    for (int top = i_hi; top > i_min; top -= 64) {
        const int i = top - lane;
        if (top != i_hi) first = query_block(at, ch, max(i, i_min), N);
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(i > i_min && needs_keys(first, own, cbase));
        if (mask) return top - __builtin_ctzll(mask);
    }
    return i_min;
}
// What block i of keys has to say to a query tile.
struct KeyValues {
    float norm, high;
};
__device__ __forceinline__ KeyValues key_values(const float* at, int i, int N) {
    const float* r = at + reach_row(i, N);
    return {r[kReachKeyNorm], r[kReachKeyHigh]};
}
// First block of keys from i_lo on that is needed, i_max if none before it is.  first: block i_lo + lane, if there is one.
__device__ __forceinline__ int first_needed_block(const float* at, int i_lo, int i_max, int N, const OwnRows& own, float cbase, int lane, KeyValues first) {
    for (int base = i_lo; base < i_max; base += 64) {
        const int i = base + lane;
        if (base != i_lo) first = key_values(at, min(i, i_max), N);
        const bool kept = i < i_max && !is_erased(first.norm, own.reach2, own.edge - kErased - (first.high - cbase) * kLog2e);
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(kept);
        if (mask) return base + __builtin_ctzll(mask);
    }
    return i_max;
}
// The two for a tile that has nothing requested yet: its own blocks and the first 64 of the other side in one trip to memory.
__device__ __forceinline__ int first_needed_block(const float* at, const float* ch, int i_lo, int i0, int i1, int N, float cbase, float sl, int lane) {
    const KeyValues first = key_values(at, min(i_lo + lane, i0), N);
    asm volatile("" ::: "memory");
    return first_needed_block(at, i_lo, i0, N, own_queries(at, ch, i0, i1, N, cbase, sl), cbase, lane, first);
}
__device__ __forceinline__ int last_needing_block(const float* at, const float* ch, int i0, int i1, int i_hi, int N, float cbase, float sl, int lane) {
    const QueryBlock first = query_block(at, ch, max(i_hi - lane, i1), N);
    asm volatile("" ::: "memory");
    return last_needing_block(at, ch, i1, i_hi, N, own_keys(at, i0, i1, N, cbase, sl), cbase, lane, first);
}
// What a row-dot workgroup has gathered of a block, `row` its place (one thread).  looked: whether it has; else the block is kept.
struct BlockValues {
    int norm, edge, key_norm, high;
};
constexpr BlockValues kNoRows = {0, 0x7fffffff, 0, (int)0x80000000};
__device__ __forceinline__ void write_block(float* row, const BlockValues& b, bool looked, bool keys) {
    row[kReachNorm] = looked ? __int_as_float(b.norm) : INFINITY;
    row[kReachEdge] = looked ? from_order(b.edge) : 0.f;
    if (!keys) return;
    row[kReachKeyNorm] = looked ? __int_as_float(b.key_norm) : INFINITY;
    row[kReachKeyHigh] = looked ? from_order(b.high) : 0.f;
}
// Over the workgroup, from all waves' lanes; at: of LDS.
template <bool KEYS>
__device__ __forceinline__ void gather_block(BlockValues* at, BlockValues b) {
    if (threadIdx.x == 0) *at = kNoRows;
    b.norm = lanes_max(b.norm), b.edge = lanes_min(b.edge);
    if (KEYS) b.key_norm = lanes_max(b.key_norm), b.high = lanes_max(b.high);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&at->norm, b.norm);
        atomicMin(&at->edge, b.edge);
        if (KEYS) {
            atomicMax(&at->key_norm, b.key_norm);
            atomicMax(&at->high, b.high);
        }
    }
    __syncthreads();
}

}  // namespace gfwa
