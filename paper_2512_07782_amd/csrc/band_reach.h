// How far the band of a tile reaches before the gate has erased it.
//
// The gate's decay grows along the band and soon outweighs what a score can add, which the norms bound: scale |q.k| <= scale |q| |k|.
// A key whose score then lies below the reference of a row by more than the binary orders that an fp32 sum resolves has no part in it:
//   kErased = 127  exp2 returns zero for every argument below -126 (the smallest normal number; measured over -120 .. -151), so the
//                  probability is exactly zero and every product it enters is zero, whatever the values are
//   kFaint = 48    and one more for every doubling by which the values that the weight would multiply outweigh those of rows close by
//                  (outweighs): the weights left out add up to less than 2^-36 of the row's (4096 keys) in these terms, so a sum misses
//                  less than 2^-36 of the values it is made of, 2^-12 of a rounding of fp32.
// (softplus(N(-2, 1)) decays by 190 over 1024 keys, unit-variance rows of d = 128 have |q| |k| / sqrt(d) of 11 to 15: the far 750 keys are
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
// Measured, us, whole bands / shortened, the pass for the norms included; gates of softplus(N(mu, 1)):
//                                        mu        -3           -2           -1
//   forward   B4 H16   N8192  d128 w1024       301 / 294    291 / 212    286 / 180
//             B1 H32   N16384 d128 w1024       314 / 300    304 / 217    302 / 185
//             B1 H32/8 N8192  d128 w4096       361 / 136    354 /  90    350 /  72
//             B4 H16   N4096  d64  causal      144 /  78    139 /  60    140 /  52
//             B2 H16   N4096  d128 w1024 fp32  351 / 324    353 / 226    353 / 181
//   backward  B4 H16   N8192  d128 w1024      1053 / 865   1016 / 613   1008 / 510
//             B1 H32   N16384 d128 w1024      1084 / 867   1059 / 618   1025 / 517
//             B1 H32/8 N8192  d128 w4096      1381 / 390   1366 / 257   1354 / 205
//             B4 H16/4 N4096  d64  causal      547 / 203    537 / 133    531 / 102
//             B4 H16/4 N4096  d64  w512        158 / 159    157 / 130    152 / 103
//             B2 H16   N4096  d128 w1024 fp32 1109 / 878   1075 / 561   1043 / 417
#pragma once
#include <initializer_list>
#include <type_traits>

#include "gfwa_internal.h"
#include "tile_stage.h"

namespace gfwa {

// Base-2 exponents below which a weight counts for nothing, with 1 for the roundings of scores and references.
constexpr float kErased = 127.f, kFaint = 49.f;
// Doublings by which rows of squared norm `far` outweigh rows of `near` (at least 0; NaN or infinite: no line but kErased holds).
__device__ __forceinline__ float outweighs(float far, float near) { return far <= near ? 0.f : 0.5f * (fast_log2(far) - fast_log2(near)); }
// Whether it can pay to read norms: `decay` over the `len` rows that see a block (that it sees).  Scores of unit-variance rows add about
// 15 to the 34 of kFaint (in units of the gate); `few` rows fewer have to be worth the reading: of one matrix of three in front of the backward,
// of two in a launch of their own in front of the forward (key_reach.hip).  (Two products compared, so that two kernels which ask the same
// always agree: there is nothing the compiler could fuse in one of them.)
constexpr float kTypicalReach = 49.f;
constexpr int kFewBackward = 128;
// The whole-tile kernels of bf16 at d = 128 run one workgroup a CU, whose look nothing overlaps: whole bands / shortened, us, B4 H16 N4096 w256, where
// mu = -1 (0.5) erases 130 (210) keys: 239 / 250 (237 / 234), at d = 64 117 / 115 (115 / 106).
__host__ __device__ constexpr int few_backward(int d) { return d == 128 ? 192 : kFewBackward; }
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
// room: what a score would have to exceed, in base-2 exponents, for a weight of 2^-kErased; heavier: doublings by which the values of the
// block outweigh others (fminf: kErased for NaN)
__device__ __forceinline__ bool is_erased(float n2, float reach2, float room, float heavier) {
    room += kErased - fminf(kFaint + heavier, kErased);
    return room > 0.f && n2 * reach2 < room * room;
}

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
// that a weight of a row is measured against, less kErased).  Values close by are those of entry 0.
__device__ __forceinline__ int first_needed_key(const KeyBlock& kb, int q0, int k_lo, int block, float reach2, float lowest, float cbase, int lane) {
    const int hi = q0 / block - 1, n = hi - k_lo / block + 1;  // (n <= 64, reach_of_forward sees to that)
    const float near_v2 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(kb.v2())));
    const bool kept = lane < n && !is_erased(kb.k2(), reach2, lowest - (kb.c - cbase) * kLog2e, outweighs(kb.v2(), near_v2));
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
    kReachEdge,      // .. lowest (c - c of the first row) + L,
    kReachG, kReachD,       // .. largest squared norm of dO and square of D,
    kReachOneK, kReachOneV,  // .. squared norms of its first key and value row: what such rows weigh here;
    kReachKeyNorm,   // and, for passes that cannot look at their keys by themselves (split kernels, fp32), the largest squared norm of its
    kReachKeyHigh,   // .. key rows, their highest gate
    kReachValue,     // .. and the largest squared norm of its value rows.
    kReachLast,      // From the whole-tile dK/dV kernel on, in the first block of its 128-key tiles: the last block of queries that needs a key.
    kReachValues
};
// Bands up to this long are not looked at: only gates of more than 0.25 (fp32 0.37) a key would erase enough of them, and the look costs 2 to 5 %
// (1 to 3 %) where it is in vain (whole step, us, whole bands / looked at: B2 H12/6 N2653 d64 w302 mu -2 66 / 69; fp32 B6 H13 N257 d128 mu -2
// 104 / 107, B5 H2 N7686 d128 w289 mu -1 493 / 437).
constexpr int shortest_reach(int d, size_t size) { return size == 2 ? few_backward(d) + 200 : kFewBackward + 132; }
// Row of dalpha from which on block i has its values: its first, or for a last block of too few rows the 17th of the one before.
__device__ __forceinline__ int reach_row(int i, int N) { return kReachRows * i + kReachValues <= N ? kReachRows * i : kReachRows * (i - 1) + 16; }

// dalpha, if the passes of a backward may leave rows out and may use it as scratch, else nullptr.
inline float* backward_reach(float* dalpha, const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* c, const float* L,
                             size_t size, int B, int H, int Hkv, int N, int d, int w, float scale) {
    const size_t rows = (size_t)B * H * N, gate = rows * sizeof(float), q = rows * d * size, kv = (size_t)B * Hkv * N * d * size;
    bool free = scale > 0.f && (w < N ? w : N) > shortest_reach(d, size);
    for (const void* m : {Q, O, dO}) free = free && !overlap(dalpha, gate, m, q);
    for (const void* m : {K, V}) free = free && !overlap(dalpha, gate, m, kv);
    for (const float* v : {c, L}) free = free && !overlap(dalpha, gate, v, gate);
    return free ? dalpha : nullptr;
}

// What the own rows of a tile are: (scale log2 e |row|)^2 of the largest, their edge relative to gate cbase in base-2 exponents (the lowest of
// queries, the highest of keys), and what rows weigh here.
struct OwnRows {
    float reach2, edge;
    float q2, g2, d2;  // (of a key tile: those of the queries at the diagonal)
    float k2, v2;      // (of a key tile: its own, 0 where the dQ pass looks by itself)
};
// Blocks i0 and i1 (the same, or next to each other) of queries.
__device__ __forceinline__ OwnRows own_queries(const float* at, const float* ch, int i0, int i1, int N, float cbase, float sl) {
    const float *r0 = at + reach_row(i0, N), *r1 = at + reach_row(i1, N);
    const int norm = max(norm_bits(r0[kReachNorm]), norm_bits(r1[kReachNorm]));
    const int edge = min(lowest_order((ch[64 * i0] - cbase) + r0[kReachEdge]), lowest_order((ch[64 * i1] - cbase) + r1[kReachEdge]));
    OwnRows own = {};
    own.k2 = fmaxf(r0[kReachOneK], r1[kReachOneK]);
    own.v2 = fmaxf(r0[kReachOneV], r1[kReachOneV]);
    own.reach2 = reach2_of(norm, sl);
    own.edge = from_order(edge) * kLog2e;
    return own;
}
// Blocks i0 and i1 of keys, and of queries at their diagonal.
__device__ __forceinline__ OwnRows own_keys(const float* at, int i0, int i1, int N, float cbase, float sl) {
    const float *r0 = at + reach_row(i0, N), *r1 = at + reach_row(i1, N);
    const int norm = max(norm_bits(r0[kReachKeyNorm]), norm_bits(r1[kReachKeyNorm]));
    const int edge = max(highest_order(r0[kReachKeyHigh] - cbase), highest_order(r1[kReachKeyHigh] - cbase));
    OwnRows own = {};
    own.reach2 = reach2_of(norm, sl);
    own.edge = from_order(edge) * kLog2e;
    own.q2 = fmaxf(r0[kReachNorm], r1[kReachNorm]);
    own.g2 = fmaxf(r0[kReachG], r1[kReachG]);
    own.d2 = fmaxf(r0[kReachD], r1[kReachD]);
    return own;
}
// What block i of queries has to say to a key tile.
struct QueryBlock {
    float norm, edge, g, d, one_k, one_v, c;
};
__device__ __forceinline__ QueryBlock query_block(const float* at, const float* ch, int i, int N) {
    const float* r = at + reach_row(i, N);
    return {r[kReachNorm], r[kReachEdge], r[kReachG], r[kReachD], r[kReachOneK], r[kReachOneV], ch[64 * i]};
}
__device__ __forceinline__ bool needs_keys(const QueryBlock& b, const OwnRows& own, float cbase) {
    // dO in dV, dS of dO and D times Q in dK; and in these queries' dQ dS of V times K
    const float here = fmaxf(outweighs(b.g, own.g2), outweighs(b.d, own.d2)) + outweighs(b.norm, own.q2);
    const float there = outweighs(own.v2, b.one_v) + outweighs(own.k2, b.one_k);
    return !is_erased(b.norm, own.reach2, ((b.c - cbase) + b.edge) * kLog2e - own.edge - kErased, fmaxf(here, there));
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
    float norm, high, value;
};
__device__ __forceinline__ KeyValues key_values(const float* at, int i, int N) {
    const float* r = at + reach_row(i, N);
    return {r[kReachKeyNorm], r[kReachKeyHigh], r[kReachValue]};
}
// First block of keys from i_lo on that is needed, i_max if none before it is.  first: block i_lo + lane, if there is one.
__device__ __forceinline__ int first_needed_block(const float* at, int i_lo, int i_max, int N, const OwnRows& own, float cbase, int lane, KeyValues first) {
    for (int base = i_lo; base < i_max; base += 64) {
        const int i = base + lane;
        if (base != i_lo) first = key_values(at, min(i, i_max), N);
        const float heavier = outweighs(first.norm, own.k2) + outweighs(first.value, own.v2);
        const bool kept = i < i_max && !is_erased(first.norm, own.reach2, own.edge - kErased - (first.high - cbase) * kLog2e, heavier);
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
    int norm, edge, g, d, one_k, one_v, key_norm, high, value;
};
__device__ __forceinline__ void write_block(float* row, const BlockValues& b, bool looked, bool keys) {
    row[kReachNorm] = looked ? __int_as_float(b.norm) : INFINITY;
    row[kReachEdge] = looked ? from_order(b.edge) : 0.f;
    row[kReachG] = looked ? __int_as_float(b.g) : 0.f;
    row[kReachD] = looked ? __int_as_float(b.d) : 0.f;
    row[kReachOneK] = looked ? __int_as_float(b.one_k) : 0.f;
    row[kReachOneV] = looked ? __int_as_float(b.one_v) : 0.f;
    if (!keys) return;
    row[kReachKeyNorm] = looked ? __int_as_float(b.key_norm) : INFINITY;
    row[kReachKeyHigh] = looked ? from_order(b.high) : 0.f;
    row[kReachValue] = looked ? __int_as_float(b.value) : 0.f;
}
// Over the workgroup, from all waves' lanes; at: of LDS.
template <bool KEYS>
__device__ __forceinline__ void gather_block(BlockValues* at, BlockValues b) {
    if (threadIdx.x == 0) *at = {0, 0x7fffffff, 0, 0, b.one_k, b.one_v, 0, (int)0x80000000, 0};
    b.norm = lanes_max(b.norm), b.edge = lanes_min(b.edge), b.g = lanes_max(b.g), b.d = lanes_max(b.d);
    if (KEYS) b.key_norm = lanes_max(b.key_norm), b.high = lanes_max(b.high), b.value = lanes_max(b.value);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&at->norm, b.norm);
        atomicMin(&at->edge, b.edge);
        atomicMax(&at->g, b.g);
        atomicMax(&at->d, b.d);
        if (KEYS) {
            atomicMax(&at->key_norm, b.key_norm);
            atomicMax(&at->high, b.high);
            atomicMax(&at->value, b.value);
        }
    }
    __syncthreads();
}

}  // namespace gfwa
