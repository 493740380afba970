// GatedFWA fused forward for bf16 storage on gfx950 (paper Alg. 2, re-designed for CDNA4), and the choice of the kernel
// that serves a problem.
//
// A workgroup of 4 waves owns 128 consecutive queries of one head, a wave 32 of them.  Key/value tiles of 64 (d = 64, or few
// workgroups) or 32 keys travel global -> LDS by direct loads (no staging registers, no LDS stores) into two ring slots each; only the
// tiles that intersect the band [q0-w+1, q0+127] are visited, from the diagonal backwards, one per step.  A wave computes
// only in the steps that hold blocks of its own band (in the others it just issues its share of the loads) and masks only
// where the band edge or the diagonal cuts.
//
// The products are formed transposed so that a lane owns one query:
//   S^T[key][query]  = g[key] + K_tile (A operand, from LDS)  x  Q^T (B operand, registers)
//   O^T[dd][query]  += V_tile^T (A operand, LDS transposing read)  x  P^T (B operand = the S^T
//                      accumulator registers converted to bf16 in place)
// so the row max / row sum of the online softmax are in-lane plus one exchange between the two
// halves of the wave, the rescale factor is a per-lane scalar, and P never leaves registers.
//
// Where the overlap comes from.  A 32 x 32 block is 8 MFMAs at d = 64 (256 cycles of the matrix pipe), 16 at d = 128 (512),
// and about 285 cycles of vector issue; at d = 64 the two together take at least 360 (measured, four waves on a SIMD
// issuing nothing else).  That is approached by many waves in different phases, not by a pipeline inside one wave: four
// (three) workgroups on a CU, 128 (168) registers, nothing carried from step to step but O, m and l.  A step is
//   d = 64    S(upper 32 keys)  ->  S(lower) beside exp(upper)  ->  O += V P(upper) beside exp(lower)  ->  O += V P(lower)
//   d = 128   S  ->  exp  ->  O += V P; with few workgroups on a CU the step of d = 64, two on a CU with 188 registers
// A step takes 420 cycles per block and SIMD at d = 64.  The kernel this one took over from, persistent, two (three) waves
// on a SIMD and three blocks in flight inside each, took 600: the branches for the mask and for the reference exponent cut
// its iterations into pieces shorter than an MFMA chain's latency.  Without effect here (1 % and less): tile loads earlier
// or later in the step, their wait moved behind the products, issue priorities around the products, a ring of more slots.
// A copy of the step for masked tiles costs more than the branch: the compiler moves the accumulators between the copies.
//
// Workgroups are not persistent.  They are dealt out longest band first, over all heads of an XCD at once, so that the
// launch ends with short ones: one head after another, the tail of the launch was a third of it.
// Forward alone, us, the persistent kernel one head after another / this one:
//   d = 64   B4 H16    N4096 w512   62.8 / 50.4     B4 H16 N4096 w2000  158 / 111     B8 H32/8 N1024 w4096  63.5 / 45.1
//            B4 H16/4  N4096 w512   62.3 / 48.3     B2 H16 N8000 w200   45.0 / 36.3   B1 H32   N16384 w1024  196 / 163
//   d = 128  B1 H32 N16384 w1024    315 / 294       B4 H16 N8192 w1024  309 / 283     B16 H16  N1000 w200   65.2 / 55.1
//            B1 H32/8 N8192 w4096   435 / 355       B2 H32 N2048 causal 101 / 73
//   and with two blocks a step
//            B1 H4  N16384 w4096    124 / 127       B1 H14 N7817  w1160  86 / 85      B1 H38  N1287 w1057 37.2 / 37.2
//
// The gate bias rides in the MFMA accumulator: S is initialised with g_i = (c_i - c_base) / scale
// straight from LDS before the K Q^T chain, so S = q.k + g_i and the probability is one fused
// multiply-add plus one exp2, sl = scale * log2(e).  The per-query term -(c_t - c_base) is
// constant along a row, cancels in the softmax, and is applied only to L.  c_base = c at the first
// query of the tile keeps the fp32 differences window-local.  The row sum is taken in fp32 over the
// unrounded probabilities with plain adds (the packed dot-product instructions run on the matrix pipe
// and would queue behind the MFMAs).
//
// Keys that the gate has erased for a whole tile are left out at the far end of its band (band_reach.h); the step knows nothing of it.
//
// Deferred running max.  exp2 is taken against the reference exponent m left by earlier blocks
// without first looking for the block's own maximum; fp32 and bf16 share their exponent range, so a
// probability may grow to 2^60 with no loss of precision.  Only when a lane's block sum exceeds that
// (always on a query block's first key block, where m is still "minus infinity") does the wave take the
// slow path: find the true maximum, raise m, rescale O and l, and redo the exponentials.  Blocks are
// visited from the diagonal backwards, where the gate bias is largest, so this is rare.
#include <stddef.h>

#include "band_reach.h"
#include "gfwa_device.h"
#include "gfwa_internal.h"
#include "split_band.h"

namespace gfwa {

constexpr int kFwdWaves = 4;
template <int D>
constexpr int kFwdBlocks = D == 64 ? 2 : 1;  // blocks of 32 keys in a step where nothing else is said
template <int D, int NB>
struct FwdSmem {
    static constexpr int kKeys = 32 * NB, kTileBytes = kKeys * D * 2;
    alignas(256) char k[2][kTileBytes];
    alignas(256) char v[2][kTileBytes];
    alignas(16) float g[2][kKeys];  // (c - c_base) / scale of the tile's keys
    int needed[kFwdWaves];           // over_waves
};

// Longest bands (the end of the sequence) first.  Heads that do not divide by the XCDs go in contiguous ranges while bands are
// short against the sequence (B1 H12 N8192 w1024 37.6 us tile after tile, 35.5 so); with longer ones a range holds long or short
// bands only, and the XCDs finish apart.  d = 64, over 200 shapes: from 0.4 N on 1.0 to 1.5 times as fast tile after tile (B2 H9
// N3795 w2727 70.0 -> 46.3 us, H30 N3284 w1803 56.0 -> 49.4; B4 H113 N162 w146 would be 11.1 -> 12.7, hence 256).  At d = 128
// the keys of all heads at once outgrow an XCD's L2 (tile after tile B2 H9 N5458 w2294 114 -> 134 us, B3 H22/11 N1219 w1138 42.4
// -> 45.3), so only causal ones, nearly causal ones with two blocks a step, and few tiles, up to 2.5 a CU, with bands of 0.3 N
// (H36/9 N2155 w1379 63.9 -> 48.8, B3 H12/3 N1845 w920 46.7 -> 37.3) or where a few tiles, not the shortest, begin another round
// (H11 N3193 w492, 275 tiles on 256 CUs, 29.6 -> 21.7, B2 H3 N5525 w364 25.1 -> 18.1; w63 13.0 -> 14.3, as other short bands).
template <int D, int NB>
__host__ __device__ __forceinline__ bool fwd_by_length(int heads, long tiles, int N, int w) {
    if (heads % 8 == 0 || w >= N) return true;
    if (D == 64) return N > 256 && 5L * w >= 2L * N;
    if (NB == 2 && N >= 1000 && 4L * w >= 3L * N) return true;
    return N > 256 && tiles > 256 && tiles <= 640 && (10L * w >= 3L * N || (w >= 192 && tiles % 256 <= 64));
}

template <int D, int NB>
__device__ __forceinline__ void fwd_tile(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const float* __restrict__ c, bf16_t* __restrict__ O, float* __restrict__ L, int N, int w, float scale_log2,
    int num_qtiles, int total, int H, int G, KeyReach reach) {
    constexpr int KC = D / 16, DB = D / 32, NV = 2 * DB;
    using Smem = FwdSmem<D, NB>;
    constexpr int kKeys = Smem::kKeys, kRowBytes = D * 2, kTileBytes = Smem::kTileBytes;
    constexpr int kChunks = kRowBytes / 16, kPieceRows = 1024 / kRowBytes, kPieces = kKeys / kFwdWaves / kPieceRows;  // per wave and matrix
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<Smem*>(smem_raw);

    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, lq = lane & 31;
    const float sl = scale_log2, inv_scale = kLog2e / scale_log2;
    const int heads = total / num_qtiles;
    int bh, qt;
    tile_of_block((int)blockIdx.x, heads, num_qtiles, fwd_by_length<D, NB>(heads, total, N, w), bh, qt);
    const int q0 = (num_qtiles - 1 - qt) * 128;
    const size_t head_off = (size_t)bh * N * D, kv_off = (size_t)kv_head_of(bh, H, G) * N * D;
    const char* Kh = reinterpret_cast<const char*>(K + kv_off);
    const char* Vh = reinterpret_cast<const char*>(V + kv_off);
    const float* ch = c + (size_t)bh * N;
    const int k_lo = max(0, q0 - w + 1), j_hi = (min(N, q0 + 128) - 1) / kKeys;
    int ntiles = j_hi - k_lo / kKeys + 1;
    const int qw0 = q0 + 32 * wv;
    int T_first = ntiles, T_end = ntiles;  // the steps this wave computes in
    if (qw0 < N) {
        T_first = j_hi - min(qw0 + 31, N - 1) / kKeys;
        T_end = j_hi - max(0, qw0 - w + 1) / kKeys + 1;
    }

    // Loads, 1 KB a piece: wave wv fills kPieces of a tile.  Only the first tile (the last of the sequence it may be) can end
    // behind the sequence, its rows past N read row N-1; the tiles behind it, and tile 0, which stands in for those past the
    // band's end, lie inside (N >= kKeys, which fwd_split_shape sees to).
    const int ld_row = lane / kChunks;
    unsigned ld_off[kPieces];  // the swizzle of a piece is that of rows 0 .. with its number in the low chunk bits
#pragma unroll
    for (int g = 0; g < kPieces; ++g)
        ld_off[g] = (unsigned)tile_off<D>(ld_row, lane % kChunks ^ ((kPieces * wv + g) & (D == 128 ? 3 : 1)));
    auto piece = [&](const char* M, char* tile, int j, int g) __attribute__((always_inline)) {
        const int at = (kPieces * wv + g) * 1024;
        dma16(M + (size_t)j * kTileBytes + at, ld_off[g], tile + at);
    };
#pragma unroll
    for (int g = 0; g < kPieces; ++g) {
        const int r = kPieceRows * (kPieces * wv + g);
        const unsigned o = (unsigned)min(j_hi * kKeys + r + ld_row, N - 1) * (unsigned)kRowBytes + (ld_off[g] - (unsigned)(ld_row * kRowBytes));
        dma16(Kh, o, sm.k[0] + r * kRowBytes);
        dma16(Vh, o, sm.v[0] + r * kRowBytes);
    }
    const int lk = lane % kKeys;
    float c_next = ch[min(j_hi * kKeys + lk, N - 1)];
    const float cbase = ch[q0];
    const int t = qw0 + lq;
    float cq, m = kNegBig, l = 0.f;
    bf16x8 qf[KC];
    {
        const int tc = min(t, N - 1);
        cq = ch[tc] - cbase;
        const bf16_t* qp = Q + head_off + (size_t)tc * D + 8 * h;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) qf[kc] = *reinterpret_cast<const bf16x8*>(qp + 16 * kc);
    }
    if (reach.block != 0 && reach_pays(cbase - ch[k_lo], q0 - k_lo, reach.few)) {  // the keys that the gate has erased for all 128 queries stay out
        const int first = forward_reach<D, kFwdWaves>(qf, K + kv_off + (size_t)min(t, N - 1) * D + 8 * h,
                                                      key_block<D>(O + head_off + (size_t)q0 * D, min(128, N - q0), lane), cq, q0, k_lo, reach.block,
                                                      cbase, sl, sm.needed, wv, lane);
        ntiles = j_hi - first / kKeys + 1;
        T_first = min(T_first, ntiles);
        T_end = min(T_end, ntiles);
    }
    unsigned ka, va, ga;  // LDS addresses of the lane's first fragments in the current slot
    {
        const unsigned base = (unsigned)(uintptr_t)smem_raw;  // 0: the kernel has no other LDS, so a slot is one address bit
        ka = base + offsetof(Smem, k) + row_frag_off<D>(lane);
        va = base + offsetof(Smem, v) + col_frag_off<D>(lane);
        ga = base + offsetof(Smem, g) + 16 * h;
    }
    static_assert(offsetof(Smem, k) % (2 * kTileBytes) == 0 && offsetof(Smem, v) % (2 * kTileBytes) == 0 &&
                      offsetof(Smem, g) % (8 * kKeys) == 0, "the two slots of a ring differ in one address bit");
    auto flip = [&]() __attribute__((always_inline)) {  // to the other ring slot
        ka ^= kTileBytes;
        va ^= kTileBytes;
        ga ^= kKeys * 4;
    };
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    constexpr float kBig = 1.152921504606846976e18f;  // 2^60

    auto expo_pair = [&](const f32x16& sb, u32x4 (&pb)[2], int cc, float nm, float& pa, float& pc) __attribute__((always_inline)) {
        const f32x2 pr = {fast_exp2(fmaf(sb[2 * cc], sl, nm)), fast_exp2(fmaf(sb[2 * cc + 1], sl, nm))};
        pa += pr[0];
        pc += pr[1];
        pb[cc >> 2][cc & 3] = __builtin_bit_cast(unsigned, __builtin_convertvector(pr, bf16x2));
    };
    // this wave's share of step T+1 has landed (and, written by every wave alike, its gate)
    auto end_step = [&](int T) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        sm.g[(T + 1) & 1][lk] = (c_next - cbase) * inv_scale;
        wg_barrier();
    };
    auto next_gate = [&](int T) __attribute__((always_inline)) { c_next = ch[max(j_hi - T - 1, 0) * kKeys + lk]; };
    end_step(-1);
    GFWA_PIN(cq);  // no load of these is pending when the loop starts: the compiler would wait for it there, and for every tile behind it
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) GFWA_PIN(qf[kc]);
    auto issue = [&](int T) __attribute__((always_inline)) {  // the loads of step T, all of this wave's share
        const int j = max(j_hi - T, 0), nb = T & 1;
#pragma unroll
        for (int g = 0; g < kPieces; ++g) {
            piece(Kh, sm.k[nb], j, g);
            piece(Vh, sm.v[nb], j, g);
        }
    };
    auto idle_step = [&](int T) __attribute__((always_inline)) {
        next_gate(T);
        issue(T + 1);
        flip();
        end_step(T);
    };
    // slow path: the block's true maximum, common to the two halves of the wave, becomes the reference
    auto raise = [&](const f32x16& sc, u32x4 (&p)[2]) __attribute__((always_inline)) -> float {
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sc[v]);
        const float mnew = fmaxf(m, xhalf_max(mx)), a = fast_exp2((m - mnew) * sl);
        m = mnew;
        l *= a;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[db][v] *= a;
        float pa = 0.f, pc = 0.f;
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) expo_pair(sc, p, cc, -mnew * sl, pa, pc);
        return pa + pc;
    };
    auto step = [&](int T) __attribute__((always_inline)) {
        const int kt0 = (j_hi - T) * kKeys;
        next_gate(T);
        f32x16 s[NB];
        u32x4 p[NB][2];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const f32x4 x = *(__attribute__((address_space(3))) const f32x4*)(uintptr_t)(ga + 32 * b * 4 + 32 * r);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[b][4 * r + e] = x[e];
            }
        // the band mask, on the initial value: a masked score stays minus infinity and its probability is exactly zero
        if (__builtin_expect(!(kt0 + kKeys - 1 <= qw0 && kt0 > qw0 + 31 - w), 0)) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = kt0 + 32 * b + acc_row(v, h);
                    s[b][v] = (i <= t && i > t - w) ? s[b][v] : -INFINITY;
                }
        }
        float pa = 0.f, pc = 0.f;
        auto scores = [&](int b, bool beside) __attribute__((always_inline)) {  // S of block b, beside the exponentials of block b + 1
            bf16x8 kf[KC];
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) kf[kc] = row_frag<D>(ka, 32 * b, kc);
            if (D == 128) __builtin_amdgcn_sched_barrier(0);  // all reads ahead of the products (2 %)
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                s[b] = mfma32(kf[kc], qf[kc], s[b]);
                if (beside)
#pragma unroll
                    for (int cc = 8 * kc / KC; cc < 8 * (kc + 1) / KC; ++cc) expo_pair(s[NB - 1], p[NB - 1], cc, -m * sl, pa, pc);
            }
        };
        auto settle = [&](int b) __attribute__((always_inline)) {  // the sums of block b: reference exponent, l
            float sum = pa + pc;
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(sum <= kBig)) != 0, 0)) sum = raise(s[b], p[b]);
            l += sum;
            pa = pc = 0.f;
        };
        auto output = [&](int b, bool beside) __attribute__((always_inline)) {  // O += V^T P of block b, beside the exponentials of block b - 1
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                o[i % DB] = mfma32(col_frag<D>(va, 32 * b + 16 * (i / DB), i % DB), __builtin_bit_cast(bf16x8, p[b][i / DB]), o[i % DB]);
                if (beside)
#pragma unroll
                    for (int cc = 8 * i / NV; cc < 8 * (i + 1) / NV; ++cc) expo_pair(s[0], p[0], cc, -m * sl, pa, pc);
            }
        };
        if constexpr (NB == 2) {
            scores(1, false);
            scores(0, true);
            issue(T + 1);
            settle(1);
            output(1, true);
        } else {
            scores(0, false);
            issue(T + 1);
#pragma unroll
            for (int cc = 0; cc < 8; ++cc) expo_pair(s[0], p[0], cc, -m * sl, pa, pc);
        }
        settle(0);
        output(0, false);
        flip();
        end_step(T);
    };
    int T = 0;
    for (; T < T_first; ++T) idle_step(T);
    for (; T < T_end; ++T) step(T);
    for (; T < ntiles; ++T) idle_step(T);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    {
        const float lt = xhalf_sum(l);
        if (t < N && h == 0) L[(size_t)bh * N + t] = (m * sl + fast_log2(lt)) * kLn2 - cq;
        store_acc_rows<DB>(o, 1.0f / lt, smem_raw + 4096 * wv, O + head_off + (size_t)qw0 * D, N - qw0, lane);
    }
}

template <int D>
__global__ __launch_bounds__(64 * kFwdWaves, D == 64 ? 4 : 3) void fwd_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const float* __restrict__ c, bf16_t* __restrict__ O, float* __restrict__ L, int N, int w, float scale_log2,
    int num_qtiles, int total, int H, int G, KeyReach reach) {
    fwd_tile<D, kFwdBlocks<D>>(Q, K, V, c, O, L, N, w, scale_log2, num_qtiles, total, H, G, reach);
}
// d = 128 with the step of d = 64, for launches that put few workgroups on a CU (fwd_two_blocks has the line and figures): with two
// waves on a SIMD the exponentials of a block have to run beside the products of the same wave's other block.
__global__ __launch_bounds__(64 * kFwdWaves, 2) void fwd_two_blocks_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const float* __restrict__ c, bf16_t* __restrict__ O, float* __restrict__ L, int N, int w, float scale_log2,
    int num_qtiles, int total, int H, int G, KeyReach reach) {
    fwd_tile<128, 2>(Q, K, V, c, O, L, N, w, scale_log2, num_qtiles, total, H, G, reach);
}

// What all 128-query tiles of a problem cost and what the longest does, counted in 64-key tiles plus two for each query tile's start
// and end, whatever the kernel's own step is: the lines below were measured against this count.
static double query_tile_steps(int BH, int N, int w, long& longest) {
    const long nq = (N + 127) / 128;
    const long band = w < N ? w : N, full = (band + 126) / 64 + 2;   // key tiles of a tile whose whole band exists
    const long ramp = nq < (full - 1) / 2 ? nq : (full - 1) / 2;      // tiles whose band the sequence's start cuts off
    longest = (2 * nq < full ? 2 * nq : full) + 2;
    return (double)BH * (double)(ramp * (ramp + 1) + 2 * ramp + (nq - ramp) * longest);
}
// The share of `slots` resident workgroups' time that holds work when the tiles are taken in rounds:
// (steps of all tiles) / (slots x rounds x steps of the longest tile).  (The dQ pass asks too.)
double query_tile_fill(int BH, int N, int w, long slots) {
    long longest;
    const double steps = query_tile_steps(BH, N, w, longest);
    const long nq = (N + 127) / 128;
    return steps / ((double)slots * (double)((BH * nq + slots - 1) / slots) * (double)longest);
}

// Whether the d = 128 forward takes steps of two blocks, two workgroups on a CU, instead of one and three.  Lines from 712 shapes
// (N 64 .. 20000, 0.3 .. 31 tiles a CU); two blocks / one, us:
//   all tiles on the CUs at once, bands not short       H4 N16384 w4096 127 / 135, H7 N8192 w3000 89 / 94 (H73 N861 w213 19.9 / 19.1;
//                                                       long sequences from 64 on: H2 N16382 w89 11.6 / 11.9, split 13.6)
//   two nearly full rounds of two, not one of three     H14 N7817 w1160 85 / 94, H7 N16106 w907 73 / 82 (H10 N7269 w557, at 2.2 tiles
//   and a rest, bands equal and not short               a CU, 48 / 39; H32 N4096 causal 146 / 138)
//   long bands that are mostly equal, from three a CU   H8 N16384 w4096 235 / 252, H9 N18120 w2021 178 / 182
//   nearly causal, heads that do not divide by the XCDs, B3 H6 N11097 574 / 624, H12 N11676 400 / 428, H36 N4466 177 / 203,
//   not many, so that every XCD streams the keys of all  H28 N6200 261 / 300 (B6 H30/15 N1407 125 / 117, H108 N801 36 / 34)
//   from 128 on where tiles go by length, N > 192        H168 N226 11.2 / 12.0, H120 N387 w200 14.8 / 15.2
// Elsewhere three waves on a SIMD are the better (B4 H16 N8192 w1024 302 / 283, B1 H32 N16384 w1024 318 / 297, B1 H124/31 N2246 w27
// 51 / 42).
// (No band here is shorter than 64, so that no sequence is shorter than a 64-key tile.)
static bool fwd_two_blocks(int BH, int N, int w) {
    const long total = (long)BH * ((N + 127) / 128), cus = device_cu_count(), band = w < N ? w : N;
    const bool by_length = fwd_by_length<128, 2>(BH, total, N, w);
    if (total <= 2 * cus) return band >= (total <= cus ? (N >= 4096 ? 64 : 128) : by_length && N > 192 ? 128 : 256);
    if (BH % 8 != 0 && BH <= 64 && 4L * w >= 3L * N && N >= 1000 && total <= 8 * cus) return true;
    long longest;
    const double even = query_tile_steps(BH, N, w, longest) / ((double)total * (double)longest);
    if (even < 0.75) return false;
    return (band >= 2048 && total > 3 * cus) || (band >= 250 && (even >= 0.9 ? 3 * total >= 10 * cus : 2 * total >= 7 * cus) && total <= 4 * cus);
}

template <int D>
static hipError_t launch_fwd(const void* Q, const void* K, const void* V, const float* c, void* O,
                             float* L, int B, int H, int Hkv, int N, int w, float scale, hipStream_t s) {
    const int nq = (N + 127) / 128, total = B * H * nq, cus = device_cu_count();
    auto kernel = fwd_bf16_kernel<D>;
    // Bands too short for two blocks a step: two workgroups on a CU by asking for more LDS, where two rounds of that are nearly
    // full and three on a CU leave a second round of less than one a CU (H25 N4803 w106 33.9 -> 32.9 us, H27 N4611 w58 30.3 -> 29.2).
    const bool two_rounds = D == 128 && 2 * total >= 7 * cus && total <= 4 * cus && 9L * w <= 4L * N;
    size_t lds = two_rounds ? (size_t)56 << 10 : sizeof(FwdSmem<D, kFwdBlocks<D>>);
    static_assert(sizeof(FwdSmem<D, kFwdBlocks<D>>) <= (56 << 10), "two workgroups of 56 KB fit a CU, three do not");
    if constexpr (D == 128) {
        if (fwd_two_blocks(B * H, N, w)) {
            kernel = fwd_two_blocks_bf16_kernel;
            lds = sizeof(FwdSmem<D, 2>);
            static DeviceOnce lds_allowed;
            if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, lds_allowed)) return e;
        }
    }
    ProfScope prof(kKernForward, s);
    KeyReach reach;
    if (hipError_t e = key_reach(reach, 128, true, Q, K, V, c, O, B, H, Hkv, N, D, w, scale, s)) return e;
    hipLaunchKernelGGL(kernel, dim3(total), dim3(64 * kFwdWaves), lds, s, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, c,
                       (bf16_t*)O, L, N, w, scale * kLog2e, nq, total, H, H / Hkv, reach);
    return hipGetLastError();
}

// Which kernel serves a problem.  The one of this file wins once a CU has so many times the steps of the longest tile to
// do (`ratio`), the split one below.
// d = 64, 1.3: over 1182 shapes the best split shape is 1.0 to 1.8 times as fast below (a mean of 1.1 at 1.2), and above between 1.3
// times as slow and equal, but where a CU has one tile or two: up to two a CU for heads that divide by the XCDs (H16/4 N3367 w1048, 1.7 a
// CU: 27.6 against 24.6 us split; B8 H3 N3313 w335 1.14 of the time, from 2.0 on 0.95 to 1.0), one and a half for others (B4 H13 N939
// w311 14.9, 12.9; at 1.6 to 2 between 0.77 and 1.13, 0.94 on average).
// d = 128, over 1766 shapes: 1.0, or 0.85 where every tile has a CU to itself or, with heads that divide by the XCDs, the band is longer
// than 1024 (B5 H4 N1921 w1282, that do not: 43.3 against 30.2 split), 0.9 for tiles by length up to two a CU (B7 H13 N437 causal 15.9
// against 20.6 split, H11 N3193 w492 21.7, 29.6; B4 H7 N1179 w381, in ranges, 20.7, 16.8) (H3 N10679 w361, at
// 0.97: 23.0 against 16.4 us split, H2 N15792 w1194, 0.93: 50.9 against 29.9; with several short bands on few of the CUs, B2 H6 N2776
// w392, 0.95, 18.7 against 21.7).  Bands that 128 queries share out well 1.05 (B2 H4/2 N5746 w1976, 1.17: 65 against 51; B2 H14
// N2021 w1786, 1.0: 44 against 55), above 2048 1.95 (H20/5 N5003 w4000, 1.91: 139 against 153; H32 N4096 causal, 2.12: 145 against
// 130), or less where the tiles fill two places on every CU: the split kernel, one on a CU, takes whole rounds (H6 N7814 w3225,
// filled to 0.58: 99 against 91; H4 N11226 w6064, 0.50: 116 against 156).
// Sequences shorter than a step's tile are the split kernel's, and there 64 queries are the better than 32 (d = 64, 512 x 4
// heads of 50: 13.7, 28.0 us).
// Inside the split kernel: one 32-query block per workgroup while that gives few workgroups, at d = 128, whose tiles are single-buffered, up
// to two and a half a CU for short bands and one and a half for long ones, which four waves share out better than 64 or 128 queries do
// (us, 32 / what 64 or 128 queries take: H1 N2100 w1300 15.0 / 20.7, w1800 18.5 / 25.9 and 32.6, H1 N8000 w1300 17.3 / 21.7, H4 N3000 w1800
// 22.9 / 26.6 and 33.6, causal 33.2 / 39.1 and 46.3; H3 N4096 w1300, at one and a half, 26.7 / 23.9); above, of even heads, 64 before 128 up to
// two and a quarter (H8 N2100 w1800 27.3 / 33.7, H2 N8000 w4096 53.1 / 63.6; H3 N6000 w1800 38.9 / 36.8, H6 N4096 w1800 39.9 / 36.8).  At
// d = 64 nearly causal bands from 1500 on take 32 up to three a CU (H8 N3000 22.6 / 30.7, H12 N2100 18.5 / 21.4, H4 N6000 w4096 36.8 / 43.9).
// 128 queries where the band is long enough to share out: at d = 64 from 2560 on
// (H15 N4000 causal: 48.5 against 71.7 us with 64; H12 N4000 w2000 38.6 against 31.4), and from 1500 on, near one tile a CU and with
// uneven bands, for heads that are no multiple of four, above all odd ones: consecutive workgroups are consecutive heads, so that every XCD
// reads the keys of all of them, half as often with 128 queries (B3 H9 N1855 causal 27.2 against 33.4, B7 H3 N2175 27.1, 36.3, H11 N3968
// w2459 35.4, 46.6; B2 H16/4 N1806 30.0, 25.6; B2 H18/9 N1517 24.8, 21.9; H6/3 N7231 w2373 52.4, 40.7; H7 N6799 w1618 45.3, 37.2).
// Bands of 1024 to 1500 in sequences of three and more of them go whole from two and three quarters a CU on (H6 N6000 w1300 37 / 56 split, H3 N8000
// 30 / 40; H16 N2100 30 / 27, H8 N4096 30 / 31).
static FwdSplit fwd_split_shape(int BH, int N, int d, int w) {
    const long cus = device_cu_count(), band = w < N ? w : N;
    long longest;
    const double ratio = query_tile_steps(BH, N, w, longest) / ((double)cus * (double)longest);
    const long tiles = (long)BH * ((N + 127) / 128);
    bool filled = ratio >= (d == 64 ? 1.3 : band > 2048 ? 1.95 : band > 1500 ? 1.05 : band > 1024 && BH % 8 == 0 ? 0.85 : 1.0);
    if (d == 64) filled &= 2 * tiles > (BH % 8 == 0 ? 4 : 3) * cus;
    if (d == 128 && band > 1500) filled |= query_tile_fill(BH, N, w, 2 * cus) >= 0.57;
    if (d == 128 && band <= 1024 && band >= (N >= 4096 ? 64 : 128)) filled |= ratio >= 0.85 && tiles <= cus;
    if (d == 128 && band <= 1024 && band >= 128 && N > 192 && fwd_by_length<128, 2>(BH, tiles, N, w)) filled |= ratio >= 0.9 && tiles <= 2 * cus;
    if (N >= 32 * (d == 64 ? kFwdBlocks<64> : kFwdBlocks<128>) && filled) return kFwdSplitNone;
    const long blocks = (long)BH * ((N + 31) / 32);
    if (blocks <= 5 * cus / 2 && (d == 64 || band <= 1024)) return kFwdSplitNarrow;
    if (d == 128 && (band > 1500 ? 5 * blocks <= 8 * cus : 2 * blocks < 3 * cus)) return kFwdSplitNarrow;
    if (d == 64 && band >= 1500 && 4 * band >= 3L * N && 8 * blocks <= 25 * cus) return kFwdSplitNarrow;
    if (d == 128 && BH % 2 == 0 && 4 * blocks <= 9 * cus) return kFwdSplitMid;
    if (d == 128 && band > 1024 && band <= 1500 && N >= 3 * band && 4 * blocks >= 11 * cus) return kFwdSplitNone;
    const bool uneven = BH % 2 != 0 ? 5L * w >= 2L * N : BH % 4 != 0 && 4L * w >= 3L * N;
    const bool wide = d == 128 || (uneven && ratio >= 0.6 && ratio <= 1.25);
    return band > (wide ? 1500 : 2560) ? kFwdSplitWide : kFwdSplitMid;
}

hipError_t forward_bf16(const void* Q, const void* K, const void* V, const float* c, void* O, float* L,
                        int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s) {
    // A grid of 2^32 work items is refused; the densest here has 256 for 64 queries.  Half of the key/value heads at a time
    // then, or of the query heads of the only one.
    if ((long)B * H * ((N + 63) / 64) >= 1L << 24) {
        const int kv = B * Hkv, G = H / Hkv, kv0 = kv > 1 ? kv / 2 : 1, g0 = kv > 1 ? G : G / 2;
        const size_t rows = (size_t)N * kv0 * g0, keys = kv > 1 ? (size_t)N * kv0 : 0;
        auto from = [&](const void* p, size_t row) { return (const char*)p + row * d * sizeof(bf16_t); };
        if (hipError_t e = forward_bf16(Q, K, V, c, O, L, kv0, g0, 1, N, d, w, scale, s)) return e;
        return forward_bf16(from(Q, rows), from(K, keys), from(V, keys), c + rows, (char*)O + rows * d * sizeof(bf16_t), L + rows,
                            kv > 1 ? kv - kv0 : 1, kv > 1 ? G : G - g0, 1, N, d, w, scale, s);
    }
    if (const FwdSplit shape = fwd_split_shape(B * H, N, d, w))
        return forward_split_bf16(shape, Q, K, V, c, O, L, B, H, Hkv, N, d, w, scale, s);
    if (d == 64) return launch_fwd<64>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    return launch_fwd<128>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
}

}  // namespace gfwa
