// GatedFWA decoding step on gfx950: one new query per (batch, head) against the cached keys and
// values of the last w positions (paper Sec. 1: O(wd) work per generated token with a KV cache; the
// arithmetic is row `pos` of the forward, Sec. 3.2 / Alg. 2).
//
// The step is bound by reading the window of the cache once (2 * w * d elements per key/value head),
// so the design is about memory traffic, not MFMA:
//   * rows of the cache are read with 16 lanes x 16 bytes (bf16, d = 128), four rows per wave
//     instruction, fully coalesced, every byte once;
//   * the G query heads that read the same key/value head are handled together (4, 2 or 1 per
//     workgroup), so the cache is read once per group, not once per head, as long as that leaves enough workgroups;
//   * the window is shared out over the 4 or 8 waves of a workgroup and, where that does not fill the chip, over
//     chunks of at least 256 keys, one workgroup each; the (reference exponent, sum, output) partials are merged across
//     the waves through LDS and, when the window has more than one chunk, across chunks by a second small kernel.
// With `alpha_t` given the kernel also advances the gate prefix, c[pos] = c[pos-1] + alpha_t, the one
// step of the scan a decoding step needs.
#include "gfwa_device.h"
#include "gfwa_internal.h"
#include <type_traits>

namespace gfwa {

constexpr int kDecChunk = 256;  // a chunk is a multiple of this many keys
constexpr float kDecNegBig = -1.0e30f;
constexpr size_t kDecOnceBytes = (size_t)24 << 20;

__device__ __forceinline__ void load8(const bf16_t* p, float (&x)[8]) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (float)v[e];
}
__device__ __forceinline__ void load8(const float* p, float (&x)[8]) {
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
}

// Partial record of one (query head, chunk): D output columns (unnormalised), then the reference
// exponent they are scaled by (log2 domain) and the sum.
__host__ __device__ constexpr int dec_record(int D) { return D + 2; }

// Eight consecutive cache elements as they arrive from memory, converted to fp32 only when used (so
// that the loads of the next step can be in flight, in few registers, while the current one is computed).
// ONCE: no other workgroup reads them, so bf16 loads are non-temporal.  A cache that holds nothing of the window yet is then read faster (us,
// three states in turn: B64 H32/8 N16384 d128 w1024 63 -> 57, H32/32 213 -> 174, B16 H32/8 w4096 57 -> 52, B4 H32/8 w1024 12.4 -> 12.4), one that
// the memory-side cache still holds in full more slowly (the first 52 -> 56): a program reads its other layers in between.  fp32 gains nothing
// (B16 H32/32 w1024 99 -> 101) and loads as before, and so do windows of less than 24 MiB in all, which the L2s may still hold (B26 H2 N1744
// d128 w992, 26 MB, 9.3 -> 9.0; B4 H8 N13281 d64 w1384, 11 MB, 9.0 -> 10.4).
template <typename T>
struct Raw8;
template <>
struct Raw8<bf16_t> {
    bf16x8 v;
    template <bool ONCE>
    __device__ __forceinline__ void load(const bf16_t* p) {
        const bf16x8* from = reinterpret_cast<const bf16x8*>(p);
        if constexpr (ONCE) v = __builtin_nontemporal_load(from);
        else v = *from;
    }
    __device__ __forceinline__ void get(float (&x)[8]) const {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = (float)v[e];
    }
};
template <>
struct Raw8<float> {
    float4 a, b;
    template <bool ONCE>
    __device__ __forceinline__ void load(const float* p) {
        a = reinterpret_cast<const float4*>(p)[0];
        b = reinterpret_cast<const float4*>(p)[1];
    }
    __device__ __forceinline__ void get(float (&x)[8]) const {
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    }
};

// Cross-lane moves on the VALU (DPP), no LDS involved, inside a row of 16 lanes.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// lane i receives the value of the N-th lane of its own aligned group of GT (1, 2 or 4) lanes
template <int GT, int N>
__device__ __forceinline__ float group_from(float x) {
    static_assert((GT == 4 || GT == 2 || GT == 1) && N < GT, "aligned groups of 1, 2 or 4 lanes");
    if (GT == 1) return x;
    constexpr int ctrl = GT == 4 ? (N | N << 2 | N << 4 | N << 6) : (N | N << 2 | (2 + N) << 4 | (2 + N) << 6);
    return dpp_mov<ctrl>(x);
}
// sum over the LPR (16 or 8) consecutive lanes that share a cache row, result in all of them
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
    static_assert(LPR == 16 || LPR == 8, "one or two cache rows per row of 16 lanes");
    if (LPR == 16) {  // rotations inside the row of 16: 0x120 + n is row_ror:n
        x += dpp_mov<0x128>(x);
        x += dpp_mov<0x124>(x);
        x += dpp_mov<0x122>(x);
        x += dpp_mov<0x121>(x);
    } else {  // lane ^ 1, lane ^ 2 inside the quads, lane ^ 4 as half-row mirror (i ^ 7) then i ^ 3
        x += dpp_mov<(1 | 0 << 2 | 3 << 4 | 2 << 6)>(x);
        x += dpp_mov<(2 | 3 << 2 | 0 << 4 | 1 << 6)>(x);
        x += dpp_mov<(3 | 2 << 2 | 1 << 4 | 0 << 6)>(dpp_mov<0x141>(x));
    }
    return x;
}

// Sum over the two halves (the four 16-lane rows) of a wave of one value per half (row): x[i] is returned summed in half
// (row) i alone.  Half the exchanges and additions of summing every value everywhere, and no trip through LDS.
__device__ __forceinline__ float half_sums(float x0, float x1) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float row_pair_sums(float x0, float x1) {  // x0 in even rows of 16 lanes, x1 in odd ones
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One workgroup of NW waves: GT query heads of one key/value head, one chunk of the window (a multiple of 256
// keys, 1 / NW of it per wave).  A step covers UN rows per lane group (4 UN or 8 UN rows per wave).
//   * every lane holds its 16-byte piece of the row and forms the partial dot products of all GT heads
//     on it; a sum over the lanes of the row (DPP adds on the VALU) leaves every lane with the GT scores;
//   * all exponentials of a wave are taken against one reference exponent per head, the score of the
//     wave's newest key (the gate bias only falls with distance).  fp32 has room for scores 2^60 above
//     it; if one ever exceeds that, the wave raises the reference and rescales (rare, wave-uniform).
//     So there is no running maximum and the output accumulators need one fused multiply-add per element;
//   * the gate prefix of a row is loaded once per head (lane j loads head j % GT) and passed round the
//     group of GT lanes by DPP;
//   * the loads of the next step are issued before the current step is computed.
template <typename T, int D, int GT, int NW, bool ONCE>
__global__ __launch_bounds__(64 * NW) void decode_partial_kernel(
    const T* __restrict__ q, const T* __restrict__ Kc, const T* __restrict__ Vc, float* __restrict__ c,
    const float* __restrict__ alpha_t, const int* __restrict__ pos, float* __restrict__ part,
    T* __restrict__ o, float* __restrict__ L, int H, int G, int Tlen, int w, float scale, int S, int chunk) {
    constexpr int LPR = D / 8;     // lanes per cache row
    constexpr int RPI = 64 / LPR;  // rows per wave instruction
    constexpr int UN = 4;          // rows per lane group and step
    constexpr int STEP_ROWS = RPI * UN;
    __shared__ __align__(16) float sm_acc[NW][GT][D];
    __shared__ float sm_m[NW][GT], sm_l[NW][GT];

    int idx = blockIdx.x;
    const int s = idx % S;
    idx /= S;
    const int gchunks = G / GT;
    const int gc = idx % gchunks;
    const int bkv = idx / gchunks;  // flat key/value head
    const int Hkv = H / G;
    const int b = bkv / Hkv;
    const int bh0 = b * H + (bkv % Hkv) * G + gc * GT;  // first of the GT query heads of this workgroup

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane / LPR, j = lane % LPR;
    const int g_own = j % GT;  // the head whose gate prefix this lane loads

    const int p = min(max(pos[b], 0), Tlen - 1);  // an out-of-range position is clamped, never followed
    const int lo = max(0, p - w + 1);
    const int k_begin = lo + s * chunk;
    const int k_end = min(p, k_begin + chunk - 1);

    // gate prefix at the query position; with alpha_t it is formed here (and stored at the end)
    float ct[GT];
#pragma unroll
    for (int g = 0; g < GT; ++g) {
        const float* crow = c + (size_t)(bh0 + g) * Tlen;
        ct[g] = alpha_t != nullptr ? (p > 0 ? crow[p - 1] : 0.f) + alpha_t[bh0 + g] : crow[p];
    }
    float ct_own = ct[0];
#pragma unroll
    for (int g = 1; g < GT; ++g) ct_own = g_own == g ? ct[g] : ct_own;
    const float* c_own = c + (size_t)(bh0 + g_own) * Tlen;

    float acc[GT][8], l[GT], mref[GT];
#pragma unroll
    for (int g = 0; g < GT; ++g) {
        l[g] = 0.f;
        mref[g] = kDecNegBig;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    }

    const int per_wave = chunk / NW;
    const int kw0 = k_begin + per_wave * wv;  // first key of this wave
    if (kw0 <= k_end) {                       // uniform over the wave
        const int kw_end = min(k_end, kw0 + per_wave - 1);
        const int nsteps = (kw_end - kw0) / STEP_ROWS + 1;
        // this lane's 8 columns of the GT queries, pre-multiplied by scale * log2(e)
        float qs[GT][8];
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            load8(q + (size_t)(bh0 + g) * D + 8 * j, qs[g]);
#pragma unroll
            for (int e = 0; e < 8; ++e) qs[g][e] *= scale * kLog2e;
        }
        const T* Kh = Kc + (size_t)bkv * Tlen * D + 8 * j;
        const T* Vh = Vc + (size_t)bkv * Tlen * D + 8 * j;

        // scores (log2 domain) of one row for the GT heads; cv_own: gate prefix of the row for head g_own
        auto scores = [&](const Raw8<T>& kr, float cv_own, float (&sc)[GT]) __attribute__((always_inline)) {
            float kx[8];
            kr.get(kx);
            const float bias_own = (cv_own - ct_own) * kLog2e;
#pragma unroll
            for (int g = 0; g < GT; ++g) {
                float dot = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) dot = fmaf(qs[g][e], kx[e], dot);
                sc[g] = row_sum<LPR>(dot);
            }
            sc[0] += group_from<GT, 0>(bias_own);
            if (GT >= 2) sc[GT >= 2 ? 1 : 0] += group_from<GT, (GT >= 2 ? 1 : 0)>(bias_own);
            if (GT == 4) {
                sc[GT == 4 ? 2 : 0] += group_from<GT, (GT == 4 ? 2 : 0)>(bias_own);
                sc[GT == 4 ? 3 : 0] += group_from<GT, (GT == 4 ? 3 : 0)>(bias_own);
            }
        };

        Raw8<T> kr[2][UN], vr[2][UN];
        float cvr[2][UN];
        auto issue = [&](int st, auto bufc) __attribute__((always_inline)) {
            constexpr int buf = decltype(bufc)::value;
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int kk = min(kw0 + st * STEP_ROWS + u * RPI + r, kw_end);  // past the range: its last row, masked
                kr[buf][u].template load<ONCE>(Kh + (size_t)kk * D);
                vr[buf][u].template load<ONCE>(Vh + (size_t)kk * D);
                cvr[buf][u] = (alpha_t != nullptr && kk == p) ? ct_own : c_own[kk];
            }
        };
        issue(0, std::integral_constant<int, 0>{});

        {  // reference exponents: the scores of the wave's newest key
            Raw8<T> k1;
            k1.template load<ONCE>(Kh + (size_t)kw_end * D);
            scores(k1, (alpha_t != nullptr && kw_end == p) ? ct_own : c_own[kw_end], mref);
#pragma unroll
            for (int g = 0; g < GT; ++g) mref[g] = fmaxf(mref[g], kDecNegBig);  // that key may be masked: a score of minus infinity
        }

        auto compute = [&](int st, auto bufc) __attribute__((always_inline)) {
            constexpr int buf = decltype(bufc)::value;
            float sc[UN][GT];
            float excess = -INFINITY;
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                scores(kr[buf][u], cvr[buf][u], sc[u]);
                const bool ok = kw0 + st * STEP_ROWS + u * RPI + r <= kw_end;
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    sc[u][g] = ok ? sc[u][g] : -INFINITY;
                    excess = fmaxf(excess, sc[u][g] - mref[g]);
                }
            }
            if (__any(excess > 60.f)) {  // a score far above the reference: raise it and rescale
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    float v = sc[0][g];
#pragma unroll
                    for (int u = 1; u < UN; ++u) v = fmaxf(v, sc[u][g]);
#pragma unroll
                    for (int off = LPR; off < 64; off <<= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
                    const float nref = fmaxf(mref[g], v);
                    const float f = fast_exp2(mref[g] - nref);
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[g][e] *= f;
                    l[g] *= f;
                    mref[g] = nref;
                }
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                float vx[8];
                vr[buf][u].get(vx);
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    const float pr = fast_exp2(sc[u][g] - mref[g]);
                    l[g] += pr;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[g][e] = fmaf(pr, vx[e], acc[g][e]);
                }
            }
        };
        for (int st = 0; st < nsteps; st += 2) {
            if (st + 1 < nsteps) issue(st + 1, std::integral_constant<int, 1>{});
            compute(st, std::integral_constant<int, 0>{});
            if (st + 1 < nsteps) {
                if (st + 2 < nsteps) issue(st + 2, std::integral_constant<int, 0>{});
                compute(st + 1, std::integral_constant<int, 1>{});
            }
        }
    }
    // One reference per head in the whole wave: plain sums over the lane groups (the lanes of a row all hold the same l).
    // With four heads head g ends in the g-th row of 16 lanes, with two in the g-th half, a single one in all lanes.
    float own[8], l_own;
    {
        auto across = [&](const float (&x)[GT]) __attribute__((always_inline)) -> float {
            if constexpr (GT == 4) return row_pair_sums(half_sums(x[0], x[2]), half_sums(x[1], x[3]));
            const float y = GT == 2 ? half_sums(x[0], x[GT - 1]) : half_sums(x[0], x[0]);
            return row_pair_sums(y, y);
        };
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float x[GT];
#pragma unroll
            for (int g = 0; g < GT; ++g) x[g] = acc[g][e];
            own[e] = across(x);
            if (LPR == 8) own[e] += dpp_mov<0x128>(own[e]);  // the two cache rows of a row of 16 lanes (row_ror:8)
        }
        l_own = across(l);
        if (LPR == 8) l_own += dpp_mov<0x128>(l_own);
    }
    // across the waves through LDS
    {
        const int g = GT == 4 ? lane >> 4 : GT == 2 ? lane >> 5 : 0;
        constexpr int kLanesPerHead = GT == 4 ? 16 : GT == 2 ? 32 : 64;
        if (lane % kLanesPerHead < LPR) {
            f32x4* to = reinterpret_cast<f32x4*>(&sm_acc[wv][g][8 * j]);
            to[0] = f32x4{own[0], own[1], own[2], own[3]};
            to[1] = f32x4{own[4], own[5], own[6], own[7]};
            if (j == 0) sm_l[wv][g] = l_own;
        }
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < GT; ++k) sm_m[wv][k] = mref[k];
        }
    }
    if (alpha_t != nullptr && s == 0 && tid < GT) c[(size_t)(bh0 + tid) * Tlen + p] = ct_own;  // thread g: head g
    __syncthreads();
    for (int x = tid; x < GT * D; x += 64 * NW) {
        const int g = x / D, col = x % D;
        float mm = sm_m[0][g];
#pragma unroll
        for (int k = 1; k < NW; ++k) mm = fmaxf(mm, sm_m[k][g]);
        float ll = 0.f, oo = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const float f = fast_exp2(sm_m[k][g] - mm);
            ll = fmaf(sm_l[k][g], f, ll);
            oo = fmaf(sm_acc[k][g][col], f, oo);
        }
        if (S == 1) {  // the whole window in one chunk: this is the result, no merge kernel follows
            o[(size_t)(bh0 + g) * D + col] = (T)(oo / ll);
            if (L != nullptr && col == 0) L[bh0 + g] = (mm + log2f(ll)) * kLn2;
        } else {
            float* rec = part + ((size_t)(bh0 + g) * S + s) * dec_record(D);
            rec[col] = oo;
            if (col == 0) {
                rec[D] = mm;
                rec[D + 1] = ll;
            }
        }
    }
}

// o = sum_s acc_s 2^(m_s - M) / sum_s l_s 2^(m_s - M),  L = (M + log2 of that sum) ln 2
template <typename T, int D>
__global__ __launch_bounds__(D) void decode_combine_kernel(const float* __restrict__ part, T* __restrict__ o,
                                                           float* __restrict__ L, int S) {
    const int bh = blockIdx.x, col = threadIdx.x;
    const float* rec = part + (size_t)bh * S * dec_record(D);
    float mm = kDecNegBig, ll = 0.f, oo = 0.f;
    constexpr int U = 8;  // records whose loads are in flight together
    for (int s0 = 0; s0 < S; s0 += U) {
        float m[U], l[U], a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float* rs = rec + (size_t)min(s0 + u, S - 1) * dec_record(D);
            m[u] = rs[D];
            l[u] = rs[D + 1];
            a[u] = rs[col];
        }
        float mn = mm;
#pragma unroll
        for (int u = 0; u < U; ++u) mn = s0 + u < S ? fmaxf(mn, m[u]) : mn;
        const float f0 = fast_exp2(mm - mn);
        ll *= f0;
        oo *= f0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float f = s0 + u < S ? fast_exp2(m[u] - mn) : 0.f;
            ll = fmaf(l[u], f, ll);
            oo = fmaf(a[u], f, oo);
        }
        mm = mn;
    }
    o[(size_t)bh * D + col] = (T)(oo / ll);
    if (L != nullptr && col == 0) L[bh] = (mm + log2f(ll)) * kLn2;
}

int decode_splits(int Tlen, int w) {
    const int span = w < Tlen ? w : Tlen;
    return (span + kDecChunk - 1) / kDecChunk;
}

size_t decode_workspace_bytes(int B, int H, int Tlen, int d, int w) {
    return (size_t)B * H * decode_splits(Tlen, w) * dec_record(d) * sizeof(float);
}

template <typename T, int D>
static hipError_t launch_decode(const T* q, const T* Kc, const T* Vc, float* c, const float* alpha_t,
                                const int* pos, T* o, float* L, float* part, int B, int H, int Hkv, int Tlen,
                                int w, float scale, hipStream_t s) {
    const int G = H / Hkv;
    // How a step is cut up, from a sweep over 12 shapes (1 to 256 sequences, groups of 1 to 4, windows 40 .. 4096):
    //   * the chip holds 8 waves per CU of the four-head kernel (198 registers), in fp32 half of that pays: one round of
    //     that many waves is the best size of a launch (B64 H32/8 w1024: 512 workgroups of 4 waves 50.6 us, 1024 61.6 us);
    //   * a step of a wave costs about as much per head as its loads do (fixed part about one head), so where even
    //     256-key chunks leave fewer waves than that, fewer heads per workgroup are faster although the cache is then read
    //     once per head (B1 H32/8 w1024: 8.4 us one head, 9.1 two, 11.9 four);
    //   * a second chunk brings the merging kernel with it, 2.8 us: worth it from about six steps of one head.
    constexpr bool kShort = sizeof(T) == 2;
    const int span = w < Tlen ? w : Tlen, round = (kShort ? 8 : 4) * device_cu_count(), max_splits = decode_splits(Tlen, w);
    int GT = G % 4 == 0 ? 4 : (G % 2 == 0 ? 2 : 1);
    while (GT > 1 && (long)B * Hkv * (G / GT) * 8 * max_splits < round) GT /= 2;
    const int items = B * Hkv * (G / GT);
    const int NW = kShort && items * 4 < round ? 8 : 4;
    int S = (round + items * NW - 1) / (items * NW);
    const int steps = (span + NW * (2048 / D) - 1) / (NW * (2048 / D));  // of a wave, with a single chunk
    if (steps * (1 + GT) <= 12) S = 1;
    if (S > max_splits) S = max_splits;
    const int chunk = ((span + S - 1) / S + kDecChunk - 1) / kDecChunk * kDecChunk;
    S = (span + chunk - 1) / chunk;
    const bool once = kShort && G == GT && (size_t)B * Hkv * span * D * 2 * sizeof(T) > kDecOnceBytes;
    {
        ProfScope prof(kKernDecode, s);
        auto launch = [&](auto gt, auto nw) {
            auto as = [&](auto once) {
                hipLaunchKernelGGL((decode_partial_kernel<T, D, decltype(gt)::value, decltype(nw)::value, decltype(once)::value>),
                                   dim3((unsigned)(items * S)), dim3(64 * decltype(nw)::value), 0, s, q, Kc, Vc, c, alpha_t, pos, part,
                                   o, L, H, G, Tlen, w, scale, S, chunk);
            };
            if (once) as(std::integral_constant<bool, kShort>{});
            else as(std::integral_constant<bool, false>{});
        };
        auto with_heads = [&](auto nw) {
            if (GT == 4) launch(std::integral_constant<int, 4>{}, nw);
            else if (GT == 2) launch(std::integral_constant<int, 2>{}, nw);
            else launch(std::integral_constant<int, 1>{}, nw);
        };
        if constexpr (kShort) {
            if (NW == 8) with_heads(std::integral_constant<int, 8>{});
            else with_heads(std::integral_constant<int, 4>{});
        } else {
            with_heads(std::integral_constant<int, 4>{});
        }
    }
    if (S > 1) {
        ProfScope prof(kKernDecodeCombine, s);
        hipLaunchKernelGGL((decode_combine_kernel<T, D>), dim3(B * H), dim3(D), 0, s, part, o, L, S);
    }
    return hipGetLastError();
}

// Scratch of the allocation-free entry point: one array per GPU, held from the moment the code object
// is loaded until the process ends.  The name `scratch` is only a host-side handle of the symbol; the
// address a kernel may use is asked for once per device and kept.
static __device__ __align__(256) float scratch[kDecodeStaticBytes / sizeof(float)];

hipError_t decode_static_scratch(float** ptr) {
    static float* per_device[64];  // nullptr: not asked for yet
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    float* p = __atomic_load_n(&per_device[dev], __ATOMIC_ACQUIRE);
    if (p == nullptr) {
        if (hipError_t e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch))) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        __atomic_store_n(&per_device[dev], p, __ATOMIC_RELEASE);
    }
    *ptr = p;
    return hipSuccess;
}

hipError_t decode(bool bf16, const void* q, const void* Kc, const void* Vc, float* c, const float* alpha_t,
                  const int* pos, void* o, float* L, float* part, int B, int H, int Hkv, int Tlen, int d, int w,
                  float scale, hipStream_t s) {
    if (bf16) {
        if (d == 128)
            return launch_decode<bf16_t, 128>((const bf16_t*)q, (const bf16_t*)Kc, (const bf16_t*)Vc, c, alpha_t, pos,
                                              (bf16_t*)o, L, part, B, H, Hkv, Tlen, w, scale, s);
        return launch_decode<bf16_t, 64>((const bf16_t*)q, (const bf16_t*)Kc, (const bf16_t*)Vc, c, alpha_t, pos,
                                         (bf16_t*)o, L, part, B, H, Hkv, Tlen, w, scale, s);
    }
    if (d == 128)
        return launch_decode<float, 128>((const float*)q, (const float*)Kc, (const float*)Vc, c, alpha_t, pos,
                                         (float*)o, L, part, B, H, Hkv, Tlen, w, scale, s);
    return launch_decode<float, 64>((const float*)q, (const float*)Kc, (const float*)Vc, c, alpha_t, pos, (float*)o,
                                    L, part, B, H, Hkv, Tlen, w, scale, s);
}

}  // namespace gfwa
