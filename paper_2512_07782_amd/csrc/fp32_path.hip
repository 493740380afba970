// fp32 storage path of GatedFWA on gfx950: forward (paper Alg. 2) and backward (Alg. 3) to fp32 accuracy, for problems that
// need it; the bf16 MFMA kernels are the throughput path.
// Two sets of kernels.  The matrix-core set (bf16 MFMAs on operands split into three pieces, the structure of the bf16
// kernels: a lane owns a query or a key, the second product takes the first one's accumulator registers as its operand)
// serves everything but tiny problems.  The one-wave-per-row set (plain FMA) has a launch's latency and serves those; forward_f32 / backward_f32 choose (f32_use_mfma).
#include <math.h>

#include <type_traits>

#include "band_reach.h"
#include "gfwa_device.h"
#include "gfwa_internal.h"
#include "split_band.h"

namespace gfwa {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// ==========================================================================================
// One-wave-per-row kernels: a wave owns one query (key) and takes the other side's rows 4 or 16 load instructions at a time,
// D / 4 lanes x 16 bytes per row.  Every lane forms its part of the dot products on the four columns it holds, a sum over the
// row's lanes by lane moves gives all of them the score, and the same registers then feed the weighted sum of those
// columns: no transposition, nothing through LDS but per-row values.  Latency bounds them, so all loads of a step go out before
// anything is waited for.  (Lanes that split the keys for the scores, then the columns, with the rows fetched one load
// after another: 512 causal rows, 4 heads, d = 128: forward 121 us, now 49; backward 366 us, now 134; prefix and forward of
// 256 rows, w = 64, d = 64: 11.1 us, now 8.9.)
// ==========================================================================================
constexpr int kF32Waves = 4;
// Load instructions per matrix and step.  Four keep a wave at 63 to 84 registers, so that up to eight share a SIMD and hide
// each other's latency, and a short window is not rounded up to a long step.  A forward of so few rows that a wave has the
// SIMD to itself is the one place where more loads in flight win (one head, d = 64, 512 causal rows: 16.4 us with 16 loads,
// 18.6 with 4; 8192 rows, w = 16, d = 128: 19.1 and 11.0; 65536 rows of 4096 sequences, d = 64: 118 and 34, backward 290
// and 82).
constexpr int kRowLoads = 4, kRowLoadsAlone = 16;

template <int CTRL>
__device__ __forceinline__ float dpp_moved(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_pair_sum(float x) {  // lane ^ 16
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float row_pair_max(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int D, int LOADS>
struct RowStep {
    static constexpr int kLanes = D / 4, kRows = 64 / kLanes;  // lanes per row, rows per load instruction
    static constexpr int kLoads = LOADS, kStep = kLoads * kRows;  // rows per step
    f32x4 x[kLoads];
    // rows row0 + u kRows + lane / kLanes, u = 0 .. kLoads - 1, of the matrix at M; past `last`: row `last`
    __device__ __forceinline__ void load(const float* M, int row0, int last, int lane) {
#pragma unroll
        for (int u = 0; u < kLoads; ++u)
            x[u] = *reinterpret_cast<const f32x4*>(M + (size_t)min(row0 + u * kRows + lane / kLanes, last) * D + 4 * (lane % kLanes));
    }
    // the rows past `last` become zero: they have weight zero, and zero times an infinity is NaN
    __device__ __forceinline__ void clear_past(int row0, int last, int lane) {
        if (row0 + kStep - 1 <= last) return;  // (the same in all lanes)
#pragma unroll
        for (int u = 0; u < kLoads; ++u)
            if (row0 + u * kRows + lane / kLanes > last) x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ float dot(const f32x4& q, int u) const {  // with the row whose columns q holds; in all its lanes
        float d = q[0] * x[u][0];
#pragma unroll
        for (int j = 1; j < 4; ++j) d = fmaf(q[j], x[u][j], d);
        d += dpp_moved<0x128>(d);  // row_ror:8, 4, 2, 1
        d += dpp_moved<0x124>(d);
        d += dpp_moved<0x122>(d);
        d += dpp_moved<0x121>(d);
        return D == 128 ? row_pair_sum(d) : d;
    }
    // sum over the row groups of a wave
    static __device__ __forceinline__ float group_sum(float v) { return xhalf_sum(D == 128 ? v : row_pair_sum(v)); }
    static __device__ __forceinline__ double group_sum(double v) {
        if (D == 64) v += __shfl_xor(v, 16, 64);
        return v + __shfl_xor(v, 32, 64);
    }
    static __device__ __forceinline__ float group_max(float v) { return xhalf_max(D == 128 ? v : row_pair_max(v)); }
    static __device__ __forceinline__ f32x4 group_sum(const f32x4& v) {
        return {group_sum(v[0]), group_sum(v[1]), group_sum(v[2]), group_sum(v[3])};
    }
};
__device__ __forceinline__ f32x4 fma4(float a, const f32x4& x, const f32x4& c) {
    return {fmaf(a, x[0], c[0]), fmaf(a, x[1], c[1]), fmaf(a, x[2], c[2]), fmaf(a, x[3], c[3])};
}

// ---- forward: online softmax over the steps of the window of row t.  Pointers are the head's.
template <int D, int LOADS>
__device__ __forceinline__ void fwd_row(const float* Qh, const float* Kh, const float* Vh, const float* ch, float* Oh, float* Lh, int t,
                                        int w, float scale, int lane) {
    using Step = RowStep<D, LOADS>;
    const int r = lane / Step::kLanes, col = 4 * (lane % Step::kLanes);
    const int lo = max(0, t - w + 1);
    Step k, v;
    float ci[Step::kLoads];
    const f32x4 q = *reinterpret_cast<const f32x4*>(Qh + (size_t)t * D + col);
    const float ct = ch[t];
    float m = -INFINITY, l = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = lo; i0 <= t; i0 += Step::kStep) {
        k.load(Kh, i0, t, lane);
#pragma unroll
        for (int u = 0; u < Step::kLoads; ++u) ci[u] = ch[min(i0 + u * Step::kRows + r, t)];
        v.load(Vh, i0, t, lane);
        float s[Step::kLoads], mx = m;
#pragma unroll
        for (int u = 0; u < Step::kLoads; ++u) {
            s[u] = fmaf(scale, k.dot(q, u), ci[u] - ct);
            s[u] = i0 + u * Step::kRows + r <= t ? s[u] : -INFINITY;
            mx = fmaxf(mx, s[u]);
        }
        v.clear_past(i0, t, lane);
        const float mnew = Step::group_max(mx);
        const float ref = mnew == -INFINITY ? 0.f : mnew;  // (every score so far is minus infinity: weight zero)
        const float a = expf(m - ref);
        l *= a;
        o *= a;
        m = mnew;
#pragma unroll
        for (int u = 0; u < Step::kLoads; ++u) {
            const float p = expf(s[u] - ref);
            l += p;
            o = fma4(p, v.x[u], o);
        }
    }
    l = Step::group_sum(l);
    o = Step::group_sum(o);
    if (r == 0) *reinterpret_cast<f32x4*>(Oh + (size_t)t * D + col) = f32x4{o[0] / l, o[1] / l, o[2] / l, o[3] / l};
    if (lane == 0) Lh[t] = m + logf(l);
}
template <int D, int LOADS>
__global__ __launch_bounds__(64 * kF32Waves) void fwd_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ c, float* __restrict__ O, float* __restrict__ L, int N, int w,
    float scale, int H, int G) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rows_per_head = (N + kF32Waves - 1) / kF32Waves;
    const int bh = blockIdx.x / rows_per_head;
    const int t = (blockIdx.x % rows_per_head) * kF32Waves + wv;
    if (t >= N) return;  // whole wave leaves; no workgroup barriers are used below
    const size_t ho = (size_t)bh * N * D, kvo = (size_t)kv_head_of(bh, H, G) * N * D, rows = (size_t)bh * N;
    fwd_row<D, LOADS>(Q + ho, K + kvo, V + kvo, c + rows, O + ho, L + rows, t, w, scale, lane);
}

// ---- dQ_t and the row sum of dS.  OWN_D: D_t = <O_t, dO_t> is formed and stored; else it is read and Oh is not.
template <int D, int LOADS, bool OWN_D>
__device__ __forceinline__ void dq_row(const float* Qh, const float* Kh, const float* Vh, const float* Oh, const float* dOh, const float* ch,
                                       const float* Lh, std::conditional_t<OWN_D, float, const float>* Dh, float* dQh, float* dc_rowh,
                                       int t, int w, float scale, int lane) {
    using Step = RowStep<D, LOADS>;
    const int r = lane / Step::kLanes, col = 4 * (lane % Step::kLanes);
    const int lo = max(0, t - w + 1);
    Step k, v;
    float ci[Step::kLoads];
    const size_t at = (size_t)t * D + col;
    const f32x4 q = *reinterpret_cast<const f32x4*>(Qh + at), g = *reinterpret_cast<const f32x4*>(dOh + at);
    const float ct = ch[t], Lt = Lh[t];
    float Dt = OWN_D ? 0.f : Dh[t];
    // fp64: the suffix sums of the gate gradient add up what this sum and the column sums of dkv_row round (with running fp32
    // sums d(alpha) of 12 heads of 300 rows, d = 128, w = 77 was off by 1.4e-6 of its norm instead of 1.0e-6)
    double rs = 0.0;
    f32x4 dq = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = lo; i0 <= t; i0 += Step::kStep) {
        k.load(Kh, i0, t, lane);
#pragma unroll
        for (int u = 0; u < Step::kLoads; ++u) ci[u] = ch[min(i0 + u * Step::kRows + r, t)];
        v.load(Vh, i0, t, lane);
        if constexpr (OWN_D)
            if (i0 == lo) {
                RowStep<D, 1> one;
                one.x[0] = *reinterpret_cast<const f32x4*>(Oh + at);
                Dt = one.dot(g, 0);
            }
        k.clear_past(i0, t, lane);
#pragma unroll
        for (int u = 0; u < Step::kLoads; ++u) {
            const float s = fmaf(scale, k.dot(q, u), ci[u] - ct);
            const float ds = i0 + u * Step::kRows + r <= t ? expf(s - Lt) * (v.dot(g, u) - Dt) : 0.f;
            rs += (double)ds;
            dq = fma4(ds, k.x[u], dq);
        }
    }
    rs = Step::group_sum(rs);
    dq = Step::group_sum(dq);
    if (r == 0) *reinterpret_cast<f32x4*>(dQh + at) = dq * scale;
    if (lane == 0) {
        if constexpr (OWN_D) Dh[t] = Dt;
        dc_rowh[t] = (float)rs;
    }
}

// ---- dK_i, dV_i (summed over the G query heads that read this key/value head, bh0 the first) and, per query head, the
// column sum of dS.  rows_s: 64 places of LDS of the wave's own, for c, L, D of a step's queries.
template <int D, int LOADS>
__device__ __forceinline__ void dkv_row(const float* Q, const float* Kh, const float* Vh, const float* dO, const float* c, const float* L,
                                        const float* Dv, float* dKh, float* dVh, float* dc_col, f32x4* rows_s, int bh0, int G, int i, int N,
                                        int w, float scale, int lane) {
    using Step = RowStep<D, LOADS>;
    const int r = lane / Step::kLanes, col = 4 * (lane % Step::kLanes);
    const size_t at = (size_t)i * D + col;
    const f32x4 k = *reinterpret_cast<const f32x4*>(Kh + at), v = *reinterpret_cast<const f32x4*>(Vh + at);
    const int t_hi = (int)min((long)N - 1, (long)i + w - 1);  // key i is seen by rows i .. i+w-1
    f32x4 dk = {0.f, 0.f, 0.f, 0.f}, dv = dk;
    Step q, d;
    for (int g = 0; g < G; ++g) {
        const size_t rows = (size_t)(bh0 + g) * N;
        const float ci = c[rows + i];
        double cs = 0.0;
        for (int t0 = i; t0 <= t_hi; t0 += Step::kStep) {
            const int tl = min(t0 + lane, t_hi);
            const f32x4 row = {c[rows + tl], L[rows + tl], Dv[rows + tl], 0.f};
            q.load(Q + rows * D, t0, t_hi, lane);
            d.load(dO + rows * D, t0, t_hi, lane);
            rows_s[lane] = row;
            q.clear_past(t0, t_hi, lane);
            d.clear_past(t0, t_hi, lane);
#pragma unroll
            for (int u = 0; u < Step::kLoads; ++u) {
                const int n = u * Step::kRows + r;
                const f32x4 x = rows_s[n];
                const float s = fmaf(scale, q.dot(k, u), ci - x[0]);
                const bool seen = t0 + n <= t_hi;
                const float p = seen ? expf(s - x[1]) : 0.f;
                const float ds = seen ? p * (d.dot(v, u) - x[2]) : 0.f;
                cs += (double)ds;
                dv = fma4(p, d.x[u], dv);
                dk = fma4(ds, q.x[u], dk);
            }
        }
        cs = Step::group_sum(cs);
        if (lane == 0) dc_col[rows + i] = (float)cs;
    }
    dk = Step::group_sum(dk);
    dv = Step::group_sum(dv);
    if (r == 0) {
        *reinterpret_cast<f32x4*>(dKh + at) = dk * scale;
        *reinterpret_cast<f32x4*>(dVh + at) = dv;
    }
}
// Both in one launch (the first workgroups take keys, the longer rows; D_t has been formed by rowdot_f32_kernel), or one of them (the
// queries, which then form D_t, first).  In two launches neither pass of a small problem fills the chip (B1 H4 N300 d64: 35.5 us,
// 24.5 in one; B4 H8 N200 w100 35.0 / 22.8; 256 rows, w = 64 14.0 / 11.8).  f32_rows_in_two_launches has the line.
enum F32Pass { kF32Both, kF32Queries, kF32Keys };
template <int D, F32Pass PASS>
__global__ __launch_bounds__(64 * kF32Waves) void bwd_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, const float* __restrict__ O,
    const float* __restrict__ dO, const float* __restrict__ c, const float* __restrict__ L, float* __restrict__ Dv, float* __restrict__ dQ,
    float* __restrict__ dK, float* __restrict__ dV, float* __restrict__ dc_col, float* __restrict__ dc_row, int N, int w, float scale,
    int key_blocks, int H, int G) {
    __shared__ f32x4 rows_s[PASS == kF32Queries ? 1 : kF32Waves][64];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rows_per_head = (N + kF32Waves - 1) / kF32Waves;
    const bool keys = PASS == kF32Both ? (int)blockIdx.x < key_blocks : PASS == kF32Keys;
    const int block = (int)blockIdx.x - (PASS == kF32Both && !keys ? key_blocks : 0);
    const int head = block / rows_per_head, row = block % rows_per_head * kF32Waves + wv;
    if (row >= N) return;  // whole wave leaves; no workgroup barriers are used
    if (keys) {
        const int Hkv = H / G;
        const size_t kvo = (size_t)head * N * D;
        dkv_row<D, kRowLoads>(Q, K + kvo, V + kvo, dO, c, L, Dv, dK + kvo, dV + kvo, dc_col, rows_s[PASS == kF32Queries ? 0 : wv],
                              (head / Hkv) * H + (head % Hkv) * G, G, row, N, w, scale, lane);
    } else {
        const size_t ho = (size_t)head * N * D, kvo = (size_t)kv_head_of(head, H, G) * N * D, rows = (size_t)head * N;
        dq_row<D, kRowLoads, PASS == kF32Queries>(Q + ho, K + kvo, V + kvo, O + ho, dO + ho, c + rows, L + rows, Dv + rows, dQ + ho,
                                                  dc_row + rows, row, w, scale, lane);
    }
}

// ==========================================================================================
// fp32 matrix-core kernels.  The part multiplies bf16 sixteen times as fast as fp32, so every product is formed from
// three bf16 pieces per operand: x = x0 + x1 + x2 holds all 24 bits of an fp32 value (each piece is what the pieces
// before it leave over, rounded to bf16; values below 2^-110 reach the end of bf16's exponent range), bf16 products are
// exact in fp32, and
//   a b = a0 b0 + (a0 b1 + a1 b0) + (a1 b1 + a0 b2 + a2 b0) + what is left out, at most 2^-23 |a b|, 2^-26 typically.
// Six bf16 MFMAs of 16 terms take 192 cycles where eight fp32 MFMAs of 2 terms take 512, and add to the accumulator
// less often: against fp64 the outputs are closer than with fp32 MFMAs (B1 H3 N1500 d128 w700, error over norm: O 1.0e-7, was
// 2.2e-7; dQ 1.7e-7, was 3.4e-7; dK 2.2e-7, was 4.1e-7; dV 1.9e-7, was 3.3e-7; dalpha 1.5e-6, was 1.9e-6).
// Layouts are those of the bf16 kernels (mfma32): a lane owns a query or a key, the second product of each kernel takes
// the first one's accumulator registers, split in place, as its B operand.  Operands are split once: resident rows
// (of Q; Q and dO; K and V) when the workgroup starts, streamed tiles on their way into LDS by the threads that fetched them.
// Measured, B2 H16 N4096 d128 w1024, with fp32 MFMAs / now: forward 642 / 334 us, dK/dV 1410 / 586 us, dQ 1001 / 470 us.
// What bounds them: executed bf16 products at 1.1 to 1.3 PFLOP/s, the matrix pipe busy 60 to 65 % of the cycles at 1.85 GHz,
// the clock the part holds under this load (2.03 GHz with the pipe at 53 %).
// ==========================================================================================

// two values -> their three bf16 pieces, packed
struct Split2 {
    unsigned p[3];
};
__device__ __forceinline__ Split2 split2(float x, float y) {
    auto pack = [](float a, float b) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2)); };
    auto lower = [](unsigned p) { return __uint_as_float(p << 16); };
    auto upper = [](unsigned p) { return __uint_as_float(p & 0xffff0000u); };
    Split2 s;
    s.p[0] = pack(x, y);
    x -= lower(s.p[0]);
    y -= upper(s.p[0]);
    s.p[1] = pack(x, y);
    s.p[2] = pack(x - lower(s.p[1]), y - upper(s.p[1]));
    return s;
}
// eight values (of a row, or the registers 8 c2 .. 8 c2 + 7 of an accumulator block) -> the pieces of an operand fragment
template <typename F>
__device__ __forceinline__ void split_frag(F&& value, bf16x8 (&f)[3]) {
    u32x4 p[3];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const Split2 t = split2(value(2 * j), value(2 * j + 1));
#pragma unroll
        for (int k = 0; k < 3; ++k) p[k][j] = t.p[k];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) f[k] = __builtin_bit_cast(bf16x8, p[k]);
}
__device__ __forceinline__ void split_row(const float* g, bf16x8 (&f)[3]) {
    const f32x4 x0 = *reinterpret_cast<const f32x4*>(g), x1 = *reinterpret_cast<const f32x4*>(g + 4);
    split_frag([&](int j) __attribute__((always_inline)) { return j < 4 ? x0[j & 3] : x1[j & 3]; }, f);
}
__device__ __forceinline__ void split_acc(const f32x16& s, int c2, bf16x8 (&f)[3]) {
    split_frag([&](int j) __attribute__((always_inline)) { return s[8 * c2 + j]; }, f);
}
// Whether the rows a wave has finished have to be formed once more by the one-wave-per-row code above, which is plain fp32
// throughout.  Two reasons.  The pieces hold every fp32 value but the infinities and those from 2^128 - 2^119 on, whose first piece is infinite and
// whose second is NaN, and products of pieces can overflow with either sign where the whole product is one infinity.  Any
// of it leaves NaN or an infinity in each result that it is part of, so the results are looked at, once, when they are done.
// And pieces end at 2^-133: a value below 2^-110 loses its low bits, of 2^-122 all but 11.  Beside values that are 2^24 times as
// large that is nothing, but a whole matrix may be that small (an unscaled gradient, say).  Then all results are, since
// each of O, dQ, dK, dV is a sum over the rows of one matrix with weights that another has made: rows that are not zero but
// below 2^-80 throughout a wave's 32 are formed again as well.  The check itself costs 0.5 % of B2 H16 N4096 d128 w1024, 10 % where
// a workgroup has no more than two or four blocks (256 sequences of 64, d = 128, backward: 37 us without, 41 with it).
struct RangeCheck {
    bool finite = true;
    float largest = 0.f;
    __device__ __forceinline__ void add(float x) { finite = finite && fabsf(x) <= 3.402823466e38f; }
    template <int DB>
    __device__ __forceinline__ void add(const f32x16 (&x)[DB]) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                add(x[db][v]);
                largest = fmaxf(largest, fabsf(x[db][v]));
            }
    }
    // (the same in all lanes; valid: this lane's row exists)
    __device__ __forceinline__ bool failed(bool valid) const {
        return __builtin_amdgcn_ballot_w64(valid && !finite) != 0 ||
               (__builtin_amdgcn_ballot_w64(valid && largest >= 8.27180613e-25f) == 0 && __builtin_amdgcn_ballot_w64(valid && largest > 0.f) != 0);
    }
};
// 32 rows of a [N, D] matrix in LDS, as three bf16 planes with the swizzle of tile_off
template <int D>
struct SplitTile {
    static constexpr int kPlane = 32 * D * 2;
    alignas(256) char p[3][kPlane];
};
// piece k of a fragment of such a tile (row_frag, col_frag of split_band.h; `at`: the lane's address in plane 0)
template <int D>
__device__ __forceinline__ bf16x8 split_row_frag(unsigned at, int kc, int k) { return row_frag<D>(at, 32 * k, kc); }
template <int D>
__device__ __forceinline__ bf16x8 split_col_frag(unsigned at, int r0, int db, int k) { return col_frag<D>(at, 32 * k + r0, db); }

// The product of the 32 rows of a tile with the resident rows b over the head dimension.  All products of smaller pieces
// come first, over the whole head dimension, then the a0 b0: added in between, the small ones lose bits to an accumulator
// that is already large (error of O 1.8e-7 of its norm instead of 1.0e-7, of dQ 2.8e-7 instead of 1.7e-7; the second
// reading of the a0 costs 1 % of the time).
// QROWS: the tile holds rows of Q or dO, b keys or values; otherwise the other way round.  Either way the same products
// are added in the same order, so that the dK/dV and the dQ kernel form the same dS, bit by bit, and its row and column
// sums cancel in the suffix sums of the gate gradient.
// A fragment is read two chunks ahead, into the registers of the one that has just been used (LDS takes 150 to 300 cycles
// with eight waves at it, a chunk's products 160).  `beside(kc)` is what else may be placed beside the products, `late` runs
// in front of the second pass (reads whose results are needed right after it).
template <int D, bool QROWS, typename F0, typename F1>
__device__ __forceinline__ f32x16 tile_dot(unsigned at, const bf16x8 (&b)[D / 16][3], F0&& beside, F1&& late) {
    constexpr int KC = D / 16;
    f32x16 c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = 0.f;
    bf16x8 f[2][3];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) f[i][k] = split_row_frag<D>(at, i, k);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
        bf16x8(&a)[3] = f[kc & 1];
        // piece k of two chunks further on; of the last two chunks' places the a0 of chunks 0 .. 3 of the second pass take four
        auto refill = [&](int k) __attribute__((always_inline)) {
            if (kc + 2 < KC) a[k] = split_row_frag<D>(at, kc + 2, k);
            else if (k < 2) a[k] = split_row_frag<D>(at, 2 * (kc & 1) + k, 0);
        };
        c = QROWS ? mfma32(a[2], b[kc][0], c) : mfma32(a[0], b[kc][2], c);
        c = QROWS ? mfma32(a[0], b[kc][2], c) : mfma32(a[2], b[kc][0], c);
        __builtin_amdgcn_sched_barrier(0);
        refill(2);
        c = mfma32(a[1], b[kc][1], c);
        c = QROWS ? mfma32(a[1], b[kc][0], c) : mfma32(a[0], b[kc][1], c);
        beside(kc);
        __builtin_amdgcn_sched_barrier(0);
        if (QROWS) refill(1);
        c = QROWS ? mfma32(a[0], b[kc][1], c) : mfma32(a[1], b[kc][0], c);
        __builtin_amdgcn_sched_barrier(0);
        if (!QROWS) refill(1);
        refill(0);
    }
    late();
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
        bf16x8& a = f[(kc >> 1) & 1][kc & 1];
        c = mfma32(a, b[kc][0], c);
        __builtin_amdgcn_sched_barrier(0);
        if (kc + 4 < KC) a = split_row_frag<D>(at, kc + 4, 0);
    }
    return c;
}
// The first fragment of a transposed tile (row half C0), to be read before tile_axpy is reached.
struct ColFrag {
    bf16x8 a0, a1, a2;
};
template <int D, int C0>
__device__ __forceinline__ ColFrag first_col(unsigned at) {
    return {split_col_frag<D>(at, 16 * C0, 0, 0), split_col_frag<D>(at, 16 * C0, 0, 1), split_col_frag<D>(at, 16 * C0, 0, 2)};
}
// acc[db] += (tile^T, 32-column block db) x over the row halves C0 .. C1 - 1, x an accumulator block as the B operand.  xf: the
// pieces of the first half; those of the second are formed between the products.  `beside(i)`: as above, (C1 - C0) D / 32
// times.
template <int D, int C0, int C1, typename F>
__device__ __forceinline__ void tile_axpy(unsigned at, const f32x16& x, bf16x8 (&xf)[3], ColFrag f, f32x16 (&acc)[D / 32], F&& beside) {
    constexpr int DB = D / 32, NF = (C1 - C0) * DB;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        const bool more = i + 1 < NF;
        const int r0 = 16 * (C0 + (i + 1) / DB), db = (i + 1) % DB;
        f32x16& c = acc[i % DB];
        c = mfma32(f.a2, xf[0], c);
        c = mfma32(f.a1, xf[1], c);
        __builtin_amdgcn_sched_barrier(0);
        if (more) f.a2 = split_col_frag<D>(at, r0, db, 2);
        c = mfma32(f.a1, xf[0], c);
        beside(i);
        __builtin_amdgcn_sched_barrier(0);
        if (more) f.a1 = split_col_frag<D>(at, r0, db, 1);
        const bf16x8 a0 = f.a0;
        if (more) f.a0 = split_col_frag<D>(at, r0, db, 0);
        c = mfma32(a0, xf[2], c);
        c = mfma32(a0, xf[1], c);
        c = mfma32(a0, xf[0], c);
        __builtin_amdgcn_sched_barrier(0);
        if (C1 - C0 == 2 && i + 1 == DB) split_acc(x, C0 + 1, xf);
    }
}

// 32-row tiles of [N, D] matrices on their way through the registers of a workgroup of T threads: 16-byte pieces, a
// thread takes every T-th (rows row, row + kStep, ..).
template <int D, int T>
struct F32TileMover {
    static constexpr int kPieces = 32 * (D / 4) / T, kStep = T / (D / 4);
    static_assert(kStep % 16 == 0 || kStep == 8, "the swizzle has period 16, eight rows further on it differs by one chunk bit (as in col_frag)");
    int row, col, at;  // first row, its column in bytes, LDS address inside a plane
    __device__ __forceinline__ void init(int tid) {
        row = tid / (D / 4);
        col = 16 * (tid % (D / 4));
        at = tile_off<D>(row, (tid % (D / 4)) >> 1) + 8 * (tid & 1);
    }
    // (`part` of n: those of the pieces that belong there)
    __device__ __forceinline__ void fetch(f32x4 (&r)[kPieces], const float* M, int row0, int N, int part = 0, int n = 1) const {  // rows past N read row N-1
        const char* first = reinterpret_cast<const char*>(M + (size_t)row0 * D);
#pragma unroll
        for (int i = part * kPieces / n; i < (part + 1) * kPieces / n; ++i)
            r[i] = *reinterpret_cast<const f32x4*>(first + (unsigned)(min(row + i * kStep, N - 1 - row0) * (D * 4) + col));
    }
    __device__ __forceinline__ void stash(const f32x4 (&r)[kPieces], SplitTile<D>& tile, int part, int n) const {
#pragma unroll
        for (int i = part * kPieces / n; i < (part + 1) * kPieces / n; ++i) {
            char* to = tile.p[0] + (kStep == 8 && (i & 1) ? at ^ (D == 128 ? 32 : 16) : at) + i * kStep * (D * 2);
            const Split2 a = split2(r[i][0], r[i][1]), b = split2(r[i][2], r[i][3]);
#pragma unroll
            for (int k = 0; k < 3; ++k) *reinterpret_cast<u32x2*>(to + k * SplitTile<D>::kPlane) = u32x2{a.p[k], b.p[k]};
        }
    }
};

// ---- forward (Alg. 2): a workgroup of NW waves owns 32 NW queries, a wave 32 of them, a lane one query (both halves of
// the wave hold it, with complementary keys).  S^T = K Q^T with the Q fragments in registers, the running maximum
// and sum per lane, O^T += V^T P^T with P^T taken from the S^T accumulator registers.
// Tiles are double buffered, the next one is split and stored between the PV products, one barrier per block.  With eight
// waves two share a SIMD, and waves 0 .. 3 have the higher issue priority: they take the matrix pipe first and do their
// softmax while the others form S, and the others do theirs beside the first ones' PV products.  (Two workgroups of four
// waves per CU instead, whose waves all come to the softmax at the same time and split every tile twice: 452 us.)
// S = 1, for short bands: one buffer, refilled between two barriers, and the LDS it saves holds further workgroups that run
// meanwhile.
template <int D, int S>
struct F32FwdSmem {
    SplitTile<D> k[S], v[S];
    alignas(16) float c[S][32];
    int needed[8];  // over_waves
};
// Order of the forward's tiles.  From the longest band to the shortest over all heads (tile_of_block), over 3418 shapes 0.95 of the
// time of one head after another (B1 H12/6 N6219 d64 w2854 374 -> 261 us, B1 H10/5 N6600 d128 w918 290 -> 189), except
//   heads that do not divide by the XCDs and are one tile each: the heads of a group on one XCD (B41 H12/3 N49 d128 21.8 -> 18.9)
//   short bands, less than a tenth of the sequence, whose lengths hardly differ: d = 64 such heads one after another too (B11 H4/2
//   N1091 w15 18.1 -> 16.0), d = 128 all heads from the sequence's start to its end (B3 H24/12 N4505 w228 397 -> 373)
template <int D>
__device__ __forceinline__ int f32_fwd_tile(int block, int heads, int tiles, int N, int w, int& head) {
    const bool short_band = 10L * w < N, by_length = heads % 8 == 0 || (tiles > 1 && (D == 128 || !short_band));
    int tile;
    tile_of_block(block, heads, tiles, by_length, head, tile);
    return by_length && (D == 64 || !short_band) ? tiles - 1 - tile : tile;
}

// LOOK, here and in the backward: reach is there.  (A look that is compiled in costs problems that never take it up to 2 %: B5 H7 N9536 d64 w58
// backward 304 / 299 us.)
template <int D, int NW, int S, bool LOOK>
__global__ __launch_bounds__(64 * NW, D == 128 && NW == 4 && S == 2 ? 1 : 2) void fwd_f32_mfma_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ c, float* __restrict__ O, float* __restrict__ L, int N, int w, float scale,
    int num_qtiles, int total_tiles, int H, int G, KeyReach reach) {
    constexpr int KC = D / 16, DB = D / 32, BQ = 32 * NW;
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<F32FwdSmem<D, S>*>(smem_raw);
    const int heads = total_tiles / num_qtiles;
    int bh;
    const int q0 = f32_fwd_tile<D>((int)blockIdx.x, heads, num_qtiles, N, w, bh) * BQ;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, lq = lane & 31;
    const int qw0 = q0 + 32 * wv, t = qw0 + lq, tc = min(t, N - 1);
    const size_t ho = (size_t)bh * N * D, kvo = (size_t)kv_head_of(bh, H, G) * N * D;
    const float *Kh = K + kvo, *Vh = V + kvo, *ch = c + (size_t)bh * N;
    if (NW == 8 && wv < 4) __builtin_amdgcn_s_setprio(1);

    const int k_lo = max(0, q0 - w + 1), jb_hi = (min(N, q0 + BQ) - 1) / 32;
    int first_key = k_lo;
    if (LOOK && reach_pays(ch[q0] - ch[k_lo], q0 - k_lo, reach.few)) {  // the keys that the gate has erased for all queries stay out
        float q2 = 0.f, k2 = 0.f, own = 0.f;
        const float *qr = Q + ho + (size_t)tc * D + 4 * h, *kr = Kh + (size_t)tc * D + 4 * h;  // (the halves take every other four columns)
#pragma unroll 8
        for (int i = 0; i < D / 8; ++i) {
            const f32x4 q = *reinterpret_cast<const f32x4*>(qr + 8 * i), k = *reinterpret_cast<const f32x4*>(kr + 8 * i);
#pragma unroll
            for (int j = 0; j < 4; ++j) q2 = fmaf(q[j], q[j], q2), k2 = fmaf(k[j], k[j], k2), own = fmaf(q[j], k[j], own);
        }
        q2 = xhalf_sum(q2);
        // the row's maximum is at least the score of the query's own key
        const float edge = (ch[tc] - ch[q0]) * kLog2e + scale * kLog2e * (xhalf_sum(own) - 1e-4f * sqrtf(q2 * xhalf_sum(k2)));
        const float reach2 = reach2_of(lanes_max<32>(norm_bits(q2)), scale * kLog2e), lowest = from_order(lanes_min<32>(lowest_order(edge))) - kErased;
        first_key = over_waves<NW, true>(first_needed_key(key_block<D>(O + ho + (size_t)q0 * D, min(BQ, N - q0), lane), q0, k_lo, reach.block, reach2,
                                                          lowest, ch[q0], lane),
                                         sm.needed, wv, lane);
    }
    const int jb_lo = first_key / 32;
    using Mover = F32TileMover<D, 64 * NW>;
    Mover mv;
    mv.init(tid);
    f32x4 kreg[Mover::kPieces], vreg[Mover::kPieces];
    float creg = 0.f;
    auto fetch = [&](int jb, int part = 0, int n = 1) __attribute__((always_inline)) {
        mv.fetch(kreg, Kh, 32 * jb, N, part, n);
        mv.fetch(vreg, Vh, 32 * jb, N, part, n);
        if (part == 0 && tid < 32) creg = ch[min(32 * jb + tid, N - 1)];
    };
    auto stash_share = [&](int buf, int i, int n) __attribute__((always_inline)) {
        mv.stash(kreg, sm.k[buf], i, n);
        mv.stash(vreg, sm.v[buf], i, n);
    };
    fetch(jb_lo);
    bf16x8 qf[KC][3];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) split_row(Q + ho + (size_t)tc * D + 16 * kc + 8 * h, qf[kc]);
    __builtin_amdgcn_sched_barrier(0);
    const float ct = ch[tc];
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    float mrun = kNegBig, lh = 0.f;  // lh: the sum over this half's keys

    int r_off = row_frag_off<D>(lane), t_off = col_frag_off<D>(lane);
    stash_share(0, 0, 1);
    if (tid < 32) sm.c[0][tid] = creg;
    wg_barrier();
    auto end_step = [&](int jb) __attribute__((always_inline)) {
        if (S == 1) {
            if (jb == jb_hi) return;
            wg_barrier();  // the tile is read by all
            stash_share(0, 0, 1);
        }
        if (tid < 32) sm.c[S == 2 ? (jb - jb_lo + 1) & 1 : 0][tid] = creg;
        wg_barrier();
    };
    auto idle_step = [&](int jb) __attribute__((always_inline)) {  // no block of this wave's band: only its share of the tile
        fetch(min(jb + 1, jb_hi));
        if (S == 2) stash_share((jb - jb_lo + 1) & 1, 0, 1);
        end_step(jb);
    };
    // (three loops: with a branch around the computing step inside one loop the compiler copies the accumulators)
    const int act_lo = qw0 < N ? max(first_key, qw0 - w + 1) / 32 : jb_hi + 1, act_hi = min(qw0 / 32, jb_hi);
    int jb = jb_lo;
    for (; jb < act_lo; ++jb) idle_step(jb);
    for (; jb <= act_hi; ++jb) {
        // (the addresses derived from these are recomputed in every block instead of living in registers across the loop)
        GFWA_PIN(r_off);
        GFWA_PIN(t_off);
        const int kb0 = 32 * jb, buf = S == 2 ? (jb - jb_lo) & 1 : 0;
        const unsigned kt = (unsigned)(uintptr_t)sm.k[buf].p[0] + r_off, vt = (unsigned)(uintptr_t)sm.v[buf].p[0] + t_off;
        f32x16 g;
        bf16x8 pf[3];
        f32x16 s = tile_dot<D, false>(
            kt, qf, [&](int kc) __attribute__((always_inline)) { fetch(min(jb + 1, jb_hi), kc, KC); },
            [&]() __attribute__((always_inline)) { acc_init_rows(g, sm.c[buf], 0, h); });
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = fmaf(scale, s[v], g[v] - ct);
        if (__builtin_expect(!(kb0 + 31 <= qw0 && kb0 > qw0 + 31 - w), 0)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = kb0 + acc_row(v, h);
                s[v] = (i <= t && i > t - w) ? s[v] : -INFINITY;
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[v]);
        // exp through the hardware exp2: the argument's rounding (2^-24 |x| log2 e) only matters for
        // probabilities that are themselves negligible
        const float mnew = fmaxf(mrun, xhalf_max(mx));
        const float a = fast_exp2((mrun - mnew) * kLog2e);
        float psum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = fast_exp2((s[v] - mnew) * kLog2e);
            psum += s[v];
        }
        lh = fmaf(lh, a, psum);
        mrun = mnew;
        if (__builtin_amdgcn_ballot_w64(a != 1.0f) != 0) {  // the maximum of some row has moved (rare after the first blocks)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[db][v] *= a;
        }
        const ColFrag f = first_col<D, 0>(vt);
        split_acc(s, 0, pf);
        tile_axpy<D, 0, 2>(vt, s, pf, f, o, [&](int i) __attribute__((always_inline)) {
            if (S == 2) stash_share(buf ^ 1, i, 2 * DB);
        });
        end_step(jb);
    }
    for (; jb <= jb_hi; ++jb) idle_step(jb);
    const float l = xhalf_sum(lh);
    RangeCheck check;
    check.add(o);  // (before the division by l, which is between 1 and the number of keys unless the next two say otherwise)
    check.add(l);
    check.add(1.0f / l);
    if (__builtin_expect(check.failed(t < N), 0)) {
#pragma unroll 1
        for (int row = qw0; row < min(N, qw0 + 32); ++row) fwd_row<D, kRowLoads>(Q + ho, Kh, Vh, ch, O + ho, L + (size_t)bh * N, row, w, scale, lane);
    } else if (t < N) {
        float* orow = O + ho + (size_t)t * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                f32x4 out;
#pragma unroll
                for (int j = 0; j < 4; ++j) out[j] = o[db][4 * i4 + j] / l;
                *reinterpret_cast<f32x4*>(orow + 32 * db + 8 * i4 + 4 * h) = out;
            }
        if (h == 0) L[(size_t)bh * N + t] = mrun + fast_log2(l) * kLn2;
    }
}

// ---- backward.  The resident rows take 96 registers per matrix at d = 128, so two waves (of eight: wv and
// wv + 4, of one SIMD) share 32 queries or keys.  Wave 0 of a pair holds the rows of the matrix that forms S and turns S into P,
// wave 1 those that form dP; what they need of each other travels through LDS.  The products with dS are one block behind
// (the tile they need, K or Q, is kept in a ring of three), so that a step has one barrier and neither wave waits for
// the other inside it: one's exponentials and splits run beside the other's MFMAs.  (In step, with a second barrier
// between the first and the second products: dK/dV 606 us, dQ 500 us.)  NP: pairs of a workgroup, four, or two for short bands.
template <int D, int NP>
struct F32BwdSmem {
    SplitTile<D> a[3], b[2];           // dK/dV: Q, dO; dQ: K, V
    f32x4 x[2][NP][4][64];              // per pair, one block behind: P (dK/dV); half of P and half of dP - D (dQ)
    alignas(16) float v[3][2][32];     // up to three values per row of the tile
};
__device__ __forceinline__ int next3(int i) { return i == 2 ? 0 : i + 1; }

// dQ and the row sums of dS (Alg. 3, query loop): the forward's layout.  S^T = K Q^T (wave 0 of a pair) and
// dP^T = V dO^T (wave 1), then both take half of the block's keys: dS^T = P^T (dP^T - D), dQ^T += K^T dS^T.
template <int D, int NP, bool LOOK>
__device__ __forceinline__ void dq_f32_mfma(
    int block, const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, const float* __restrict__ dO,
    const float* __restrict__ c, const float* __restrict__ L, const float* __restrict__ Dv, float* __restrict__ dQ,
    float* __restrict__ dc_row, const float* __restrict__ reach, int N, int w, float scale, int num_qtiles, int total_tiles, int H, int G) {
    constexpr int KC = D / 16, DB = D / 32;
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<F32BwdSmem<D, NP>*>(smem_raw);
    const int heads = total_tiles / num_qtiles;
    int bh, qt;
    tile_of_block(block, heads, num_qtiles, true, bh, qt);
    const int q0 = (num_qtiles - 1 - qt) * 32 * NP;  // longest bands first
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, lq = lane & 31;
    const int qg = wv % NP;
    auto run = [&](auto role_c) __attribute__((always_inline)) {
        constexpr int role = decltype(role_c)::value;
        const int qw0 = q0 + 32 * qg, t = qw0 + lq, tc = min(t, N - 1);
        const size_t ho = (size_t)bh * N * D, kvo = (size_t)kv_head_of(bh, H, G) * N * D;
        const float *Kh = K + kvo, *Vh = V + kvo, *ch = c + (size_t)bh * N;

        int first_key = max(0, q0 - w + 1);
        if (LOOK && reach_pays(ch[q0] - ch[first_key], q0 - first_key, kFewBackward)) {  // the keys that the gate has erased for all queries stay out
            const float* at = reach + (size_t)bh * N;
            first_key = max(first_key, 64 * first_needed_block(at, ch, first_key / 64, q0 / 64, (min(N, q0 + 32 * NP) - 1) / 64, N, ch[q0], scale * kLog2e, lane));
        }
        const int jb_lo = first_key / 32, jb_hi = (min(N, q0 + 32 * NP) - 1) / 32;
        using Mover = F32TileMover<D, 128 * NP>;
        Mover mv;
        mv.init(tid);
        f32x4 kreg[Mover::kPieces], vreg[Mover::kPieces];
        float creg = 0.f;
        auto fetch = [&](int jb, int part = 0, int n = 1) __attribute__((always_inline)) {
            mv.fetch(kreg, Kh, 32 * jb, N, part, n);
            mv.fetch(vreg, Vh, 32 * jb, N, part, n);
            if (part == 0 && tid < 32) creg = ch[min(32 * jb + tid, N - 1)];
        };
        int buf = 0, a_slot = 0;  // of the current tile
        auto stash_share = [&](int i, int n) __attribute__((always_inline)) {  // into the next one's
            mv.stash(kreg, sm.a[next3(a_slot)], i, n);
            mv.stash(vreg, sm.b[buf ^ 1], i, n);
        };
        fetch(jb_lo);
        bf16x8 rf[KC][3];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) split_row((role == 0 ? Q : dO) + ho + (size_t)tc * D + 16 * kc + 8 * h, rf[kc]);
        __builtin_amdgcn_sched_barrier(0);
        const float ct = ch[tc], Lt = L[(size_t)bh * N + tc], Dt = Dv[(size_t)bh * N + tc];
        f32x16 acc[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;
        float rs = 0.f;
        int r_off = row_frag_off<D>(lane), t_off = col_frag_off<D>(lane) + 16 * role * (D * 2);
        mv.stash(kreg, sm.a[0], 0, 1);
        mv.stash(vreg, sm.b[0], 0, 1);
        if (tid < 32) sm.v[0][0][tid] = creg;
        wg_barrier();
        auto end_step = [&]() __attribute__((always_inline)) {
            buf ^= 1;
            a_slot = next3(a_slot);
            if (tid < 32) sm.v[0][buf][tid] = creg;
            wg_barrier();
        };
        auto idle_step = [&](int jb) __attribute__((always_inline)) {  // no block of this wave's band: only its share of the tile
            fetch(min(jb + 1, jb_hi));
            stash_share(0, 1);
            end_step();
        };
        f32x4 own[2];  // P (wave 0) or dP - D (wave 1) of this wave's half of the block
        auto first_products = [&](int jb) __attribute__((always_inline)) {
            const int kb0 = 32 * jb;
            f32x16 g;
            const unsigned at = (unsigned)(uintptr_t)(role == 0 ? sm.a[a_slot].p[0] : sm.b[buf].p[0]) + r_off;
            f32x16 s = tile_dot<D, false>(
                at, rf, [&](int kc) __attribute__((always_inline)) { stash_share(kc, KC); },
                [&]() __attribute__((always_inline)) {
                    if (role == 0) acc_init_rows(g, sm.v[0][buf], 0, h);
                });
            if (role == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = fast_exp2((fmaf(scale, s[v], g[v] - ct) - Lt) * kLog2e);
                if (__builtin_expect(!(kb0 + 31 <= qw0 && kb0 > qw0 + 31 - w), 0)) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int i = kb0 + acc_row(v, h);
                        s[v] = (i <= t && i > t - w) ? s[v] : 0.f;
                    }
                }
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] -= Dt;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int mine = 8 * role + 4 * i, other = 8 * (1 - role) + 4 * i;
                own[i] = f32x4{s[mine], s[mine + 1], s[mine + 2], s[mine + 3]};
                sm.x[buf][qg][2 * role + i][lane] = f32x4{s[other], s[other + 1], s[other + 2], s[other + 3]};
            }
        };
        auto second_product = [&](int fetched) __attribute__((always_inline)) {  // of the block before the current tile
            const unsigned at = (unsigned)(uintptr_t)sm.a[a_slot == 0 ? 2 : a_slot - 1].p[0] + t_off;
            const ColFrag f = first_col<D, 0>(at);
            float part = 0.f, ds[8];  // (a block's sum by itself first: the suffix sums of the gate gradient add up every rounding)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const f32x4 o = sm.x[buf ^ 1][qg][2 * (1 - role) + i][lane];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    part = fmaf(own[i][j], o[j], part);
                    ds[4 * i + j] = own[i][j] * o[j];
                }
            }
            rs += part;
            bf16x8 sf[3];
            split_frag([&](int j) __attribute__((always_inline)) { return ds[j]; }, sf);
            tile_axpy<D, 0, 1>(at, acc[0], sf, f, acc, [&](int i) __attribute__((always_inline)) { fetch(fetched, i, DB); });  // (one half: its pieces are in sf)
        };
        // (the loop that computes has no branch around the accumulators: with one the compiler copies them)
        const int act_lo = qw0 < N ? max(first_key, qw0 - w + 1) / 32 : jb_hi + 1, act_hi = min(qw0 / 32, jb_hi);
        __builtin_amdgcn_s_setprio(role == 0);  // has the exponentials to do behind its MFMAs
        int jb = jb_lo;
        for (; jb < act_lo; ++jb) idle_step(jb);
        if (jb <= act_hi) {
            fetch(min(jb + 1, jb_hi));
            first_products(jb);
            end_step();
            for (++jb; jb <= act_hi; ++jb) {
                // (the addresses derived from these are recomputed in every block instead of living in registers across the loop)
                GFWA_PIN(r_off);
                GFWA_PIN(t_off);
                second_product(min(jb + 1, jb_hi));
                first_products(jb);
                end_step();
            }
            second_product(min(jb, jb_hi));
        }
        for (; jb <= jb_hi; ++jb) idle_step(jb);
        wg_barrier();
        // wave 1 of a pair hands its sums over, wave 0 adds and stores (the tiles' space is free)
        f32x4* xch = reinterpret_cast<f32x4*>(smem_raw) + qg * (4 * DB + 1) * 64;
        if (role == 1) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    xch[(4 * db + i4) * 64 + lane] = f32x4{acc[db][4 * i4], acc[db][4 * i4 + 1], acc[db][4 * i4 + 2], acc[db][4 * i4 + 3]};
            xch[4 * DB * 64 + lane] = f32x4{rs, 0.f, 0.f, 0.f};
        }
        wg_barrier();
        if (role == 0) {
            rs = xhalf_sum(rs + xch[4 * DB * 64 + lane][0]);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const f32x4 x = xch[(4 * db + i4) * 64 + lane];
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[db][4 * i4 + j] = scale * (acc[db][4 * i4 + j] + x[j]);
                }
            RangeCheck check;
            check.add(acc);
            check.add(rs);
            if (__builtin_expect(check.failed(t < N), 0)) {
                const size_t rows = (size_t)bh * N;
#pragma unroll 1
                for (int row = qw0; row < min(N, qw0 + 32); ++row)
                    dq_row<D, kRowLoads, false>(Q + ho, Kh, Vh, nullptr, dO + ho, ch, L + rows, Dv + rows, dQ + ho, dc_row + rows, row, w, scale,
                                                lane);
            } else if (t < N) {
                float* out = dQ + ho + (size_t)t * D;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4)
                        *reinterpret_cast<f32x4*>(out + 32 * db + 8 * i4 + 4 * h) =
                            f32x4{acc[db][4 * i4], acc[db][4 * i4 + 1], acc[db][4 * i4 + 2], acc[db][4 * i4 + 3]};
                if (h == 0) dc_row[(size_t)bh * N + t] = rs;
            }
        }
    };
    if (wv < NP) run(std::integral_constant<int, 0>{});
    else run(std::integral_constant<int, 1>{});
}

// dK, dV (summed over the G query heads of a group) and, per query head, the column sums of dS (Alg. 3, key loop): a
// workgroup owns 32 NP keys, a pair of waves 32 of them, a lane one key.  S = Q K^T (wave 0) and dP = dO V^T (wave 1) with
// 32-query tiles of Q and dO from LDS, then dV^T += dO^T P (wave 0) and, a block later, dK^T += Q^T dS (wave 1).
template <int D, int NP, bool LOOK>
__device__ __forceinline__ void dkv_f32_mfma(
    int block, const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, const float* __restrict__ dO,
    const float* __restrict__ c, const float* __restrict__ L, const float* __restrict__ Dv, float* __restrict__ dK,
    float* __restrict__ dV, float* __restrict__ dc_col, const float* __restrict__ reach, int N, int w, float scale, int num_ktiles, int total_tiles,
    int H, int G) {
    constexpr int KC = D / 16, DB = D / 32;
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<F32BwdSmem<D, NP>*>(smem_raw);
    const int heads = total_tiles / num_ktiles;
    int bkv, kt;  // flat key/value head; the sequence's end, which few queries see, last
    tile_of_block(block, heads, num_ktiles, true, bkv, kt);
    const int k0 = kt * 32 * NP;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, lk = lane & 31;
    const int kg = wv % NP;
    auto run = [&](auto role_c) __attribute__((always_inline)) {
        constexpr int role = decltype(role_c)::value;
        const int kw0 = k0 + 32 * kg, i = kw0 + lk, ic = min(i, N - 1);
        const int Hkv = H / G;
        const int bh0 = (bkv / Hkv) * H + (bkv % Hkv) * G;  // first query head of the group
        const size_t kvo = (size_t)bkv * N * D;

        // query blocks that see a key of the tile: rows k0 .. k0 + 32 NP - 1 + w - 1, of every query head of the group in turn
        const int qb_lo = k0 / 32;
        const int t_hi = (int)min((long)N - 1, (long)k0 + 32 * NP - 1 + w - 1);
        auto blocks_of = [&](int g) __attribute__((always_inline)) {  // of query head g, without those that the gate has erased all keys for
            int qb_hi = t_hi / 32;
            const size_t rows = (size_t)(bh0 + g) * N;
            const float* ch = c + rows;
            const int k1 = min(k0 + 32 * NP, N) - 1, i_min = k1 / 64;
            if (LOOK && t_hi / 64 > i_min && reach_pays(ch[t_hi] - ch[k1], t_hi - k1, kFewBackward)) {
                qb_hi = min(qb_hi, 2 * last_needing_block(reach + rows, ch, k0 / 64, i_min, t_hi / 64, N, ch[k0], scale * kLog2e, lane) + 1);
            }
            return __builtin_amdgcn_readfirstlane(qb_hi) - qb_lo + 1;
        };
        int nblk = blocks_of(0);  // of the query head at hand
        using Mover = F32TileMover<D, 128 * NP>;
        Mover mv;
        mv.init(tid);
        f32x4 qreg[Mover::kPieces], greg[Mover::kPieces];
        float creg = 0.f, lreg = 0.f, dreg = 0.f;
        auto fetch = [&](int g, int b, int part, int n) __attribute__((always_inline)) {  // query block b of the group's query head g
            const int first = 32 * (qb_lo + b);
            const size_t rows = (size_t)(bh0 + g) * N;
            mv.fetch(qreg, Q + rows * D, first, N, part, n);
            mv.fetch(greg, dO + rows * D, first, N, part, n);
            if (part == 0 && tid < 32) {
                const unsigned r = (unsigned)min(first + tid, N - 1);
                creg = (c + rows)[r];
                lreg = (L + rows)[r];
                dreg = (Dv + rows)[r];
            }
        };
        auto fetch_next = [&](int g, int b, int part = 0, int n = 1) __attribute__((always_inline)) {  // (behind the last block: that one again)
            const bool same = b + 1 < nblk;
            fetch(same ? g : min(g + 1, G - 1), same ? b + 1 : g + 1 < G ? 0 : b, part, n);
        };
        int buf = 0, a_slot = 0;  // of the current tile
        auto stash_share = [&](int p, int n) __attribute__((always_inline)) {  // into the next one's
            mv.stash(qreg, sm.a[next3(a_slot)], p, n);
            mv.stash(greg, sm.b[buf ^ 1], p, n);
        };
        auto stash_rows = [&]() __attribute__((always_inline)) {
            if (tid < 32) {
                sm.v[0][buf][tid] = creg;
                sm.v[1][buf][tid] = lreg;
                sm.v[2][buf][tid] = dreg;
            }
        };
        fetch(0, 0, 0, 1);
        bf16x8 rf[KC][3];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) split_row((role == 0 ? K : V) + kvo + (size_t)ic * D + 16 * kc + 8 * h, rf[kc]);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 acc[DB];  // dV of the keys (wave 0), dK (wave 1)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;
        int r_off = row_frag_off<D>(lane), t_off = col_frag_off<D>(lane);
        mv.stash(qreg, sm.a[0], 0, 1);
        mv.stash(greg, sm.b[0], 0, 1);
        stash_rows();
        wg_barrier();
        auto end_step = [&]() __attribute__((always_inline)) {
            buf ^= 1;
            a_slot = next3(a_slot);
            stash_rows();
            wg_barrier();
        };
        auto idle_step = [&](int g, int b) __attribute__((always_inline)) {  // a query block that sees none of this pair's keys
            fetch_next(g, b);
            stash_share(0, 1);
            end_step();
        };
        RangeCheck check;
        for (int g = 0; g < G; ++g) {  // query heads
            if (g > 0) nblk = blocks_of(g);
            const int b_lo = kw0 < N ? kg : nblk, b_hi = (int)min((long)nblk - 1, ((long)kw0 + 30 + w) / 32 - qb_lo);
            int b = 0;
            for (; b < b_lo; ++b) idle_step(g, b);
            if constexpr (role == 0) {
                const float ci = c[(size_t)(bh0 + g) * N + ic];
                for (; b <= b_hi; ++b) {
                    // (the addresses derived from these are recomputed in every block instead of living in registers across the loop)
                    GFWA_PIN(r_off);
                    GFWA_PIN(t_off);
                    const int qb0 = 32 * (qb_lo + b);
                    const unsigned gt = (unsigned)(uintptr_t)sm.b[buf].p[0] + t_off;
                    f32x16 x, l;
                    f32x16 s = tile_dot<D, true>(
                        (unsigned)(uintptr_t)sm.a[a_slot].p[0] + r_off, rf,
                        [&](int kc) __attribute__((always_inline)) { fetch_next(g, b, kc, KC); },
                        [&]() __attribute__((always_inline)) { acc_init_rows(x, sm.v[0][buf], 0, h); });
                    acc_init_rows(l, sm.v[1][buf], 0, h);
#pragma unroll
                    for (int v = 0; v < 16; ++v) s[v] = fast_exp2((fmaf(scale, s[v], ci - x[v]) - l[v]) * kLog2e);
                    if (__builtin_expect(!(kw0 + 31 <= qb0 && (long)kw0 > (long)qb0 + 31 - w && qb0 + 31 < N), 0)) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int tq = qb0 + acc_row(v, h);
                            s[v] = (i <= tq && i > tq - w && tq < N) ? s[v] : 0.f;
                        }
                    }
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4)
                        sm.x[buf][kg][i4][lane] = f32x4{s[4 * i4], s[4 * i4 + 1], s[4 * i4 + 2], s[4 * i4 + 3]};
                    const ColFrag f = first_col<D, 0>(gt);
                    bf16x8 xf[3];
                    split_acc(s, 0, xf);
                    tile_axpy<D, 0, 2>(gt, s, xf, f, acc, [&](int p) __attribute__((always_inline)) { stash_share(p, 2 * DB); });
                    end_step();
                }
            } else {
                float colsum = 0.f;
                f32x16 s;  // dP - D of the block
                auto first_product = [&]() __attribute__((always_inline)) {
                    f32x16 x;
                    s = tile_dot<D, true>(
                        (unsigned)(uintptr_t)sm.b[buf].p[0] + r_off, rf,
                        [&](int kc) __attribute__((always_inline)) { stash_share(kc, KC); },
                        [&]() __attribute__((always_inline)) { acc_init_rows(x, sm.v[2][buf], 0, h); });
#pragma unroll
                    for (int v = 0; v < 16; ++v) s[v] -= x[v];
                };
                auto second_product = [&](int cur) __attribute__((always_inline)) {  // of the block before the current tile
                    const unsigned qt = (unsigned)(uintptr_t)sm.a[a_slot == 0 ? 2 : a_slot - 1].p[0] + t_off;
                    const ColFrag f = first_col<D, 0>(qt);
                    float part = 0.f;  // (a block's sum by itself first: the suffix sums of the gate gradient add up every rounding)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const f32x4 p = sm.x[buf ^ 1][kg][i4][lane];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            part = fmaf(p[j], s[4 * i4 + j], part);
                            float ds = s[4 * i4 + j] * p[j];
                            GFWA_PIN(ds);  // formed here, so that P does not stay in registers until the second half is split
                            s[4 * i4 + j] = ds;
                        }
                        GFWA_PIN(part);  // (nor until the sum, which nothing waits for)
                    }
                    colsum += part;
                    __builtin_amdgcn_sched_barrier(0);
                    bf16x8 xf[3];
                    split_acc(s, 0, xf);
                    tile_axpy<D, 0, 2>(qt, s, xf, f, acc, [&](int p) __attribute__((always_inline)) { fetch_next(g, cur, p, 2 * DB); });
                };
                if (b <= b_hi) {
                    fetch_next(g, b);
                    first_product();
                    end_step();
                    for (++b; b <= b_hi; ++b) {
                        GFWA_PIN(r_off);
                        GFWA_PIN(t_off);
                        second_product(b);
                        first_product();
                        end_step();
                    }
                    second_product(min(b, nblk - 1));  // (its tile and its P are still there in the step that follows, whatever that is)
                }
                const float cs_all = xhalf_sum(colsum);
                check.add(cs_all);
                if (i < N && h == 0) dc_col[(size_t)(bh0 + g) * N + i] = cs_all;
            }
            for (; b < nblk; ++b) idle_step(g, b);
        }
        if (role == 1)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[db][v] *= scale;
        check.add(acc);
        const bool failed = check.failed(i < N);
        wg_barrier();  // the tiles and the exchange are read, their space is free
        int* verdict = reinterpret_cast<int*>(smem_raw);  // [pair][role]
        if (lane == 0) verdict[2 * kg + role] = failed;
        wg_barrier();
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(verdict[2 * kg] | verdict[2 * kg + 1]), 0)) {
            // both results of the pair's keys, by the wave that has already stored column sums of them
            f32x4* rows_s = reinterpret_cast<f32x4*>(smem_raw + 1024) + 64 * kg;
            if (role == 1)
#pragma unroll 1
                for (int key = kw0; key < min(N, kw0 + 32); ++key)
                    dkv_row<D, kRowLoads>(Q, K + kvo, V + kvo, dO, c, L, Dv, dK + kvo, dV + kvo, dc_col, rows_s, bh0, G, key, N, w, scale, lane);
        } else if (i < N) {
            float* out = (role == 0 ? dV : dK) + kvo + (size_t)i * D;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    *reinterpret_cast<f32x4*>(out + 32 * db + 8 * i4 + 4 * h) =
                        f32x4{acc[db][4 * i4], acc[db][4 * i4 + 1], acc[db][4 * i4 + 2], acc[db][4 * i4 + 3]};
        }
    };
    if (wv < NP) run(std::integral_constant<int, 0>{});
    else run(std::integral_constant<int, 1>{});
}

// Both passes in one launch, the first dkv_tiles workgroups the dK/dV pass, whose chains are the longer ones with grouped heads:
// the dQ pass fills the CUs that those leave idle, at the end of a large problem or beside all of a small one.  Two launches /
// one, whole backward: B1 H8 N1000 d128 w500 149 / 87 us, B1 H2 N2000 d64 causal 240 / 139, B1 H4 N4000 d128 w1000 250 / 155,
// B2 H8/2 N515 d64 181 / 150, B2 H16 N1000 d128 causal 236 / 176, B2 H16 N4096 d128 w1024 1108 / 1065.
// Both passes deal out their tiles by length, whatever the shape: over 1557 shapes 1.00 to 1.02 of the time of the best order in every
// class of them, one head after another 1.0 to 1.19 (B1 H2 N10498 d128 w1236 326 -> 308).
template <int D, int NP, bool LOOK>
__global__ __launch_bounds__(128 * NP, NP == 4 ? 1 : 2) void bwd_f32_mfma_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, const float* __restrict__ dO,
    const float* __restrict__ c, const float* __restrict__ L, const float* __restrict__ Dv, float* __restrict__ dQ, float* __restrict__ dK,
    float* __restrict__ dV, float* __restrict__ dc_col, float* __restrict__ dc_row, const float* __restrict__ reach, int N, int w, float scale,
    int tiles_per_head, int dkv_tiles, int dq_tiles, int H, int G) {
    const int b = (int)blockIdx.x;
    if (b < dkv_tiles) dkv_f32_mfma<D, NP, LOOK>(b, Q, K, V, dO, c, L, Dv, dK, dV, dc_col, reach, N, w, scale, tiles_per_head, dkv_tiles, H, G);
    else dq_f32_mfma<D, NP, LOOK>(b - dkv_tiles, Q, K, V, dO, c, L, Dv, dQ, dc_row, reach, N, w, scale, tiles_per_head, dq_tiles, H, G);
}

// ---- D_t = <O_t, dO_t>
template <int D>
__global__ __launch_bounds__(256) void rowdot_f32_kernel(const float* __restrict__ O, const float* __restrict__ dO,
                                                         float* __restrict__ Dv, long rows) {
    using Step = RowStep<D, 1>;
    const int lane = threadIdx.x & 63;
    const long row = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * Step::kRows + lane / Step::kLanes;
    if (row - lane / Step::kLanes >= rows) return;  // the whole wave
    const size_t at = (size_t)min(row, rows - 1) * D + 4 * (lane % Step::kLanes);
    Step o;
    o.x[0] = *reinterpret_cast<const f32x4*>(O + at);
    const float d = o.dot(*reinterpret_cast<const f32x4*>(dO + at), 0);
    if (row < rows && lane % Step::kLanes == 0) Dv[row] = d;
}

// The same in front of the matrix-core kernels, with what these ask of a block of 64 rows (band_reach.h): squared norms of Q and K, the lowest
// edge of the queries and the highest gate of the keys, where the gate decays enough that they are asked for.  A value row or a D that
// is not finite keeps its block.  reach: dalpha.
template <int D>
__global__ __launch_bounds__(256, 4) void rowdot_reach_f32_kernel(const float* __restrict__ O, const float* __restrict__ dO,
                                                               const float* __restrict__ Q, const float* __restrict__ K,
                                                               const float* __restrict__ V, const float* __restrict__ c,
                                                               const float* __restrict__ L, float* __restrict__ Dv, float* __restrict__ reach,
                                                               int N, int w, int blocks, int H, int G) {
    using Step = RowStep<D, 1>;
    constexpr int kLanes = Step::kLanes, kRows = 4 * Step::kRows, kPasses = kReachRows / kRows;
    __shared__ BlockValues values;
    const int lane = threadIdx.x & 63, bh = (int)blockIdx.x / blocks, t0 = (int)blockIdx.x % blocks * kReachRows;
    const size_t head = (size_t)bh * N, kv = (size_t)kv_head_of(bh, H, G) * N;
    const int r0 = t0 + threadIdx.x / kLanes, col = 4 * (lane % kLanes);
    auto row_of = [&](int p) { return min(r0 + p * kRows, N - 1); };
    const float* ch = c + head;
    const int far = max(0, t0 - w + 1), end = (int)min((long)N - 1, (long)t0 + kReachRows - 2 + w);
    // (all of them requested before the first is used: a workgroup alone on its CU waits for them one after another otherwise, 13 us)
    Step o[kPasses], go[kPasses];
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        o[p].x[0] = *reinterpret_cast<const f32x4*>(O + (head + row_of(p)) * D + col);
        go[p].x[0] = *reinterpret_cast<const f32x4*>(dO + (head + row_of(p)) * D + col);
    }
    const bool look = reach_pays(ch[t0] - ch[far], t0 - far, kFewBackward) || reach_pays(ch[end] - ch[t0], end - t0, kFewBackward);
    float d[kPasses];
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
        d[p] = o[p].dot(go[p].x[0], 0);
        if (r0 + p * kRows < N && lane % kLanes == 0) Dv[head + row_of(p)] = d[p];
    }
    if (look) {
        auto norm_of = [&](const float* row) {
            Step x;
            x.x[0] = *reinterpret_cast<const f32x4*>(row + col);
            return x.dot(x.x[0], 0);
        };
        BlockValues mine = kNoRows;
#pragma unroll
        for (int p = 0; p < kPasses; ++p) {
            const int row = row_of(p);
            const float v2 = norm_of(V + (kv + row) * D);
            mine.norm = max(mine.norm, finite(d[p]) ? norm_bits(norm_of(Q + (head + row) * D)) : kInfBits);
            mine.edge = min(mine.edge, lowest_order((ch[row] - ch[t0]) + L[head + row]));
            mine.key_norm = max(mine.key_norm, finite(v2) ? norm_bits(norm_of(K + (kv + row) * D)) : kInfBits);
            mine.high = max(mine.high, highest_order(ch[row]));
        }
        gather_block<true>(&values, mine);
    }
    if (threadIdx.x == 0) write_block(reach + head + reach_row(t0 / kReachRows, N), values, look, true);
}

// Bands that workgroups of 64 queries (keys) serve better than larger ones: d = 64, at most 128 long.  A workgroup walks
// band + rows - 1 keys, of which a wave needs band + 31, and the LDS of the small one lets four (backward: two) share a CU.
// (64- / 128- / 256-query workgroups, B1 H64 N4096 w8: forward 64 / 73 / 103 us, backward with 64 / 128: 231 / 294; B4 H16 N2000
// w128: 56 / 57 / 65, 167 / 191; w256: 77 / 78 / 83, 233 / 251; B2 H16 N2000 w512: 63 / 60 / 58, 194 / 187.)
static bool f32_short_band(int N, int d, int w) { return d == 64 && (w < N ? w : N) <= 128; }

// How the matrix-core forward is cut up: 256 queries per workgroup (two waves per SIMD) once that gives every CU one, 128
// before and where a sequence ends within them.  More such sequences than CUs give up the second tile buffer at d = 128, for a
// second workgroup on the CU (512 sequences of 32: 11.8 us, 17.0 with 256-query workgroups; 2048 of 64: 81, 98; 256 of 64: 14.5,
// 13.1).  Between 65 and 128 long bands of d = 64 are one workgroup's (512 sequences of 128: 20.2 us with 64 queries, 19.7).
enum F32Fwd { kF32Fwd64, kF32Fwd128, kF32Fwd128Double, kF32Fwd256Double };  // queries per workgroup, tile buffers
static F32Fwd f32_fwd_shape(long BH, int N, int d, int w) {
    if (f32_short_band(N, d, w) && (w <= 64 || N <= 64 || N > 128)) return kF32Fwd64;
    if (N <= 128) return d == 128 && BH > device_cu_count() ? kF32Fwd128 : kF32Fwd128Double;
    return BH * ((N + 255) / 256) >= device_cu_count() ? kF32Fwd256Double : kF32Fwd128Double;
}

// Which kernels serve a problem.  Forward, by estimates of the two in us, fitted to 166 shapes (1 to 4096 sequences of 1 to 5001, w 1 ..
// 2000; where the choice costs more than 8 % it costs at most 7 us).  A row of the one-wave-per-row kernels takes 0.25 ns and 0.3 ns per step
// of 16 (d = 64) or 8 keys, and the longest row's steps follow one another.  The matrix-core kernels walk a tile's band one 32-row block
// after another, in rounds of as many workgroups as the chip holds.  (Row / matrix-core kernels: 256 rows, w = 64, d = 64: 4.5 / 12 us; 512
// causal rows, 4 heads, d = 128: 48 / 51; 1100 rows, w = 400, 4 heads, d = 128: 68 / 57; 4096 sequences of 16, d = 64: 34 / 25; 2048 of 8, d = 128:
// 10 / 33; 2048 of 64, d = 128: 299 / 81.)
// Backward, a line on the safe side of the row kernels, whose gate gradient is the more exact one: they form the same dS in both passes
// and add it up in fp64 (against fp64, error over norm, 26 shapes of 60 to 1100 rows: dQ, dK, dV 1.3e-7 to 3.2e-7 with either, d(alpha) 2.7e-7
// to 1.9e-6 and 4.2e-7 to 2.5e-6, 1.1 to 3.9 times as much with the matrix cores at 25 of them).  The terms are those of the two passes one
// after another, the key side walking the G query heads in turn.  Over 10315 shapes (1 to 64 sequences of 1 to 16384, 1 to 8 query heads on a
// key/value head), one launch for both passes, the row kernels serve 6344, and are slower by more than a tenth at 185 of those (up to
// 1.56: B3 H1 N885 d64 97 / 69 us, B3 H14 N89 d128 36 / 26); of the others the matrix-core kernels are slower by more than 8 % at 52 (up to 1.28:
// B9 H18/3 N134 d64 w36 49 / 62).
static bool f32_use_mfma(bool backward, int B, int H, int Hkv, int N, int d, int w) {
    const double cus = device_cu_count(), BH = (double)B * H, wc = w < N ? w : N, G = H / Hkv, wide = d / 64.0;
    const double step = kRowLoads * 256.0 / d, longest = ceil(wc / step), rows = BH * N * 1e-3;
    const double steps = (wc - wc * (wc - 1.0) / (2.0 * N)) / step;  // of a row, on average, before they are rounded up
    if (!backward) {
        const F32Fwd shape = f32_fwd_shape((long)B * H, N, d, w);
        const int q = shape == kF32Fwd64 ? 64 : shape == kF32Fwd256Double ? 256 : 128;
        const double blocks = ceil(fmin((double)N, wc + q - 1.0) / 32.0);
        double per_cu = BH * ((N + q - 1) / q) / cus;
        if (q == 256) per_cu = ceil(per_cu);  // one workgroup on a CU at a time
        return 2.5 + 2.0 * wide + blocks * fmax(d == 128 ? 2.75 : 1.5, (d == 128 ? 4.5 : q == 64 ? 1.3 : q == 128 ? 1.8 : 2.5) * per_cu) <
               3.0 + rows * (0.25 + 0.3 * fmax(1.0, steps + 0.5)) + 0.36 * longest;
    }
    const int k = f32_short_band(N, d, w) ? 64 : 128;
    const double tiles = (N + k - 1) / k, slots = cus * (k == 64 ? 2 : 1), blocks = ceil(fmin((double)N, wc + k - 1.0) / 32.0);
    const double fixed = 4.0 * wide, block = d == 128 ? 1.6 : 1.0;
    return 7.0 + ceil(BH * tiles / slots) * (fixed + 1.7 * block * blocks) + ceil(BH / G * tiles / slots) * (fixed + 2.0 * G * block * blocks) <
           8.0 + rows * (0.5 + 0.66 * fmin(longest, steps + 1.0)) + (0.35 + 0.5 * G) * (d == 128 ? 1.3 : 1.0) * longest;
}

template <int D, int NW, int S>
static hipError_t launch_fwd_f32_mfma(const float* Q, const float* K, const float* V, const float* c, float* O, float* L, int B,
                                      int H, int Hkv, int N, int w, float scale, hipStream_t s) {
    constexpr size_t lds = sizeof(F32FwdSmem<D, S>);
    const int nq = (N + 32 * NW - 1) / (32 * NW), total = B * H * nq;
    KeyReach reach = {0, 0};
    if constexpr (S == 2)  // (short sequences and bands never look)
        if (hipError_t e = key_reach(reach, 32 * NW, false, Q, K, V, c, O, B, H, Hkv, N, D, w, scale, s)) return e;
    auto with = [&](auto look) -> hipError_t {
        constexpr auto kernel = fwd_f32_mfma_kernel<D, NW, S, decltype(look)::value>;
        static DeviceOnce lds_allowed;
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, lds_allowed)) return e;
        hipLaunchKernelGGL(kernel, dim3(total), dim3(64 * NW), lds, s, Q, K, V, c, O, L, N, w, scale, nq, total, H, H / Hkv, reach);
        return hipGetLastError();
    };
    if constexpr (S == 2)
        if (reach.block != 0) return with(std::true_type{});
    return with(std::false_type{});
}

template <int D, int LOADS>
static void launch_fwd_f32_rows(const float* Q, const float* K, const float* V, const float* c, float* O, float* L, int B, int H, int Hkv,
                                int N, int w, float scale, hipStream_t s) {
    hipLaunchKernelGGL((fwd_f32_kernel<D, LOADS>), dim3(B * H * ((N + kF32Waves - 1) / kF32Waves)), dim3(64 * kF32Waves), 0, s, Q, K, V, c, O,
                       L, N, w, scale, H, H / Hkv);
}

template <int D>
static hipError_t launch_fwd_f32(const float* Q, const float* K, const float* V, const float* c, float* O, float* L, int B, int H, int Hkv,
                                 int N, int w, float scale, hipStream_t s) {
    if (!f32_use_mfma(false, B, H, Hkv, N, D, w)) {
        if ((long)B * H * N <= 4L * device_cu_count()) launch_fwd_f32_rows<D, kRowLoadsAlone>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        else launch_fwd_f32_rows<D, kRowLoads>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        return hipGetLastError();
    }
    switch (f32_fwd_shape(B * H, N, D, w)) {
        case kF32Fwd64:
            if constexpr (D == 64) return launch_fwd_f32_mfma<D, 2, 1>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
            [[fallthrough]];
        case kF32Fwd128: return launch_fwd_f32_mfma<D, 4, 1>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        case kF32Fwd128Double: return launch_fwd_f32_mfma<D, 4, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        default: return launch_fwd_f32_mfma<D, 8, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    }
}

hipError_t forward_f32(const float* Q, const float* K, const float* V, const float* c, float* O, float* L,
                       int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s) {
    ProfScope prof(kKernForward, s);
    return d == 128 ? launch_fwd_f32<128>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s)
                    : launch_fwd_f32<64>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
}

template <int D>
static void launch_rowdot_f32(const float* O, const float* dO, float* Dv, long rows, hipStream_t s) {
    constexpr int kRows = 4 * RowStep<D, 1>::kRows;
    hipLaunchKernelGGL((rowdot_f32_kernel<D>), dim3((unsigned)((rows + kRows - 1) / kRows)), dim3(256), 0, s, O, dO, Dv, rows);
}

// One launch(key_blocks, blocks) for both passes of the backward, or one for each where a grid with all blocks would hold the 2^32
// work items at which a launch is refused (MHA, 2^23 sequences of up to four tokens).
template <class Launch>
static void launch_passes(long key_blocks, long query_blocks, int threads, Launch launch) {
    if ((key_blocks + query_blocks) * threads < 1L << 32) return launch((int)key_blocks, (int)(key_blocks + query_blocks));
    launch((int)key_blocks, (int)key_blocks);
    launch(0, (int)query_blocks);
}

// One launch for both passes of the row kernels, unless the chip is full anyway and a row is one step (d = 128, 8 keys): then the
// row-dot launch's second reading of dO and the registers of the longer pass, which the query rows take too, are all that is left of
// it.  Two launches / one, us: B48 H24/6 N695 w5 939 / 1051, B57 H6 N1480 w7 796 / 853, B15 H6 N739 w4 91 / 95; 16384 rows of
// w <= 8 equal, of grouped heads 1.02 (H32/8 N686 w7 38 / 35); with windows of 9 to 32 one launch is up to 1.2 times as fast at every size, at d = 64 always.
static bool f32_rows_in_two_launches(long rows, int N, int w) { return (w < N ? w : N) <= 8 && rows > 32768; }

template <int D>
static hipError_t launch_bwd_f32_rows(const float* Q, const float* K, const float* V, const float* O, const float* dO, const float* c,
                                      const float* L, float* Dv, float* dQ, float* dK, float* dV, float* dc_col, float* dc_row, int B,
                                      int H, int Hkv, int N, int w, float scale, hipStream_t s) {
    const int per_head = (N + kF32Waves - 1) / kF32Waves;
    auto launch = [&](auto kernel, int key_blocks, int blocks) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * kF32Waves), 0, s, Q, K, V, O, dO, c, L, Dv, dQ, dK, dV, dc_col, dc_row, N, w, scale,
                           key_blocks, H, H / Hkv);
    };
    if constexpr (D == 128)
        if (f32_rows_in_two_launches((long)B * H * N, N, w)) {
            {
                ProfScope prof(kKernDq, s);
                launch(bwd_f32_kernel<D, kF32Queries>, 0, B * H * per_head);
            }
            ProfScope prof(kKernDkv, s);
            launch(bwd_f32_kernel<D, kF32Keys>, 0, B * Hkv * per_head);
            return hipGetLastError();
        }
    ProfScope prof(kKernDkv, s);  // one record for the two launches
    launch_rowdot_f32<D>(O, dO, Dv, (long)B * H * N, s);
    launch_passes((long)B * Hkv * per_head, (long)B * H * per_head, 64 * kF32Waves,
                  [&](int key_blocks, int blocks) { launch(bwd_f32_kernel<D, kF32Both>, key_blocks, blocks); });
    return hipGetLastError();
}

template <int D, int NP>
static hipError_t launch_bwd_f32_mfma(const float* Q, const float* K, const float* V, const float* O, const float* dO, const float* c,
                                      const float* L, float* Dv, float* dQ, float* dK, float* dV, float* dc_col, float* dc_row, float* reach,
                                      int B, int H, int Hkv, int N, int w, float scale, hipStream_t s) {
    constexpr size_t lds = sizeof(F32BwdSmem<D, NP>);
    const int nt = (N + 32 * NP - 1) / (32 * NP);
    reach = NP == 4 ? backward_reach(reach, Q, K, V, O, dO, c, L, sizeof(float), B, H, Hkv, N, D, w, scale) : nullptr;  // (64-row tiles are for short bands)
    {
        ProfScope prof(kKernRowDot, s);
        const int blocks = (N + kReachRows - 1) / kReachRows;
        if (reach == nullptr) launch_rowdot_f32<D>(O, dO, Dv, (long)B * H * N, s);
        else
            hipLaunchKernelGGL((rowdot_reach_f32_kernel<D>), dim3((unsigned)(B * H) * blocks), dim3(256), 0, s, O, dO, Q, K, V, c, L, Dv, reach, N, w,
                               blocks, H, H / Hkv);
    }
    auto with = [&](auto look) -> hipError_t {
        constexpr auto kernel = bwd_f32_mfma_kernel<D, NP, decltype(look)::value>;
        static DeviceOnce lds_allowed;
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, lds_allowed)) return e;
        ProfScope prof(kKernDkv, s);
        launch_passes((long)B * Hkv * nt, (long)B * H * nt, 128 * NP, [&](int dkv_tiles, int blocks) {
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(128 * NP), lds, s, Q, K, V, dO, c, L, Dv, dQ, dK, dV, dc_col, dc_row, reach, N, w, scale, nt,
                               dkv_tiles, blocks - dkv_tiles, H, H / Hkv);
        });
        return hipGetLastError();
    };
    if constexpr (NP == 4)
        if (reach != nullptr) return with(std::true_type{});
    return with(std::false_type{});
}

template <int D>
static hipError_t launch_bwd_f32(const float* Q, const float* K, const float* V, const float* O, const float* dO, const float* c,
                                 const float* L, float* Dv, float* dQ, float* dK, float* dV, float* dc_col, float* dc_row, float* reach, int B,
                                 int H, int Hkv, int N, int w, float scale, hipStream_t s) {
    if (!f32_use_mfma(true, B, H, Hkv, N, D, w))
        return launch_bwd_f32_rows<D>(Q, K, V, O, dO, c, L, Dv, dQ, dK, dV, dc_col, dc_row, B, H, Hkv, N, w, scale, s);
    auto with = [&](auto launch) { return launch(Q, K, V, O, dO, c, L, Dv, dQ, dK, dV, dc_col, dc_row, reach, B, H, Hkv, N, w, scale, s); };
    if constexpr (D == 64)
        if (f32_short_band(N, D, w)) return with(launch_bwd_f32_mfma<D, 2>);
    return with(launch_bwd_f32_mfma<D, 4>);
}

hipError_t backward_f32(const float* Q, const float* K, const float* V, const float* O, const float* dO,
                        const float* c, const float* L, float* dQ, float* dK, float* dV, float* dalpha,
                        float* ws, int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s) {
    const size_t rows = (size_t)B * H * N;
    float* Dv = ws;
    float* dc_col = ws + rows;
    float* dc_row = ws + 2 * rows;
    const hipError_t e = d == 128 ? launch_bwd_f32<128>(Q, K, V, O, dO, c, L, Dv, dQ, dK, dV, dc_col, dc_row, dalpha, B, H, Hkv, N, w, scale, s)
                                  : launch_bwd_f32<64>(Q, K, V, O, dO, c, L, Dv, dQ, dK, dV, dc_col, dc_row, dalpha, B, H, Hkv, N, w, scale, s);
    if (e != hipSuccess) return e;
    // behind the three vectors as the workspace query sizes them (each padded to 256 bytes)
    const size_t one = ((rows * sizeof(float)) + 255) & ~(size_t)255;
    return gate_grad_scan(dc_col, dc_row, dalpha, reinterpret_cast<double*>(reinterpret_cast<char*>(ws) + 3 * one), B * H, N, s);
}

}  // namespace gfwa
