// GatedFWA fused forward for bf16 storage, 64-wide heads (paper Alg. 2).
//
// A workgroup of 4 waves owns 128 consecutive queries of one head, a wave 32 of them; key/value tiles of 64 keys travel
// global -> LDS by direct loads into two ring slots each, from the diagonal backwards.  Products, layouts, gate and
// softmax are those of fwd_bf16.hip (a lane owns one query, S^T = K Q^T starts from the gate, O^T += V^T P^T takes the S
// accumulators as its operand, deferred running maximum); what differs is where the overlap comes from.  At d = 64 a
// 32 x 32 block is 8 MFMAs (256 cycles of the matrix pipe) and about 285 cycles of vector issue, and the two together
// take at least 360 (measured, four waves on a SIMD issuing nothing else).  That is reached by many waves in different
// phases rather than by a pipeline inside one wave: 128 registers, four workgroups on a CU, one step
//   S(upper 32 keys)  ->  S(lower) beside exp(upper)  ->  O += V P(upper) beside exp(lower)  ->  O += V P(lower)
// with nothing carried from step to step but O, m and l, and no code twice (a masked copy of the step makes the
// compiler move the accumulators about).  A step takes 420 cycles per block and SIMD; the pipelined kernel it took over
// from, three waves on a SIMD, 600.
//
// Workgroups are not persistent.  They are dealt out longest band first, over all heads of an XCD at once, so that the
// launch ends with short ones: one head after another, the tail of the launch was a third of it.
// Forward alone, us, before / head after head / as it is:
//   B4 H16    N4096 w512   62.8 / 54.9 / 50.4     B4 H16 N4096  w2000  158 / 130 / 111     B8 H32/8 N1024  w4096  63.5 / 59.5 / 45.1
//   B4 H16/4  N4096 w512   62.3 / 51.3 / 48.3     B2 H16 N8000  w200   45.0 / 39.6 / 36.3  B1 H32   N16384 w1024  196 / 163 / 166
#include <stddef.h>

#include "gfwa_device.h"
#include "gfwa_internal.h"
#include "split_band.h"

namespace gfwa {

namespace {
constexpr int D = 64, kWaves = 4;
constexpr int kRowBytes = D * 2, kTileBytes = kTileRows * kRowBytes;
struct FwdD64Smem {
    alignas(256) char k[2][kTileBytes];
    alignas(256) char v[2][kTileBytes];
    alignas(16) float g[2][kTileRows];  // (c - c_base) / scale of the tile's keys
};
}  // namespace

__global__ __launch_bounds__(64 * kWaves, 4) void fwd_d64_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const float* __restrict__ c, bf16_t* __restrict__ O, float* __restrict__ L, int N, int w, float scale_log2,
    int num_qtiles, int total, int H, int G) {
    constexpr int KC = D / 16, DB = D / 32, NV = 2 * DB;
    constexpr int kChunks = kRowBytes / 16, kPieceRows = 1024 / kRowBytes, kPieces = kTileRows / kWaves / kPieceRows;  // per wave and matrix
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<FwdD64Smem*>(smem_raw);

    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, lq = lane & 31;
    const float sl = scale_log2, inv_scale = kLog2e / scale_log2;
    // Longest bands (the end of the sequence) first.  Heads that do not divide by the XCDs: B1 H12 N8192 w1024 37.6 us tile
    // after tile, 35.5 in contiguous ranges; B3 H11 N4096 causal 105 and 107 us.
    const int heads = total / num_qtiles;
    int bh, qt;
    tile_of_block(heads, num_qtiles, heads % 8 == 0 || w >= N, bh, qt);
    const int q0 = (num_qtiles - 1 - qt) * 128;
    const size_t head_off = (size_t)bh * N * D, kv_off = (size_t)kv_head_of(bh, H, G) * N * D;
    const char* Kh = reinterpret_cast<const char*>(K + kv_off);
    const char* Vh = reinterpret_cast<const char*>(V + kv_off);
    const float* ch = c + (size_t)bh * N;
    const int j_lo = max(0, q0 - w + 1) / kTileRows, j_hi = (min(N, q0 + 128) - 1) / kTileRows, ntiles = j_hi - j_lo + 1;
    const int qw0 = q0 + 32 * wv;
    int T_first = ntiles, T_end = ntiles;  // the steps this wave computes in
    if (qw0 < N) {
        T_first = j_hi - min(qw0 + 31, N - 1) / kTileRows;
        T_end = j_hi - max(0, qw0 - w + 1) / kTileRows + 1;
    }

    // Loads, 1 KB a piece: wave wv fills rows 16 wv .. of a tile.  Only the first tile (the last of the sequence it may be)
    // can end behind the sequence, its rows past N read row N-1; the tiles behind it, and tile 0, which stands in for those
    // past the band's end, lie inside (N >= 64).
    const int ld_row = lane / kChunks;
    unsigned ld_off[2];  // even and odd pieces differ in the swizzle
#pragma unroll
    for (int g = 0; g < 2; ++g) ld_off[g] = (unsigned)tile_off<D>(ld_row, lane % kChunks ^ g);
    static_assert(kPieceRows == 8, "row bit 3 is the swizzle's lowest chunk bit");
    auto piece = [&](const char* M, char* tile, int j, int g) __attribute__((always_inline)) {
        const int at = (16 * wv + kPieceRows * g) * kRowBytes;
        dma16(M + (size_t)j * kTileBytes + at, ld_off[g & 1], tile + at);
    };
#pragma unroll
    for (int g = 0; g < kPieces; ++g) {
        const int r = 16 * wv + kPieceRows * g;
        const unsigned o = (unsigned)min(j_hi * kTileRows + r + ld_row, N - 1) * (unsigned)kRowBytes + (ld_off[g & 1] - (unsigned)(ld_row * kRowBytes));
        dma16(Kh, o, sm.k[0] + r * kRowBytes);
        dma16(Vh, o, sm.v[0] + r * kRowBytes);
    }
    float c_next = ch[min(j_hi * kTileRows + lane, N - 1)];
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
    unsigned ka, va, ga;  // LDS addresses of the lane's first fragments in the current slot
    {
        const unsigned base = (unsigned)(uintptr_t)smem_raw;  // 0: the kernel has no other LDS, so a slot is one address bit
        ka = base + offsetof(FwdD64Smem, k) + row_frag_off<D>(lane);
        va = base + offsetof(FwdD64Smem, v) + col_frag_off<D>(lane);
        ga = base + offsetof(FwdD64Smem, g) + 16 * h;
    }
    static_assert(offsetof(FwdD64Smem, k) % (2 * kTileBytes) == 0 && offsetof(FwdD64Smem, v) % (2 * kTileBytes) == 0 &&
                      offsetof(FwdD64Smem, g) % (8 * kTileRows) == 0, "the two slots of a ring differ in one address bit");
    auto flip = [&]() __attribute__((always_inline)) {  // to the other ring slot
        ka ^= kTileBytes;
        va ^= kTileBytes;
        ga ^= kTileRows * 4;
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
        sm.g[(T + 1) & 1][lane] = (c_next - cbase) * inv_scale;
        wg_barrier();
    };
    auto next_gate = [&](int T) __attribute__((always_inline)) { c_next = ch[max(j_hi - T - 1, 0) * kTileRows + lane]; };
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
        const int kt0 = (j_hi - T) * kTileRows;
        next_gate(T);
        f32x16 s[2];
        u32x4 p[2][2];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const f32x4 x = *(__attribute__((address_space(3))) const f32x4*)(uintptr_t)(ga + 32 * b * 4 + 32 * r);
#pragma unroll
                for (int e = 0; e < 4; ++e) s[b][4 * r + e] = x[e];
            }
        if (__builtin_expect(!(kt0 + 63 <= qw0 && kt0 > qw0 + 31 - w), 0)) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = kt0 + 32 * b + acc_row(v, h);
                    s[b][v] = (i <= t && i > t - w) ? s[b][v] : -INFINITY;
                }
        }
        bf16x8 kf[2][KC], vf[NV];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kf[1][kc] = row_frag<D>(ka, 32, kc);
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) s[1] = mfma32(kf[1][kc], qf[kc], s[1]);
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) kf[0][kc] = row_frag<D>(ka, 0, kc);
        float pa = 0.f, pc = 0.f;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            s[0] = mfma32(kf[0][kc], qf[kc], s[0]);
            expo_pair(s[1], p[1], 2 * kc, -m * sl, pa, pc);
            expo_pair(s[1], p[1], 2 * kc + 1, -m * sl, pa, pc);
        }
        issue(T + 1);
        float sum = pa + pc;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(sum <= kBig)) != 0, 0)) sum = raise(s[1], p[1]);
        l += sum;
        pa = pc = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            vf[i] = col_frag<D>(va, 32 + 16 * (i / DB), i % DB);
            o[i % DB] = mfma32(vf[i], __builtin_bit_cast(bf16x8, p[1][i / DB]), o[i % DB]);
            expo_pair(s[0], p[0], 2 * i, -m * sl, pa, pc);
            expo_pair(s[0], p[0], 2 * i + 1, -m * sl, pa, pc);
        }
        sum = pa + pc;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(sum <= kBig)) != 0, 0)) sum = raise(s[0], p[0]);
        l += sum;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            vf[i] = col_frag<D>(va, 16 * (i / DB), i % DB);
            o[i % DB] = mfma32(vf[i], __builtin_bit_cast(bf16x8, p[0][i / DB]), o[i % DB]);
        }
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
        store_acc_rows<DB>(o, 1.0f / lt, sm.k[0] + 4096 * wv, O + head_off + (size_t)qw0 * D, N - qw0, lane);
    }
}

hipError_t forward_d64_bf16(const void* Q, const void* K, const void* V, const float* c, void* O, float* L, int B, int H,
                             int Hkv, int N, int w, float scale, hipStream_t s) {
    const int nq = (N + 127) / 128, total = B * H * nq;
    ProfScope prof(kKernForward, s);
    hipLaunchKernelGGL(fwd_d64_bf16_kernel, dim3(total), dim3(64 * kWaves), sizeof(FwdD64Smem), s, (const bf16_t*)Q,
                       (const bf16_t*)K, (const bf16_t*)V, c, (bf16_t*)O, L, N, w, scale * kLog2e, nq, total, H, H / Hkv);
    return hipGetLastError();
}

}  // namespace gfwa
