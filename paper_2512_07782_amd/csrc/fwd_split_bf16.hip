// GatedFWA fused forward for bf16 storage, for problems with too few query tiles to fill the chip (paper Alg. 2).
//
// The kernel of fwd_bf16.hip gives 128 queries to a workgroup of 4 waves and walks their band one key
// tile after another: with few query tiles, or tiles of very different bands, most SIMDs hold one wave or none and the
// launch lasts as long as its longest chain of tiles.  Here a workgroup of NW waves owns QW blocks of 32 queries, and
// KW = NW / QW groups of QW waves take every KW-th key tile (KB blocks of 32 keys) of the band each; the partial
// (reference exponent, sum, output) of the groups are merged through LDS at the end.  The band then takes 1 / KW
// of the steps, at the price of K and V travelling to LDS once per 32 QW queries and of the merge (about 1.5 us).
// What bounds it at these sizes is latency: launch, first loads, the first pass through the code (instruction
// cache), then about 0.8 us per step.  Three shapes (which one: fwd_split_shape in fwd_bf16.hip), forward alone, us,
// and beside them a persistent kernel of 128-query tiles, the predecessor of the one in fwd_bf16.hip:
//                                       persistent   wide (8 waves, 4x2)   mid (4 waves, 2x2)   narrow (4 waves, 1x4)
//   B1 H32/8 N700  d128 w1024              17.5            16.1                 14.4                 16.8
//   B1 H4    N1000 d128 w333               16.1            14.2                 10.4                  7.5
//   B2 H8/2  N515  d64  w512               11.7             9.9                  8.6                  6.6
//   B1 H8    N5003 d128 w3000              63.2            51.5                 56.7                 69.8
//   B1 H16   N5003 d128 w3000             136.6           100.1                104.7                134.9
//   B1 H4    N16384 d128 w1024             42.2            52.6                 52.0                 66.9
//
// Products, layouts, gate and softmax are those of fwd_bf16.hip (a lane owns one query, S^T = K Q^T starts from the
// gate, O^T += V^T P^T takes the S accumulators as its operand, deferred running maximum).  Steps outside a wave's own band only load, so that the loop that computes has no
// branch around the accumulators (with one the compiler copies all of them twice per step).
#include "band_reach.h"
#include "gfwa_device.h"
#include "gfwa_internal.h"
#include "split_band.h"

namespace gfwa {

// LOOK: whether reach is there.  (Short problems never have it, and a look that is compiled in costs them: B1 H32/8 N700 d128 w1024, with the gate's
// scan, 19.2 / 19.1 us.)
template <int D, int NW, int QW, int KB, int RING, bool LOOK>
__global__ __launch_bounds__(64 * NW, D == 64 && NW == 4 ? 3 : 2) void fwd_split_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const float* __restrict__ c, bf16_t* __restrict__ O, float* __restrict__ L, int N, int w, float scale_log2,
    int num_qtiles, int BH, int H, int G, KeyReach reach) {
    using Band = SplitBand<D, NW, QW, KB, RING>;
    constexpr int KC = D / 16, DB = D / 32, KW = Band::KW;
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<typename Band::Smem*>(smem_raw);

    const float sl = scale_log2;
    // longest bands first (they start at the end of the sequence); the heads of one XCD stay on it when 8 divides BH
    const int bh = (int)(blockIdx.x % BH);
    const int q0 = (num_qtiles - 1 - (int)(blockIdx.x / BH)) * 32 * QW;
    const size_t head_off = (size_t)bh * N * D, kv_off = (size_t)kv_head_of(bh, H, G) * N * D;
    Band band(sm);
    band.open(K + kv_off, V + kv_off, c + (size_t)bh * N, N, w, q0, kLog2e / scale_log2);
    const int lane = band.lane, h = lane >> 5;
    const int qw0 = q0 + 32 * band.qi, t = qw0 + (lane & 31), tc = min(t, N - 1);
    const float cq = band.ch[tc] - band.cbase;
    bf16x8 qf[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
        qf[kc] = *reinterpret_cast<const bf16x8*>(Q + head_off + (size_t)tc * D + 8 * h + 16 * kc);
    const int k_off = row_frag_off<D>(lane), v_off = col_frag_off<D>(lane);
    // used up here, so that the compiler does not wait for these loads (and every later one) inside the loop
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) GFWA_PIN(qf[kc]);
    const int k_lo = max(0, q0 - w + 1);
    if (LOOK && reach_pays(band.cbase - band.ch[k_lo], q0 - k_lo, reach.few))  // what the gate has erased for all queries stays out
        band.from(forward_reach<D, NW>(qf, K + kv_off + (size_t)tc * D + 8 * h, key_block<D>(O + head_off + (size_t)q0 * D, min(32 * QW, N - q0), lane), cq,
                                       q0, k_lo, reach.block, band.cbase, sl, sm.needed, band.wv, lane),
                  q0, w);

    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    float m = kNegBig, l = 0.f;
    constexpr float kBig = 1.152921504606846976e18f;  // 2^60

    int s = 0;
    for (; s < band.s_first; ++s) band.idle_step(s);
    for (; s < band.s_end; ++s) {
        band.open_step(s);
        const int s_next = band.requested(s), k0 = band.first_key(s);
        const unsigned kt = (unsigned)(uintptr_t)sm.t.k[band.kg][s % RING] + k_off;
        const unsigned vt = (unsigned)(uintptr_t)sm.t.v[band.kg][s % RING] + v_off;
        const bool cut = band.cut(k0, qw0, w);
        f32x16 sc[KB];
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            acc_init_rows(sc[b], sm.g[band.wv][s & 1], 32 * b, h);
            if (__builtin_expect(cut, 0)) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = k0 + 32 * b + acc_row(v, h);
                    sc[b][v] = (i <= t && i > t - w) ? sc[b][v] : -INFINITY;
                }
            }
            bf16x8 kf[KC];  // all reads ahead of the products: a lone read's latency is four MFMAs
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) kf[kc] = row_frag<D>(kt, 32 * b, kc);
            __builtin_amdgcn_sched_barrier(0);
            // the loads of a later step go out one by one between the products
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                sc[b] = mfma32(kf[kc], qf[kc], sc[b]);
                if (RING > 1) {
                    constexpr int P = 2 * Band::kLoads;
#pragma unroll
                    for (int i = P * (KC * b + kc) / (KC * KB); i < P * (KC * b + kc + 1) / (KC * KB); ++i)
                        band.issue_piece(s_next, s + 1, i);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        bf16x8 vf[KB][2 * DB];  // in flight during the softmax
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int i = 0; i < 2 * DB; ++i) vf[b][i] = col_frag<D>(vt, 32 * b + 16 * (i / DB), i % DB);
        __builtin_amdgcn_sched_barrier(0);
        float p[KB][16], psum = 0.f;
        auto expo = [&]() __attribute__((always_inline)) {
            const float nm = -m * sl;
            psum = 0.f;
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    p[b][v] = fast_exp2(fmaf(sc[b][v], sl, nm));
                    psum += p[b][v];
                }
        };
        expo();
        // first tile of a lane, or a score far above the reference
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(psum <= kBig)) != 0, 0)) {
            float mx = -INFINITY;
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sc[b][v]);
            const float mnew = fmaxf(m, xhalf_max(mx));
            const float a = fast_exp2((m - mnew) * sl);
            m = mnew;
            l *= a;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[db][v] *= a;
            expo();
        }
        l += psum;
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            bf16x8 pf[2];
            acc_to_bfrag(p[b], pf);
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int db = 0; db < DB; ++db) o[db] = mfma32(vf[b][c2 * DB + db], pf[c2], o[db]);
        }
        band.close_step(s);
    }
    for (; s < band.steps; ++s) band.idle_step(s);

    band.merge(
        o, m, l,
        [&](const float (&mk)[KW], const float (&lk)[KW], float (&f)[KW]) __attribute__((always_inline)) {
            float mm = kNegBig, lt = 0.f;
#pragma unroll
            for (int k = 0; k < KW; ++k) mm = fmaxf(mm, mk[k]);
#pragma unroll
            for (int k = 0; k < KW; ++k) {
                f[k] = fast_exp2((mk[k] - mm) * sl);
                lt = fmaf(lk[k], f[k], lt);
            }
            lt = xhalf_sum(lt);  // the two halves of a wave hold complementary keys
            if (band.kg == 0 && h == 0 && t < N) L[(size_t)bh * N + t] = (mm * sl + fast_log2(lt)) * kLn2 - cq;
            return 1.0f / lt;
        },
        O + head_off + (size_t)q0 * D, N - q0);
}

template <int D, int NW, int QW, int KB, int RING>
static hipError_t launch_split(const void* Q, const void* K, const void* V, const float* c, void* O, float* L, int B,
                               int H, int Hkv, int N, int w, float scale, hipStream_t s) {
    using Smem = SplitBandSmem<D, NW, QW, KB, RING>;
    const int nq = (N + 32 * QW - 1) / (32 * QW);
    ProfScope prof(kKernForward, s);
    KeyReach reach;
    if (hipError_t e = key_reach(reach, 32 * QW, true, Q, K, V, c, O, B, H, Hkv, N, D, w, scale, s)) return e;
    auto with = [&](auto look) -> hipError_t {
        constexpr auto kernel = fwd_split_bf16_kernel<D, NW, QW, KB, RING, decltype(look)::value>;
        static DeviceOnce lds_allowed;
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), sizeof(Smem), lds_allowed)) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)(B * H) * nq), dim3((64 * NW)), sizeof(Smem), s, (const bf16_t*)Q, (const bf16_t*)K,
                           (const bf16_t*)V, c, (bf16_t*)O, L, N, w, scale * kLog2e, nq, B * H, H, H / Hkv, reach);
        return hipGetLastError();
    };
    return reach.block != 0 ? with(std::true_type{}) : with(std::false_type{});
}

hipError_t forward_split_bf16(FwdSplit shape, const void* Q, const void* K, const void* V, const float* c, void* O,
                              float* L, int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s) {
    if (d == 128) {
        if (shape == kFwdSplitWide) return launch_split<128, 8, 4, 2, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        if (shape == kFwdSplitMid) return launch_split<128, 4, 2, 1, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        return launch_split<128, 4, 1, 1, 1>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    }
    if (shape == kFwdSplitWide) return launch_split<64, 8, 4, 2, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    if (shape == kFwdSplitMid) return launch_split<64, 4, 2, 1, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    return launch_split<64, 4, 1, 1, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
}

}  // namespace gfwa
