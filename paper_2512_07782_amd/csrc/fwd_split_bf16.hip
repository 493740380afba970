// GatedFWA fused forward for bf16 storage, for problems with too few query tiles to fill the chip (paper Alg. 2).
//
// The persistent kernel of fwd_bf16.hip gives 128 queries to a workgroup of 4 waves and walks their band one key
// tile after another: with few query tiles, or tiles of very different bands, most SIMDs hold one wave or none and the
// launch lasts as long as its longest chain of tiles.  Here a workgroup of NW waves owns QW blocks of 32 queries, and
// KW = NW / QW groups of QW waves take every KW-th key tile (KB blocks of 32 keys) of the band each; the partial
// (reference exponent, sum, output) of the groups are merged through LDS at the end.  The band then takes 1 / KW
// of the steps, at the price of K and V travelling to LDS once per 32 QW queries and of the merge (about 1.5 us).
// What bounds it at these sizes is latency: launch, first loads, the first pass through the code (instruction
// cache), then about 0.8 us per step.  Three shapes (which one: fwd_split_shape in fwd_bf16.hip), forward alone, us:
//                                       persistent   wide (8 waves, 4x2)   mid (4 waves, 2x2)   narrow (4 waves, 1x4)
//   B1 H32/8 N700  d128 w1024              17.5            16.1                 14.4                 16.8
//   B1 H4    N1000 d128 w333               16.1            14.2                 10.4                  7.5
//   B2 H8/2  N515  d64  w512               11.7             9.9                  8.6                  6.6
//   B1 H8    N5003 d128 w3000              63.2            51.5                 56.7                 69.8
//   B1 H16   N5003 d128 w3000             136.6           100.1                104.7                134.9
//   B1 H4    N16384 d128 w1024             42.2            52.6                 52.0                 66.9
//
// Products, layouts, gate and softmax are those of fwd_bf16.hip (a lane owns one query, S^T = K Q^T starts from the
// gate, O^T += V^T P^T takes the S accumulators as its operand, deferred running maximum), without the
// software pipeline inside the wave.  Steps outside a wave's own band only load, so that the loop that computes has no
// branch around the accumulators (with one the compiler copies all of them twice per step).
#include "gfwa_device.h"
#include "gfwa_internal.h"
#include "tile_stage.h"

namespace gfwa {

template <int D, int NW, int QW, int KB, int RING>
struct FwdSplitSmem {
    static constexpr int KW = NW / QW;
    union {
        struct {
            alignas(16) char k[KW][RING][32 * KB * D * 2];  // KB 32-key blocks per group and ring slot
            alignas(16) char v[KW][RING][32 * KB * D * 2];
        } t;
        f32x4 xch[NW][D / 8][64];                // merge: accumulators, [wave][register group][lane]
        alignas(16) char out[32 * QW * (D * 2 + 16)];     // then the finished rows on their way to memory
    };
    float m[NW][64], l[NW][64];
    alignas(16) float g[NW][2][32 * KB];  // (c - c_base) / scale of the keys of a wave's blocks
};

template <int D, int NW, int QW, int KB, int RING>
__global__ __launch_bounds__(64 * NW, D == 64 ? (NW == 4 ? 3 : 2) : 2) void fwd_split_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const float* __restrict__ c, bf16_t* __restrict__ O, float* __restrict__ L, int N, int w, float scale_log2,
    int num_qtiles, int BH, int H, int G) {
    static_assert(RING > 1 || QW == 1, "a slot that other waves read is refilled behind a barrier");
    constexpr int KW = NW / QW;
    constexpr int KC = D / 16, DB = D / 32;
    using Smem = FwdSplitSmem<D, NW, QW, KB, RING>;
    extern __shared__ __align__(256) char smem_raw[];  // tiles start at multiples of 256 bytes (see k_off)
    Smem& sm = *reinterpret_cast<Smem*>(smem_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = wv % QW, kg = wv / QW;
    const int h = lane >> 5, lq = lane & 31;
    const float sl = scale_log2, inv_scale = kLog2e / scale_log2;

    // longest bands first (they start at the end of the sequence); the heads of one XCD stay on it when 8 divides BH
    const int bh = (int)(blockIdx.x % BH);
    const int q0 = (num_qtiles - 1 - (int)(blockIdx.x / BH)) * 32 * QW;
    const size_t head_off = (size_t)bh * N * D;
    const size_t kv_off = (size_t)kv_head_of(bh, H, G) * N * D;
    const char* Kh = reinterpret_cast<const char*>(K + kv_off);
    const char* Vh = reinterpret_cast<const char*>(V + kv_off);
    const float* ch = c + (size_t)bh * N;
    const int qw0 = q0 + 32 * qi, t = qw0 + lq;

    // key tiles of KB 32-key blocks that meet the band, in visiting order kt_hi, kt_hi - 1, ..; group kg takes numbers
    // kg, kg + KW, ..
    constexpr int kKeys = 32 * KB;
    const int kt_hi = (min(N, q0 + 32 * QW) - 1) / kKeys, kt_lo = max(0, q0 - w + 1) / kKeys;
    const int ntile = kt_hi - kt_lo + 1;
    const int mine = ntile > kg ? (ntile - kg + KW - 1) / KW : 0;  // steps of this group
    const int steps = (ntile + KW - 1) / KW;                       // steps of the workgroup

    // a group's tile travels global -> LDS by 1 KB loads, shared out over its QW waves
    constexpr int kRowBytes = D * 2, kCpr = kRowBytes / 16, kRowsPerLoad = 1024 / kRowBytes;
    constexpr int kLoads = kKeys / kRowsPerLoad / QW;  // per wave and matrix
    constexpr int kPieces = 2 * kLoads;
    const int ld_row = lane / kCpr, ld_chunk = swz_chunk<D>(ld_row, lane % kCpr) * 16;
    auto issue_piece = [&](int s, int slot, int i) __attribute__((always_inline)) {  // even i: keys, odd i: values
        const int k0 = (kt_hi - (s * KW + kg)) * kKeys, buf = slot % RING;
        const int j = qi * kLoads + i / 2;  // 1 KB piece of the tile: its swizzle is that of piece 0 with j in the low chunk bits
        const unsigned off = (unsigned)min(k0 + j * kRowsPerLoad + ld_row, N - 1) * (unsigned)kRowBytes +
                             (unsigned)(ld_chunk ^ (16 * (j & (D == 128 ? 3 : 1))));
        if (i & 1) dma16(Vh, off, sm.t.v[kg][buf] + j * 1024);
        else dma16(Kh, off, sm.t.k[kg][buf] + j * 1024);
    };
    auto issue = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) issue_piece(s, s, i);
    };
    auto gate_of = [&](int s) __attribute__((always_inline)) {
        return ch[min((kt_hi - (s * KW + kg)) * kKeys + (KB == 1 ? lq : lane), N - 1)];
    };
    float c_next = mine > 0 ? gate_of(0) : 0.f;
#pragma unroll
    for (int s = 0; s < (RING > 1 ? RING - 1 : 1); ++s)
        if (s < mine) issue(s);

    const float cbase = ch[q0];
    const int tc = min(t, N - 1);
    const float cq = ch[tc] - cbase;
    bf16x8 qf[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
        qf[kc] = *reinterpret_cast<const bf16x8*>(Q + head_off + (size_t)tc * D + 8 * h + 16 * kc);

    // byte offsets of this lane's first fragments in a tile; the others differ by an exclusive or of the chunk bits
    // and by multiples of 16 rows (the swizzle's period)
    const int k_off = tile_off<D>(lq, h);
    const int v_off = tile_off<D>(4 * h + ((lane & 15) >> 2), 2 * (lq >> 4) + ((lane & 3) >> 1)) + 8 * (lane & 1);
    auto key_frag = [&](unsigned at, int b, int kc) __attribute__((always_inline)) {
        return *(__attribute__((address_space(3))) const bf16x8*)(uintptr_t)((at ^ (32 * kc)) + 32 * b * kRowBytes);
    };
    auto value_frag = [&](unsigned at, int b, int c2, int db) __attribute__((always_inline)) {
        constexpr int k8 = D == 128 ? 32 : 16;  // what eight rows further on does to the swizzle
        const int rows = (32 * b + 16 * c2) * kRowBytes;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)((at ^ (64 * db)) + rows));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)((at ^ (64 * db) ^ k8) + rows + 8 * kRowBytes));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // used up here, so that the compiler does not wait for these loads (and every later one) inside the loop
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) GFWA_PIN(qf[kc]);

    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    float m = kNegBig, l = 0.f;
    constexpr float kBig = 1.152921504606846976e18f;  // 2^60

    // start of a step: the group's tile of step s has landed, the readers of the slot that is filled next are done
    auto open_step = [&](int s) __attribute__((always_inline)) {
        if (s < mine) sm.g[wv][s & 1][KB == 1 ? lq : lane] = (c_next - cbase) * inv_scale;
        if (RING > 2 && s + 2 < mine) {  // the loads of later steps stay in flight
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((RING - 2) * 2 * kLoads) : "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        if (QW > 1) wg_barrier();
        if (s + 1 < mine) c_next = gate_of(s + 1);
    };
    auto idle_step = [&](int s) __attribute__((always_inline)) {  // no block of this wave's band: only its share of the loads
        open_step(s);
        const int s_next = s + (RING > 1 ? RING - 1 : 1);
        if (s_next < mine) issue(s_next);
    };
    // steps of the group whose tile meets this wave's band: s_first .. s_end - 1
    int s_first = 0, s_end = 0;
    if (qw0 < N) {
        const int n_first = kt_hi - (qw0 + 31) / kKeys, n_last = kt_hi - max(0, qw0 - w + 1) / kKeys;  // tiles, in visiting order
        s_first = n_first > kg ? (n_first - kg + KW - 1) / KW : 0;
        s_end = n_last >= kg ? min(mine, (n_last - kg) / KW + 1) : 0;
    }
    int s = 0;
    for (; s < min(s_first, steps); ++s) idle_step(s);
    for (; s < s_end; ++s) {
        open_step(s);
        const int buf = s % RING;
        // the step whose tile is requested now; past the end its last one again, into a slot that nothing reads any more
        const int s_next = min(s + RING - 1, mine - 1);
        const int k0 = (kt_hi - (s * KW + kg)) * kKeys;
        {
            const unsigned kt = (unsigned)(uintptr_t)sm.t.k[kg][buf] + k_off;
            const unsigned vt = (unsigned)(uintptr_t)sm.t.v[kg][buf] + v_off;
            const bool cut = !(k0 + kKeys - 1 <= qw0 && k0 > qw0 + 31 - w);  // the diagonal or the window edge cuts the tile
            f32x16 sc[KB];
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                acc_init_rows(sc[b], sm.g[wv][s & 1], 32 * b, h);
                if (__builtin_expect(cut, 0)) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int i = k0 + 32 * b + acc_row(v, h);
                        sc[b][v] = (i <= t && i > t - w) ? sc[b][v] : -INFINITY;
                    }
                }
                bf16x8 kf[KC];  // all reads ahead of the products: a lone read's latency is four MFMAs
#pragma unroll
                for (int kc = 0; kc < KC; ++kc) kf[kc] = key_frag(kt, b, kc);
                __builtin_amdgcn_sched_barrier(0);
                // the loads of a later step go out one by one between the products: issued in a row they would hold the
                // wave up for as long as the load unit takes to work them off
#pragma unroll
                for (int kc = 0; kc < KC; ++kc) {
                    sc[b] = mfma32(kf[kc], qf[kc], sc[b]);
                    if (RING > 1) {
#pragma unroll
                        for (int i = kPieces * (KC * b + kc) / (KC * KB); i < kPieces * (KC * b + kc + 1) / (KC * KB); ++i)
                            issue_piece(s_next, s + RING - 1, i);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            bf16x8 vf[KB][2 * DB];  // in flight during the softmax
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int i = 0; i < 2 * DB; ++i) vf[b][i] = value_frag(vt, b, i / DB, i % DB);
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
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(psum <= kBig)) != 0, 0)) {  // first tile of a lane, or a score far above the reference
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
                    for (int db = 0; db < DB; ++db)
                        o[db] = mfma32(vf[b][c2 * DB + db], pf[c2], o[db]);
            }
        }
        if (RING == 1 && s + 1 < mine) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave's reads of the slot are done
            issue(s + 1);
        }
    }

    for (; s < steps; ++s) idle_step(s);

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // a tile requested in vain has landed too
    // ---- merge of the KW groups: every wave hands its accumulators over and takes 1 / KW of its queries' columns
    __syncthreads();
    sm.m[wv][lane] = m;
    sm.l[wv][lane] = l;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            sm.xch[wv][4 * db + r][lane] = f32x4{o[db][4 * r], o[db][4 * r + 1], o[db][4 * r + 2], o[db][4 * r + 3]};
    __syncthreads();
    float mm = kNegBig, lt = 0.f, f[KW];
#pragma unroll
    for (int k = 0; k < KW; ++k) mm = fmaxf(mm, sm.m[k * QW + qi][lane]);
#pragma unroll
    for (int k = 0; k < KW; ++k) {
        f[k] = fast_exp2((sm.m[k * QW + qi][lane] - mm) * sl);
        lt = fmaf(sm.l[k * QW + qi][lane], f[k], lt);
    }
    lt = xhalf_sum(lt);  // the two halves of a wave hold complementary keys
    const float inv = 1.0f / lt;
    constexpr int kOwn = D / 8 / KW;  // register groups (of 4 columns) this wave finishes
    f32x4 own[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        own[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            const f32x4 x = sm.xch[k * QW + qi][kOwn * kg + i][lane];
#pragma unroll
            for (int j = 0; j < 4; ++j) own[i][j] = fmaf(x[j], f[k], own[i][j]);
        }
    }
    if (kg == 0 && h == 0 && t < N) L[(size_t)bh * N + t] = (mm * sl + fast_log2(lt)) * kLn2 - cq;
    __syncthreads();  // the exchange is read; its space takes the rows
    constexpr int kPitch = D * 2 + 16;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const f32x4 x4 = {own[i][0] * inv, own[i][1] * inv, own[i][2] * inv, own[i][3] * inv};
        *reinterpret_cast<bf16x4*>(sm.out + (32 * qi + lq) * kPitch + 16 * (kOwn * kg + i) + 8 * h) =
            __builtin_convertvector(x4, bf16x4);
    }
    __syncthreads();
    bf16_t* Oh = O + head_off + (size_t)q0 * D;
    for (int x = tid; x < 32 * QW * kCpr; x += (64 * NW)) {
        const int row = x / kCpr, cc = x % kCpr;
        if (q0 + row < N)
            *reinterpret_cast<bf16x8*>(Oh + (size_t)row * D + 8 * cc) =
                *reinterpret_cast<const bf16x8*>(sm.out + row * kPitch + 16 * cc);
    }
}

template <int D, int NW, int QW, int KB, int RING>
static hipError_t launch_split(const void* Q, const void* K, const void* V, const float* c, void* O, float* L, int B,
                               int H, int Hkv, int N, int w, float scale, hipStream_t s) {
    using Smem = FwdSplitSmem<D, NW, QW, KB, RING>;
    static DeviceOnce lds_allowed;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&fwd_split_bf16_kernel<D, NW, QW, KB, RING>), sizeof(Smem),
                                         lds_allowed))
        return e;
    const int nq = (N + 32 * QW - 1) / (32 * QW);
    ProfScope prof(kKernForward, s);
    hipLaunchKernelGGL((fwd_split_bf16_kernel<D, NW, QW, KB, RING>), dim3((unsigned)(B * H) * nq), dim3((64 * NW)), sizeof(Smem),
                       s, (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, c, (bf16_t*)O, L, N, w, scale * kLog2e, nq,
                       B * H, H, H / Hkv);
    return hipGetLastError();
}

hipError_t forward_split_bf16(FwdSplit shape, const void* Q, const void* K, const void* V, const float* c, void* O,
                              float* L, int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s) {
    if (d == 128) {
        if (shape == kFwdSplitWide) return launch_split<128, 8, 4, 2, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        if (shape == kFwdSplitMid) return launch_split<128, 4, 2, 1, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
        return launch_split<128, 4, 1, 1, 1>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    }
    if (shape == kFwdSplitWide) return launch_split<64, 8, 4, 2, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    if (shape == kFwdSplitMid) return launch_split<64, 4, 2, 1, 3>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
    return launch_split<64, 4, 1, 1, 2>(Q, K, V, c, O, L, B, H, Hkv, N, w, scale, s);
}

}  // namespace gfwa
