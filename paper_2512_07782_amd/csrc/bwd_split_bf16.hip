// GatedFWA backward for bf16 storage, for problems whose 128-query or 128-key tiles are too few or too uneven to
// fill the chip (paper App. E.2 / Alg. 3).  The arithmetic, layouts and roundings are those of bwd_bf16.hip (dS formed
// twice, no stored blocks); what differs is who does it:
//   dQ   a workgroup owns 32 QW queries and splits the key tiles of their band over groups of waves (split_band.h)
//   dKV  a workgroup owns 32 keys; each of its NW waves streams its own share of the 32-query blocks that see them - of
//        all query heads of the group - through LDS of its own, without a barrier, and the NW partial dK, dV are
//        summed through LDS at the end
// Latency bounds these sizes (first loads, first pass through the code, about 1 us per step of a wave), not a rate.
// Where the workgroups of the two passes together are one a CU, or up to about two of long bands, they go in one launch, D_t formed by
// both (bwd_in_one_launch in bwd_bf16.hip has the line and more figures).
// Whole backward, us, with the 128-row kernels / with the kernels here, one launch each (B2 H8/2 N515 d64 in one: 22.2):
//   B2 H8/2 N515 d64 w512   63.4 / 26.6      B2 H8/2 N515 d128 w512   80.7 / 47.9     B1 H4 N1000 d128 w333    39.9 / 24.9
//   B1 H8 N700 d128 w1024   46.9 / 31.7      B1 H4 N5003 d64 w3000   117.6 / 74.2     B1 H16/4 N5003 d64 w3000  323 / 223 (dKV only)
#include "band_reach.h"
#include "gfwa_device.h"
#include "gfwa_internal.h"
#include "split_band.h"

namespace gfwa {

constexpr float kPosBig = 1.0e30f;

// ---- D_t = <O_t, dO_t>, dQ, row sums of dS.  Workgroup `block` of the pass.  LOOK, here and below: a.reach is there.  (Short problems never have it, and a
// look that is compiled in costs them: step B2 H8/2 N515 d64 w512 35.2 / 35.0 us.)
template <int D, int NW, int QW, int KB, int RING, bool LOOK>
__device__ __forceinline__ void dq_split(const BwdBf16& a, int num_qtiles, int block) {
    using Band = SplitBand<D, NW, QW, KB, RING>;
    constexpr int KC = D / 16, DB = D / 32, KW = Band::KW;
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<typename Band::Smem*>(smem_raw);

    const bf16_t *__restrict__ Q = a.Q, *__restrict__ K = a.K, *__restrict__ V = a.V, *__restrict__ O = a.O, *__restrict__ dO = a.dO;
    const float *__restrict__ c = a.c, *__restrict__ L = a.L;
    float *__restrict__ Dv = a.Dv, *__restrict__ dc_row = a.dc_row;
    bf16_t* __restrict__ dQ = a.dQ;
    const int N = a.N, w = a.w, BH = a.B * a.H, H = a.H, G = a.H / a.Hkv;
    const float scale = a.scale, sl = scale * kLog2e;
    const int bh = block % BH;  // longest bands first
    const int q0 = (num_qtiles - 1 - block / BH) * 32 * QW;
    const size_t head_off = (size_t)bh * N * D, kv_off = (size_t)kv_head_of(bh, H, G) * N * D;
    Band band(sm);
    band.open(K + kv_off, V + kv_off, c + (size_t)bh * N, N, w, q0, 1.0f / scale);
    const int lane = band.lane, h = lane >> 5;
    const int qw0 = q0 + 32 * band.qi, t = qw0 + (lane & 31), tc = min(t, N - 1);
    bf16x8 qf[KC], gf[KC];
    float dsum = 0.f;  // this half's part of D_t
    {
        const size_t roff = head_off + (size_t)tc * D + 8 * h;
        bf16x8 of[KC];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            qf[kc] = *reinterpret_cast<const bf16x8*>(Q + roff + 16 * kc);
            gf[kc] = *reinterpret_cast<const bf16x8*>(dO + roff + 16 * kc);
            of[kc] = *reinterpret_cast<const bf16x8*>(O + roff + 16 * kc);
        }
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
#pragma unroll
            for (int e = 0; e < 8; ++e) dsum = fmaf((float)of[kc][e], (float)gf[kc][e], dsum);
    }
    const float dt = xhalf_sum(dsum);
    if (band.kg == 0 && h == 0 && t < N) Dv[(size_t)bh * N + t] = dt;
    int first = max(0, q0 - w + 1);
    if (LOOK && reach_pays(band.cbase - band.ch[first], q0 - first, kFewBackward)) {  // the keys that the gate has erased for all queries stay out
        const float* at = a.reach + (size_t)bh * N;
        first = max(first, 64 * first_needed_block(at, band.ch, first / 64, q0 / 64, (min(N, q0 + 32 * QW) - 1) / 64, N, band.cbase, sl, lane));
        band.from(__builtin_amdgcn_readfirstlane(first), q0, w);
    }
    // rows past N get an exponent of -big, i.e. p = 0
    const float nlsub = t < N ? -(L[(size_t)bh * N + tc] + (band.ch[tc] - band.cbase)) * kLog2e : -kPosBig;
    const int k_off = row_frag_off<D>(lane), v_off = col_frag_off<D>(lane);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {  // no load of these is pending when the loop starts
        GFWA_PIN(qf[kc]);
        GFWA_PIN(gf[kc]);
    }

    f32x16 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;
    float rowsum = 0.f;

    int s = 0;
    for (; s < band.s_first; ++s) band.idle_step(s);
    for (; s < band.s_end; ++s) {
        band.open_step(s);
        const int s_next = band.requested(s), k0 = band.first_key(s);
        const unsigned kt = (unsigned)(uintptr_t)sm.t.k[band.kg][s % RING], vt = (unsigned)(uintptr_t)sm.t.v[band.kg][s % RING];
        const bool cut = band.cut(k0, qw0, w);
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            f32x16 sc, dp;
            acc_init_rows(sc, sm.g[band.wv][s & 1], 32 * b, h);
#pragma unroll
            for (int v = 0; v < 16; ++v) dp[v] = -dt;
            bf16x8 kf[KC], vf[KC];
            auto requests = [&](int i0, int i1) __attribute__((always_inline)) {  // of the loads of a later step
                if (RING > 1)
#pragma unroll
                    for (int i = i0; i < i1; ++i) band.issue_piece(s_next, s + 1, i);
            };
            constexpr int P = 2 * Band::kLoads;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) kf[kc] = row_frag<D>(kt + k_off, 32 * b, kc);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kc = 0; kc < KC / 2; ++kc) vf[kc] = row_frag<D>(vt + k_off, 32 * b, kc);
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                sc = mfma32(kf[kc], qf[kc], sc);
                requests(P * (2 * KC * b + kc) / (2 * KC * KB), P * (2 * KC * b + kc + 1) / (2 * KC * KB));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kc = KC / 2; kc < KC; ++kc) vf[kc] = row_frag<D>(vt + k_off, 32 * b, kc);
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                dp = mfma32(vf[kc], gf[kc], dp);
                requests(P * (2 * KC * b + KC + kc) / (2 * KC * KB), P * (2 * KC * b + KC + kc + 1) / (2 * KC * KB));
            }
            bf16x8 tf[2 * DB];  // K^T, in flight during the exponentials
#pragma unroll
            for (int i = 0; i < 2 * DB; ++i) tf[i] = col_frag<D>(kt + v_off, 32 * b + 16 * (i / DB), i % DB);
            __builtin_amdgcn_sched_barrier(0);
            float p[16], ds[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) p[v] = fast_exp2(fmaf(sc[v], sl, nlsub));
            if (__builtin_expect(cut, 0)) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = k0 + 32 * b + acc_row(v, h);
                    p[v] = (i <= t && i > t - w) ? p[v] : 0.f;
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                ds[v] = p[v] * dp[v];
                rowsum += ds[v];
            }
            bf16x8 dsf[2];
            acc_to_bfrag(ds, dsf);
#pragma unroll
            for (int i = 0; i < 2 * DB; ++i) acc[i % DB] = mfma32(tf[i], dsf[i / DB], acc[i % DB]);
        }
        band.close_step(s);
    }
    for (; s < band.steps; ++s) band.idle_step(s);

    band.merge(
        acc, rowsum, 0.f,
        [&](const float (&rs)[KW], const float (&)[KW], float (&f)[KW]) __attribute__((always_inline)) {
            float all = 0.f;
#pragma unroll
            for (int k = 0; k < KW; ++k) {
                all += rs[k];
                f[k] = 1.f;
            }
            all = xhalf_sum(all);
            if (band.kg == 0 && h == 0 && t < N) dc_row[(size_t)bh * N + t] = all;
            return scale;
        },
        dQ + head_off + (size_t)q0 * D, N - q0);
}

template <int D, int NW, int QW, int KB, int RING, bool LOOK>
__global__ __launch_bounds__(64 * NW, D == 64 && NW == 4 ? 3 : 2) void bwd_dq_split_bf16_kernel(BwdBf16 a, int num_qtiles) {
    dq_split<D, NW, QW, KB, RING, LOOK>(a, num_qtiles, (int)blockIdx.x);
}

// ---- dK, dV (summed over the query heads of a group), column sums of dS per query head.  OWN_D: D_t is formed here too, from
// the rows of O, in the order of additions of dq_split, instead of read.
template <int D, int NW>
struct DkvSplitSmem {
    union {
        struct {
            alignas(256) char q[NW][2][32 * D * 2];  // a wave's own ring of 32-query blocks of Q
            alignas(256) char g[NW][2][32 * D * 2];  // and of dO
        } t;
        f32x4 xch[NW][2 * (D / 8)][64];                   // reduction: dK, then dV accumulators
        alignas(16) char out[2][32 * (D * 2 + 16)];
    };
    alignas(16) float nl[NW][2][32];    // -(L_t + c_t - c_base) / scale of the block's rows; -big past N
    alignas(16) float dvec[NW][2][32];  // -D_t
    float col[NW][kDkvSplitMaxGroup][32];
};

template <int D, int NW, bool OWN_D, bool LOOK>
__device__ __forceinline__ void dkv_split(const BwdBf16& a, int block) {
    constexpr int KC = D / 16, DB = D / 32;
    extern __shared__ __align__(256) char smem_raw[];
    auto& sm = *reinterpret_cast<DkvSplitSmem<D, NW>*>(smem_raw);
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, lk = lane & 31;
    const bf16_t *__restrict__ Q = a.Q, *__restrict__ K = a.K, *__restrict__ V = a.V, *__restrict__ O = a.O, *__restrict__ dO = a.dO;
    const float *__restrict__ c = a.c, *__restrict__ L = a.L, *__restrict__ Dv = a.Dv;
    bf16_t *__restrict__ dK = a.dK, *__restrict__ dV = a.dV;
    float* __restrict__ dc_col = a.dc_col;
    const int N = a.N, w = a.w, BHkv = a.B * a.Hkv, H = a.H, G = a.H / a.Hkv;
    const float scale = a.scale, sl = scale * kLog2e, inv_scale = 1.0f / scale;

    const int bkv = block % BHkv, k0 = block / BHkv * 32;  // whole bands first, the sequence's end last
    const int Hkv = H / G, bh0 = (bkv / Hkv) * H + (bkv % Hkv) * G;
    const size_t kv_off = (size_t)bkv * N * D;
    const int key = k0 + lk, keyc = min(key, N - 1);

    // 32-query blocks that see one of the keys, of every query head of the group in turn; wave wv takes every NW-th
    const int qb_lo = k0 >> 5, t_hi = (int)min((long)N - 1, (long)k0 + 31 + w - 1);
    int nblk = (t_hi >> 5) - qb_lo + 1;
    if constexpr (LOOK) {  // up to the last that one of the heads needs: the gate has erased the keys for those behind it
        const int k1 = min(k0 + 32, N) - 1, i_min = k1 / 64;
        int last = i_min;
        for (int g = 0; g < G && last < t_hi / 64; ++g) {
            const size_t rows = (size_t)(bh0 + g) * N;
            const float* ch = c + rows;
            if (reach_pays(ch[t_hi] - ch[k1], t_hi - k1, kFewBackward)) {
                last = max(last, last_needing_block(a.reach + rows, ch, k0 / 64, i_min, t_hi / 64, N, ch[k0], sl, lane));
            } else {
                last = t_hi / 64;
            }
        }
        nblk = __builtin_amdgcn_readfirstlane(min(t_hi >> 5, 2 * last + 1)) - qb_lo + 1;
    }
    const int items = G * nblk, mine = items > wv ? (items - wv + NW - 1) / NW : 0;
    PieceLoader<D> loader;
    loader.init(lane);
    float l_next = 0.f, c_next = 0.f, d_next = 0.f, ck_next = 0.f;
    bf16x8 o_next[OWN_D ? KC : 1];  // OWN_D: this lane's half row of O, the elements that row_frag has of dO
    auto issue = [&](int s, int slot) __attribute__((always_inline)) {
        const int it = wv + s * NW, bh = bh0 + it / nblk, t0 = (qb_lo + it % nblk) * 32;
        const size_t rows = (size_t)bh * N;
        const char* Qh = reinterpret_cast<const char*>(Q + rows * D);
        const char* Gh = reinterpret_cast<const char*>(dO + rows * D);
        const int tc = min(t0 + lk, N - 1);
        l_next = L[rows + tc];
        c_next = c[rows + tc];
        if constexpr (OWN_D) {
            const bf16_t* orow = O + (rows + tc) * D + 8 * h;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) o_next[kc] = *reinterpret_cast<const bf16x8*>(orow + 16 * kc);
        } else {
            d_next = Dv[rows + tc];
        }
        ck_next = c[rows + keyc];
#pragma unroll
        for (int j = 0; j < 32 / PieceLoader<D>::kRows; ++j) {
            loader.load(Qh, t0, j, N, sm.t.q[wv][slot & 1]);
            loader.load(Gh, t0, j, N, sm.t.g[wv][slot & 1]);
        }
    };
    if (mine > 0) issue(0, 0);
    for (int i = lane; i < kDkvSplitMaxGroup * 32; i += 64) (&sm.col[wv][0][0])[i] = 0.f;

    bf16x8 kf[KC], vf[KC];
    {
        const size_t roff = kv_off + (size_t)keyc * D + 8 * h;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            kf[kc] = *reinterpret_cast<const bf16x8*>(K + roff + 16 * kc);
            vf[kc] = *reinterpret_cast<const bf16x8*>(V + roff + 16 * kc);
        }
    }
    const int r_off = row_frag_off<D>(lane), t_off = col_frag_off<D>(lane);
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {  // no load of these is pending when the loop starts
        GFWA_PIN(kf[kc]);
        GFWA_PIN(vf[kc]);
    }
    f32x16 dk[DB], dv[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) dk[db][v] = dv[db][v] = 0.f;
    float colsum = 0.f;

    for (int s = 0; s < mine; ++s) {
        const int it = wv + s * NW, g = it / nblk, t0 = (qb_lo + it % nblk) * 32;
        const float cbase = __shfl(ck_next, 0, 64), ckl = (ck_next - cbase) * kLog2e;  // c_base: the head's c at the first key
        sm.nl[wv][s & 1][lk] = t0 + lk < N ? -(l_next + (c_next - cbase)) * inv_scale : -kPosBig;
        if (!OWN_D) sm.dvec[wv][s & 1][lk] = -d_next;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if constexpr (OWN_D) {
            const unsigned gt = (unsigned)(uintptr_t)sm.t.g[wv][s & 1];
            float dsum = 0.f;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const bf16x8 ga = row_frag<D>(gt + row_frag_off<D>(lane), 0, kc);
#pragma unroll
                for (int e = 0; e < 8; ++e) dsum = fmaf((float)o_next[kc][e], (float)ga[e], dsum);
            }
            sm.dvec[wv][s & 1][lk] = -xhalf_sum(dsum);
        }
        issue(min(s + 1, mine - 1), s + 1);  // (the last block once more at the end, into a slot nothing reads)
        const unsigned qt = (unsigned)(uintptr_t)sm.t.q[wv][s & 1], gt = (unsigned)(uintptr_t)sm.t.g[wv][s & 1];
        f32x16 sc, dp;
        acc_init_rows(sc, sm.nl[wv][s & 1], 0, h);
        acc_init_rows(dp, sm.dvec[wv][s & 1], 0, h);
        {
            bf16x8 qa[KC], ga[KC];
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) qa[kc] = row_frag<D>(qt + r_off, 0, kc);
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) ga[kc] = row_frag<D>(gt + r_off, 0, kc);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                sc = mfma32(qa[kc], kf[kc], sc);
                dp = mfma32(ga[kc], vf[kc], dp);
            }
        }
        bf16x8 gt_f[2 * DB], qt_f[2 * DB];  // dO^T and Q^T, in flight during the exponentials
#pragma unroll
        for (int i = 0; i < 2 * DB; ++i) gt_f[i] = col_frag<D>(gt + t_off, 16 * (i / DB), i % DB);
#pragma unroll
        for (int i = 0; i < 2 * DB; ++i) qt_f[i] = col_frag<D>(qt + t_off, 16 * (i / DB), i % DB);
        __builtin_amdgcn_sched_barrier(0);
        float p[16], ds[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) p[v] = fast_exp2(fmaf(sc[v], sl, ckl));
        if (__builtin_expect(!(k0 + 31 <= t0 && k0 > t0 + 31 - w), 0)) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = t0 + acc_row(v, h);
                p[v] = (key <= t && key > t - w) ? p[v] : 0.f;
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            ds[v] = p[v] * dp[v];
            colsum += ds[v];
        }
        bf16x8 pf[2], dsf[2];
        acc_to_bfrag(p, pf);
        acc_to_bfrag(ds, dsf);
#pragma unroll
        for (int i = 0; i < 2 * DB; ++i) {
            dv[i % DB] = mfma32(gt_f[i], pf[i / DB], dv[i % DB]);
            dk[i % DB] = mfma32(qt_f[i], dsf[i / DB], dk[i % DB]);
        }
        if (s + 1 == mine || (it + NW) / nblk != g) {  // the wave's last block of this query head
            const float cs = xhalf_sum(colsum);
            if (h == 0) sm.col[wv][g][lk] = cs;
            colsum = 0.f;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the block requested in vain has landed too
    __syncthreads();
    for (int i = threadIdx.x; i < G * 32; i += 64 * NW) {
        float cs = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) cs += sm.col[k][i / 32][i % 32];
        if (k0 + i % 32 < N) dc_col[(size_t)(bh0 + i / 32) * N + k0 + i % 32] = cs;
    }
    // ---- sum of the NW partial dK, dV: every wave hands its accumulators over and finishes 1 / NW of the columns
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            sm.xch[wv][4 * db + r][lane] = f32x4{dk[db][4 * r], dk[db][4 * r + 1], dk[db][4 * r + 2], dk[db][4 * r + 3]};
            sm.xch[wv][D / 8 + 4 * db + r][lane] = f32x4{dv[db][4 * r], dv[db][4 * r + 1], dv[db][4 * r + 2], dv[db][4 * r + 3]};
        }
    __syncthreads();
    constexpr int kOwn = 2 * (D / 8) / NW;
    f32x4 own[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        own[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            const f32x4 x = sm.xch[k][kOwn * wv + i][lane];
#pragma unroll
            for (int j = 0; j < 4; ++j) own[i][j] += x[j];
        }
    }
    __syncthreads();  // the exchange is read; its space takes the rows
    constexpr int kPitch = D * 2 + 16, kCpr = D / 8;
    const int mat = wv / (NW / 2);  // 0: dK, 1: dV
    const float post = mat == 0 ? scale : 1.0f;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const f32x4 x4 = {own[i][0] * post, own[i][1] * post, own[i][2] * post, own[i][3] * post};
        *reinterpret_cast<bf16x4*>(sm.out[mat] + lk * kPitch + 16 * (kOwn * (wv % (NW / 2)) + i) + 8 * h) =
            __builtin_convertvector(x4, bf16x4);
    }
    __syncthreads();
    for (int x = threadIdx.x; x < 2 * 32 * kCpr; x += 64 * NW) {
        const int which = x / (32 * kCpr), row = x / kCpr % 32, cc = x % kCpr;
        bf16_t* out = (which == 0 ? dK : dV) + kv_off + (size_t)(k0 + row) * D + 8 * cc;
        if (k0 + row < N)
            *reinterpret_cast<bf16x8*>(out) = *reinterpret_cast<const bf16x8*>(sm.out[which] + row * kPitch + 16 * cc);
    }
}

template <int D, int NW, bool LOOK>
__global__ __launch_bounds__(64 * NW, D == 64 ? 2 : 1) void bwd_dkv_split_bf16_kernel(BwdBf16 a) {
    dkv_split<D, NW, false, LOOK>(a, (int)blockIdx.x);
}

// Both passes in one launch, for problems of few workgroups: one after the other each leaves most of the chip idle and pays for its own
// launch.  The first dkv_blocks workgroups, the longer chains, are the dK/dV pass.  Every workgroup asks for the LDS of the larger half, about
// 140 KB, so one is resident on a CU, and a second round starts behind the shortest of the first.
template <int D, int NW, bool LOOK>
__global__ __launch_bounds__(64 * NW, D == 64 ? 2 : 1) void bwd_both_split_bf16_kernel(BwdBf16 a, int dkv_blocks, int num_qtiles) {
    if ((int)blockIdx.x < dkv_blocks) dkv_split<D, NW, true, LOOK>(a, (int)blockIdx.x);
    else dq_split<D, NW, 2, 1, 2, LOOK>(a, num_qtiles, (int)blockIdx.x - dkv_blocks);
}

template <int D, int NW, int QW, int KB, int RING, bool LOOK>
static hipError_t launch_dq_split_as(const BwdBf16& a, hipStream_t s) {
    using Smem = SplitBandSmem<D, NW, QW, KB, RING>;
    constexpr auto kernel = bwd_dq_split_bf16_kernel<D, NW, QW, KB, RING, LOOK>;
    static DeviceOnce lds_allowed;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), sizeof(Smem), lds_allowed)) return e;
    const int nq = (a.N + 32 * QW - 1) / (32 * QW), BH = a.B * a.H;
    ProfScope prof(kKernDq, s);
    hipLaunchKernelGGL(kernel, dim3((unsigned)BH * nq), dim3(64 * NW), sizeof(Smem), s, a, nq);
    return hipGetLastError();
}
template <int D, int NW, int QW, int KB, int RING>
static hipError_t launch_dq_split(const BwdBf16& a, hipStream_t s) {
    return a.reach != nullptr ? launch_dq_split_as<D, NW, QW, KB, RING, true>(a, s) : launch_dq_split_as<D, NW, QW, KB, RING, false>(a, s);
}

hipError_t bwd_dq_split_bf16(FwdSplit shape, const BwdBf16& a, int d, hipStream_t s) {
    if (d == 128) {
        if (shape == kFwdSplitMid) return launch_dq_split<128, 4, 2, 1, 2>(a, s);
        return launch_dq_split<128, 4, 1, 1, 1>(a, s);
    }
    if (shape == kFwdSplitMid) return launch_dq_split<64, 4, 2, 1, 2>(a, s);
    return launch_dq_split<64, 4, 1, 1, 2>(a, s);
}

template <int D, int NW, bool LOOK>
static hipError_t launch_dkv_split(const BwdBf16& a, hipStream_t s) {
    using Smem = DkvSplitSmem<D, NW>;
    constexpr auto kernel = bwd_dkv_split_bf16_kernel<D, NW, LOOK>;
    static DeviceOnce lds_allowed;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), sizeof(Smem), lds_allowed)) return e;
    ProfScope prof(kKernDkv, s);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.B * a.Hkv) * ((a.N + 31) / 32)), dim3(64 * NW), sizeof(Smem), s, a);
    return hipGetLastError();
}

hipError_t bwd_dkv_split_bf16(const BwdBf16& a, int d, hipStream_t s) {
    if (a.reach != nullptr) return d == 128 ? launch_dkv_split<128, 4, true>(a, s) : launch_dkv_split<64, 8, true>(a, s);
    return d == 128 ? launch_dkv_split<128, 4, false>(a, s) : launch_dkv_split<64, 8, false>(a, s);
}

template <int D, int NW, bool LOOK>
static hipError_t launch_both_split(const BwdBf16& a, hipStream_t s) {
    using DkvSmem = DkvSplitSmem<D, NW>;
    using DqSmem = SplitBandSmem<D, NW, 2, 1, 2>;
    constexpr size_t lds = sizeof(DkvSmem) > sizeof(DqSmem) ? sizeof(DkvSmem) : sizeof(DqSmem);
    constexpr auto kernel = bwd_both_split_bf16_kernel<D, NW, LOOK>;
    static DeviceOnce lds_allowed;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds, lds_allowed)) return e;
    const int nq = (a.N + 63) / 64, nk = a.B * a.Hkv * ((a.N + 31) / 32);
    ProfScope prof(kKernDkv, s);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(nk + a.B * a.H * nq)), dim3(64 * NW), lds, s, a, nk, nq);
    return hipGetLastError();
}

hipError_t bwd_both_split_bf16(const BwdBf16& a, int d, hipStream_t s) {
    if (a.reach != nullptr) return d == 128 ? launch_both_split<128, 4, true>(a, s) : launch_both_split<64, 8, true>(a, s);
    return d == 128 ? launch_both_split<128, 4, false>(a, s) : launch_both_split<64, 8, false>(a, s);
}

}  // namespace gfwa
