// Shared parts of the kernels that split the band of a query tile over groups of waves (fwd_split_bf16.hip and the dQ
// kernel of bwd_split_bf16.hip): a workgroup of NW waves owns QW blocks of 32 queries, KW = NW / QW groups of QW waves
// take every KW-th key tile (KB blocks of 32 keys) each, and their partial results are merged through LDS.
#pragma once
#include "tile_stage.h"

namespace gfwa {

// Operand fragments of a bf16 tile with the swizzle of tile_off.  `at` is the LDS address of the lane's first fragment
// (tile + row_frag_off or tile + col_frag_off, tiles starting at multiples of 256 bytes): the other fragments differ
// from it by an exclusive or of the chunk bits and by multiples of 16 rows, the swizzle's period, so that a lane
// carries two offsets instead of one address per fragment.
template <int D>
__device__ __forceinline__ int row_frag_off(int lane) { return tile_off<D>(lane & 31, lane >> 5); }
template <int D>
__device__ __forceinline__ int col_frag_off(int lane) {
    return tile_off<D>(4 * (lane >> 5) + ((lane & 15) >> 2), 2 * ((lane & 31) >> 4) + ((lane & 3) >> 1)) + 8 * (lane & 1);
}
// as lds_read_frag: row r0 + lane % 32, elements 16 kc + 8 (lane / 32) + 0..7
template <int D>
__device__ __forceinline__ bf16x8 row_frag(unsigned at, int r0, int kc) {
    return *(__attribute__((address_space(3))) const bf16x8*)(uintptr_t)((at ^ (32 * kc)) + r0 * (D * 2));
}
// as lds_read_tr_frag: the transpose's fragment of rows r0 .. r0 + 15, 32-column block db
template <int D>
__device__ __forceinline__ bf16x8 col_frag(unsigned at, int r0, int db) {
    constexpr int k8 = D == 128 ? 32 : 16;  // what eight rows further on do to the swizzle
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)((at ^ (64 * db)) + r0 * (D * 2)));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)((at ^ (64 * db) ^ k8) + (r0 + 8) * (D * 2)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// 1 KB pieces of a tile by direct global -> LDS loads: piece j of a tile that starts at row `row0` (rows at or beyond N
// read row N-1); a piece's swizzle is that of piece 0 with j in the low chunk bits.
template <int D>
struct PieceLoader {
    static constexpr int kRowBytes = D * 2, kChunks = kRowBytes / 16, kRows = 1024 / kRowBytes;
    int row, chunk;
    __device__ __forceinline__ void init(int lane) {
        row = lane / kChunks;
        chunk = swz_chunk<D>(row, lane % kChunks) * 16;
    }
    __device__ __forceinline__ void load(const char* M, int row0, int j, int N, char* tile) const {
        const unsigned off = (unsigned)min(row0 + j * kRows + row, N - 1) * (unsigned)kRowBytes +
                             (unsigned)(chunk ^ (16 * (j & (D == 128 ? 3 : 1))));
        dma16(M, off, tile + j * 1024);
    }
};

template <int D, int NW, int QW, int KB, int RING>
struct SplitBandSmem {
    static constexpr int KW = NW / QW;
    union {
        struct {
            alignas(256) char k[KW][RING][32 * KB * D * 2];  // one key tile per group and ring slot
            alignas(256) char v[KW][RING][32 * KB * D * 2];
        } t;
        f32x4 xch[NW][D / 8][64];                      // merge: accumulators, [wave][register group][lane]
        alignas(16) char out[32 * QW * (D * 2 + 16)];  // then the finished rows on their way to memory
    };
    float m[NW][64], l[NW][64];
    alignas(16) float g[NW][2][32 * KB];  // (c - c_base) / scale of the keys of a wave's tile
    int needed[NW];                       // over_waves
};

template <int D, int NW, int QW, int KB, int RING>
struct SplitBand {
    static_assert(RING == 2 || (RING == 1 && QW == 1), "a slot that other waves read is refilled behind a barrier");
    static constexpr int KW = NW / QW, kKeys = 32 * KB, KC = D / 16, DB = D / 32;
    static constexpr int kLoads = kKeys / PieceLoader<D>::kRows / QW;  // per wave and matrix
    using Smem = SplitBandSmem<D, NW, QW, KB, RING>;

    Smem& sm;
    const char *Kh, *Vh;
    const float* ch;
    int N, lane, wv, qi, kg;
    int kt_hi;           // last key tile of the band; group kg takes tiles kt_hi - kg, kt_hi - kg - KW, ..
    int mine, steps;     // steps of this group, of the workgroup
    int s_first, s_end;  // steps whose tile meets this wave's own band
    float cbase, inv_scale, c_next;
    PieceLoader<D> loader;

    __device__ __forceinline__ explicit SplitBand(Smem& s) : sm(s) {}

    // the tile of 32 QW queries from q0 of a head whose keys and values start at K, V and whose gate prefix is c
    __device__ __forceinline__ void open(const bf16_t* K, const bf16_t* V, const float* c, int n, int w, int q0, float inv_sc) {
        Kh = reinterpret_cast<const char*>(K);
        Vh = reinterpret_cast<const char*>(V);
        ch = c;
        N = n;
        inv_scale = inv_sc;
        lane = threadIdx.x & 63;
        wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        qi = wv % QW;
        kg = wv / QW;
        loader.init(lane);
        kt_hi = (min(N, q0 + 32 * QW) - 1) / kKeys;
        from(max(0, q0 - w + 1), q0, w);
        c_next = mine > 0 ? gate_of(0) : 0.f;
        if (mine > 0) issue(0);
        cbase = ch[q0];
    }
    // The steps of a band that starts at key k_lo, in the window or behind what the gate has erased (at q0 at most).  Called again before
    // the first step: tiles past the new start may have been requested then, and are waited for in merge.
    __device__ __forceinline__ void from(int k_lo, int q0, int w) {
        const int kt_lo = k_lo / kKeys, qw0 = q0 + 32 * qi, ntile = kt_hi - kt_lo + 1;
        mine = ntile > kg ? (ntile - kg + KW - 1) / KW : 0;
        steps = (ntile + KW - 1) / KW;
        s_first = s_end = 0;
        if (qw0 < N) {
            const int n_first = kt_hi - (qw0 + 31) / kKeys, n_last = kt_hi - max(k_lo, qw0 - w + 1) / kKeys;
            s_first = n_first > kg ? min((n_first - kg + KW - 1) / KW, steps) : 0;
            s_end = n_last >= kg ? min(mine, (n_last - kg) / KW + 1) : 0;
        }
    }
    __device__ __forceinline__ int first_key(int s) const { return (kt_hi - (s * KW + kg)) * kKeys; }
    __device__ __forceinline__ float gate_of(int s) const { return ch[min(first_key(s) + (KB == 1 ? lane & 31 : lane), N - 1)]; }
    // 1 KB of step s's tile into the ring slot of step `slot`; even i: keys, odd i: values
    __device__ __forceinline__ void issue_piece(int s, int slot, int i) const {
        if (i & 1) loader.load(Vh, first_key(s), qi * kLoads + i / 2, N, sm.t.v[kg][slot % RING]);
        else loader.load(Kh, first_key(s), qi * kLoads + i / 2, N, sm.t.k[kg][slot % RING]);
    }
    __device__ __forceinline__ void issue(int s) const {
#pragma unroll
        for (int i = 0; i < 2 * kLoads; ++i) issue_piece(s, s, i);
    }
    // start of a step: the group's tile of step s has landed, the readers of the slot that is filled next are done
    __device__ __forceinline__ void open_step(int s) {
        if (s < mine) sm.g[wv][s & 1][KB == 1 ? lane & 31 : lane] = (c_next - cbase) * inv_scale;
        // (The next step's gate value is a load that the compiler waits for by itself, with vmcnt(0): a tile requested two
        // steps ahead, into a third slot, would be waited for as well.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (QW > 1) wg_barrier();
        if (s + 1 < mine) c_next = gate_of(s + 1);
    }
    // a step with no block of this wave's band: only its share of the loads
    __device__ __forceinline__ void idle_step(int s) {
        open_step(s);
        if (s + 1 < mine) issue(s + 1);
    }
    // the step whose tile is requested during step s; past the end the last one again, into a slot that nothing reads any more
    __device__ __forceinline__ int requested(int s) const { return min(s + 1, mine - 1); }
    // RING == 1: the slot's reads by this wave (its only reader) are done, refill it
    __device__ __forceinline__ void close_step(int s) const {
        if (RING == 1 && s + 1 < mine) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue(s + 1);
        }
    }
    __device__ __forceinline__ bool cut(int k0, int qw0, int w) const {  // the diagonal or the window edge cuts the tile
        return !(k0 + kKeys - 1 <= qw0 && k0 > qw0 + 31 - w);
    }

    // Every wave hands its accumulators over (a lane owns a query, register 4 g + j of them column 8 g + 4 (lane / 32) + j)
    // and takes 1 / KW of its queries' columns: sum over the groups k of f[k] times their accumulators, times post,
    // stored as rows of 2 D bytes from `out` on (row 0 of the workgroup's tile; rows_valid of them exist).
    // m and l of the groups are exchanged before f is asked for, by f_of(m_k, l_k), which runs between the barriers.
    template <typename F>
    __device__ __forceinline__ void merge(const f32x16 (&acc)[DB], float m, float l, F&& f_of, bf16_t* out, int rows_valid) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // a tile requested in vain has landed too
        __syncthreads();
        sm.m[wv][lane] = m;
        sm.l[wv][lane] = l;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                sm.xch[wv][4 * db + r][lane] = f32x4{acc[db][4 * r], acc[db][4 * r + 1], acc[db][4 * r + 2], acc[db][4 * r + 3]};
        __syncthreads();
        float mk[KW], lk[KW], f[KW];
#pragma unroll
        for (int k = 0; k < KW; ++k) {
            mk[k] = sm.m[k * QW + qi][lane];
            lk[k] = sm.l[k * QW + qi][lane];
        }
        const float post = f_of(mk, lk, f);
        constexpr int kOwn = D / 8 / KW;  // register groups this wave finishes
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
        __syncthreads();  // the exchange is read; its space takes the rows
        constexpr int kPitch = D * 2 + 16, kCpr = D / 8;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
            const f32x4 x4 = {own[i][0] * post, own[i][1] * post, own[i][2] * post, own[i][3] * post};
            *reinterpret_cast<bf16x4*>(sm.out + (32 * qi + (lane & 31)) * kPitch + 16 * (kOwn * kg + i) + 8 * (lane >> 5)) =
                __builtin_convertvector(x4, bf16x4);
        }
        __syncthreads();
        for (int x = threadIdx.x; x < 32 * QW * kCpr; x += 64 * NW) {
            const int row = x / kCpr, cc = x % kCpr;
            if (row < rows_valid)
                *reinterpret_cast<bf16x8*>(out + (size_t)row * D + 8 * cc) =
                    *reinterpret_cast<const bf16x8*>(sm.out + row * kPitch + 16 * cc);
        }
    }
};

}  // namespace gfwa
