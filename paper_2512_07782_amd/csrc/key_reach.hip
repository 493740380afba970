// Norms and gates of the key blocks in front of the query tiles of a forward (band_reach.h): largest squared norms and highest gate of
// every block of keys, written into the rows of O of the tiles that see it.
//
// Memory bounds it where it reads (K and V once: B4 H16 N8192 d128, 268 MB, 43 us, 6.2 TB/s), the launch where no tile asks.
#include "band_reach.h"
#include "gfwa_internal.h"

namespace gfwa {

__device__ __forceinline__ float square8(const bf16_t* p, float x) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(p);
    return dot8(v, v, x);
}
__device__ __forceinline__ float square8(const float* p, float x) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(p + 4 * i);
#pragma unroll
        for (int j = 0; j < 4; ++j) x = fmaf(v[j], v[j], x);
    }
    return x;
}

// A wave takes one block of keys of one key/value head and serves the G query heads that read it.  (Workgroups of one wave: all of them
// are resident at once, and where nothing is read the launch is over after two dependent loads; 4096 workgroups of four waves 9 us.)
template <int D, typename T>
__global__ __launch_bounds__(64) void key_reach_kernel(const T* __restrict__ K, const T* __restrict__ V, const float* __restrict__ c,
                                                       T* __restrict__ O, int N, int w, int blocks, int block, int tile, int H, int G) {
    constexpr int kLanes = D / 8, kRows = 64 / kLanes, U = 16 / sizeof(T);  // lanes of a row, rows at a time, times in flight
    const int lane = threadIdx.x;
    const int bkv = (int)blockIdx.x / blocks, kb = (int)blockIdx.x % blocks, k0 = kb * block, k1 = min(N, k0 + block);
    const int Hkv = H / G, bh0 = (bkv / Hkv) * H + (bkv % Hkv) * G;
    // the tiles that start behind the block and within the window of its last key
    const int t_lo = (k0 + block + tile - 1) / tile, t_hi = (int)(min((long)N - 1, (long)k0 + block - 2 + w) / tile);
    if (t_lo > t_hi) return;
    const int nt = t_hi - t_lo + 1;
    // The tiles that will look at their blocks (the forward kernels ask the same), and whether there is one.
    auto asks = [&](int g, int t) __attribute__((always_inline)) {
        const float* ch = c + (size_t)(bh0 + g) * N;
        const int q0 = (t_lo + t) * tile, k_lo = max(0, q0 - w + 1);
        return reach_pays(ch[q0] - ch[k_lo], q0 - k_lo, kFewForward);
    };
    bool any = false;
    for (int g = 0; g < G; ++g)
        for (int t = lane; t < nt; t += 64) any |= asks(g, t);
    if (__builtin_amdgcn_ballot_w64(any) == 0) return;
    int norm = 0, value = 0;
    const size_t at = (size_t)bkv * N * D + 8 * (lane % kLanes);
    for (int r0 = k0 + lane / kLanes; r0 - lane / kLanes < k1; r0 += U * kRows) {
        float nk[U], nv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const size_t row = at + (size_t)min(r0 + u * kRows, k1 - 1) * D;
            nk[u] = square8(K + row, 0.f);
            nv[u] = square8(V + row, 0.f);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float v2 = row_sum<kLanes>(nv[u]);
            norm = max(norm, finite(v2) ? norm_bits(row_sum<kLanes>(nk[u])) : kInfBits);  // (a value row that is not finite keeps its block)
            value = max(value, norm_bits(v2));
        }
    }
    const unsigned norms = pack_norms(lanes_max(norm), lanes_max(value));
    for (int g = 0; g < G; ++g) {
        const float* ch = c + (size_t)(bh0 + g) * N;
        int high = (int)0x80000000;
        for (int i = k0 + lane; i < k1; i += 64) high = max(high, highest_order(ch[i]));
        high = lanes_max(high);
        for (int t = lane; t < nt; t += 64) {
            const int q0 = (t_lo + t) * tile, e = q0 / block - 1 - kb;
            if (asks(g, t) && e < key_blocks_in<D, T>(min(tile, N - q0)))
                reinterpret_cast<KeyBlock*>(O + ((size_t)(bh0 + g) * N + q0) * D)[e] = {norms, from_order(high)};
        }
    }
}

// Whether a forward looks at the reach of its keys, and by what blocks.  Where the gate then decays too little the launch is in vain, 2 to 3 us:
// 2 to 3 % of the shortest forwards that take it for a window that only gates of more than 0.1 a key erase in part, and up to 10 % for
// windows that all but the slowest do, where a forward of 30 us is one of 15 with mu = -2.  (us: at the rate of long forwards, which short
// ones do not reach.)  Below 600 keys hardly any gate does.
static int reach_block_of(int BH, int N, int d, int w, bool bf16) {
    const long band = w < N ? w : N;
    const double us = 4e-6 * BH * (double)N * band * d / (bf16 ? d == 128 ? 900.0 : 700.0 : 150.0) / (2 * band > N ? 2.0 : 1.0);
    if (band < 600 || us < (band < 900 ? 100.0 : band < 1300 ? 50.0 : 20.0)) return 0;
    long block = 64;
    while ((band + block) / block + 1 > 64) block *= 2;  // (an entry for each lane of a wave)
    return (int)block;
}

template <int D, typename T>
static void launch(int block, int tile, const void* K, const void* V, const float* c, void* O, int B, int H, int Hkv, int N, int w, hipStream_t s) {
    const int blocks = (N + block - 1) / block;
    hipLaunchKernelGGL((key_reach_kernel<D, T>), dim3((unsigned)(B * Hkv) * blocks), dim3(64), 0, s, (const T*)K, (const T*)V, c, (T*)O, N, w, blocks,
                       block, tile, H, H / Hkv);
}
hipError_t key_reach(int& block, int tile, bool bf16, const void* Q, const void* K, const void* V, const float* c, void* O, int B, int H, int Hkv,
                     int N, int d, int w, float scale, hipStream_t s) {
    const size_t row = (size_t)d * (bf16 ? 2 : 4), out = (size_t)B * H * N * row, keys = (size_t)B * Hkv * N * row;
    block = scale > 0.f ? reach_block_of(B * H, N, d, w, bf16) : 0;
    if (overlap(O, out, Q, out) || overlap(O, out, K, keys) || overlap(O, out, V, keys) || overlap(O, out, c, (size_t)B * H * N * sizeof(float)))
        block = 0;
    if (block == 0) return hipSuccess;
    if (bf16) d == 128 ? launch<128, bf16_t>(block, tile, K, V, c, O, B, H, Hkv, N, w, s) : launch<64, bf16_t>(block, tile, K, V, c, O, B, H, Hkv, N, w, s);
    else d == 128 ? launch<128, float>(block, tile, K, V, c, O, B, H, Hkv, N, w, s) : launch<64, float>(block, tile, K, V, c, O, B, H, Hkv, N, w, s);
    return hipGetLastError();
}

}  // namespace gfwa
