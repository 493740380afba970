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
                                                       T* __restrict__ O, int N, int w, int blocks, int block, int few, int tile, int H, int G) {
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
        return reach_pays(ch[q0] - ch[k_lo], q0 - k_lo, few);
    };
    bool any = false;
    for (int i = lane; i < G * nt; i += 64) any |= asks(i / nt, i % nt);
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
    for (int g0 = 0; g0 < G; g0 += 4) {  // four heads' gates at once, and their tiles over the lanes
        int high[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) high[j] = (int)0x80000000;
        for (int i = k0 + lane; i < k1; i += 64)
#pragma unroll
            for (int j = 0; j < 4; ++j) high[j] = max(high[j], highest_order(c[(size_t)(bh0 + min(g0 + j, G - 1)) * N + i]));
#pragma unroll
        for (int j = 0; j < 4; ++j) high[j] = lanes_max(high[j]);
        for (int i = lane; i < min(4, G - g0) * nt; i += 64) {
            const int j = i / nt, t = i % nt, q0 = (t_lo + t) * tile, e = q0 / block - 1 - kb;
            const int top = j < 2 ? (j == 0 ? high[0] : high[1]) : (j == 2 ? high[2] : high[3]);
            if (asks(g0 + j, t) && e < key_blocks_in<D, T>(min(tile, N - q0)))
                reinterpret_cast<KeyBlock*>(O + ((size_t)(bh0 + g0 + j) * N + q0) * D)[e] = {norms, from_order(top)};
        }
    }
}

// Whether a forward looks at the reach of its keys, by what blocks, and what a tile has to save.
// A tile's band has to lose 100 keys that tiles and blocks do not divide (steps of 32 or 64 keys, 64-key blocks, the tile's own queries), and
// as many as the forward streams while the pass reads K and V (few).  A launch in which no tile asks costs 2 to 3 us: there is one where the keys
// beyond these and the first 500, which only gates above 0.2 a key erase, take sixteen times as long, so that slow gates lose 4 % at most.
// (Times at the rates of large problems, with fewer than two tiles a CU accordingly less, at least half.)
// Whole bands / with the launch, us, gates of softplus(N(mu, 1)):                mu    -6          -3          -2          -1
//   taken      B1 H8    N5003  d128 w3000                                           52 / 55     52 / 56     52 / 46     53 / 39
//              B1 H12   N6000  d128 w4096                                          117 / 119   113 / 82    114 / 69    114 / 58
//              B1 H4    N16384 d128 w4096                                          139 / 142   134 / 76    135 / 49    136 / 38
//              B2 H16   N4096  d128 w1024 fp32                                     344 / 347   345 / 347   348 / 301   349 / 210
//   not taken  B4 H16   N4096  d64  w1024                                           79 / 82     79 / 82     76 / 72     75 / 56
//              B1 H32   N4096  d128 w1024                                           76 / 78     75 / 78     73 / 73     72 / 57
//              B1 H20   N3000  d128 causal                                          61 / 63     60 / 65     59 / 50     58 / 43
//              B1 H12   N4096  d64  causal                                          41 / 43     41 / 44     41 / 33     41 / 28
//              B4 H16/4 N8192  d64  w512                                            99 / 102    99 / 102    98 / 100    93 / 84
//              B1 H32   N4096  d128 w700 fp32                                      263 / 266   262 / 266   263 / 272   265 / 210
static KeyReach reach_of(int B, int H, int Hkv, int N, int d, int w, bool bf16) {
    const double band = w < N ? w : N, mean = band - band * band / (2.0 * N), rows = (double)B * H * N;
    const double tiles = rows / (128 * 512), fill = tiles < 0.5 ? 0.5 : tiles < 1 ? tiles : 1;
    const double rate = bf16 ? d == 128 ? 900e6 : 700e6 : 150e6;  // FLOP/us
    const double per_key = 4 * rows * d / rate / fill;            // us for a key of the band
    const double few = 100 + 2.0 * B * Hkv * N * d * (bf16 ? 2 : 4) / 6.2e6 / per_key;
    if (per_key * (mean - few - 500) < 40) return {0, 0};
    long block = 64;
    while (((long)band + block) / block + 1 > 64) block *= 2;  // (an entry for each lane of a wave)
    return {(int)block, (int)few};
}

template <int D, typename T>
static void launch(KeyReach reach, int tile, const void* K, const void* V, const float* c, void* O, int B, int H, int Hkv, int N, int w, hipStream_t s) {
    const int blocks = (N + reach.block - 1) / reach.block;
    hipLaunchKernelGGL((key_reach_kernel<D, T>), dim3((unsigned)(B * Hkv) * blocks), dim3(64), 0, s, (const T*)K, (const T*)V, c, (T*)O, N, w, blocks,
                       reach.block, reach.few, tile, H, H / Hkv);
}
hipError_t key_reach(KeyReach& reach, int tile, bool bf16, const void* Q, const void* K, const void* V, const float* c, void* O, int B, int H, int Hkv,
                     int N, int d, int w, float scale, hipStream_t s) {
    const size_t row = (size_t)d * (bf16 ? 2 : 4), out = (size_t)B * H * N * row, keys = (size_t)B * Hkv * N * row;
    reach = scale > 0.f ? reach_of(B, H, Hkv, N, d, w, bf16) : KeyReach{0, 0};
    if (overlap(O, out, Q, out) || overlap(O, out, K, keys) || overlap(O, out, V, keys) || overlap(O, out, c, (size_t)B * H * N * sizeof(float)))
        reach.block = 0;
    if (reach.block == 0) return hipSuccess;
    if (bf16) d == 128 ? launch<128, bf16_t>(reach, tile, K, V, c, O, B, H, Hkv, N, w, s) : launch<64, bf16_t>(reach, tile, K, V, c, O, B, H, Hkv, N, w, s);
    else d == 128 ? launch<128, float>(reach, tile, K, V, c, O, B, H, Hkv, N, w, s) : launch<64, float>(reach, tile, K, V, c, O, B, H, Hkv, N, w, s);
    return hipGetLastError();
}

}  // namespace gfwa
