// Gate prefix scans on gfx950 (paper Sec. 3.2 definition of the cumulative gate; Alg. 1, the
// cumulative-sum / carry steps; Sec. 3.3 for the reverse scan that turns d(prefix) into d(alpha)).
//
// One workgroup of 4 or 16 waves (scan_four_waves) streams one (b,h) row in chunks of 4096 elements, cut into 16 runs of 256 consecutive ones:
// float4 per lane, in-lane prefix, scan of the lane totals by DPP moves; the totals of runs and waves are added up in
// fp64, across the waves through LDS, and a carry is kept in fp64 across chunks.  Every element is read once and written
// once (8 bytes of HBM traffic per element).  Short rows are bound by latency: the loads of a chunk go out before
// anything else (before the carry of a segment is formed, before the previous chunk is finished), there is one barrier
// per chunk and no shuffle through LDS.  (With 16 waves throughout, shuffles and two barriers: 300 rows of 8192 7.6 us, now
// 5.3; 1024 rows of 65536 114 us, now 105; 100 rows of 262144 with the activation 156 us, now 127.)
//
// The same kernel also fuses the gate activation of Alg. 1 in front of the scan: with the
// pre-activation h and the amplitude beta as inputs it forms
//   alpha = softplus(beta h) / (beta + eps),  softplus(z) = nu + log(exp(z - nu) + exp(-nu)), nu = max(z, 0)
// (evaluated as nu + log1p(exp(-|z|)), the same sum; see softplus_parts)
// on the fly (12 bytes per element, no alpha or z tensor in HBM), which is the paper's one-pass
// gate preprocessing as a whole.
#include "gfwa_device.h"
#include "gfwa_internal.h"

namespace gfwa {

constexpr int kScanChunk = 4096;  // elements a workgroup takes at a time: 16 runs of 256, shared out over its waves
constexpr int kScanRuns = kScanChunk / 256;
constexpr int kScanTargetWorkgroups = 2048;  // scan-then-propagate: segments are cut until about this many exist

// Softplus of z in the overflow-safe form of Alg. 1, nu + log(exp(z - nu) + exp(-nu)) with nu = max(z, 0).
// One of the two exponentials is exp(0) = 1 and the other is e = exp(-|z|), so the logarithm is
// log(1 + e), 0 < e <= 1.  Built on the hardware exp2 / log2 / reciprocal (about 1 ulp each) so that
// the kernels stay bound by memory traffic, and arranged so that a small result keeps its
// relative accuracy:
//   e       = 2^(x log2(e)) with the rounding error of the product x log2(e) carried as a correction,
//   log1p(e) = log(u) * e / (u - 1),  u = fl(1 + e)   (= e when u rounds to 1),
// the second being the classical cure for the rounding of 1 + e.  Returns softplus(z); *e_out = e.
__device__ __forceinline__ float softplus_parts(float z, float* e_out) {
    constexpr float kLog2eHi = 1.44269502162933349609375f;  // fl(log2(e))
    constexpr float kLog2eLo = 1.92596299e-8f;              // log2(e) - kLog2eHi
    constexpr float kLn2 = 0.693147182464599609375f;
    const float x = fmaxf(-fabsf(z), -128.f);               // below -128 e is 0 in fp32 anyway
    const float t = x * kLog2eHi;
    const float t_lo = fmaf(x, kLog2eHi, -t) + x * kLog2eLo;
    const float p = __builtin_amdgcn_exp2f(t);
    const float e = fmaf(p, t_lo * kLn2, p);
    const float u = 1.0f + e;
    const float um1 = u - 1.0f;
    const float l = __builtin_amdgcn_logf(u) * kLn2;        // log(u), u in [1, 2]
    const float log1p_e = um1 == 0.f ? e : l * (e * __builtin_amdgcn_rcpf(um1));
    *e_out = e;
    return fmaxf(z, 0.f) + log1p_e;
}

// alpha of one element (Alg. 1, on-chip steps)
__device__ __forceinline__ float gate_alpha(float h, float beta, float eps) {
    float e;
    return softplus_parts(beta * h, &e) * __builtin_amdgcn_rcpf(beta + eps);
}

enum ScanInput { kScanPlain = 0, kScanDiff = 1, kScanGate = 2 };

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp_or_zero(float x) {  // lanes without a source, or in a row that ROWS leaves out, get 0
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROWS, 0xf, false));
}
// inclusive scan over the 64 lanes: shifts inside the rows of 16 lanes, then the totals of the rows before
__device__ __forceinline__ float wave_scan(float x) {
    x += dpp_or_zero<0x111>(x);
    x += dpp_or_zero<0x112>(x);
    x += dpp_or_zero<0x114>(x);
    x += dpp_or_zero<0x118>(x);
    x += dpp_or_zero<0x142, 0xa>(x);  // lane 15 (47) to row 1 (3)
    x += dpp_or_zero<0x143, 0xc>(x);  // lane 31 to rows 2, 3
    return x;
}
__device__ __forceinline__ float lane_value(float x, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// Four floats in one access at any multiple of 4 bytes: rows of odd length start anywhere.  (Element by element, rows of
// such a length took four times the load and store instructions: 8 rows of 5003 5.75 -> 4.18 us, 1024 of 515 4.80 -> 4.05,
// 300 of 999 with the activation 5.33 -> 4.57, 3 of 100001 with it in segments 9.75 -> 7.46.)
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));

// The four elements at logical positions p .. p + 3 of a row, zero at and beyond `end`.  Position p of the scan is memory index
// p (forward) or N - 1 - p (reverse).  MODE kScanDiff: the scanned value is a[idx] - b[idx]; kScanGate: gate_alpha(a[idx],
// b[idx], eps).  Loading and evaluation are apart so that the loads of a chunk are in flight while something else is computed.
template <bool REVERSE, int MODE>
struct ScanQuad {
    f32x4 x, y;
    __device__ __forceinline__ void load(const float* ar, const float* br, int N, int p, int end) {
        constexpr bool TWO = MODE != kScanPlain;
        x = y = f32x4{0.f, 0.f, 0.f, 0.f};
        if (p + 3 < end) {
            const int idx = REVERSE ? N - 4 - p : p;
            x = *reinterpret_cast<const float4_any*>(ar + idx);
            if (TWO) y = *reinterpret_cast<const float4_any*>(br + idx);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (p + e < end) {
                    const int idx = REVERSE ? N - 1 - (p + e) : p + e, to = REVERSE ? 3 - e : e;
                    x[to] = ar[idx];
                    if (TWO) y[to] = br[idx];
                }
        }
    }
    __device__ __forceinline__ void values(float (&v)[4], float eps, int p, int end) const {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int from = REVERSE ? 3 - e : e;
            v[e] = MODE == kScanPlain ? x[from] : MODE == kScanDiff ? x[from] - y[from] : p + e < end ? gate_alpha(x[from], y[from], eps) : 0.f;
        }
    }
};
// first logical position of run r of this lane's wave in the chunk that starts at `base`
template <int WAVES>
__device__ __forceinline__ int run_start(int base, int wv, int r, int lane) { return base + (wv * (kScanRuns / WAVES) + r) * 256 + 4 * lane; }

// A workgroup takes segment blockIdx.x % P of row blockIdx.x / P, seg_len logical positions long, and starts from the sum of the
// row's earlier segments: from `partial` (scan-then-propagate), or, ALONE, from the row itself (scan_rows_alone).
template <bool REVERSE, int MODE, int WAVES, bool ALONE>
__device__ __forceinline__ void scan_rows(const float* __restrict__ a, const float* __restrict__ b, float* __restrict__ out, int N, float eps,
                                          const double* __restrict__ partial, int seg_len, int P, bool by_runs) {
    constexpr int RUNS = kScanRuns / WAVES;
    __shared__ double wave_tot[2][WAVES];
    // (a row that is one workgroup's does not wait for the divisions, 0.1 us: B2 H8/2 N515 d64 step 35.1 / 35.0)
    const int seg = P > 1 ? (int)(blockIdx.x % P) : 0;
    const size_t row = (size_t)(P > 1 ? blockIdx.x / P : blockIdx.x) * N;
    const int begin = seg * seg_len, end = min(N, begin + seg_len);
    const float* ar = a + row;
    const float* br = MODE != kScanPlain ? b + row : nullptr;
    float* outr = out + row;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;

    ScanQuad<REVERSE, MODE> quad[RUNS];
    auto load = [&](int base) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) quad[r].load(ar, br, N, run_start<WAVES>(base, wv, r, lane), end);
    };
    load(begin);
    double carry = 0.0;
    if (!ALONE && partial != nullptr && seg > 0) {  // sum of the earlier segments of this row, fp64, in every wave by itself
        const double* pr = partial + (size_t)(blockIdx.x / P) * P;
        double acc = 0.0;
        for (int q = lane; q < seg; q += 64) acc += pr[q];
        carry = wave_sum(acc);
    }
    if (ALONE && seg > 0) {
        // of its elements: fp32 over four and fp64 across, as segment_sum_kernel, or (by_runs) fp32 over runs and fp64 across, as a whole row
        // in one workgroup: the prefix of a call without a workspace does not depend on the way it is formed
        double acc = 0.0;
        constexpr int U = 4 / RUNS > 1 ? 4 / RUNS : 1;  // chunks in flight
        for (int base = 0; base < begin; base += U * kScanChunk) {
            ScanQuad<REVERSE, MODE> q[U][RUNS];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < RUNS; ++r) q[u][r].load(ar, br, N, run_start<WAVES>(base + u * kScanChunk, wv, r, lane), begin);
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < RUNS; ++r) {
                    float v[4];
                    q[u][r].values(v, eps, run_start<WAVES>(base + u * kScanChunk, wv, r, lane), begin);
                    if (by_runs) acc += (double)lane_value(wave_scan(((v[0] + v[1]) + v[2]) + v[3]), 63);
                    else acc += (double)((v[0] + v[1]) + (v[2] + v[3]));
                }
        }
        if (!by_runs) acc = wave_sum(acc);
        if (lane == 0) wave_tot[1][wv] = acc;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < WAVES; ++k) carry += wave_tot[1][k];  // (the first chunk's totals go to the other place)
    }
    int buf = 0;
    for (int base = begin; base < end; base += kScanChunk, buf ^= 1) {
        float v[RUNS][4], excl[RUNS];  // excl: sum of the lanes before, in the run
        double before[RUNS], total = 0.0;   // before: sum of the wave's runs before
#pragma unroll
        for (int r = 0; r < RUNS; ++r) quad[r].values(v[r], eps, run_start<WAVES>(base, wv, r, lane), end);
        if (base + kScanChunk < end) load(base + kScanChunk);
#pragma unroll
        for (int r = 0; r < RUNS; ++r) {
            v[r][1] += v[r][0];
            v[r][2] += v[r][1];
            v[r][3] += v[r][2];
            const float incl = wave_scan(v[r][3]);
            excl[r] = incl - v[r][3];
            before[r] = total;
            total += (double)lane_value(incl, 63);
        }
        if (lane == 0) wave_tot[buf][wv] = total;
        __syncthreads();  // (the totals alternate between two places: the next chunk's writers need no second barrier)
        double start = carry;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            const double t = wave_tot[buf][k];
            if (k < wv) start += t;
            carry += t;
        }
#pragma unroll
        for (int r = 0; r < RUNS; ++r) {
            const int p = run_start<WAVES>(base, wv, r, lane);
            const double from = start + before[r] + (double)excl[r];
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (float)(from + (double)v[r][e]);
            if (p + 3 < end) {
                const int idx = REVERSE ? N - 4 - p : p;
                *reinterpret_cast<float4_any*>(outr + idx) = REVERSE ? f32x4{y[3], y[2], y[1], y[0]} : f32x4{y[0], y[1], y[2], y[3]};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (p + e < end) outr[REVERSE ? N - 1 - (p + e) : p + e] = y[e];
            }
        }
    }
}

template <bool REVERSE, int MODE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void scan_rows_kernel(const float* __restrict__ a, const float* __restrict__ b, float* __restrict__ out, int N,
                                                                 float eps, const double* __restrict__ partial, int seg_len, int P) {
    scan_rows<REVERSE, MODE, WAVES, false>(a, b, out, N, eps, partial, seg_len, P, false);
}
// (A kernel of its own: the loads in flight for the row in front take 23 registers, with which one workgroup of 16 waves is left of two on a CU.
// With the activation, us, one kernel for both / two: 1000 rows of 16384 34.4 / 31.6, 1024 of 12000 28.0 / 24.9, 300 of 65536 51.8 / 47.4.)
template <bool REVERSE, int MODE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void scan_rows_alone_kernel(const float* __restrict__ a, const float* __restrict__ b, float* __restrict__ out,
                                                                       int N, float eps, int P, bool by_runs) {
    scan_rows<REVERSE, MODE, WAVES, true>(a, b, out, N, eps, nullptr, kScanChunk, P, by_runs);
}

// Phase 1 of scan-then-propagate (App. "Preprocessing via Scan-Then-Propagate"): the sum of every
// segment, the activation recomputed on the fly when the input is (h, beta).  fp32 over four elements, fp64 across.
template <bool REVERSE, int MODE, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void segment_sum_kernel(const float* __restrict__ a,
                                                                   const float* __restrict__ b,
                                                                   double* __restrict__ partial, int N, float eps,
                                                                   int seg_len, int P) {
    constexpr int RUNS = kScanRuns / WAVES;
    __shared__ double wave_tot[WAVES];
    const int seg = (int)(blockIdx.x % P);
    const size_t row = (size_t)(blockIdx.x / P) * N;
    const int begin = seg * seg_len, end = min(N, begin + seg_len);
    const float* ar = a + row;
    const float* br = MODE != kScanPlain ? b + row : nullptr;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    double acc = 0.0;
    for (int base = begin; base < end; base += kScanChunk) {
        ScanQuad<REVERSE, MODE> quad[RUNS];
#pragma unroll
        for (int r = 0; r < RUNS; ++r) quad[r].load(ar, br, N, run_start<WAVES>(base, wv, r, lane), end);
#pragma unroll
        for (int r = 0; r < RUNS; ++r) {
            float v[4];
            quad[r].values(v, eps, run_start<WAVES>(base, wv, r, lane), end);
            acc += (double)((v[0] + v[1]) + (v[2] + v[3]));
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) wave_tot[wv] = acc;
    __syncthreads();
    if (tid == 0) {
        double all = 0.0;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) all += wave_tot[k];
        partial[blockIdx.x] = all;
    }
}

// Four waves with four runs of a chunk each, or sixteen with one.  Four have less to exchange and more loads in flight per
// wave: better for rows of one or two chunks once CUs have several (320 rows of 4096: 3.4 against 4.3 us; 1024 rows of 515:
// 4.3 against 6.5; 300 rows of 8192: 5.3 against 6.6), and for segments (scan and sums of 8 rows of 32768: 5.8 against 6.2).
// A workgroup alone on its CU has no other to hide its vector work and its scattered accesses behind, and sixteen waves
// share them out: up to one per CU, sixteen are better with the activation (64 rows of 4096: 3.4 against 3.8 us, of 8192:
// 4.9 against 6.3) and for whole rows (64 rows of 515: 2.9 against 3.2; of 4096, in front of a forward that displaces the inputs: the
// pair 67.7 against 68.8; of 6000, two chunks: 4.0 against 4.2, of exactly two 3.96 against 3.86).
// Longer rows keep a CU busy with one workgroup after another's barrier, and the activation is bound by vector work: sixteen
// waves cover that (100 rows of 262144 with the activation: 127 against 249 us; sums of 512 segments with it: 7.0 against 8.0).
static bool scan_four_waves(bool activation, bool segment, long workgroups, int len) {
    if (workgroups <= device_cu_count() && (activation || !segment)) return false;
    return len <= 2 * kScanChunk;
}
// Few rows of three chunks or more go in segments of one chunk that each add up the row before them by themselves: one launch, no scratch,
// the row read (P + 1) / 2 times out of the L2.  Up to a workgroup a CU, with the activation, which is formed again as often, three on four, and
// 16 segments.  us, one workgroup a row / scan-then-propagate / this:
//               1 row of 12000    16384            32768            65536             32 rows of 12000   16384            24576            32768
//   plain       4.5 / 8.1 / 4.1   5.4 / 8.0 / 4.3  9.3 / 8.1 / 6.1  17.1 / 8.1 / 9.9   5.0 / 8.4 / 4.3   5.9 / 8.4 / 4.6   7.9 / 8.5 / 5.8  10.0 / 8.6 /  8.2
//   activation  5.8 / 8.1 / 5.7   7.2 / 8.1 / 6.2 12.7 / 8.1 / 9.6  23.7 / 8.2 / 15.9  6.3 / 8.4 / 6.2   7.7 / 8.5 / 6.8  10.5 / 8.6 / 9.6  13.5 / 8.8 / 14.9
// (96 rows of 16384, 384 segments: 6.5 / 8.9 / 6.8, 8.3 / 10.5 / 13.4.)
// (With the sums by runs, which the prefix without a workspace keeps: 1 row of 65536 14.0, 32 rows of 16384 5.2, 8 of 32768 7.9; 17.2, 6.8, 10.2 with the
// activation; 17.4, 5.8, 9.5 and 24.0, 7.6, 12.9 in one workgroup a row.)
static bool scan_rows_alone(bool activation, int rows, int N) {
    const int P = (N + kScanChunk - 1) / kScanChunk;
    return P >= 3 && P <= 16 && (activation ? 4 : 3) * (long)rows * P <= 3L * device_cu_count();
}
// Whether scan-then-propagate, and the gate gradient of few rows, which sum up the chunks in front of a segment by fours in fp64, take this instead of
// their two launches: up to 8 chunks, 4 with the activation.  (One workgroup a row is faster than two launches up to 6 chunks, too, but sums
// chunks up by runs in fp32, the coarser: against fp64, d(alpha) of B4 H16 N8192 d128 w1024 2.0e-6 by fours, 2.3e-6 by runs.)
static bool scan_in_one_launch(bool activation, int rows, int N) {
    const int P = (N + kScanChunk - 1) / kScanChunk;
    return P == 1 || (P <= (activation ? 4 : 8) && scan_rows_alone(activation, rows, N));
}
// (out over an input: the segments behind still need what the ones in front overwrite)
static bool scan_in_place(const float* a, const float* b, const float* out, int rows, int N) {
    const size_t bytes = (size_t)rows * N * sizeof(float);
    return overlap(out, bytes, a, bytes) || (b != nullptr && overlap(out, bytes, b, bytes));
}
template <bool REVERSE, int MODE>
static void launch_scan(const float* a, const float* b, float* out, int rows, int N, float eps, const double* partial, int seg_len,
                        int P, bool by_runs, hipStream_t s) {
    if (partial == nullptr) {
        if (scan_rows_alone(MODE == kScanGate, rows, N) && !scan_in_place(a, b, out, rows, N)) {
            constexpr int kWaves = MODE == kScanGate ? 16 : 4;  // (scan_four_waves of one chunk and few workgroups)
            P = (N + kScanChunk - 1) / kScanChunk;
            hipLaunchKernelGGL((scan_rows_alone_kernel<REVERSE, MODE, kWaves>), dim3((unsigned)(rows * P)), dim3(64 * kWaves), 0, s, a, b, out, N, eps, P,
                               by_runs);
            return;
        }
        seg_len = N;
        P = 1;
    }
    const unsigned wgs = (unsigned)(rows * P);
    if (scan_four_waves(MODE == kScanGate, P > 1, wgs, seg_len))
        hipLaunchKernelGGL((scan_rows_kernel<REVERSE, MODE, 4>), dim3(wgs), dim3(256), 0, s, a, b, out, N, eps, partial, seg_len, P);
    else
        hipLaunchKernelGGL((scan_rows_kernel<REVERSE, MODE, 16>), dim3(wgs), dim3(1024), 0, s, a, b, out, N, eps, partial, seg_len, P);
}
template <bool REVERSE, int MODE>
static void launch_segment_sum(const float* a, const float* b, double* partial, int rows, int N, float eps, int seg_len, int P, hipStream_t s) {
    const unsigned wgs = (unsigned)(rows * P);
    if (MODE != kScanGate && seg_len <= 2 * kScanChunk)
        hipLaunchKernelGGL((segment_sum_kernel<REVERSE, MODE, 4>), dim3(wgs), dim3(256), 0, s, a, b, partial, N, eps, seg_len, P);
    else
        hipLaunchKernelGGL((segment_sum_kernel<REVERSE, MODE, 16>), dim3(wgs), dim3(1024), 0, s, a, b, partial, N, eps, seg_len, P);
}

hipError_t gate_prefix(const float* alpha, float* c, int rows, int N, hipStream_t s) {
    ProfScope prof(kKernGatePrefix, s);
    launch_scan<false, kScanPlain>(alpha, nullptr, c, rows, N, 0.f, nullptr, 0, 1, true, s);
    return hipGetLastError();
}

hipError_t gate_activation_prefix(const float* hpre, const float* beta, float eps, float* c, int rows, int N,
                                  hipStream_t s) {
    ProfScope prof(kKernGateActPrefix, s);
    launch_scan<false, kScanGate>(hpre, beta, c, rows, N, eps, nullptr, 0, 1, true, s);
    return hipGetLastError();
}

// Scan-then-propagate for few, very long rows: P segments per row, each a workgroup of its own.
int scan_segments(int rows, int N, int* seg_len) {
    const int chunks = (N + kScanChunk - 1) / kScanChunk;
    int P = (kScanTargetWorkgroups + rows - 1) / rows;
    if (P > chunks) P = chunks;
    if (P < 1) P = 1;
    const int seg_chunks = (chunks + P - 1) / P;
    *seg_len = seg_chunks * kScanChunk;
    return (chunks + seg_chunks - 1) / seg_chunks;
}

size_t gate_scan_workspace_bytes(int rows, int N) {
    return (size_t)rows * ((N + kScanChunk - 1) / kScanChunk) * sizeof(double);  // at most one segment per chunk
}

hipError_t gate_prefix_stp(const float* in, const float* beta, float eps, float* c, double* partial, int rows,
                           int N, hipStream_t s) {
    if (scan_in_one_launch(beta != nullptr, rows, N) && (N <= kScanChunk || !scan_in_place(in, beta, c, rows, N))) {
        ProfScope prof(beta != nullptr ? kKernGateActPrefix : kKernGatePrefix, s);
        if (beta != nullptr) launch_scan<false, kScanGate>(in, beta, c, rows, N, eps, nullptr, 0, 1, false, s);
        else launch_scan<false, kScanPlain>(in, nullptr, c, rows, N, 0.f, nullptr, 0, 1, false, s);
        return hipGetLastError();
    }
    int seg_len = 0;
    const int P = scan_segments(rows, N, &seg_len);
    {
        ProfScope prof(kKernScanSegmentSum, s);
        if (beta != nullptr) launch_segment_sum<false, kScanGate>(in, beta, partial, rows, N, eps, seg_len, P, s);
        else launch_segment_sum<false, kScanPlain>(in, beta, partial, rows, N, eps, seg_len, P, s);
    }
    {
        ProfScope prof(kKernScanPropagate, s);
        if (beta != nullptr) launch_scan<false, kScanGate>(in, beta, c, rows, N, eps, partial, seg_len, P, false, s);
        else launch_scan<false, kScanPlain>(in, beta, c, rows, N, eps, partial, seg_len, P, false, s);
    }
    return hipGetLastError();
}

// d(alpha) -> d(h), d(beta): elementwise chain rule on the gate's definition
//   sigma = 1 / (1 + exp(-z)),  d alpha/d h = sigma beta / (beta + eps),
//   d alpha/d beta = sigma h / (beta + eps) - softplus(z) / (beta + eps)^2
__device__ __forceinline__ void gate_grad(float h, float b, float g, float eps, float& dh, float& dbeta) {
    const float z = b * h;
    float e;
    const float sp = softplus_parts(z, &e);
    const float sig = (z >= 0.f ? 1.0f : e) * __builtin_amdgcn_rcpf(1.0f + e);  // sigma(z), no overflow
    const float rbe = __builtin_amdgcn_rcpf(b + eps);
    const float gs = g * sig * rbe;
    dh = gs * b;
    dbeta = gs * h - g * sp * rbe * rbe;
}

// VEC: every pointer is 16-byte aligned, the body moves float4; the last n % 4 elements go one by one
template <bool VEC>
__global__ __launch_bounds__(256) void gate_activation_bwd_kernel(const float* __restrict__ hpre,
                                                                  const float* __restrict__ beta,
                                                                  const float* __restrict__ dalpha,
                                                                  float* __restrict__ dh,
                                                                  float* __restrict__ dbeta, size_t n, float eps) {
    const size_t tid = (size_t)blockIdx.x * 256 + threadIdx.x, nthr = (size_t)gridDim.x * 256;
    const size_t n4 = VEC ? n / 4 : 0;
    for (size_t i = tid; i < n4; i += nthr) {
        const float4 h = reinterpret_cast<const float4*>(hpre)[i];
        const float4 b = reinterpret_cast<const float4*>(beta)[i];
        const float4 g = reinterpret_cast<const float4*>(dalpha)[i];
        float4 oh, ob;
        gate_grad(h.x, b.x, g.x, eps, oh.x, ob.x);
        gate_grad(h.y, b.y, g.y, eps, oh.y, ob.y);
        gate_grad(h.z, b.z, g.z, eps, oh.z, ob.z);
        gate_grad(h.w, b.w, g.w, eps, oh.w, ob.w);
        reinterpret_cast<float4*>(dh)[i] = oh;
        reinterpret_cast<float4*>(dbeta)[i] = ob;
    }
    for (size_t i = n4 * 4 + tid; i < n; i += nthr) gate_grad(hpre[i], beta[i], dalpha[i], eps, dh[i], dbeta[i]);
}

hipError_t gate_activation_backward(const float* hpre, const float* beta, float eps, const float* dalpha,
                                    float* dh, float* dbeta, size_t n, hipStream_t s) {
    ProfScope prof(kKernGateActBwd, s);
    const bool vec = (((uintptr_t)hpre | (uintptr_t)beta | (uintptr_t)dalpha | (uintptr_t)dh | (uintptr_t)dbeta) & 15) == 0;
    const size_t want = ((vec ? n / 4 + 3 : n) + 255) / 256;
    const unsigned grid = (unsigned)(want < 8192 ? (want ? want : 1) : 8192);
    if (vec)
        hipLaunchKernelGGL(gate_activation_bwd_kernel<true>, dim3(grid), dim3(256), 0, s, hpre, beta, dalpha, dh,
                           dbeta, n, eps);
    else
        hipLaunchKernelGGL(gate_activation_bwd_kernel<false>, dim3(grid), dim3(256), 0, s, hpre, beta, dalpha, dh,
                           dbeta, n, eps);
    return hipGetLastError();
}

// Few long rows leave most of the chip idle with one workgroup per row: then the rows are cut into segments
// (scan-then-propagate, as gate_prefix_stp does for the forward prefix), which needs `partial`.
bool gate_grad_scan_wants_segments(int rows, int N) {
    return rows < device_cu_count() && N >= 2 * kScanChunk && !scan_in_one_launch(false, rows, N);
}

hipError_t gate_grad_scan(const float* dc_col, const float* dc_row, float* dalpha, double* partial, int rows, int N,
                          hipStream_t s) {
    if (partial != nullptr && gate_grad_scan_wants_segments(rows, N)) {
        int seg_len = 0;
        const int P = scan_segments(rows, N, &seg_len);
        {
            ProfScope prof(kKernGateGradSegmentSum, s);
            launch_segment_sum<true, kScanDiff>(dc_col, dc_row, partial, rows, N, 0.f, seg_len, P, s);
        }
        ProfScope prof(kKernGateGrad, s);
        launch_scan<true, kScanDiff>(dc_col, dc_row, dalpha, rows, N, 0.f, partial, seg_len, P, false, s);
        return hipGetLastError();
    }
    ProfScope prof(kKernGateGrad, s);
    launch_scan<true, kScanDiff>(dc_col, dc_row, dalpha, rows, N, 0.f, nullptr, 0, 1, false, s);
    return hipGetLastError();
}

}  // namespace gfwa
