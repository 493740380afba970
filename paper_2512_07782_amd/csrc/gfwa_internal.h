// Host-side launch functions behind the C ABI (one per kernel family).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace gfwa {

// Whether two ranges of bytes share one: outputs that a caller puts over inputs do not serve as scratch before these are read.
inline bool overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
    return (const char*)a < (const char*)b + b_bytes && (const char*)b < (const char*)a + a_bytes;
}

// c = inclusive prefix sum of alpha along N, one row per (b,h).
hipError_t gate_prefix(const float* alpha, float* c, int rows, int N, hipStream_t s);
hipError_t gate_activation_prefix(const float* hpre, const float* beta, float eps, float* c, int rows, int N,
                                  hipStream_t s);
hipError_t gate_activation_backward(const float* hpre, const float* beta, float eps, const float* dalpha,
                                    float* dh, float* dbeta, size_t n, hipStream_t s);
// The same prefix (beta == nullptr: of `in` itself; else of the gate activation of (in, beta)) in two
// launches that cut every row into segments (scan-then-propagate); partial: gate_scan_workspace_bytes().
size_t gate_scan_workspace_bytes(int rows, int N);
hipError_t gate_prefix_stp(const float* in, const float* beta, float eps, float* c, double* partial, int rows,
                           int N, hipStream_t s);
// dalpha = reverse inclusive prefix sum of (col - row) along N.  partial: gate_scan_workspace_bytes(rows, N) of
// scratch (or nullptr); with it, few long rows are scanned in segments.
hipError_t gate_grad_scan(const float* dc_col, const float* dc_row, float* dalpha, double* partial, int rows, int N,
                          hipStream_t s);

// Q, O, dO, dQ: [B,H,N,d]; K, V, dK, dV: [B,Hkv,N,d] with Hkv dividing H (query head h reads head h / (H/Hkv));
// c, L, dalpha: [B,H,N].
hipError_t forward_bf16(const void* Q, const void* K, const void* V, const float* c, void* O, float* L,
                        int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s);
double query_tile_fill(int BH, int N, int w, long slots);  // how full rounds of `slots` 128-query tiles are, 0 .. 1
// The same for few or uneven query tiles, the band of a tile split over groups of waves (fwd_split_bf16.hip).
enum FwdSplit { kFwdSplitNone = 0, kFwdSplitNarrow, kFwdSplitMid, kFwdSplitWide };  // 32, 64, 128 queries per workgroup
hipError_t forward_split_bf16(FwdSplit shape, const void* Q, const void* K, const void* V, const float* c, void* O,
                              float* L, int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s);
// Values of the key blocks in front of the forward's query tiles (band_reach.h), in O.
// key_reach: launches the pass for tiles of `tile` queries if it pays, and says by what blocks (0: it does not) and how many keys have to be
// erased for reading their norms to pay.
struct KeyReach {
    int block, few;
};
hipError_t key_reach(KeyReach& reach, int tile, bool bf16, const void* Q, const void* K, const void* V, const float* c, void* O, int B, int H, int Hkv,
                     int N, int d, int w, float scale, hipStream_t s);
hipError_t forward_f32(const float* Q, const float* K, const float* V, const float* c, float* O,
                       float* L, int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s);

// Arguments of the bf16 backward kernels (device pointers and sizes as in gfwa_backward_gqa; Dv, dc_col, dc_row: workspace).
struct BwdBf16 {
    const __bf16 *Q, *K, *V, *O, *dO;
    const float *c, *L;
    float* Dv;
    __bf16 *dQ, *dK, *dV;
    float *dc_col, *dc_row;
    const float* reach;  // norms of the row blocks (band_reach.h), or nullptr
    int B, H, Hkv, N, w;
    float scale;
};
constexpr int kDkvSplitMaxGroup = 8;  // query heads per key/value head bwd_dkv_split_bf16 has room for
// The two passes for few or uneven tiles (bwd_split_bf16.hip).  The dQ pass also forms D_t, so it goes first.
hipError_t bwd_dq_split_bf16(FwdSplit shape, const BwdBf16& a, int d, hipStream_t s);
hipError_t bwd_dkv_split_bf16(const BwdBf16& a, int d, hipStream_t s);
hipError_t bwd_both_split_bf16(const BwdBf16& a, int d, hipStream_t s);  // in one launch

// Workspace layout of the backward: three fp32 vectors of B*H*N (each padded to 256 bytes): D, dc_col,
// dc_row; gate_scan_workspace_bytes(B*H, N) (padded to 256) of segment sums for the gate-gradient scan; with `spill` (bf16, d = 128 only) backward_bf16_spill_bytes() more for the dS blocks.
size_t backward_bf16_spill_bytes(int B, int H, int N, int d, int w);  // 0: no such variant for this shape
hipError_t backward_bf16(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                         const float* c, const float* L, void* dQ, void* dK, void* dV, float* dalpha,
                         float* ws, bool spill, int B, int H, int Hkv, int N, int d, int w, float scale,
                         hipStream_t s);
hipError_t backward_f32(const float* Q, const float* K, const float* V, const float* O, const float* dO,
                        const float* c, const float* L, float* dQ, float* dK, float* dV, float* dalpha,
                        float* ws, int B, int H, int Hkv, int N, int d, int w, float scale, hipStream_t s);

// Decoding step: q, o [B,H,d]; caches Kc, Vc [B,Hkv,T,d]; c [B,H,T] (entry pos[b] written when alpha_t is
// given); pos [B] device ints; part: decode_workspace_bytes() of scratch.
size_t decode_workspace_bytes(int B, int H, int Tlen, int d, int w);
hipError_t decode(bool bf16, const void* q, const void* Kc, const void* Vc, float* c, const float* alpha_t,
                  const int* pos, void* o, float* L, float* part, int B, int H, int Hkv, int Tlen, int d, int w,
                  float scale, hipStream_t s);

// Device address, on the current device, of the library's own decode scratch of kDecodeStaticBytes
// (looked up on the first call per device, no allocation).
constexpr size_t kDecodeStaticBytes = (size_t)32 << 20;
hipError_t decode_static_scratch(float** ptr);

// Calibration kernels (probe.hip): a pure bf16 MFMA loop and a plain 16-byte copy.
hipError_t probe_mfma(float* sink, int iterations, int workgroups, int random_operands, double* flops, hipStream_t s);
hipError_t probe_copy(const void* src, void* dst, size_t bytes, hipStream_t s);

// Kernel ids for the optional per-kernel event timing (see gfwa_profile_* in include/gfwa.h).
enum KernelId { kKernGatePrefix = 0, kKernForward, kKernRowDot, kKernDkv, kKernDq, kKernGateGrad, kKernGateActPrefix,
                kKernGateActBwd, kKernDecode, kKernDecodeCombine, kKernScanSegmentSum,
                kKernScanPropagate, kKernGateGradSegmentSum, kKernCount };

// Per-device launch set-up, done once per device and kernel (`done`: one bit per device id, owned by the caller):
// lets `kernel` use `bytes` of dynamic LDS on the current device.
struct DeviceOnce { unsigned long long bits = 0; };
hipError_t allow_dynamic_lds(const void* kernel, size_t bytes, DeviceOnce& done);
// Compute units of the current device (256 if the query fails).
int device_cu_count();

// RAII pair of HIP events around one kernel launch on stream s; a no-op unless profiling is on.
struct ProfScope {
    ProfScope(int kernel, hipStream_t s);
    ~ProfScope();
    int slot_;
    hipStream_t s_;
};


}  // namespace gfwa
