// Host-side launchers of the gfx950 kernels (internal; the public ABI is in
// include/moe_resident.h).  Each launcher assumes validated arguments and
// only enqueues work on `stream`; it returns hipGetLastError().
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "common.h"
#include "moe_resident.h"

namespace moe {

hipError_t launch_route_fwd(const void* x, const void* w, const float* bias, int bf16, int T,
                            int d, int E, int k, float inv_tau, int gate, const uint8_t* resident,
                            float* logits, int32_t* idx, float* tw, int32_t* local,
                            hipStream_t s);

size_t route_bwd_ws_bytes(int T, int d, int E);
hipError_t launch_route_bwd(const void* x, const void* w, int bf16, int T, int d, int E, int k,
                            float inv_tau, int gate, const int32_t* idx, const float* tw,
                            const float* logits, const float* dtw, float* dz, float* dw_router,
                            float* d_bias, void* dx, int accumulate_dx, void* ws,
                            hipStream_t s);

size_t dispatch_ws_bytes(int T, int k, int E_r);
hipError_t launch_dispatch(const void* x, int bf16, int T, int d, int k, int E_r,
                           const int32_t* local, int32_t* counts, int32_t* offsets,
                           int32_t* perm, int32_t* inv_perm, void* xp, void* ws, hipStream_t s);
// The same counting sort with its workspace in a library-owned device array
// of kDispatchScratchBytes (one per device); dispatch_ws_bytes() of the call
// must not exceed it.
constexpr size_t kDispatchScratchBytes = MOE_DISPATCH_NOALLOC_MAX_WS;
hipError_t launch_dispatch_noalloc(const void* x, int bf16, int T, int d, int k, int E_r,
                                   const int32_t* local, int32_t* counts, int32_t* offsets,
                                   int32_t* perm, int32_t* inv_perm, void* xp, hipStream_t s);
hipError_t launch_dispatch_bwd(const void* dxp, int bf16, int T, int d, int k, int cap,
                               const int32_t* inv_perm, void* dx, int accumulate, hipStream_t s);

hipError_t launch_combine_fwd(const void* yp, int bf16, int T, int d, int k, int cap,
                              const float* tw, const int32_t* inv_perm, const void* y_add, void* y,
                              hipStream_t s);
hipError_t launch_combine_bwd(const void* dy, const void* yp, int bf16, int T, int d, int k,
                              int cap, const float* tw, const int32_t* inv_perm, void* dyp,
                              float* dtw, hipStream_t s);

// Grouped SwiGLU FFN over 1 or 2 expert sets (moe_ffn_set of the public
// header), one launch per GEMM kind.  ws: NULL (no K parts) or
// ffn_fwd_ws_bytes() bytes, 256-byte aligned; its contents on entry are ignored.
size_t ffn_fwd_ws_bytes(const moe_ffn_set* sets, int n_sets, int bf16, int d);
hipError_t launch_ffn_fwd_sets(const moe_ffn_set* sets, int n_sets, int bf16, int d, void* ws,
                               hipStream_t s);
// ws: NULL (static tile dealing, no split-K) or ffn_bwd_ws_bytes() bytes,
// 256-byte aligned; its contents on entry are ignored.
size_t ffn_bwd_ws_bytes(const moe_ffn_set* sets, int n_sets, int bf16, int d);
hipError_t launch_ffn_bwd_sets(const moe_ffn_set* sets, int n_sets, int bf16, int d,
                               int accumulate_dw, void* ws, hipStream_t s);

int num_cus();

// Blocks (256 threads, 16 bytes per access) of an elementwise stream over n fp32
// elements: a vector per thread, up to 8192 blocks, and per_cu blocks per CU from
// `few` elements on.  Few blocks read and write few DRAM pages at a time, and the
// arrays are far larger than the caches; but enough loads have to be in flight, and
// of small arrays the many blocks' are quicker.  Measured (us, nothing in the caches):
//   256 / 512 / 1024 / 8192 blocks   8 M              25 M                    138 M
//   AdamW                     52 / 52 / 55 / 49  143 / 136 / 152 / 140  746 / 788 / 865 / 954
//   outer step                40 / 40 / 42 / 40  114 / 116 / 126 / 119  660 / 667 / 794 / 887
// Delta and mean add the peers one after another, so a thread has few loads in flight:
//   512 / 1024 / 4096 / 8192 blocks
//   delta of 1 peer           33 / 31 / 32 / 32   88 / 88 / 91 / 88    501 / 501 / 586 / 610
//   delta of 3                50 / 41 / 42 / 43  140 / 115 / 122 / 125 774 / 675 / 751 / 767
//   delta of 7                84 / 64 / 67 / 66  245 / 183 / 198 / 206 1369 / 1079 / 1137 / 1160
//   mean of 1                 25 / 20 / 20 / 21   68 / 50 / 51 / 52    359 / 269 / 277 / 283
//   mean of 3                 43 / 31 / 30 / 30  118 / 82 / 85 / 85    664 / 484 / 474 / 499
//   mean of 7                 76 / 52 / 51 / 51  222 / 152 / 150 / 155 1249 / 910 / 892 / 892
// (4 M, mean of 7: 28 us with 1024 blocks, 27 with 8192; 67 M, mean of 15: 862 with
// 1024, 790 with 4096.  1280 blocks against 1024, 138 M: mean of 3 454 against 483, of 7
// 852 against 919, delta of 3 684 against 698.  Four peers' loads at once were slower
// at every number of blocks but the smallest, whose times hang on where the arrays
// lie: mean of 7, 25 M, 158 to 183, delta of 3, 138 M, 667 to 827 with 256 blocks.)
inline int stream_blocks(size_t n, size_t few, int per_cu) {
  const size_t want = (n / 4 + 255) / 256;
  const size_t most = n < few ? 8192 : (size_t)num_cus() * per_cu;
  return (int)std::max<size_t>(1, std::min<size_t>(want, most));
}
// AdamW and the outer step; the delta and the mean over peers.
constexpr size_t kFewBlocks = 16u << 20, kFewBlocksPeers = 8u << 20;
inline int peer_stream_blocks(size_t n, int n_peers, int per_cu) {
  return stream_blocks(n, kFewBlocksPeers, n_peers <= 7 ? per_cu : 16);
}

constexpr int kMaxPeers = 16;
hipError_t launch_expert_delta(const float* start, const float* now, const float* const* peers,
                               int n_peers, size_t n, float* dl, float* avg, hipStream_t s);

// Optimisers (optim.hip); c1, c2 = the step's AdamW bias corrections.
hipError_t launch_adamw(float* theta, const float* grad, float* m, float* v, size_t n, float lr,
                        float beta1, float beta2, float eps, float wd, float c1, float c2,
                        void* theta_bf16, hipStream_t s);
hipError_t launch_outer_nesterov(float* start, float* now, const float* delta, float* mom,
                                 size_t n, float lr, float mu, void* theta_bf16, hipStream_t s);
hipError_t launch_replica_mean(const float* local, const float* const* peers, int n_peers,
                               size_t n, float* out, hipStream_t s);

// Placement and migration (placement.hip).  gen_placement: false when the
// constraints cannot be met.  launch_copy_expert_rows: src_row / dst_row are
// host arrays of n_rows <= 256 entries (dst_row NULL = 0..n_rows-1).
bool gen_placement(int N_e, int O_e, int M, const int32_t* expert_perm,
                   const int32_t* worker_perm, int32_t* sets);
hipError_t launch_copy_expert_rows(const float* src, const int32_t* src_row, float* dst,
                                   const int32_t* dst_row, int n_rows, size_t row_len,
                                   void* dst_bf16, hipStream_t s);

}  // namespace moe
