// Internal declarations shared by the HIP sources of libultratex.so.
#pragma once

// Host-side declarations only (api.cpp builds with a plain C++ compiler too);
// the kernel sources include hip_runtime.h themselves.
#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "ultratex.h"

namespace ut {

// Records a message for ut_last_error() and returns `st`.
ut_status fail(ut_status st, const char* fmt, ...);
// Maps a HIP error (if any) to UT_ERR_HIP with context; UT_OK otherwise.
ut_status check_hip(hipError_t e, const char* what);

// Brackets the kernel launches of its lifetime with HIP events on `s` while
// tracing is on (ut_trace_enable); name base<a,b> (a, b < 0: omitted).
class TraceScope {
 public:
  TraceScope(hipStream_t s, const char* base, int a = -1, int b = -1);
  ~TraceScope();
  TraceScope(const TraceScope&) = delete;
  TraceScope& operator=(const TraceScope&) = delete;

 private:
  hipStream_t stream_;
  hipEvent_t start_ = nullptr;
  char name_[48] = "";
};

// Host checks of the validate mode, on host copies of the arguments.
// Compressed lists: ptr[0] = 0, ptr non-decreasing, ptr[rows] = n_idx, and
// every row strictly ascending within [0, limit). With idx = NULL only the
// first two properties are checked.
ut_status check_lists(const char* fn, const char* what, const int32_t* ptr, const int32_t* idx,
                      int64_t n_idx, int64_t rows, int32_t limit);
// Sample offsets: cu[0] = 0, cu[B] = T, non-decreasing, no sample > max_seqlen.
ut_status check_cu_seqlens(const char* fn, const int32_t* cu, int32_t B, int64_t T,
                           int32_t max_seqlen);

// ---- Background Token Dropping (btd.hip) ----
constexpr int kCompactTile = 4096;   // mask bytes per workgroup of the scan
int64_t compact_tiles(int64_t L);
hipError_t launch_compact(const uint8_t* mask, int64_t L, int64_t capacity, int32_t* kept_idx,
                          int32_t* inv_idx, int32_t* n_kept, int32_t* tile_scratch,
                          hipStream_t s);
hipError_t launch_gather(const void* x_full, int64_t row_bytes, void* x_packed, int64_t capacity,
                         const int32_t* kept_idx, const int32_t* n_kept, hipStream_t s);
hipError_t launch_scatter(const void* x_packed, const int32_t* kept_idx, int64_t n_kept,
                          int64_t row_bytes, void* x_full, hipStream_t s);

// ---- Block index (block_index.hip) ----
hipError_t launch_block_index(const uint8_t* mask, int B, int H, int Nq, int Nk,
                              int32_t* q_rowptr, int32_t* q_cols, int32_t* kv_colptr,
                              int32_t* kv_rows, int64_t cap, hipStream_t s);

// ---- Attention (bsattn_fwd.hip, bsattn_bwd.hip) ----
struct AttnShape {
  int B, N, H, D, block, nblk;   // N: tokens per sample (the longest, with cu)
  float scale;
  const int32_t* cu = nullptr;   // [B + 1] sample offsets, or null for a uniform batch
  int64_t T = 0;                 // packed tokens (B N when uniform)
};
// Whether the attention kernels give each XCD whole heads (tile_of) or take
// the tiles in plain order, all XCDs on the same heads. A workgroup streams
// two [N, D] tensors of its head (K and V, or Q and dO): with whole heads an
// XCD's workgroups share them in its own 4 MiB of L2, in plain order every
// XCD reads every head from the last-level cache behind the L2s. Measured in
// ms, plain / by head: forward at 24 x 6,552 x 128 (3.4 MB a head) 0.181 /
// 0.169, dK/dV at 32 x 9,011 x 64 (2.3 MB) 0.312 / 0.303, dense forward at
// 24 x 12,801 x 128 (6.6 MB) 1.91 / 1.89, but forward at 24 x 77,586 x 128
// (39 MB) 7.05 / 7.52 and dK/dV there 13.4 / 13.9: eight heads at once then
// overflow the last-level cache too. The head count has to divide by 8 so
// that every XCD gets as many heads of every sample, and the eight heads that
// run side by side have to be alike (heads_alike, below).
constexpr int64_t kXcdHeadBytes = (int64_t)8 << 20;
inline bool heads_by_xcd(const AttnShape& sh) {
  return sh.H % 8 == 0 && (int64_t)sh.N * sh.D * 4 <= kXcdHeadBytes;
}
// The same for dQ from the stored tiles. By head an XCD reads the tiles that it
// wrote itself, and finds them in its L2 where a head's fit: plain / by head 35 / 31
// us at 24 x 2,000 x 128 with block 64, density 0.4 (3.4 MB of tiles a head), 75 / 71
// at 6,000, 0.1 (7.5), 31 / 29 at 24 x 4,000 x 64, 0.1 (3.5), but 86 / 91 there at
// 0.4 (13), 84 / 88 at 8,000, 0.1 (13), 161 / 173 at 6,000 x 64 with block 128, 0.4
// (29) and 1,060 / 1,164 at 22,879 x 64. At head_dim 128, block 128, it is never
// behind: 181 / 178 at 24 x 6,552 (27), 545 / 542 at 15,000 (90). `pairs`: the room
// for tiles, which is all that is known of their number here.
constexpr int64_t kXcdTileBytes = (int64_t)8 << 20;
inline bool stored_dq_by_head(const AttnShape& sh, int64_t pairs) {
  return heads_by_xcd(sh) && ((sh.D == 128 && sh.block == 128) ||
                              pairs * 2 * sh.block * sh.block <= kXcdTileBytes * sh.B * sh.H);
}
// Whether a column list of n entries, of `all` entries in the launch, is a serial
// chain more than twice as long as what each of the 512 workgroups that fit takes
// (so fewer than 256 lists are). Backward with stored tiles, one dense column in
// each head, chains with the 64-key pass / apart in ms (32-key pass for all lists):
// 24 x 22,879, lists of 9, 2.08 / 2.06 and 2.12 / 2.06 (2.00, column 7 and 170);
// of 3, 1.54 / 1.45 (1.40); 24 x 12,000, lists of 5, 0.911 / 0.893 (0.868);
// 24 x 77,060, lists of 9, 7.93 / 7.44 (7.50); 4 heads, lists of 30, 5.33 / 5.00
// (4.99). Looking for chains costs about 10 us where there are none.
constexpr bool chain_list(int64_t n, int64_t all) { return n * 256 > all; }
// First tile of the group of eight heads (8 nblk workgroups in a row) that
// workgroup wg, of head wg / nblk in plain order, belongs to.
constexpr unsigned group_tile(unsigned head, unsigned nblk) { return (head & ~7u) * nblk; }
// Workgroups go round-robin to the 8 XCDs, so in a group workgroup 8 k + x is
// the k-th of XCD x: by head it takes tile k of the group's head x.
constexpr unsigned head_tile(unsigned wg, unsigned first, unsigned nblk) {
  return first + ((wg - first) & 7) * nblk + ((wg - first) >> 3);
}
// Whether the longest of the group's eight heads, by list entries (at(x): list
// offset of head x's first tile, at(8) the group's end), is within 1/32 of their mean: by head the XCD with the
// longest one ends last. Heads that keep equally many blocks, as Top-K
// selection gives, are equal. Taken by head all the same, one dense head among
// 8 (6,552 x 128, the others 3 blocks a row) took 166 us in the forward where
// plain order takes 124, and three dense ones on one XCD among 24 took 415
// where it takes 186; even heads gain 2 to 7%, hence the small margin.
template <typename At>
constexpr bool heads_alike(At at) {
  int32_t most = 0;
  for (int x = 0; x < 8; ++x) {
    const int32_t n = at(x + 1) - at(x);
    most = n > most ? n : most;
  }
  const int64_t total = (int64_t)at(8) - at(0);
  return 32 * (8 * (int64_t)most - total) <= total;
}
hipError_t launch_bsattn_fwd(const void* q, const void* k, const void* v, void* o, float* lse,
                             const AttnShape& sh, const int32_t* rowptr, const int32_t* cols,
                             hipStream_t s);
// Where the backward keeps stored dS tiles (max_pairs = 0: none; dQ is then
// recomputed for every query block).
struct DsTiles {
  int32_t* row_ok = nullptr;   // [B H Nq] query block takes dQ from the tiles
  int32_t* map = nullptr;      // [max_pairs] row-list entry -> tile (column-list position)
  char* tiles = nullptr;       // [max_pairs][2 block^2] bf16 dS
  int64_t max_pairs = 0;
};
// Backward. `aux` holds the two statistics planes (8 bytes per query row).
hipError_t launch_bsattn_bwd(const void* q, const void* k, const void* v, const void* o,
                             const void* dout, const float* lse, void* dq, void* dk, void* dv,
                             const AttnShape& sh, const int32_t* rowptr, const int32_t* cols,
                             const int32_t* colptr, const int32_t* rows, float* aux,
                             const DsTiles& ds, hipStream_t s);

// Scratch of ut_bsattn_bwd_noalloc: a file-scope device array in
// bsattn_bwd.hip, one copy per GPU, holding the backward's two statistics
// planes (8 bytes per query row).
constexpr size_t kNoallocScratchBytes = (size_t)32 << 20;
// Device address of that array on the device that `s` belongs to (the current
// device for the null stream), looked up once per device.
hipError_t noalloc_scratch(hipStream_t s, float** ptr);

// ---- Top-K block selection (topk_mask.hip) ----
constexpr int64_t kTopkMaxLds = 65536;   // LDS bytes of one selection workgroup
// Query blocks per selection workgroup (16, 4 or 1), 0 if one row does not fit.
int topk_rows_per_group(int D, int nblk);
hipError_t launch_topk_block_mask(const void* q, const void* k, int B, int N, int H, int D,
                                  int block, int k_keep, int prefix, uint8_t* mask, float* pooled,
                                  hipStream_t s);

// ---- Foreground Euler update and loss (fg_step.hip) ----
constexpr int kLossParts = 1024;   // partial sums of the loss (fixed order)
hipError_t launch_euler_fg(float* z, int64_t L, int64_t C, const void* v, bool v_bf16,
                           const int32_t* kept, int64_t n, float dt, hipStream_t s);
hipError_t launch_fg_loss(const void* v, bool v_bf16, const void* eps, const void* z0,
                          bool x_bf16, int64_t L, int64_t C, const int32_t* kept, int64_t n,
                          float* loss, float* grad, double* partial, hipStream_t s);

// ---- Composite latent and token masks (composite.hip) ----
hipError_t launch_composite(const void* packed, int64_t n_kept, const int32_t* inv, int64_t L,
                            const void* bg, int64_t bg_rows, int64_t row_bytes, void* out,
                            hipStream_t s);
hipError_t launch_token_mask(const uint8_t* alpha, int V, int Hp, int Wp, int patch, int thr,
                             int radius, uint8_t* out, uint8_t* pooled, hipStream_t s);

}  // namespace ut
