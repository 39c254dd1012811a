// Block lists from a binary block mask on gfx950 (paper Sec. 3.3, Eq. 7 and
// the selected sets S_i of Eq. 8).
//
// Row lists (S_i, ascending j) feed the forward and the dQ pass; column lists
// (query blocks selecting key block j, ascending i) feed the dK/dV pass. Both
// are built without atomics, so the output is unique and deterministic, in
// two launches:
//   1. the count of every row and every column, stored as ~count in the
//      pointer array (negative, so that it can't be taken for an offset);
//   2. fill: each workgroup adds up the counts before its own rows or columns,
//      replaces its own counts by offsets, and writes its lists.
// A list array of more than kPrefixMax entries takes a scan launch in between
// (one workgroup per array) instead of the sums in launch 2.
// Launches 1 and 2 each build both kinds of list: their first workgroups take
// a 64-column slab of one (b, h) each (column lists), the rest take 64 mask
// rows each (row lists). Lists are put together in LDS and written coalesced: a
// row by its wave, a slab's columns, one contiguous run of the output, by the
// workgroup.
#include <hip/hip_runtime.h>

#include "common.h"

namespace ut {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kRowCols = 1024;    // columns of a row per load: 16 a lane
constexpr int kRowsPerWave = 4;   // mask rows per wave in the row lists
constexpr int kLists = 64;        // lists per workgroup: rows, or columns of a slab
static_assert(kLists == kWaves * kRowsPerWave, "row lists per workgroup");
constexpr int kPrefixPer = 16;    // counts per thread of the sums in the fill
// At 14,472 rows and columns (24 heads, 603 blocks, density 0.1) the sums add
// about 4 us to the fill and save a scan launch of 7.8 us. The two launches now
// take 11.7 + 15.3 us there between events (8.9 + 12.7 in a kernel trace; three
// launches, with a load per mask byte and a store per 64 columns, between events:
// 11.3 + 7.8 + 23.7); both are bound by the vector instructions and the latencies
// of one pass over 8.7 MB, not by bandwidth.
constexpr int64_t kPrefixMax = kPrefixPer * kThreads;
// Entries (uint16) of a slab's columns that LDS holds; longer runs, and block
// indices past 65535, are written straight to the output. Such columns are
// dense, so that their stores are nearly coalesced as they are.
constexpr int kStage = 28 * 1024;

__device__ inline uint64_t lanes_below_mask() {
  const int lane = threadIdx.x & 63;
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// kBytes mask bytes (4 or 16) at `at`, any alignment, of a mask of `total`
// bytes; bytes past the mask read as 0. One unguarded load, clamped to the
// mask's last kBytes (a guarded load is waited for before the next one is
// issued); past_end then shifts what was clamped into place, for the few waves
// that read there. A mask shorter than kBytes is read byte by byte.
// Offsets fit 32 bits (masks stay below 2^31 bytes), which keeps the addresses
// of many loads in few registers.
template <int kBytes, bool kTiny, typename T>
__device__ inline T load_bytes(const uint8_t* __restrict__ mask, uint32_t at, uint32_t total) {
  T x = {};
  if constexpr (kTiny) {
    uint32_t w[kBytes / 4] = {};
    for (uint32_t b = 0; b < kBytes; ++b)
      if (at + b < total) w[b / 4] |= (uint32_t)mask[at + b] << (8 * (b % 4));
    __builtin_memcpy(&x, w, kBytes);
  } else {
    __builtin_memcpy(&x, mask + min(at, total - kBytes), kBytes);
  }
  return x;
}
__device__ inline void past_end(uint32_t& x, uint32_t at, uint32_t total) {
  if (at <= total - 4) return;
  x = at < total ? x >> (8 * (at + 4 - total)) : 0u;
}
__device__ inline void past_end(u32x4& x, uint32_t at, uint32_t total) {
  if (at <= total - 16) return;
  const uint32_t gone = at < total ? at + 16 - total : 16;   // bytes before `at` in x
  for (uint32_t b = 0; b < gone / 4; ++b) x = u32x4{x[1], x[2], x[3], 0u};
#pragma unroll
  for (int e = 0; e < 4; ++e)   // (the double word above the last is 0)
    x[e] = (uint32_t)((((uint64_t)(e < 3 ? x[e + 1] : 0u) << 32) | x[e]) >> (8 * (gone % 4)));
}

// Bit 8 b + 7 set when byte b of x is nonzero.
__device__ inline uint32_t nonzero_bytes(uint32_t x) {
  return (((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u;
}

// Between the LDS writes of a wave's lanes and the reads of others of its
// lanes: the hardware runs a wave's LDS operations in order, the fences keep the
// compiler from moving them across (wave_barrier alone orders no memory).
__device__ inline void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive sum over the wave's lanes.
__device__ inline int wave_scan(int x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

__device__ inline uint64_t readlane64(uint64_t v, int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

struct FillShared {
  int off[kLists + 1];   // offsets of this workgroup's lists
  int red[kWaves];
  uint16_t stage[kStage];
};

// Offsets of the workgroup's lists l0 .. l0 + n - 1 into sh.off[0 .. n]. With
// kScanned ptr holds offsets already. Otherwise it holds ~count for the lists
// that no workgroup has converted yet and offsets for the others: a thread may
// see either, each one 4-byte value. The last offset seen before l0 (ptr[0] = 0
// is one from the start) plus the counts after it is this workgroup's base.
// Its own lists' counts are converted by itself alone, after the reads.
template <bool kScanned>
__device__ __forceinline__ void list_offsets(int32_t* ptr, int64_t l0, int n, FillShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if constexpr (kScanned) {
    if (tid <= n) sh.off[tid] = ptr[l0 + tid];
    __syncthreads();
    return;
  }
  const int own = tid < n ? ~ptr[l0 + 1 + tid] : 0;
  // entries 1 + 4 tid + 4096 k + (0..3), clamped to the array's start instead
  // of guarded, so that all loads are in flight at once; 0 counts past l0
  u32x4 v[kPrefixPer / 4];
  if (l0 >= 4) {   // entries 0..3 exist
#pragma unroll
    for (int k = 0; k < kPrefixPer / 4; ++k) {
      const int x = 1 + 4 * tid + 4 * kThreads * k;
      __builtin_memcpy(&v[k], ptr + (x + 3 <= l0 ? x : 0), sizeof(u32x4));
    }
  }
  uint32_t all = ~0u;   // its sign stays while only counts are seen
  int sum = 0;
#pragma unroll
  for (int k = 0; k < kPrefixPer / 4; ++k) {
    const int x = 1 + 4 * tid + 4 * kThreads * k;
    if (x + 3 > l0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[k][e] = x + e <= l0 ? (uint32_t)ptr[x + e] : ~0u;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      all &= v[k][e];
      sum += (int)~v[k][e];
    }
  }
  if (__syncthreads_or((int)all >= 0)) {   // some list before l0 is converted
    int seen = 0;
#pragma unroll
    for (int k = 0; k < kPrefixPer; ++k)
      if ((int)v[k / 4][k % 4] >= 0) seen = 1 + 4 * tid + 4 * kThreads * (k / 4) + k % 4;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) seen = max(seen, __shfl_xor(seen, o, 64));
    if (lane == 0) sh.red[w] = seen;
    __syncthreads();
    for (int x = 0; x < kWaves; ++x) seen = max(seen, sh.red[x]);
    sum = 0;
#pragma unroll
    for (int k = 0; k < kPrefixPer; ++k) {
      const int x = 1 + 4 * tid + 4 * kThreads * (k / 4) + k % 4;
      const int y = (int)v[k / 4][k % 4];
      sum += x > seen ? ~y : x == seen ? y : 0;
    }
    __syncthreads();
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (lane == 0) sh.red[w] = sum;
  __syncthreads();
  if (w == 0) {
    int base = 0;
    for (int x = 0; x < kWaves; ++x) base += sh.red[x];
    const int incl = wave_scan(own);
    if (lane == 0) sh.off[0] = base;
    if (lane < n) {
      sh.off[lane + 1] = base + incl;
      __hip_atomic_store(ptr + l0 + 1 + lane, base + incl, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
}

// The staged run of n entries from offset `base` of the output.
__device__ inline void write_run(const FillShared& sh, int base, int n, int32_t* __restrict__ out,
                                 int64_t cap) {
  for (int k = threadIdx.x; k < n; k += kThreads)
    if ((int64_t)base + k < cap) out[(int64_t)base + k] = sh.stage[k];
}

// Row lists: each wave takes kRowsPerWave consecutive mask rows (of B*H*Nq), 16
// columns per lane: a scan of the lanes' counts places each lane's entries.
template <bool kFill, bool kScanned, bool kTiny>
__device__ __forceinline__ void row_lists(const uint8_t* __restrict__ mask, int64_t rows, int Nk, int32_t* rowptr,
                          int32_t* __restrict__ cols, int64_t cap, int64_t wg, int* __restrict__ next,
                          FillShared* sh) {
  const int64_t w0 = wg * kLists;   // the workgroup's first row
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = w0 + w * kRowsPerWave;
  const int lane = threadIdx.x & 63;
  const int own = (int)min((int64_t)kLists, rows - w0);
  // the next entry of each of the wave's rows, in LDS (the wave's own words)
  int* const at = next + w * kRowsPerWave;
  uint16_t* const mine = kFill ? sh->stage + w * (kStage / kWaves) : nullptr;
  static_assert(kStage / kWaves >= kRowCols, "one row's piece");
  if (lane < kRowsPerWave) at[lane] = kFill ? sh->off[min((int)(r0 - w0) + lane, own)] : 0;
  wave_lds_order();
  const uint32_t total = (uint32_t)rows * Nk;
#pragma unroll 1
  for (int j0 = 0; j0 < Nk && r0 < rows; j0 += kRowCols) {
    const int j = j0 + 16 * lane;   // this lane's 16 columns
    u32x4 f[kRowsPerWave];
#pragma unroll
    for (int q = 0; q < kRowsPerWave; ++q)
      f[q] = load_bytes<16, kTiny, u32x4>(mask, (uint32_t)min(r0 + q, rows - 1) * Nk + j, total);
    if (!kTiny && (uint32_t)min(r0 + kRowsPerWave - 1, rows - 1) * Nk + j0 + 16 * 63 > total - 16) {
#pragma unroll
      for (int q = 0; q < kRowsPerWave; ++q) past_end(f[q], (uint32_t)min(r0 + q, rows - 1) * Nk + j, total);
    }
    // one row at a time, the next ones' bytes moved up
#pragma unroll 1
    for (int q = 0; q < kRowsPerWave && r0 + q < rows; ++q) {
      uint32_t m = 0;   // bit e: column j + e
#pragma unroll
      for (int e = 0; e < 4; ++e)   // the four flags, 7 bits apart, to bits 28..31
        m |= ((nonzero_bytes(f[0][e]) >> 7) * 0x10204080u >> 28) << (4 * e);
      m &= j + 16 <= Nk ? 0xffffu : j < Nk ? (1u << (Nk - j)) - 1u : 0u;
      const int incl = wave_scan(__popc(m)), p = at[q];
      if constexpr (kFill) {
        // the row's piece in the wave's own part of the stage, then coalesced
        int k = incl - __popc(m);
#pragma unroll 1
        for (; m; m &= m - 1) mine[k++] = (uint16_t)(16 * lane + __builtin_ctz(m));
        wave_lds_order();
        const int n = __builtin_amdgcn_readlane(incl, 63);
        for (int x = lane; x < n; x += 64)
          if ((int64_t)p + x < cap) cols[(int64_t)p + x] = j0 + mine[x];
        wave_lds_order();
      }
      if (lane == 63) at[q] = p + incl;
      wave_lds_order();   // before the row's next piece, and the counts below
#pragma unroll
      for (int x = 0; x + 1 < kRowsPerWave; ++x) f[x] = f[x + 1];
    }
  }
  if constexpr (!kFill) {
    if (r0 == 0 && lane == 0) rowptr[0] = 0;
    if (lane < kRowsPerWave && r0 + lane < rows)
      rowptr[r0 + lane + 1] = kScanned ? at[lane] : ~at[lane];
  }
}

// Column lists: the workgroup owns columns j0..j0+63 of one (b, h); lane c is
// column j0 + c. Wave w walks a contiguous range of 64-row tiles and gathers a
// tile's 64 x 64 bits with 16 loads of 4 bytes per lane. The waves' counts,
// added in wave order through LDS, place each wave's rows within its columns'
// lists; filling then takes each lane's set bits in turn into the staged run.
// Lists too long for it take the columns one at a time with the lanes as rows, so
// each column's new entries are written contiguously.
template <bool kFill, bool kScanned, bool kTiny>
__device__ __forceinline__ void col_lists(const uint8_t* __restrict__ mask, int Nq, int Nk, int32_t* colptr,
                          int32_t* __restrict__ rows_out, int64_t cap, int64_t wg, int slabs,
                          int64_t bhs, int* __restrict__ part, uint32_t* __restrict__ turn,
                          FillShared* sh) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t bh = wg / slabs;
  const int j = (int)(wg % slabs) * 64 + lane;
  const bool col_ok = j < Nk;
  const int ntiles = (Nq + 63) / 64;
  const int per = (ntiles + kWaves - 1) / kWaves;
  const int t0 = min(ntiles, w * per), t1 = min(ntiles, t0 + per);
  // Bit r of lane c's result: row 64 t + r of column j0 + c. Lane l first takes
  // rows 16 (l / 16) .. +15 of columns 4 (l % 16) .. +3 with one 4-byte load a
  // row, collects eight rows' flags per byte, and LDS hands each column its
  // eight bytes.
  const uint32_t total = (uint32_t)bhs * Nq * Nk, row0 = (uint32_t)bh * Nq;
  const int jl = (int)(wg % slabs) * 64 + 4 * (lane & 15);
  uint32_t* const my = turn + w * 128;
  auto bits = [&](int t) __attribute__((always_inline)) {
    const int i0 = 64 * t + 16 * (lane >> 4);
    uint32_t f[16];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      f[u] = load_bytes<4, kTiny, uint32_t>(mask, (row0 + min(i0 + u, Nq - 1)) * Nk + jl, total);
    if (!kTiny && (row0 + min(64 * t + 63, Nq - 1)) * Nk + (uint32_t)(wg % slabs) * 64 + 60 > total - 4) {
#pragma unroll
      for (int u = 0; u < 16; ++u) past_end(f[u], (row0 + min(i0 + u, Nq - 1)) * Nk + jl, total);
    }
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const uint32_t own = i0 + u < Nq ? ~0u : 0u;
      (u < 8 ? lo : hi) |= (nonzero_bytes(f[u]) & own) >> (7 - u % 8);
    }
    // through a wave's own 512 bytes
    my[(lane >> 4) * 32 + (lane & 15)] = lo;
    my[(lane >> 4) * 32 + 16 + (lane & 15)] = hi;
    wave_lds_order();
    const uint8_t* const by = reinterpret_cast<const uint8_t*>(my);
    uint64_t m = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) m |= (uint64_t)by[64 * k + lane] << (8 * k);
    wave_lds_order();
    return col_ok ? m : 0ull;
  };
  // a wave with one tile (Nq <= 1024) keeps its mask for the fill
  uint64_t one = 0;
  int cnt = 0;
#pragma unroll 1
  for (int t = t0; t < t1; ++t) {
    one = bits(t);
    cnt += __popcll(one);
  }
  part[w * 64 + lane] = cnt;
  __syncthreads();
  if constexpr (!kFill) {
    if (w == 0 && col_ok) {
      int tot = 0;
      for (int x = 0; x < kWaves; ++x) tot += part[x * 64 + lane];
      if (wg == 0 && lane == 0) colptr[0] = 0;
      colptr[bh * Nk + j + 1] = kScanned ? tot : ~tot;
    }
  } else {
    const int own = min(64, Nk - (int)(wg % slabs) * 64);
    const int base = sh->off[0], n = sh->off[own] - base;
    // this wave's first entry of the lane's column: the column's offset plus
    // the entries of the earlier waves' (lower) rows
    int pos = sh->off[min(lane, own)] - base;
    for (int x = 0; x < w; ++x) pos += part[x * 64 + lane];
    const bool staged = n <= kStage && Nq <= 65536;
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
      if (t1 - t0 > 1) one = bits(t);
      if (staged) {
#pragma unroll 1
        for (uint64_t m = one; m; m &= m - 1)
          sh->stage[pos++] = (uint16_t)(64 * t + __builtin_ctzll(m));
        continue;
      }
      // one column at a time, the lanes as the tile's rows: the column's set
      // rows go to consecutive entries
#pragma unroll 8
      for (int c = 0; c < 64; ++c) {
        const uint64_t mc = readlane64(one, c);   // column j0 + c, rows 64 t .. +63
        if (mc == 0) continue;
        const int64_t pc = (int64_t)base + __builtin_amdgcn_readlane(pos, c);
        if ((mc >> lane) & 1) {
          const int64_t k = pc + __popcll(mc & lanes_below_mask());
          if (k < cap) rows_out[k] = 64 * t + lane;
        }
      }
      pos += __popcll(one);
    }
    __syncthreads();
    if (staged) write_run(*sh, base, n, rows_out, cap);
  }
}

// Counts and fill: workgroups [0, col_wgs) build column lists, the rest row
// lists. kScanned: counts and offsets are plain, with the scan in between.
// Two workgroups on a CU (8 waves a SIMD, 64 registers): the 466 workgroups of
// the 2K lists run in one round.
template <bool kFill, bool kScanned, bool kTiny>
__global__ __launch_bounds__(kThreads, 8) void index_pass(const uint8_t* __restrict__ mask, int64_t rows,
                                                       int Nq, int Nk, int slabs, int64_t col_wgs,
                                                       int32_t* rowptr, int32_t* __restrict__ cols,
                                                       int32_t* colptr,
                                                       int32_t* __restrict__ rows_out, int64_t cap) {
  __shared__ int part[kThreads];
  __shared__ uint32_t turn[kWaves * 128];
  FillShared* sh = nullptr;
  if constexpr (kFill) {
    __shared__ FillShared fill;
    sh = &fill;
  }
  const int64_t wg = blockIdx.x;
  if constexpr (kFill) {   // one copy of the code for both kinds of list
    const bool col = wg < col_wgs;
    const int64_t j0 = wg % slabs * 64, r0 = (wg - col_wgs) * kLists;
    list_offsets<kScanned>(col ? colptr : rowptr, col ? wg / slabs * Nk + j0 : r0,
                           (int)min((int64_t)kLists, col ? Nk - j0 : rows - r0), *sh);
  }
  if (wg < col_wgs)
    col_lists<kFill, kScanned, kTiny>(mask, Nq, Nk, colptr, rows_out, cap, wg, slabs, rows / Nq, part,
                              turn, sh);
  else
    row_lists<kFill, kScanned, kTiny>(mask, rows, Nk, rowptr, cols, cap, wg - col_wgs, part, sh);
}

// In-place scan: ptr[1..n] holds counts -> ptr[0..n] holds offsets.
// blockIdx.x selects one of two arrays. Each pass stages 16K counts in LDS
// with coalesced loads, scans 16 consecutive counts per thread, and writes
// the offsets back coalesced (one pass for the lists of a 2K canvas).
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 16;
constexpr int kScanChunk = kScanThreads * kScanPer;

__global__ __launch_bounds__(kScanThreads) void scan_counts(int32_t* __restrict__ a, int64_t na,
                                                            int32_t* __restrict__ b, int64_t nb) {
  int32_t* p = blockIdx.x == 0 ? a : b;
  const int64_t n = blockIdx.x == 0 ? na : nb;
  // logical count L at buf[L + L / 16]: conflict-free both for the
  // coalesced order (consecutive L per lane) and for 16 consecutive counts
  // per thread (lane stride 17)
  __shared__ int buf[kScanChunk + kScanChunk / 16];
  auto at = [](int L) { return L + (L >> 4); };
  __shared__ int wsum[kScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int carry = 0;
  if (tid == 0) p[0] = 0;
  for (int64_t c0 = 1; c0 <= n; c0 += kScanChunk) {
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) {
      const int64_t i = c0 + e * kScanThreads + tid;
      buf[at(e * kScanThreads + tid)] = i <= n ? p[i] : 0;
    }
    __syncthreads();
    int x[kScanPer];
    int s = 0;
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) {
      s += buf[at(tid * kScanPer + e)];
      x[e] = s;   // inclusive within the thread
    }
    int incl = s;   // inclusive over the wave's threads
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int off = carry + incl - s, tot = 0;
    for (int i = 0; i < kScanThreads / 64; ++i) {
      off += (i < w) ? wsum[i] : 0;
      tot += wsum[i];
    }
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) buf[at(tid * kScanPer + e)] = off + x[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kScanPer; ++e) {
      const int64_t i = c0 + e * kScanThreads + tid;
      if (i <= n) p[i] = buf[at(e * kScanThreads + tid)];
    }
    carry += tot;
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_block_index(const uint8_t* mask, int B, int H, int Nq, int Nk,
                              int32_t* q_rowptr, int32_t* q_cols, int32_t* kv_colptr,
                              int32_t* kv_rows, int64_t cap, hipStream_t s) {
  const int64_t rows = (int64_t)B * H * Nq;
  const int slabs = (Nk + 63) / 64;
  const int64_t col_wgs = (int64_t)slabs * B * H;
  const int64_t row_wgs = (rows + kWaves * kRowsPerWave - 1) / (kWaves * kRowsPerWave);
  const dim3 grid((unsigned)(col_wgs + row_wgs));
  const bool scan = rows > kPrefixMax || (int64_t)B * H * Nk > kPrefixMax;
  auto pass = [&](auto kernel, const char* name) {
    TraceScope ts_(s, name);
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, mask, rows, Nq, Nk, slabs, col_wgs,
                       q_rowptr, q_cols, kv_colptr, kv_rows, cap);
  };
  if (rows * Nk < 16) {   // shorter than one load: byte by byte
    pass(index_pass<false, false, true>, "index_count");
    pass(index_pass<true, false, true>, "index_fill");
    return hipGetLastError();
  }
  if (!scan) {
    pass(index_pass<false, false, false>, "index_count");
    pass(index_pass<true, false, false>, "index_fill");
    return hipGetLastError();
  }
  pass(index_pass<false, true, false>, "index_count");
  {
    TraceScope ts_(s, "index_scan");
    hipLaunchKernelGGL(scan_counts, dim3(2), dim3(kScanThreads), 0, s, q_rowptr, rows, kv_colptr,
                       (int64_t)B * H * Nk);
  }
  pass(index_pass<true, true, false>, "index_fill");
  return hipGetLastError();
}

}  // namespace ut
