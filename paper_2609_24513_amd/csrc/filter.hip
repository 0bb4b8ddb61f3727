// filter_aabb_pairs and compact_pairs.
//
// Filter: all (i, j) whose closed mesh boxes overlap (touching boxes count),
// optionally restricted to pairs whose common box part meets a closed query
// box.  With a query box and datasets of up to kSmallScan meshes, two kernels
// keep the meshes that meet it and pair them (any number of boxes at once);
// larger ones are reduced to the kept meshes first (a flag pass and a device
// scan).  Without one, up to kFastCols columns and kFastRows rows, two kernels
// produce the pairs (a count pass and a write pass over blocks of 64 rows,
// the block totals summed in front of each block).  Everything else takes the
// general path: one wave per kept row of A against LDS tiles of the kept boxes
// of B, a scan of the row counts and a second pass that writes each row's
// pairs.  Either way the output is
// sorted by (i, j) and identical run to run.  The exact total is always
// written; output beyond `cap` is dropped (the caller relaunches with a
// larger buffer, as the paper does for its result structure, Section 3.5).
//
// Compaction (Section 3.5 result materialisation): pairs whose flag is 1,
// in input order, in tiles of kScanTile pairs: the flag count of every tile,
// then every tile writes its pairs from the counts of the tiles before it.
// The prefix sums are the library's own (scan.h).
#include <hip/hip_runtime.h>

#include "common.h"
#include "scan.h"

namespace pr {
namespace {

constexpr int kBlock = 256;
constexpr int kScanBlock = 1024;        // threads of the single-block scans
constexpr int kScanItems = 4;           // consecutive items per thread per tile
constexpr int64_t kSmallScan = 65536;   // single-block scans up to this many items

__device__ __forceinline__ const MeshDesc* meshes_of(const void* blob) {
  const BlobHeader* h = reinterpret_cast<const BlobHeader*>(blob);
  return reinterpret_cast<const MeshDesc*>(reinterpret_cast<const char*>(blob) + h->off_mesh);
}

__device__ __forceinline__ bool meet(const float* a, const float* b) {
  return a[0] <= b[3] && b[0] <= a[3] && a[1] <= b[4] && b[1] <= a[4] && a[2] <= b[5] && b[2] <= a[5];
}

__global__ void k_keep(const void* blob, int64_t M, const float* query, int32_t* flag) {
  const MeshDesc* md = meshes_of(blob);
  int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (; m < M; m += (int64_t)gridDim.x * blockDim.x) {
    bool ok = md[m].n_tris > 0;
    if (query) ok = ok && meet(md[m].box, query);
    flag[m] = ok ? 1 : 0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) flag[M] = 0;
}

// Kept meshes: their ids and a compact copy of their boxes (24 bytes each,
// read coalesced by the row kernels instead of 64-byte descriptors).
__global__ void k_list(const void* blob, const int32_t* flag, const int32_t* pos, int64_t M, int32_t* ids,
                       float* boxes) {
  const MeshDesc* md = meshes_of(blob);
  int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (; m < M; m += (int64_t)gridDim.x * blockDim.x)
    if (flag[m]) {
      const int32_t k = pos[m];
      ids[k] = (int32_t)m;
      for (int c = 0; c < 6; ++c) boxes[6 * (int64_t)k + c] = md[m].box[c];
    }
}

// Without a query box every mesh is a row (A) or a column (B): boxes copied
// in index order, an empty mesh given an inverted box (+inf lows, -inf
// highs) that meets nothing; ids are the identity.
__global__ void k_boxes_all(const void* blob_a, int64_t MA, int32_t* ids_a, float* box_a, int32_t* cnt_a,
                            const void* blob_b, int64_t MB, int32_t* ids_b, float* box_b, int32_t* cnt_b) {
  const int64_t n = MA + MB;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const bool a = i < MA;
    const int64_t m = a ? i : i - MA;
    const MeshDesc& d = meshes_of(a ? blob_a : blob_b)[m];
    float* bx = (a ? box_a : box_b) + 6 * m;
    const bool ok = d.n_tris > 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      bx[c] = ok ? d.box[c] : INFINITY;
      bx[3 + c] = ok ? d.box[3 + c] : -INFINITY;
    }
    (a ? ids_a : ids_b)[m] = (int32_t)m;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *cnt_a = (int32_t)MA;
    *cnt_b = (int32_t)MB;
  }
}

// Exclusive scan of the row counts (at most kSmallScan rows) in one block,
// over the first *n_live rows only (the kept rows); the total goes to
// off[n] (n the rows scanned) and to the caller's count.
__global__ __launch_bounds__(kScanBlock) void k_rowscan_small(const int64_t* cnt, int64_t rows, const int32_t* n_live,
                                                              int64_t* off, int64_t* total_out) {
  __shared__ int64_t s_scan[kScanBlock / 64];
  const int64_t live = *n_live;
  const int64_t n = live < 0 ? 0 : (live < rows ? live : rows);
  int64_t running = 0;
  for (int64_t base = 0; base < n; base += kScanBlock * kScanItems) {
    const int64_t r0 = base + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t sum = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      v[i] = r0 + i < n ? cnt[r0 + i] : 0;
      sum += v[i];
    }
    int64_t total = 0;
    int64_t o = running + block_exclusive_sum<kScanBlock>(sum, s_scan, total);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i)
      if (r0 + i < n) {
        off[r0 + i] = o;
        o += v[i];
      }
    running += total;
  }
  if (threadIdx.x == 0) {
    off[n] = running;
    *total_out = running;
  }
}

struct RowArgs {
  const float* box_a;  // compact boxes of the kept meshes
  const float* box_b;
  const int32_t* ids_a;
  const int32_t* ids_b;
  const int32_t* na;  // device counts
  const int32_t* nb;
  const float* query;
  int64_t rows;       // capacity of the row arrays (n_meshes_a)
  bool live_only;     // counts only for the kept rows (the scan reads no more)
  int64_t* rowcnt;    // [rows + 1]
  const int64_t* rowoff;
  int32_t* pairs;
  int64_t cap;
};

// Row kernels: a block takes kRowsPerBlock kept rows of A (one per wave) and
// walks the kept boxes of B in tiles of kTile staged in LDS (one copy per
// tile for the block's rows instead of one L2 read per row); each wave tests
// its row against the tile, 64 columns at a time.
constexpr int kRowsPerBlock = kBlock / 64;
constexpr int kTile = 1024;

__device__ __forceinline__ bool test_box(const float* a, const float* q, float l0, float l1, float l2, float h0,
                                         float h1, float h2) {
  if (q) {
    return fmaxf(fmaxf(a[0], l0), q[0]) <= fminf(fminf(a[3], h0), q[3]) &&
           fmaxf(fmaxf(a[1], l1), q[1]) <= fminf(fminf(a[4], h1), q[4]) &&
           fmaxf(fmaxf(a[2], l2), q[2]) <= fminf(fminf(a[5], h2), q[5]);
  }
  return a[0] <= h0 && l0 <= a[3] && a[1] <= h1 && l1 <= a[4] && a[2] <= h2 && l2 <= a[5];
}

__device__ __forceinline__ void load_tile(float (*t)[kTile], const float* box_b, int32_t t0, int32_t nb) {
  for (int i = threadIdx.x; i < kTile; i += kBlock) {
    const int32_t k = t0 + i;
    if (k < nb) {
#pragma unroll
      for (int c = 0; c < 6; ++c) t[c][i] = box_b[6 * (int64_t)k + c];
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_row_count(RowArgs r) {
  __shared__ float tile[6][kTile];
  const int32_t na = *r.na, nb = *r.nb;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t nrows = r.live_only ? (na < r.rows ? (int64_t)na : r.rows) : r.rows;
  const int64_t groups = (nrows + kRowsPerBlock - 1) / kRowsPerBlock;
  for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
    const int64_t row = g * kRowsPerBlock + wv;
    const bool live = row < na;
    float a[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) a[c] = live ? r.box_a[6 * row + c] : 0.f;
    unsigned long long cnt = 0;
    if (g * kRowsPerBlock < na) {  // uniform over the block
      for (int32_t t0 = 0; t0 < nb; t0 += kTile) {
        __syncthreads();
        load_tile(tile, r.box_b, t0, nb);
        __syncthreads();
        if (live) {
          const int32_t n = min(kTile, nb - t0);
          for (int32_t i = lane; i < n; i += 64)
            cnt += test_box(a, r.query, tile[0][i], tile[1][i], tile[2][i], tile[3][i], tile[4][i], tile[5][i]) ? 1
                                                                                                             : 0;
        }
      }
    }
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0 && row < nrows) r.rowcnt[row] = (int64_t)cnt;
  }
  if (!r.live_only && blockIdx.x == 0 && threadIdx.x == 0) r.rowcnt[r.rows] = 0;
}

__global__ __launch_bounds__(kBlock) void k_row_write(RowArgs r) {
  __shared__ float tile[6][kTile];
  const int32_t na = *r.na, nb = *r.nb;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t groups = ((int64_t)na + kRowsPerBlock - 1) / kRowsPerBlock;
  for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {
    const int64_t row = g * kRowsPerBlock + wv;
    const bool live = row < na;
    float a[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) a[c] = live ? r.box_a[6 * row + c] : 0.f;
    const int32_t ia = live ? r.ids_a[row] : 0;
    int64_t out = live ? r.rowoff[row] : 0;
    for (int32_t t0 = 0; t0 < nb; t0 += kTile) {
      __syncthreads();
      load_tile(tile, r.box_b, t0, nb);
      __syncthreads();
      if (!live) continue;
      const int32_t n = min(kTile, nb - t0);
      for (int32_t i0 = 0; i0 < n; i0 += 64) {
        const int32_t i = i0 + lane;
        const bool ok =
            i < n && test_box(a, r.query, tile[0][i], tile[1][i], tile[2][i], tile[3][i], tile[4][i], tile[5][i]);
        const uint64_t m = __ballot(ok);
        if (ok) {
          const int64_t pos = out + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
          if (pos < r.cap) {
            r.pairs[2 * pos] = ia;
            r.pairs[2 * pos + 1] = r.ids_b[t0 + i];
          }
        }
        out += __popcll(m);
      }
    }
  }
}

// Pair kernels for the common shape (at most kFastCols columns, at most
// kFastRows rows).  A block owns kRT = 64 consecutive rows, one per lane;
// each of its kPairWaves waves holds the rows' boxes and walks a contiguous
// slice of the columns, 64 at a time: one vector load per lane stages the
// chunk in the wave's LDS area, then every column is read back as an LDS
// broadcast and tested by all 64 rows at once (six compares per 64 tests),
// each lane counting its row's hits in a register.  The count pass stores
// the (row, slice) counts and the block's total; the write pass scans the
// block's counts in row-major order, adds the totals of the blocks before
// it and walks the slices again, each lane writing its row's pairs in
// ascending column order: the same sorted list as the general path's.  The
// kernels read the mesh descriptors directly (an empty mesh pairs with
// nothing).
constexpr int kRT = 64;
constexpr int kPairBlock = 1024;
constexpr int kPairWaves = kPairBlock / 64;
constexpr int64_t kFastCols = 8192;
constexpr int64_t kFastGrid = 2048;
constexpr int64_t kFastRows = kRT * kFastGrid;

struct PairArgs {
  const void* blob_a;
  const void* blob_b;
  int64_t MA, MB;
  int32_t* cnt;       // [grid * kRT * kPairWaves]: (row, slice) counts
  int32_t* blocksum;  // [grid]
  int32_t* pairs;
  int64_t cap;
  int64_t* count;
};

// Box of row i of A or column i of B; an empty mesh gets an inverted box
// (+inf lows, -inf highs), which meets nothing.
__device__ __forceinline__ void mesh_box(const void* blob, int64_t i, float* b) {
  const cptr_t<MeshDesc> d = cview(meshes_of(blob)) + i;
  const bool ok = d->n_tris > 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    b[c] = ok ? d->box[c] : INFINITY;
    b[3 + c] = ok ? d->box[3 + c] : -INFINITY;
  }
}

// Column slice of wave w: [lo, hi).
__device__ __forceinline__ void slice_of(int64_t nb, int w, int64_t& lo, int64_t& hi) {
  const int64_t per = (nb + kPairWaves - 1) / kPairWaves;
  lo = per * w < nb ? per * w : nb;
  hi = lo + per < nb ? lo + per : nb;
}

// Closed overlap of row box a and a column box, without branches.
__device__ __forceinline__ bool overlap(const float* a, float l0, float l1, float l2, float h0, float h1, float h2) {
  return (a[0] <= h0) & (l0 <= a[3]) & (a[1] <= h1) & (l1 <= a[4]) & (a[2] <= h2) & (l2 <= a[5]);
}

// A staged column: box (lo xyz, hi xyz) and id.
struct alignas(16) ColBox {
  float lo[3];
  float hi0;
  float hi1, hi2;
  int32_t id, pad;
};

// Walks the wave's slice [lo, hi) in chunks of 64 staged in `st` (the
// wave's 64-entry LDS area) for the lane's row box rb; with WRITE, each hit
// (row id ia, column id) goes to pairs[out++] while out < cap.  Returns the
// number of hits.
template <bool WRITE>
__device__ __forceinline__ int32_t walk(const PairArgs& a, ColBox* st, int64_t lo, int64_t hi, const float* rb,
                                        int32_t ia, int64_t out) {
  const int lane = threadIdx.x & 63;
  int32_t n = 0;
  for (int64_t c0 = lo; c0 < hi; c0 += 64) {
    const int m = (int)(hi - c0 < 64 ? hi - c0 : 64);
    if (lane < m) {
      float b[6];
      mesh_box(a.blob_b, c0 + lane, b);
      st[lane] = ColBox{{b[0], b[1], b[2]}, b[3], b[4], b[5], (int32_t)(c0 + lane), 0};
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int u = 0; u < m; ++u) {
      const ColBox c = st[u];
      const bool ok = overlap(rb, c.lo[0], c.lo[1], c.lo[2], c.hi0, c.hi1, c.hi2);
      if (WRITE && ok) {
        if (out < a.cap) {
          a.pairs[2 * out] = ia;
          a.pairs[2 * out + 1] = c.id;
        }
        ++out;
      }
      n += ok ? 1 : 0;
    }
    __builtin_amdgcn_wave_barrier();  // the chunk is read before the next one is staged
  }
  return n;
}

template <bool WRITE>
__global__ __launch_bounds__(kPairBlock) void k_pairs(PairArgs a) {
  __shared__ int64_t s_red[kPairWaves];
  __shared__ int32_t s_scan[kPairWaves];
  __shared__ ColBox s_col[kPairWaves][64];
  __shared__ int64_t s_base;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int32_t)(threadIdx.x >> 6));
  const int64_t r0 = (int64_t)blockIdx.x * kRT;
  const int64_t na = a.MA, nb = a.MB;
  const int64_t row = r0 + lane;
  float rb[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  const int32_t ia = (int32_t)row;
  if (row < na) mesh_box(a.blob_a, row, rb);
  int64_t lo, hi;
  slice_of(nb, w, lo, hi);
  const bool any = r0 < na;  // uniform over the block
  int32_t* cnt = a.cnt + (int64_t)blockIdx.x * kPairBlock;
  if (!WRITE) {
    const int32_t n = any ? walk<false>(a, s_col[w], lo, hi, rb, ia, 0) : 0;
    cnt[lane * kPairWaves + w] = n;  // row-major (row, slice)
    const int64_t t = block_sum<kPairBlock>((int64_t)n, s_red);
    if (threadIdx.x == 0) a.blocksum[blockIdx.x] = (int32_t)t;
    return;
  }
  int32_t total = 0;
  const int32_t pre = block_exclusive_sum<kPairBlock>(cnt[threadIdx.x], s_scan, total);
  int64_t before = 0;
  for (int64_t b = threadIdx.x; b < (int64_t)blockIdx.x; b += kPairBlock) before += a.blocksum[b];
  before = block_sum<kPairBlock>(before, s_red);
  if (threadIdx.x == 0) s_base = before;
  __syncthreads();
  // the offset of (row = lane, slice = w) sits with thread lane * kPairWaves + w
  __shared__ int32_t s_off[kPairBlock];
  s_off[threadIdx.x] = pre;
  __syncthreads();
  if (any) walk<true>(a, s_col[w], lo, hi, rb, ia, s_base + s_off[lane * kPairWaves + w]);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *a.count = s_base + total;
}


// Query boxes over datasets of at most kSmallScan meshes, any number of boxes
// in two launches (a launch of its own for the kept lists, the counts, their
// scan and the pairs took 20 us a box).  k_query_keep holds one mesh per
// thread and tests it against every box: each wave's ballot is stored (word w
// of a dataset covers meshes 64 w ... 64 w + 63), with the control words of
// the second kernel cleared.  k_query_pairs gives each box up to kQBlocks
// blocks, a few boxes more of them.  A block scans the box's ballots, takes a
// contiguous share of the kept rows (by ticket, so that a block only ever
// waits for blocks that run already), finds their pairs with the kept columns
// staged in LDS, publishes their number, adds up the numbers of the shares
// before it, and writes its pairs in place, sorted by (i, j): from LDS, or when
// they are too many for it by walking its rows again.  Two kept boxes
// that overlap share a point with the query box on every axis (three
// pairwise-meeting intervals, none empty, have a common point; an empty query
// box keeps nothing), so the boxes' own overlap is the whole test.
// Bound by latency for usual boxes (a few hundred rows), by the staging of the
// columns for those that keep most meshes.  One box: with 32 blocks for it and
// two walks 8.5 us for a few hundred kept meshes and 8.0 ms for all of 25,000 x
// 25,000 (2.6 for 25,000 x 8,000, 53 for 65,536 x 65,536); this 9.3 us and 1.0
// ms (0.37, 6.3); 512 blocks 13 us and 0.53 ms.  Shares of kQRows rows keep
// every wave busy; where the staging of many column tiles is most of a share's
// time, kQRowsWide spread it over more blocks (2,000 x 60,000: 2.1 -> 0.6 ms).
constexpr int kQWords = (int)(kSmallScan / 64);
constexpr int kQBlocks = 32;                              // of each box, at least, and for a call of
constexpr int kQBlocksAll = 128;                          // few boxes together
constexpr int kQRows = 16;                                // rows of a share, at least,
constexpr int kQRowsWide = 4;                             // and with many column tiles
constexpr int kQWide = 4;                                 // tiles
constexpr int kQShare = (int)(kSmallScan / kQBlocks);     // rows of a share, at most
constexpr int kQRowTile = 256, kQColTile = 1024;
constexpr int kQHits = 1024;                              // pairs of a share that LDS keeps
constexpr uint64_t kPublished = 1ull << 63;
static_assert(kSmallScan <= 65536 && kQShare <= 4096, "a mesh in 16 bits, a row in 12, a place in 20");
static_assert(kQWords == kScanBlock && kQShare <= 2 * kScanBlock, "one word and two rows per thread");
static_assert(kQBlocksAll <= kScanBlock, "one earlier share a thread");

__global__ __launch_bounds__(kScanBlock) void k_query_keep(const void* blob_a, int64_t MA, const void* blob_b,
                                                           int64_t MB, const float* boxes, int32_t n, uint64_t* bits,
                                                           unsigned long long* ctl, int32_t n_ctl) {
  const int64_t tiles_a = (MA + kScanBlock - 1) / kScanBlock;
  const bool first = (int64_t)blockIdx.x < tiles_a;
  const int64_t tile = first ? (int64_t)blockIdx.x : (int64_t)blockIdx.x - tiles_a;
  const int64_t M = first ? MA : MB;
  const int64_t m = tile * kScanBlock + threadIdx.x;
  float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  bool live = false;
  if (m < M) {
    const float4* p4 = reinterpret_cast<const float4*>(meshes_of(first ? blob_a : blob_b) + m);
    const float4 u = p4[0], v = p4[1], w = p4[2];  // box, node base/count, tri base/count
    b[0] = u.x; b[1] = u.y; b[2] = u.z; b[3] = u.w; b[4] = v.x; b[5] = v.y;
    live = __float_as_int(w.y) > 0;
  }
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < n_ctl; i += kScanBlock) ctl[i] = 0ull;
  uint64_t* out = bits + (first ? 0 : kQWords) + (m >> 6);
  const cptr_t<float> qs = cview(boxes);
  for (int32_t q = 0; q < n; ++q) {
    float qb[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) qb[c] = qs[6 * q + c];
    const uint64_t w = __ballot(live && meet(b, qb));
    if ((threadIdx.x & 63) == 0 && m < ((M + 63) & ~(int64_t)63)) out[(int64_t)q * (2 * kQWords)] = w;
  }
}

// The kept meshes first ... first + n - 1 of a dataset (kept order) into id:
// each thread writes those of its own word.
__device__ __forceinline__ void kept_ids(const uint64_t* words, const int32_t* before, int32_t first, int32_t n,
                                         int32_t* id) {
  uint64_t w = words[threadIdx.x];
  for (int32_t k = before[threadIdx.x] - first; w && k < n; w &= w - 1, ++k)
    if (k >= 0) id[k] = 64 * (int32_t)threadIdx.x + __builtin_ctzll(w);
}

__global__ __launch_bounds__(kScanBlock, 8) void k_query_pairs(const void* blob_a, int64_t MA, const void* blob_b,
                                                            int64_t MB, const float* boxes, const uint64_t* bits,
                                                            unsigned long long* ctl, int32_t* pairs, int64_t cap,
                                                            int64_t* counts) {
  __shared__ uint64_t s_wa[kQWords], s_wb[kQWords];
  __shared__ int32_t s_pa[kQWords], s_pb[kQWords];
  __shared__ float s_col[6][kQColTile], s_rbox[6][kQRowTile];
  __shared__ int32_t s_cid[kQColTile], s_rid[kQRowTile];
  __shared__ int32_t s_row[2 * kScanBlock + 2];  // pairs of each row of the share, then their places
  __shared__ int32_t s_i32[kScanBlock / 64];
  __shared__ int64_t s_i64[kScanBlock / 64];
  __shared__ uint32_t s_hit[kQHits][2];  // row | place in it << 12, mesh of A | mesh of B << 16
  __shared__ int32_t s_hits;
  __shared__ int32_t s_ticket;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t q = blockIdx.y;
  const int32_t blocks = (int32_t)gridDim.x;
  ctl += q * (blocks + 1);  // the shares' published counts, then the ticket
  pairs += 2 * q * cap;
  const uint64_t* wa = bits + q * (2 * kQWords);
  // an inverted box is empty, though a mesh box that spans both of its planes passes the closed compares
  const cptr_t<float> qb = cview(boxes) + 6 * q;
  const bool some = qb[0] <= qb[3] && qb[1] <= qb[4] && qb[2] <= qb[5];
  if (t == 0) s_ticket = (int32_t)atomicAdd(ctl + blocks, 1ull);
  const uint64_t a = t < (MA + 63) / 64 ? wa[t] : 0ull, b = t < (MB + 63) / 64 ? wa[kQWords + t] : 0ull;
  s_wa[t] = a;
  s_wb[t] = b;
  int32_t na, nb;
  s_pa[t] = block_exclusive_sum<kScanBlock>((int32_t)__popcll(a), s_i32, na);
  s_pb[t] = block_exclusive_sum<kScanBlock>((int32_t)__popcll(b), s_i32, nb);
  if (!some) na = 0;
  s_row[2 * t] = 0;
  s_row[2 * t + 1] = 0;
  if (t == 0) {
    s_row[2 * kScanBlock] = 0;
    s_hits = 0;
  }
  __syncthreads();
  const int32_t most = nb > kQWide * kQColTile ? (na + kQRowsWide - 1) / kQRowsWide : (na + kQRows - 1) / kQRows;
  const int32_t share = s_ticket, shares = max(1, min(blocks, most));
  if (share >= shares) return;
  const int32_t r0 = (int32_t)((int64_t)na * share / shares), r1 = (int32_t)((int64_t)na * (share + 1) / shares);
  const MeshDesc *ma = meshes_of(blob_a), *mb = meshes_of(blob_b);
  int32_t staged = -1;  // first column of the tile in LDS
  int64_t base = 0;
  for (int pass = 0; pass < 2; ++pass) {
    for (int32_t rt = r0; rt < r1; rt += kQRowTile) {
      const int32_t nr = min(kQRowTile, r1 - rt);
      __syncthreads();
      kept_ids(s_wa, s_pa, rt, nr, s_rid);
      __syncthreads();
      if (t < nr) {
        const MeshDesc& d = ma[s_rid[t]];
#pragma unroll
        for (int c = 0; c < 6; ++c) s_rbox[c][t] = d.box[c];
      }
      for (int32_t ct = 0; ct < nb; ct += kQColTile) {
        const int32_t nc = min(kQColTile, nb - ct);
        if (staged != ct) {
          __syncthreads();
          kept_ids(s_wb, s_pb, ct, nc, s_cid);
          __syncthreads();
          if (t < nc) {
            const MeshDesc& d = mb[s_cid[t]];
#pragma unroll
            for (int c = 0; c < 6; ++c) s_col[c][t] = d.box[c];
          }
          staged = ct;
        }
        __syncthreads();
        for (int32_t r = w; r < nr; r += kScanBlock / 64) {
          float x[6];
#pragma unroll
          for (int c = 0; c < 6; ++c) x[c] = s_rbox[c][r];
          const int32_t ia = s_rid[r], row = rt - r0 + r;
          int32_t at = s_row[row];
          for (int32_t i0 = 0; i0 < nc; i0 += 64) {
            const int32_t i = i0 + lane;
            const bool ok = i < nc && overlap(x, s_col[0][i], s_col[1][i], s_col[2][i], s_col[3][i], s_col[4][i],
                                              s_col[5][i]);
            const uint64_t m = __ballot(ok);
            if (!m) continue;
            const int32_t before = (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (pass == 0) {
              int32_t h = 0;
              if (lane == 0) h = atomicAdd(&s_hits, __popcll(m));
              h = __builtin_amdgcn_readfirstlane(h) + before;
              if (ok && h < kQHits) {
                s_hit[h][0] = (uint32_t)row | (uint32_t)(at + before) << 12;
                s_hit[h][1] = (uint32_t)ia | (uint32_t)s_cid[i] << 16;
              }
            } else if (ok) {
              const int64_t pos = base + at + before;
              if (pos < cap) {
                pairs[2 * pos] = ia;
                pairs[2 * pos + 1] = s_cid[i];
              }
            }
            at += __popcll(m);
          }
          if (lane == 0) s_row[row] = at;
        }
      }
    }
    if (pass == 1) break;
    __syncthreads();
    const int32_t v0 = s_row[2 * t], v1 = s_row[2 * t + 1];
    int64_t total;
    const int64_t pre = block_exclusive_sum<kScanBlock>((int64_t)v0 + v1, s_i64, total);
    if (t == 0) __hip_atomic_store(ctl + share, kPublished | (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int64_t earlier = 0;
    if (t < share) {
      uint64_t v;
      do v = __hip_atomic_load(ctl + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      while (!(v & kPublished));
      earlier = (int64_t)(v & ~kPublished);
    }
    base = block_sum<kScanBlock>(earlier, s_i64);
    s_row[2 * t] = (int32_t)pre;
    s_row[2 * t + 1] = (int32_t)(pre + v0);
    if (t == 0 && share == shares - 1) counts[q] = base + total;
    if (total == 0) return;
    __syncthreads();
    if (total <= kQHits) {
      for (int k = t; k < (int)total; k += kScanBlock) {
        const int64_t pos = base + s_row[s_hit[k][0] & 4095u] + (s_hit[k][0] >> 12);
        if (pos < cap) {
          pairs[2 * pos] = (int32_t)(s_hit[k][1] & 0xffffu);
          pairs[2 * pos + 1] = (int32_t)(s_hit[k][1] >> 16);
        }
      }
      return;
    }
  }
}

__global__ void k_set_i64(int64_t* out, int64_t v) { *out = v; }

__device__ __forceinline__ int64_t clamped_n(int64_t n, const int64_t* n_dev) {
  return n_dev ? (*n_dev < 0 ? 0 : (*n_dev < n ? *n_dev : n)) : n;
}

// Compaction, pass 1: the number of flagged pairs of each tile (pairs at
// or beyond the device count, when one is given, are not flagged).
__global__ __launch_bounds__(kTileThreads) void k_cflag_tiles(const uint8_t* flags, int64_t n, const int64_t* n_dev,
                                                              int64_t* tsum) {
  __shared__ int64_t s[kTileThreads / 64];
  const int64_t m = clamped_n(n, n_dev);
  const int64_t i0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kTileItems;
  int64_t c = 0;
#pragma unroll
  for (int k = 0; k < kTileItems; ++k) c += i0 + k < m && flags[i0 + k] ? 1 : 0;
  const int64_t t = block_sum<kTileThreads>(c, s);
  if (threadIdx.x == 0) tsum[blockIdx.x] = t;
}

// The flags (bytes other than 0) among the first n, summed over the threads
// of a block: 16 at a time where the pointer is aligned, all of a thread's
// reads in flight.
template <int B, int N>
__device__ __forceinline__ int64_t count_flags(const uint8_t* flags, int64_t n, int64_t* s) {
  int64_t c = 0;
  if ((reinterpret_cast<uintptr_t>(flags) & 15) == 0) {
    const uint4* f4 = reinterpret_cast<const uint4*>(flags);
    uint4 v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int64_t i = threadIdx.x + (int64_t)k * B;
      v[k] = 16 * i + 16 <= n ? f4[i] : make_uint4(0u, 0u, 0u, 0u);
    }
    auto set = [](uint32_t x) { return __popc((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) & 0x80808080u); };
#pragma unroll
    for (int k = 0; k < N; ++k) c += set(v[k].x) + set(v[k].y) + set(v[k].z) + set(v[k].w);
    if ((int64_t)threadIdx.x < (n & 15)) c += flags[(n & ~(int64_t)15) + threadIdx.x] ? 1 : 0;
  } else {
    for (int64_t i = threadIdx.x; i < n; i += B) c += flags[i] ? 1 : 0;
  }
  return block_sum<B>(c, s);
}

// Compaction, pass 2: tile b writes its flagged pairs in order from its
// offset.  BASE 1: tsum already holds the tiles' offsets (scanned by
// k_scan_top, which also wrote the count); otherwise the last tile writes the
// count and the tile adds up the counts of the tiles before it (BASE 0) or
// counts their flags itself (BASE 2, for at most kOneTiles tiles: no pass 1;
// 2,000 pairs 7.4 + 4.6 us and a gap -> 8.6 us).
// kTileItems consecutive pairs per thread; their flagged pairs are read
// before the scan, so that every load is in flight at once.
constexpr int64_t kOneTiles = 16;

template <int BASE>
__global__ __launch_bounds__(kTileThreads) void k_cflag_write(const int32_t* pairs, const uint8_t* flags, int64_t n,
                                                              const int64_t* n_dev, const int64_t* tsum, int32_t* out,
                                                              int64_t cap, int64_t* count) {
  __shared__ int64_t s[kTileThreads / 64];
  const int64_t m = clamped_n(n, n_dev);
  const int64_t i0 = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kTileItems;
  uint32_t f = 0;
#pragma unroll
  for (int k = 0; k < kTileItems; ++k) f |= (i0 + k < m && flags[i0 + k] ? 1u : 0u) << k;
  int32_t pv[kTileItems][2];
#pragma unroll
  for (int k = 0; k < kTileItems; ++k)
    if ((f >> k) & 1u) {
      pv[k][0] = pairs[2 * (i0 + k)];
      pv[k][1] = pairs[2 * (i0 + k) + 1];
    }
  int64_t base;
  if (BASE == 1) {
    base = tsum[blockIdx.x];
  } else if (BASE == 2) {
    constexpr int N = (int)((kOneTiles * kScanTile / 16 + kTileThreads - 1) / kTileThreads);
    const int64_t before = (int64_t)blockIdx.x * kScanTile;
    base = count_flags<kTileThreads, N>(flags, before < m ? before : m, s);
  } else {
    int64_t b = 0;
    for (int64_t j = threadIdx.x; j < (int64_t)blockIdx.x; j += kTileThreads) b += tsum[j];
    base = block_sum<kTileThreads>(b, s);
  }
  int64_t all = 0;
  int64_t pos = base + block_exclusive_sum<kTileThreads>((int64_t)__popc(f), s, all);
#pragma unroll
  for (int k = 0; k < kTileItems; ++k)
    if ((f >> k) & 1u) {
      if (pos < cap) {
        out[2 * pos] = pv[k][0];
        out[2 * pos + 1] = pv[k][1];
      }
      ++pos;
    }
  if (BASE != 1 && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *count = base + all;
}

// Tiles up to which pass 2 adds up the earlier tiles' counts itself.
constexpr int64_t kDirectTiles = 1024;

// Concatenation of the leading pairs of n fixed-size regions (the candidate
// lists that one filter call per query leaves in its own region), in region
// order, with the counts read on the device: one block per region sums the
// clamped counts of the regions before it, then copies its rows.
__global__ __launch_bounds__(kBlock) void k_gather(const int32_t* regions, int64_t region_cap, const int64_t* counts,
                                                  int64_t n, int32_t* out, int64_t cap, int64_t* total) {
  __shared__ int64_t s_red[kBlock / 64];
  __shared__ int64_t s_off;
  const int64_t k = blockIdx.x;
  if (n == 0) {
    if (threadIdx.x == 0) *total = 0;
    return;
  }
  auto clamped = [&](int64_t j) {
    const int64_t c = counts[j];
    return c < 0 ? (int64_t)0 : (c < region_cap ? c : region_cap);
  };
  int64_t part = 0;
  for (int64_t j = threadIdx.x; j < k; j += kBlock) part += clamped(j);
  part = block_sum<kBlock>(part, s_red);
  if (threadIdx.x == 0) s_off = part;
  __syncthreads();
  const int64_t off = s_off, c = clamped(k);
  const int32_t* src = regions + 2 * k * region_cap;
  for (int64_t i = threadIdx.x; i < c; i += kBlock)
    if (off + i < cap) {
      out[2 * (off + i)] = src[2 * i];
      out[2 * (off + i) + 1] = src[2 * i + 1];
    }
  if (k == n - 1 && threadIdx.x == 0) *total = off + c;
}

// A batch's results into pinned host memory, as many pairs and flags as the
// device count says: one launch writes what four copies of the buffers' full
// size did (32 requests of up to 5,000 pairs: 36 -> 5.4 us).  Bound by the
// link to the host, which few blocks fill.
constexpr int kHostBlocks = 64;

struct HostOut {
  const int32_t* pairs;
  const uint8_t* flags;
  const int64_t *total, *counts;
  const int32_t* status;
  int64_t cap, n;
  int32_t* h_pairs;
  uint8_t* h_flags;
  int64_t* h_counts;
  int32_t* h_status;
};

// bytes [0, n) of src to dst, 16 at a time where both are aligned.
__device__ __forceinline__ void copy_out(void* dst, const void* src, int64_t n) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  int64_t done = 0;
  if (((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15) == 0) {
    done = n & ~(int64_t)15;
    for (int64_t i = t; i < n >> 4; i += step) reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(src)[i];
  }
  for (int64_t i = done + t; i < n; i += step)
    reinterpret_cast<uint8_t*>(dst)[i] = reinterpret_cast<const uint8_t*>(src)[i];
}

__global__ __launch_bounds__(kBlock) void k_to_host(HostOut o) {
  const int64_t m = clamped_n(o.cap, o.total);
  copy_out(o.h_pairs, o.pairs, 8 * m);
  copy_out(o.h_flags, o.flags, m);
  copy_out(o.h_counts, o.counts, 8 * o.n);
  if (blockIdx.x == 0 && threadIdx.x == 0) *o.h_status = *o.status;
}

// Boxes that one pair of launches takes, and the blocks of each of n boxes.
int64_t boxes_at_once(int64_t n) { return n < 1 ? 1 : (n < 1024 ? n : 1024); }
int64_t query_blocks(int64_t n) { return kQBlocksAll / n > kQBlocks ? kQBlocksAll / n : kQBlocks; }

struct FilterWs {
  int32_t *flag_a, *flag_b, *pos_a, *pos_b, *ids_a, *ids_b;
  float *box_a, *box_b;
  int64_t *rowcnt, *rowoff;
  int32_t *blocksum, *paircnt;
  int64_t* tsum;  // tile sums of the device-wide scans
  uint64_t* qbits;            // query-box ballots, [n][2][kQWords]
  unsigned long long* qctl;   // [n][blocks + 1]
};

int carve_filter(Carve& cv, FilterWs& w, int64_t MA, int64_t MB, int64_t n_boxes) {
  w.flag_a = cv.take<int32_t>(MA + 1);
  w.flag_b = cv.take<int32_t>(MB + 1);
  w.pos_a = cv.take<int32_t>(MA + 1);
  w.pos_b = cv.take<int32_t>(MB + 1);
  w.ids_a = cv.take<int32_t>(MA + 1);
  w.ids_b = cv.take<int32_t>(MB + 1);
  w.box_a = cv.take<float>(6 * (MA + 1));
  w.box_b = cv.take<float>(6 * (MB + 1));
  w.rowcnt = cv.take<int64_t>(MA + 1);
  w.rowoff = cv.take<int64_t>(MA + 1);
  w.blocksum = cv.take<int32_t>(kFastGrid);
  const int64_t fast_rows = MA <= kFastRows ? MA : 0;
  w.paircnt = cv.take<int32_t>((fast_rows + kRT - 1) / kRT * kPairBlock);
  const int64_t mx = MA > MB ? MA : MB;
  w.tsum = cv.take<int64_t>(scan_tiles_of(mx + 1));
  w.qbits = cv.take<uint64_t>(n_boxes * 2 * kQWords);
  // a call's last chunk of fewer boxes has up to kQBlocksAll + n words, less than a full chunk
  w.qctl = cv.take<unsigned long long>(n_boxes * (query_blocks(n_boxes) + 1));
  return PR_OK;
}

// Query boxes over datasets of at most kSmallScan meshes; box q's pairs start
// at pairs[q * cap].
bool small_query(int64_t MA, int64_t MB) { return MA <= kSmallScan && MB <= kSmallScan; }

void launch_query(hipStream_t s, const void* blob_a, int64_t MA, const void* blob_b, int64_t MB, const float* boxes,
                  int32_t n, int32_t* pairs, int64_t cap, int64_t* counts, const FilterWs& w) {
  const int64_t tiles = (MA + kScanBlock - 1) / kScanBlock + (MB + kScanBlock - 1) / kScanBlock;
  // a small dataset needs fewer blocks
  const int64_t least = MB > kQWide * kQColTile ? kQRowsWide : kQRows, most = query_blocks(n);
  const int64_t blocks = MA / least + 1 < most ? MA / least + 1 : most;
  hipLaunchKernelGGL(k_query_keep, dim3((unsigned)(tiles > 0 ? tiles : 1)), dim3(kScanBlock), 0, s, blob_a, MA, blob_b,
                     MB, boxes, n, w.qbits, w.qctl, (int32_t)(n * (blocks + 1)));
  hipLaunchKernelGGL(k_query_pairs, dim3((unsigned)blocks, (unsigned)n), dim3(kScanBlock), 0, s, blob_a, MA, blob_b, MB,
                     boxes, (const uint64_t*)w.qbits, w.qctl, pairs, cap, counts);
}

struct CompactWs {
  int64_t* tsum;  // flag count (then offset) of each tile
};

int carve_compact(Carve& cv, CompactWs& w, int64_t n) {
  w.tsum = cv.take<int64_t>(scan_tiles_of(n) + 1);
  return PR_OK;
}

}  // namespace
}  // namespace pr

using namespace pr;

extern "C" int filter_aabb_pairs_ws_bytes(int64_t n_meshes_a, int64_t n_meshes_b, size_t* ws_bytes) {
  if (n_meshes_a < 0 || n_meshes_b < 0 || !ws_bytes) { set_error("bad argument"); return PR_E_ARG; }
  if (n_meshes_a >= ((int64_t)1 << 30) || n_meshes_b >= ((int64_t)1 << 30)) { set_error("too many meshes"); return PR_E_UNSUPPORTED; }
  Carve cv{nullptr, 0};
  FilterWs w{};
  int r = carve_filter(cv, w, n_meshes_a, n_meshes_b, 1);
  if (r) return r;
  *ws_bytes = cv.used + 256;
  return PR_OK;
}

extern "C" int filter_aabb_pairs(const void* blob_a, int64_t n_meshes_a, const void* blob_b, int64_t n_meshes_b,
                                 const float* query_box, int32_t* pairs, int64_t cap, int64_t* dev_count, void* ws,
                                 size_t ws_bytes, void* stream) {
  if (!blob_a || !blob_b || !dev_count || !ws || cap < 0 || (cap > 0 && !pairs) || n_meshes_a < 0 || n_meshes_b < 0) {
    set_error("bad argument");
    return PR_E_ARG;
  }
  if (n_meshes_a >= ((int64_t)1 << 30) || n_meshes_b >= ((int64_t)1 << 30)) { set_error("too many meshes"); return PR_E_UNSUPPORTED; }
  hipStream_t s = (hipStream_t)stream;
  Carve cv{(char*)ws, ws_bytes};
  FilterWs w{};
  int r = carve_filter(cv, w, n_meshes_a, n_meshes_b, 1);
  if (r) return r;
  if (cv.used > ws_bytes) { set_error("ws_bytes %zu < required %zu", ws_bytes, cv.used); return PR_E_CAPACITY; }
  const int64_t MA = n_meshes_a, MB = n_meshes_b;
  if (query_box && small_query(MA, MB)) {
    launch_query(s, blob_a, MA, blob_b, MB, query_box, 1, pairs, cap, dev_count, w);
    PR_HIP(hipGetLastError());
    return PR_OK;
  }
  if (!query_box && MA > 0 && MB > 0 && MA <= kFastRows && MB <= kFastCols) {
    PairArgs pa{};
    pa.MA = MA;
    pa.MB = MB;
    pa.blocksum = w.blocksum;
    pa.cnt = w.paircnt;
    pa.pairs = pairs;
    pa.cap = cap;
    pa.count = dev_count;
    pa.blob_a = blob_a;
    pa.blob_b = blob_b;
    const int grid = (int)((MA + kRT - 1) / kRT);
    hipLaunchKernelGGL(k_pairs<false>, dim3(grid), dim3(kPairBlock), 0, s, pa);
    hipLaunchKernelGGL(k_pairs<true>, dim3(grid), dim3(kPairBlock), 0, s, pa);
    PR_HIP(hipGetLastError());
    return PR_OK;
  }
  if (!query_box) {
    hipLaunchKernelGGL(k_boxes_all, dim3(grid_for(MA + MB, kBlock)), dim3(kBlock), 0, s, blob_a, MA, w.ids_a,
                       w.box_a, w.pos_a + MA, blob_b, MB, w.ids_b, w.box_b, w.pos_b + MB);
  } else {
    hipLaunchKernelGGL(k_keep, dim3(grid_for(MA + 1, kBlock)), dim3(kBlock), 0, s, blob_a, MA, query_box, w.flag_a);
    hipLaunchKernelGGL(k_keep, dim3(grid_for(MB + 1, kBlock)), dim3(kBlock), 0, s, blob_b, MB, query_box, w.flag_b);
    PR_HIP(device_exclusive_scan(w.flag_a, w.pos_a, MA + 1, w.tsum, (int64_t*)nullptr, s));
    PR_HIP(device_exclusive_scan(w.flag_b, w.pos_b, MB + 1, w.tsum, (int64_t*)nullptr, s));
    hipLaunchKernelGGL(k_list, dim3(grid_for(MA, kBlock)), dim3(kBlock), 0, s, blob_a, (const int32_t*)w.flag_a,
                       (const int32_t*)w.pos_a, MA, w.ids_a, w.box_a);
    hipLaunchKernelGGL(k_list, dim3(grid_for(MB, kBlock)), dim3(kBlock), 0, s, blob_b, (const int32_t*)w.flag_b,
                       (const int32_t*)w.pos_b, MB, w.ids_b, w.box_b);
  }
  RowArgs ra{};
  ra.box_a = w.box_a;
  ra.box_b = w.box_b;
  ra.query = query_box;
  ra.ids_a = w.ids_a;
  ra.ids_b = w.ids_b;
  ra.na = w.pos_a + MA;
  ra.nb = w.pos_b + MB;
  ra.rows = MA;
  ra.live_only = MA <= kSmallScan;
  ra.rowcnt = w.rowcnt;
  ra.rowoff = w.rowoff;
  ra.pairs = pairs;
  ra.cap = cap;
  const int64_t row_groups = (MA + kRowsPerBlock - 1) / kRowsPerBlock;
  const int rows_grid = (int)(row_groups < 2048 ? (row_groups > 0 ? row_groups : 1) : 2048);
  hipLaunchKernelGGL(k_row_count, dim3(rows_grid), dim3(kBlock), 0, s, ra);
  if (MA <= kSmallScan) {
    hipLaunchKernelGGL(k_rowscan_small, dim3(1), dim3(kScanBlock), 0, s, (const int64_t*)w.rowcnt, MA,
                       (const int32_t*)(w.pos_a + MA), w.rowoff, dev_count);
    hipLaunchKernelGGL(k_row_write, dim3(rows_grid), dim3(kBlock), 0, s, ra);
  } else {
    PR_HIP(device_exclusive_scan((const int64_t*)w.rowcnt, w.rowoff, MA + 1, w.tsum, dev_count, s));
    hipLaunchKernelGGL(k_row_write, dim3(rows_grid), dim3(kBlock), 0, s, ra);
  }
  PR_HIP(hipGetLastError());
  return PR_OK;
}

extern "C" int filter_aabb_pairs_batch_ws_bytes(int64_t n_meshes_a, int64_t n_meshes_b, int64_t n_boxes,
                                                size_t* ws_bytes) {
  if (n_meshes_a < 0 || n_meshes_b < 0 || n_boxes < 0 || !ws_bytes) { set_error("bad argument"); return PR_E_ARG; }
  if (n_meshes_a >= ((int64_t)1 << 30) || n_meshes_b >= ((int64_t)1 << 30)) { set_error("too many meshes"); return PR_E_UNSUPPORTED; }
  Carve cv{nullptr, 0};
  FilterWs w{};
  int r = carve_filter(cv, w, n_meshes_a, n_meshes_b, boxes_at_once(n_boxes));
  if (r) return r;
  *ws_bytes = cv.used + 256;
  return PR_OK;
}

extern "C" int filter_aabb_pairs_batch(const void* blob_a, int64_t n_meshes_a, const void* blob_b, int64_t n_meshes_b,
                                       const float* query_boxes, int64_t n_boxes, int32_t* regions, int64_t region_cap,
                                       int64_t* dev_counts, void* ws, size_t ws_bytes, void* stream) {
  size_t need = 0;
  int r = filter_aabb_pairs_batch_ws_bytes(n_meshes_a, n_meshes_b, n_boxes, &need);
  if (r) return r;
  if (!blob_a || !blob_b || !ws || region_cap < 0 || (n_boxes > 0 && (!query_boxes || !dev_counts)) ||
      (n_boxes > 0 && region_cap > 0 && !regions)) {
    set_error("bad argument");
    return PR_E_ARG;
  }
  if (n_boxes == 0) return PR_OK;
  if (!small_query(n_meshes_a, n_meshes_b)) {
    for (int64_t k = 0; k < n_boxes; ++k) {
      r = filter_aabb_pairs(blob_a, n_meshes_a, blob_b, n_meshes_b, query_boxes + 6 * k, regions + 2 * k * region_cap,
                            region_cap, dev_counts + k, ws, ws_bytes, stream);
      if (r) return r;
    }
    return PR_OK;
  }
  Carve cv{(char*)ws, ws_bytes};
  FilterWs w{};
  const int64_t chunk = boxes_at_once(n_boxes);
  r = carve_filter(cv, w, n_meshes_a, n_meshes_b, chunk);
  if (r) return r;
  if (cv.used > ws_bytes) { set_error("ws_bytes %zu < required %zu", ws_bytes, cv.used); return PR_E_CAPACITY; }
  for (int64_t k = 0; k < n_boxes; k += chunk)
    launch_query((hipStream_t)stream, blob_a, n_meshes_a, blob_b, n_meshes_b, query_boxes + 6 * k,
                 (int32_t)(n_boxes - k < chunk ? n_boxes - k : chunk), regions + 2 * k * region_cap, region_cap,
                 dev_counts + k, w);
  PR_HIP(hipGetLastError());
  return PR_OK;
}

extern "C" int compact_pairs_ws_bytes(int64_t n_pairs, size_t* ws_bytes) {
  if (n_pairs < 0 || !ws_bytes) { set_error("bad argument"); return PR_E_ARG; }
  if (n_pairs >= ((int64_t)1 << 30)) { set_error("n_pairs >= 2^30"); return PR_E_UNSUPPORTED; }
  Carve cv{nullptr, 0};
  CompactWs w{};
  int r = carve_compact(cv, w, n_pairs);
  if (r) return r;
  *ws_bytes = cv.used + 256;
  return PR_OK;
}

extern "C" int compact_pairs(const int32_t* pairs, const uint8_t* flags, int64_t n_pairs, const int64_t* dev_n_pairs,
                             int32_t* out, int64_t cap, int64_t* dev_count, void* ws, size_t ws_bytes, void* stream) {
  if (n_pairs < 0 || cap < 0 || !dev_count || !ws || (n_pairs > 0 && (!pairs || !flags)) || (cap > 0 && !out)) {
    set_error("bad argument");
    return PR_E_ARG;
  }
  if (n_pairs >= ((int64_t)1 << 30)) { set_error("n_pairs >= 2^30"); return PR_E_UNSUPPORTED; }
  hipStream_t s = (hipStream_t)stream;
  Carve cv{(char*)ws, ws_bytes};
  CompactWs w{};
  int r = carve_compact(cv, w, n_pairs);
  if (r) return r;
  if (cv.used > ws_bytes) { set_error("ws_bytes %zu < required %zu", ws_bytes, cv.used); return PR_E_CAPACITY; }
  const int64_t nt = scan_tiles_of(n_pairs);
  if (nt == 0) {
    hipLaunchKernelGGL(k_set_i64, dim3(1), dim3(1), 0, s, dev_count, (int64_t)0);
    PR_HIP(hipGetLastError());
    return PR_OK;
  }
  if (nt <= kOneTiles) {
    hipLaunchKernelGGL(k_cflag_write<2>, dim3((unsigned)nt), dim3(kTileThreads), 0, s, pairs, flags, n_pairs,
                       dev_n_pairs, (const int64_t*)w.tsum, out, cap, dev_count);
    PR_HIP(hipGetLastError());
    return PR_OK;
  }
  hipLaunchKernelGGL(k_cflag_tiles, dim3((unsigned)nt), dim3(kTileThreads), 0, s, flags, n_pairs, dev_n_pairs, w.tsum);
  if (nt <= kDirectTiles) {
    hipLaunchKernelGGL(k_cflag_write<0>, dim3((unsigned)nt), dim3(kTileThreads), 0, s, pairs, flags, n_pairs,
                       dev_n_pairs, (const int64_t*)w.tsum, out, cap, dev_count);
  } else {
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kTopThreads), 0, s, w.tsum, nt, dev_count);
    hipLaunchKernelGGL(k_cflag_write<1>, dim3((unsigned)nt), dim3(kTileThreads), 0, s, pairs, flags, n_pairs,
                       dev_n_pairs, (const int64_t*)w.tsum, out, cap, dev_count);
  }
  PR_HIP(hipGetLastError());
  return PR_OK;
}

extern "C" int gather_pair_regions(const int32_t* regions, int64_t region_cap, const int64_t* dev_counts,
                                   int64_t n_regions, int32_t* out, int64_t cap, int64_t* dev_total, void* stream) {
  if (region_cap < 0 || n_regions < 0 || cap < 0 || !dev_total ||
      (n_regions > 0 && (!regions || !dev_counts)) || (cap > 0 && !out)) {
    set_error("bad argument");
    return PR_E_ARG;
  }
  if (n_regions > ((int64_t)1 << 20)) { set_error("n_regions > 2^20"); return PR_E_UNSUPPORTED; }
  hipLaunchKernelGGL(k_gather, dim3(n_regions > 0 ? (unsigned)n_regions : 1u), dim3(kBlock), 0, (hipStream_t)stream,
                     regions, region_cap, dev_counts, n_regions, out, cap, dev_total);
  PR_HIP(hipGetLastError());
  return PR_OK;
}

extern "C" int results_to_host(const int32_t* pairs, const uint8_t* flags, const int64_t* dev_total, int64_t cap,
                               const int64_t* dev_counts, int64_t n_counts, const int32_t* dev_status,
                               int32_t* host_pairs, uint8_t* host_flags, int64_t* host_counts, int32_t* host_status,
                               void* stream) {
  if (cap < 0 || n_counts < 0 || !dev_total || !dev_status || !host_status ||
      (cap > 0 && (!pairs || !flags || !host_pairs || !host_flags)) || (n_counts > 0 && (!dev_counts || !host_counts))) {
    set_error("bad argument");
    return PR_E_ARG;
  }
  HostOut o{};
  o.pairs = pairs; o.flags = flags; o.total = dev_total; o.counts = dev_counts; o.status = dev_status;
  o.cap = cap; o.n = n_counts;
  // device addresses of the pinned buffers: memory that is not pinned is refused here
  struct { void* host; void** dev; } map[] = {{host_pairs, (void**)&o.h_pairs}, {host_flags, (void**)&o.h_flags},
                                              {host_counts, (void**)&o.h_counts}, {host_status, (void**)&o.h_status}};
  for (auto& m : map) {
    if (!m.host) continue;
    if (hipHostGetDevicePointer(m.dev, m.host, 0) != hipSuccess || !*m.dev) {
      (void)hipGetLastError();
      set_error("a host buffer is not pinned");
      return PR_E_ARG;
    }
  }
  hipLaunchKernelGGL(k_to_host, dim3(kHostBlocks), dim3(kBlock), 0, (hipStream_t)stream, o);
  PR_HIP(hipGetLastError());
  return PR_OK;
}
