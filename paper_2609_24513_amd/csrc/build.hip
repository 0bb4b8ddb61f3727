// build_mesh_bvh: per-mesh wide BVHs and unique-edge segments for a dataset.
//
// Steps (all on the device, one batched pass over every mesh; a mesh's faces
// are handled in chunks, one block each, so that large and small meshes load
// the chip alike):
//  1. plan: per mesh, where its chunks, sort cells and node slots begin;
//  2. validate faces (ids in range, finite coordinates, not exactly
//     collinear), per-mesh exact boxes and FP32-safe flags;
//  3. sort the triangles of each mesh by the Morton code of their centroid
//     (ties by face index), and its half-edges by the Morton code of their
//     midpoint (ties by vertex ids): a counting pass over cells (the code's
//     top bits), then units of consecutive cells that fit LDS are sorted
//     there, cells that do not fit divided before.  Copies of one edge share
//     midpoint and ids, so they end up side by side and are merged in the same
//     kernel (Section 3.1: duplicate edges of one mesh are merged);
//  4. per mesh, a binary radix tree over the sorted codes (Karras 2012,
//     "Maximizing parallelism in the construction of BVHs, octrees, and k-d
//     trees"; numbering of nodes from there), ties broken by position, with
//     exact min/max boxes, bottom up from neighbours' common prefixes (Apetrei
//     2014, "Fast and simple agglomerative LBVH construction"): the nodes that
//     lie inside a chunk in LDS, the others after them;
//  5. collapse to width W: each wide node starts from a binary node and
//     repeatedly opens the child with the largest box surface among those
//     holding more than L triangles, until it has W children; children of at
//     most L triangles become leaves (a Karras subtree is a contiguous range
//     of the sorted order, so a leaf is a range of leaf-order triangles);
//  6. the unique edges as FP32 endpoints in groups of 64 consecutive ones,
//     with the exact box of each group.
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>

#include "scan.h"

#include <climits>
#include <cstdio>

#include <type_traits>

#include "common.h"
#include "predicates.h"

namespace pr {
namespace {

constexpr int kBlock = 256;
constexpr int kTreeChunk = 512;    // sorted positions (and faces) of one tree block
constexpr int kCodeChunk = 2048;   // faces of one counting block
constexpr int kLdsCells = 1 << 14; // cells counted in LDS
constexpr int kUnit = 1280;        // sort unit: the cells that start in this many items (2 x 106 M half-edges: 1,024 3.2, this 3.0 ms)
constexpr int kUnitCap = 2048;     // items a unit may hold to be sorted in LDS
constexpr int kBins = 2048;        // bins of the LDS sort
constexpr int kBinMax = 128;       // items of a bin that are placed by comparing them with each other
constexpr int kSplitBits = 14;     // bins of one split of an overfull cell, at most (as a power of two)
constexpr int kSplitBlock = 1024;
// Sort units that one launch takes, triangles' and half-edges': fewer than the
// chip holds twice over are bound by launches (2 x 173 meshes of 320 faces: a
// launch less is 2 % of build and join); a build of 2 x 35 M triangles takes 3.0
// ms in two launches and 3.5 in one.
constexpr int64_t kSortOne = 2048;
constexpr int kLdsBlock = 512;     // threads of a sort block (the same sort, at 79 registers: 256 3.0, this 2.74, 1,024 5.5 ms)
constexpr int kTreeBlock = 512;    // threads of a tree block, one position each
constexpr int kMaxRoots = 128;     // subtrees that tile a chunk: at most two per tree level (62 levels)
constexpr int kTopUnits = 512;     // subtrees of chunks that one pass of a top block joins
constexpr int kTopLists = 256;     // root lists it takes at most
constexpr int kSubtree = kTreeChunk;  // binary subtrees of at most this many triangles are collapsed in LDS
constexpr int kPack = 1024;      // positions of the subtrees that a block collapses together
constexpr int kPackBlock = 256;

__device__ __forceinline__ uint32_t spread10(uint32_t v) {
  v &= 0x3ffu;
  v = (v | (v << 16)) & 0x030000ffu;
  v = (v | (v << 8)) & 0x0300f00fu;
  v = (v | (v << 4)) & 0x030c30c3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

__device__ __forceinline__ uint32_t quant10(float c, float lo, float hi) {
  float ext = hi - lo;
  if (!(ext > 0.f)) return 0;
  float t = (c - lo) / ext * 1024.f;
  int q = (int)t;
  return (uint32_t)(q < 0 ? 0 : (q > 1023 ? 1023 : q));
}

__device__ __forceinline__ uint32_t morton3(f3 c, const float* box) {
  return (spread10(quant10(c.x, box[0], box[3])) << 2) | (spread10(quant10(c.y, box[1], box[4])) << 1) |
         spread10(quant10(c.z, box[2], box[5]));
}

__device__ __forceinline__ int lanes_before(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ bool safe_coord(float c) {
  float a = fabsf(c);
  return c == 0.f || (a >= kSafeLo && a <= kSafeHi);
}

__device__ __forceinline__ f3 load_v(const float* verts, int64_t g) {
  return f3{verts[3 * g], verts[3 * g + 1], verts[3 * g + 2]};
}

// Per mesh: its faces and the first of its entries in each table.  When a
// mesh's offsets are inconsistent no mesh has faces or entries: the build
// fails through the status word, and ranges that overlap, which each look
// sound, cannot add up to more than the tables hold.
struct MeshPlan {
  int64_t v0;       // first vertex
  int32_t nv;       // vertices
  int32_t f0;       // first face
  int32_t n;        // faces
  int32_t tchunk;   // tree chunks of kTreeChunk faces
  int32_t tunit;    // triangle sort units of kUnit faces
  int32_t eunit;    // edge sort units of kUnit half-edges
  int32_t tcell;    // triangle cells
  int32_t ecell;    // edge cells
  int32_t node;     // node slots (nodes_bound of them)
  int32_t rchunk;   // root lists: one per chunk of a mesh of several
  int32_t cchunk;   // counting chunks of kCodeChunk faces of a mesh of several cells
  int32_t pad;
};

// A binary node: the boxes of its two children and the sorted positions
// [lo, split] and [split + 1, hi] that they cover (relative to the mesh).  The
// child over one position is a leaf; an inner left child is node `split`, an
// inner right child node split + 1.
struct alignas(64) BinNode {
  float box[2][6];
  int32_t lo, split, hi, pad;
};

// A subtree whose parent lies outside its chunk.
struct RootRec {
  float box[6];
  int32_t hi;  // its last position (its first follows the subtree before it)
  int32_t d;   // prefix length across its end
};

// A subtree for one block of the collapse: its first position, the slot of its
// wide node, and depth | triangles << 8 | (its binary node is its last
// position's) << 31.
struct SubItem {
  int32_t mesh, lo, slot;
  uint32_t info;
};

// An item of a sort: its code, then the words that order equal codes.
struct Item {
  uint32_t k, x, y;
};

struct BuildArgs {
  const float* verts;
  const int64_t* vert_off;
  const int32_t* faces;
  const int64_t* face_off;
  int64_t n_meshes, v_total, f_total;
  int width, leaf;
  int builder;           // 0: open the largest-area child, 1: the largest area x triangle count
  // blob sections
  char* blob;
  MeshDesc* mesh;
  char* nodes;
  float* tris;
  int32_t* triid;
  float* seg;
  int32_t* edge;
  float* cbox;
  int32_t* cmesh;
  float* rep;            // [M][4] representative vertex of each mesh
  float* rbox;           // [chunk_cap][8] box of each run of 64 groups, at the run's first group
  int64_t node_cap, chunk_cap;
  // workspace
  int32_t* status;       // min bad face (INT_MAX if none)
  int32_t* exps;         // [2] lowest, highest coordinate bit exponent
  int32_t* ctr;          // [0] meshes in `big`, [1] entries of `subs`, [2] of `over`, [3] of `packed`
  uint64_t* psum;        // [kPlanBlocks][4] entries of each plan block's meshes
  MeshPlan* plan;        // [M + 1], totals at [M]
  uint32_t* mm;          // [M][8] ordered box bits (lo xyz, hi xyz), [6] != 0: a coordinate out of the safe range
  int32_t* used;         // [M] node slots in use
  int32_t* depth;        // [M] deepest node level
  int32_t* nedges;       // [M] unique edges
  int64_t* groups;       // [M + 1] group counts, then scanned
  int64_t* etotal;       // [1] unique edges of the dataset
  int32_t* big;          // [M] meshes of more than kSubtree triangles
  int32_t* tmap;         // [tchunk] mesh of each tree chunk
  int32_t* tumap;        // [tunit] mesh of each triangle unit
  int32_t* emap;         // [eunit] mesh of each edge unit
  int32_t* cmap;         // [cchunk] mesh of each counting chunk
  uint32_t* hist;        // triangle cells, then edge cells: counts
  uint32_t* start;       // their exclusive scan
  int64_t cells_t, cells_all;  // capacity of the triangle cells, of both
  int64_t* tsum;         // tile sums of the scan
  uint32_t* key;         // [F] Morton code of each face
  uint32_t* rank;        // [F] place within its cell
  uint2* tcells;         // [F] (code, face) in cell order
  uint32_t* sk;          // [F] sorted codes
  uint32_t* sv;          // [F] sorted faces
  uint32_t* ekey;        // [3F] Morton code of each half-edge's midpoint
  uint32_t* erank;       // [3F]
  Item* ecells;          // [3F] (code, lower, higher vertex id) in cell order
  uint32_t* ul;          // [3F] unique edges of each unit, at its first item
  uint32_t* uh;
  int2* over;            // cells of more than kUnitCap items: mesh, cell (half-edges: the sign bit set)
  int32_t* packed;       // sort units for k_sort_packed (half-edges: the sign bit set)
  int32_t* tfirst;       // [tunit] of an overfull cell's parts that start in a unit the first start, the last
  int32_t* tlast;
  int32_t* efirst;       // [eunit]
  int32_t* elast;
  int32_t* ustart;       // [eunit] first item of each unit (from the mesh's first)
  int32_t* ucount;       // [eunit] unique edges of each unit
  int32_t* uoff;         // [eunit] unique edges of the mesh before the unit
  BinNode* bin;          // [F]
  RootRec* roots;        // [rchunk][kMaxRoots]
  int32_t* nroots;       // [rchunk]
  int32_t* items;        // [F][3] work lists of the top collapse (node, slot, depth)
  SubItem* subs;         // subtrees for the wave-wise collapse
};

// ---- ordered float bits (min and max by integer atomics) -----------------------

__device__ __forceinline__ uint32_t to_ordered(float x) {
  const uint32_t b = __float_as_uint(x);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float from_ordered(uint32_t u) {
  return __uint_as_float(u & 0x80000000u ? u & 0x7fffffffu : ~u);
}

// ---- step 1: plan ----------------------------------------------------------------

// Cells of a sort of n items, as a power of two: one while a unit holds them
// all, then a sixteenth to an eighth of n.  A closed surface meets about
// cells^(2/3) of them, so an occupied cell of 10^5 items holds some 200.
__host__ __device__ __forceinline__ int cell_bits(int64_t n) {
  if (n <= kUnitCap) return 0;
  return 63 - __builtin_clzll((uint64_t)n) - 3;
}

__device__ __forceinline__ int32_t div_up(int64_t n, int d) { return (int32_t)((n + d - 1) / d); }

// Grids of one block a table entry: a launch takes less than 2^32 threads a
// dimension, which 8.4 M meshes of a chunk each exceed, so the blocks are
// numbered over two.
constexpr int64_t kGridX = 1 << 22;
__device__ __forceinline__ int32_t block_id() { return (int32_t)(blockIdx.y * gridDim.x + blockIdx.x); }
inline dim3 grid_of(int64_t n) {
  return n <= kGridX ? dim3((unsigned)n) : dim3((unsigned)kGridX, (unsigned)((n + kGridX - 1) / kGridX));
}

// Entries of mesh m (in: there is one) in every table, two 32-bit numbers to a
// word (every total is below 2^31); false when its offsets are inconsistent.
__device__ __forceinline__ bool plan_entries(const BuildArgs& a, int64_t m, bool in, MeshPlan& p, uint64_t* c) {
  p = MeshPlan{};
  bool ok = true;
  if (in) {
    const int64_t f0 = a.face_off[m], f1 = a.face_off[m + 1], v0 = a.vert_off[m], v1 = a.vert_off[m + 1];
    ok = f0 >= 0 && f1 >= f0 && f1 <= a.f_total && v0 >= 0 && v1 >= v0 && v1 <= a.v_total;
    if (m == 0) ok = ok && f0 == 0 && v0 == 0;
    if (m == a.n_meshes - 1) ok = ok && f1 == a.f_total && v1 == a.v_total;
    if (ok) {
      p.v0 = v0;
      p.nv = (int32_t)(v1 - v0);
      p.f0 = (int32_t)f0;
      p.n = (int32_t)(f1 - f0);
    }
  }
  const uint32_t n = (uint32_t)p.n, chunks = (n + kTreeChunk - 1) / kTreeChunk;
  const uint32_t nodes = nodes_bound(n, (uint32_t)a.width, (uint32_t)a.leaf);
  auto two = [](uint32_t hi, uint32_t lo) { return ((uint64_t)hi << 32) | lo; };
  c[0] = two(chunks, (n + kUnit - 1) / kUnit);
  c[1] = two((3 * n + kUnit - 1) / kUnit, n > (uint32_t)kTreeChunk ? chunks : 0u);
  c[2] = in ? two(1u << cell_bits(n), 1u << cell_bits(3 * (int64_t)n)) : 0ull;
  c[3] = two(cell_bits(3 * (int64_t)n) ? (n + kCodeChunk - 1) / kCodeChunk : 0u, nodes);
  return ok;
}

// The plan of many meshes is made by several blocks, `span` meshes each (a
// multiple of 1,024), after k_plan_sums has summed every block's entries (one
// block for 1 M meshes 5.1 ms).
constexpr int64_t kPlanOne = 2048;  // meshes that one block plans alone, at most
constexpr int64_t kPlanBlocks = 512;

__global__ __launch_bounds__(1024) void k_plan_sums(BuildArgs a, int64_t span) {
  __shared__ int64_t s[16];
  int64_t sum[4] = {0, 0, 0, 0};
  bool bad = false;
  const int64_t m0 = blockIdx.x * span, m1 = m0 + span < a.n_meshes ? m0 + span : a.n_meshes;
#pragma unroll 1
  for (int64_t m = m0 + threadIdx.x; m < m1; m += 1024) {
    MeshPlan p;
    uint64_t c[4];
    bad |= !plan_entries(a, m, true, p, c);
    for (int q = 0; q < 4; ++q) sum[q] += (int64_t)c[q];
  }
  for (int q = 0; q < 4; ++q) {
    const int64_t t = block_sum<1024>(sum[q], s);
    if (threadIdx.x == 0) a.psum[4 * blockIdx.x + q] = (uint64_t)t;
  }
  if (bad) *a.status = 0;
}

// The exclusive sums over the meshes of every table's entries.  One mesh a
// thread and rolled loops: a lone block runs each instruction once, so its time
// is the fetch of its code (unrolled over four meshes a thread 37 us for 173
// meshes).
__global__ __launch_bounds__(1024) void k_plan(BuildArgs a, int64_t span) {
  __shared__ uint64_t s_sum[4][16], s_run[4];
  __shared__ int s_bad;  // a mesh's offsets are inconsistent
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const bool last = blockIdx.x == gridDim.x - 1;
  const int64_t m0 = blockIdx.x * span, m1 = last ? a.n_meshes : m0 + span;
  if (threadIdx.x < 4) s_run[threadIdx.x] = 0ull;
  if (threadIdx.x == 0) s_bad = gridDim.x > 1 && *a.status != INT_MAX;
  __syncthreads();
  if (blockIdx.x > 0 && threadIdx.x < 4) {
    uint64_t run = 0;
#pragma unroll 8
    for (uint32_t b = 0; b < blockIdx.x; ++b) run += a.psum[4 * b + threadIdx.x];
    s_run[threadIdx.x] = run;
  }
#pragma unroll 1
  for (int64_t base = m0; base < m1; base += 1024) {
    const int64_t m = base + threadIdx.x;
    const bool in = m < m1;
    MeshPlan p;
    uint64_t c[4];
    if (!plan_entries(a, m, in, p, c)) s_bad = 1;
    uint64_t inc[4] = {c[0], c[1], c[2], c[3]};
#pragma unroll 1
    for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint64_t y = __shfl_up(inc[q], o);
        inc[q] += lane >= o ? y : 0ull;
      }
    }
    if (lane == 63) {
#pragma unroll
      for (int q = 0; q < 4; ++q) s_sum[q][w] = inc[q];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
      uint64_t run = s_run[threadIdx.x];
#pragma unroll 1
      for (int k = 0; k < 16; ++k) {
        const uint64_t x = s_sum[threadIdx.x][k];
        s_sum[threadIdx.x][k] = run;
        run += x;
      }
      s_run[threadIdx.x] = run;
    }
    __syncthreads();
    uint64_t at[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) at[q] = s_sum[q][w] + inc[q] - c[q];
    p.tchunk = (int32_t)(at[0] >> 32);
    p.tunit = (int32_t)(uint32_t)at[0];
    p.eunit = (int32_t)(at[1] >> 32);
    p.rchunk = (int32_t)(uint32_t)at[1];
    p.tcell = (int32_t)(at[2] >> 32);
    p.ecell = (int32_t)(uint32_t)at[2];
    p.node = (int32_t)(uint32_t)at[3];
    p.cchunk = (int32_t)(at[3] >> 32);
    if (in) a.plan[m] = p;
    __syncthreads();  // s_sum is written again
  }
  __syncthreads();
  if (last && threadIdx.x == 0) {
    MeshPlan t{};
    t.tchunk = (int32_t)(s_run[0] >> 32);
    t.tunit = (int32_t)(uint32_t)s_run[0];
    t.eunit = (int32_t)(s_run[1] >> 32);
    t.rchunk = (int32_t)(uint32_t)s_run[1];
    t.tcell = (int32_t)(s_run[2] >> 32);
    t.ecell = (int32_t)(uint32_t)s_run[2];
    t.node = (int32_t)(uint32_t)s_run[3];
    t.cchunk = (int32_t)(s_run[3] >> 32);
    a.plan[a.n_meshes] = t;
  }
  if (!s_bad) return;
  if (threadIdx.x == 0) *a.status = 0;
  __syncthreads();  // the totals are written
#pragma unroll 1
  for (int64_t m = m0 + threadIdx.x; m < (last ? m1 + 1 : m1); m += 1024) a.plan[m] = MeshPlan{};
}

// Everything that starts at a fixed value.
__global__ void k_build_init(BuildArgs a) {
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = i0; i < a.cells_all; i += step) a.hist[i] = 0u;
  for (int64_t i = i0; i < 8 * a.n_meshes; i += step) a.mm[i] = (i & 7) < 3 ? 0xffffffffu : 0u;
  for (int64_t i = i0; i < a.n_meshes; i += step) a.depth[i] = 0;
  if (i0 == 0) {
    *a.status = INT_MAX;
    a.exps[0] = INT_MAX;
    a.exps[1] = INT_MIN;
    a.ctr[0] = 0;
    a.ctr[1] = 0;
    a.ctr[2] = 0;
    a.ctr[3] = 0;
  }
}

// The mesh of every chunk and unit, one wave per mesh.
__global__ __launch_bounds__(kBlock) void k_maps(BuildArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t m = (blockIdx.x * (int64_t)kBlock + threadIdx.x) >> 6; m < a.n_meshes; m += nw) {
    const MeshPlan p = a.plan[m], q = a.plan[m + 1];
    for (int32_t i = p.tchunk + lane; i < q.tchunk; i += 64) a.tmap[i] = (int32_t)m;
    for (int32_t i = p.tunit + lane; i < q.tunit; i += 64) {
      a.tumap[i] = (int32_t)m;
      a.tfirst[i] = INT_MAX;
      a.tlast[i] = -1;
    }
    for (int32_t i = p.eunit + lane; i < q.eunit; i += 64) {
      a.emap[i] = (int32_t)m;
      a.efirst[i] = INT_MAX;
      a.elast[i] = -1;
    }
    for (int32_t i = p.cchunk + lane; i < q.cchunk; i += 64) a.cmap[i] = (int32_t)m;
  }
}

// ---- step 2: faces and mesh boxes ------------------------------------------------

// Exponents of the lowest and highest set bit of a finite non-zero FP32 value.
__device__ __forceinline__ int bit_lo(float x) {
  const uint32_t b = __float_as_uint(x) & 0x7fffffffu;
  const uint32_t e = b >> 23, m = b & 0x7fffffu;
  return e == 0 ? -149 + __builtin_ctz(m) : (int)e - 150 + __builtin_ctz(m | 0x800000u);
}
__device__ __forceinline__ int bit_hi(float x) {
  const uint32_t b = __float_as_uint(x) & 0x7fffffffu;
  const uint32_t e = b >> 23, m = b & 0x7fffffu;
  return e == 0 ? -149 + (31 - __builtin_clz(m)) : (int)e - 127;
}

__global__ __launch_bounds__(kBlock) void k_prep(BuildArgs a) {
  const int32_t block = block_id();
  __shared__ int s_lo[kBlock / 64], s_hi[kBlock / 64];
  if (block >= a.plan[a.n_meshes].tchunk) return;
  const int32_t m = a.tmap[block];
  const MeshPlan p = a.plan[m];
  const int32_t c0 = (block - p.tchunk) * kTreeChunk, c1 = min(p.n, c0 + kTreeChunk);
  int elo = INT_MAX, ehi = INT_MIN;  // bit exponents over this thread's coordinates
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool unsafe = false;
  for (int32_t i = c0 + (int32_t)threadIdx.x; i < c1; i += kBlock) {
    const int64_t f = (int64_t)p.f0 + i;
    const int32_t id[3] = {a.faces[3 * f], a.faces[3 * f + 1], a.faces[3 * f + 2]};
    bool bad = false;
    for (int k = 0; k < 3; ++k) bad |= id[k] < 0 || id[k] >= p.nv;
    if (bad) {
      atomicMin(a.status, (int32_t)f);
      unsafe = true;
      continue;
    }
    const f3 p0 = load_v(a.verts, p.v0 + id[0]), p1 = load_v(a.verts, p.v0 + id[1]), p2 = load_v(a.verts, p.v0 + id[2]);
    const float cs[9] = {p0.x, p0.y, p0.z, p1.x, p1.y, p1.z, p2.x, p2.y, p2.z};
    bool fin = true;
    for (int k = 0; k < 9; ++k) { fin &= isfinite(cs[k]); unsafe |= !safe_coord(cs[k]); }
    if (!fin) {
      atomicMin(a.status, (int32_t)f);
      unsafe = true;
    } else {
      for (int k = 0; k < 9; ++k)
        if (cs[k] != 0.f) {
          elo = min(elo, bit_lo(cs[k]));
          ehi = max(ehi, bit_hi(cs[k]));
        }
      // exactly collinear iff all three coordinate-plane orientations vanish
      ExactCounters cnt{0};
      const bool degen = sign_orient2d(p0, p1, p2, 1, 2, cnt) == 0 && sign_orient2d(p0, p1, p2, 2, 0, cnt) == 0 &&
                         sign_orient2d(p0, p1, p2, 0, 1, cnt) == 0;
      if (degen) atomicMin(a.status, (int32_t)f);
    }
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], fminf(fminf(cs[k], cs[3 + k]), cs[6 + k]));
      hi[k] = fmaxf(hi[k], fmaxf(fmaxf(cs[k], cs[3 + k]), cs[6 + k]));
    }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int o = 32; o > 0; o >>= 1) {
    elo = min(elo, __shfl_xor(elo, o));
    ehi = max(ehi, __shfl_xor(ehi, o));
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], __shfl_xor(lo[k], o));
      hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], o));
    }
  }
  const bool any_unsafe = __ballot(unsafe) != 0;
  uint32_t* mm = a.mm + 8 * (int64_t)m;
  if (lane == 0) {
    s_lo[w] = elo;
    s_hi[w] = ehi;
    if (lo[0] <= hi[0]) {
      for (int k = 0; k < 3; ++k) {
        atomicMin(mm + k, to_ordered(lo[k]));
        atomicMax(mm + 3 + k, to_ordered(hi[k]));
      }
    }
    if (any_unsafe) atomicOr(mm + 6, 1u);
  }
  __syncthreads();
  // one counter pair serves every block: an atomic only where it changes
  // (one each per wave took 0.27 of the 0.28 ms of a 5 M-face build's pass)
  if (threadIdx.x == 0) {
    for (int k = 1; k < kBlock / 64; ++k) {
      elo = min(elo, s_lo[k]);
      ehi = max(ehi, s_hi[k]);
    }
    if (elo < __hip_atomic_load(a.exps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(a.exps, elo);
    if (ehi > __hip_atomic_load(a.exps + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(a.exps + 1, ehi);
  }
}

// Descriptors of the meshes; the root of a mesh of at most L triangles; the
// work lists of the collapse.
template <int W>
__global__ void k_desc(BuildArgs a) {
  for (int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; m < a.n_meshes;
       m += (int64_t)gridDim.x * blockDim.x) {
    const MeshPlan p = a.plan[m];
    const uint32_t* mm = a.mm + 8 * m;
    MeshDesc d;
    for (int k = 0; k < 3; ++k) {
      const bool any = mm[k] <= mm[3 + k];
      d.box[k] = any ? from_ordered(mm[k]) : INFINITY;
      d.box[3 + k] = any ? from_ordered(mm[3 + k]) : -INFINITY;
    }
    d.node_base = p.node;
    d.n_nodes = p.n > 0 ? 1 : 0;
    d.tri_base = p.f0;
    d.n_tris = p.n;
    d.chunk_base = 0; d.n_chunks = 0; d.n_edges = 0;
    d.depth = p.n > 0 ? 1 : 0;
    d.root = p.n > 0 ? p.node : kEmpty;
    d.flags = mm[6] == 0u ? kMeshSafe : 0;
    a.mesh[m] = d;
    // representative vertex for the point-in-mesh test: the first corner of
    // the mesh's first face (a bad id fails the build through the status word)
    float4 rv = make_float4(0.f, 0.f, 0.f, 0.f);
    if (p.n > 0) {
      const int32_t id = a.faces[3 * (int64_t)p.f0];
      if (id >= 0 && id < p.nv) {
        const float* x = a.verts + 3 * (p.v0 + id);
        rv = make_float4(x[0], x[1], x[2], 1.f);
      }
    }
    reinterpret_cast<float4*>(a.rep)[m] = rv;
    a.used[m] = 1;
    // a sort in one cell needs no counting pass
    if (cell_bits(p.n) == 0) a.hist[p.tcell] = (uint32_t)p.n;
    if (cell_bits(3 * (int64_t)p.n) == 0) a.hist[a.cells_t + p.ecell] = 3u * (uint32_t)p.n;
    if (p.n > 0 && p.n <= a.leaf) {
      Node<W> nd;
      for (int c = 0; c < W; ++c) {
        for (int k = 0; k < 3; ++k) { nd.lo[k][c] = INFINITY; nd.hi[k][c] = -INFINITY; }
        nd.child[c] = kEmpty;
        nd.pad[c] = 0;
      }
      for (int k = 0; k < 3; ++k) { nd.lo[k][0] = d.box[k]; nd.hi[k][0] = d.box[3 + k]; }
      nd.child[0] = leaf_ref(p.f0, p.n);
      reinterpret_cast<Node<W>*>(a.nodes)[p.node] = nd;
    } else if (p.n > kSubtree) {
      a.big[atomicAdd(a.ctr, 1)] = (int32_t)m;
    } else if (p.n > 0) {
      a.subs[atomicAdd(a.ctr + 1, 1)] = SubItem{(int32_t)m, 0, 0, 1u | (uint32_t)p.n << 8};
    }
  }
}

// ---- step 3: sorts ------------------------------------------------------------------

__device__ __forceinline__ void half_edge(const int32_t* id, int k, uint32_t& lo, uint32_t& hi) {
  const uint32_t u = (uint32_t)id[k], v = (uint32_t)id[k == 2 ? 0 : k + 1];
  lo = u < v ? u : v;
  hi = u < v ? v : u;
}

// Morton codes of a face's centroid and of its half-edges' midpoints.
__device__ __forceinline__ void face_codes(const BuildArgs& a, const MeshPlan& p, const float* box, int64_t f,
                                           uint32_t* key) {
  f3 v[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) v[k] = load_v(a.verts, p.v0 + a.faces[3 * f + k]);
  key[0] = morton3(f3{0.5f * (fminf(fminf(v[0].x, v[1].x), v[2].x) + fmaxf(fmaxf(v[0].x, v[1].x), v[2].x)),
                      0.5f * (fminf(fminf(v[0].y, v[1].y), v[2].y) + fmaxf(fmaxf(v[0].y, v[1].y), v[2].y)),
                      0.5f * (fminf(fminf(v[0].z, v[1].z), v[2].z) + fmaxf(fmaxf(v[0].z, v[1].z), v[2].z))},
                   box);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const f3 x = v[k], y = v[k == 2 ? 0 : k + 1];
    key[1 + k] = morton3(f3{0.5f * (x.x + y.x), 0.5f * (x.y + y.y), 0.5f * (x.z + y.z)}, box);
  }
}

// The codes of meshes of several cells, and each item's place within its cell.  A
// block counts its kCodeChunk faces in LDS, and the first item of each cell
// fetches the cell's places for all of the block's: atomics in memory run at
// some 50 per ns over the chip (one for each run of equal cells in a wave
// took 0.43 ms for 5.5 M faces).  A mesh of more than kLdsCells cells takes
// them in memory one by one, or a wave's at once if they are of one cell
// (atomics on one address take some 9 ns each: the 4 M of a mesh of 1 M faces
// that lie in one cell 35 ms, so 0.7).
__global__ __launch_bounds__(1024) void k_codes_cells(BuildArgs a) {
  constexpr int R = kCodeChunk / 1024;
  __shared__ uint32_t s_cnt[kLdsCells];
  if (*a.status != INT_MAX) return;
  if ((int32_t)blockIdx.x >= a.plan[a.n_meshes].cchunk) return;
  const int32_t m = a.cmap[blockIdx.x];
  const MeshPlan p = a.plan[m];
  const int32_t c0 = ((int32_t)blockIdx.x - p.cchunk) * kCodeChunk;
  const int tb = cell_bits(p.n), eb = cell_bits(3 * (int64_t)p.n);
  float box[6];
  for (int k = 0; k < 6; ++k) box[k] = a.mesh[m].box[k];
  uint32_t key[R][4];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int32_t i = c0 + r * 1024 + (int32_t)threadIdx.x;
    if (i >= p.n) continue;
    const int64_t f = (int64_t)p.f0 + i;
    face_codes(a, p, box, f, key[r]);
    a.key[f] = key[r][0];
#pragma unroll
    for (int k = 0; k < 3; ++k) a.ekey[3 * f + k] = key[r][1 + k];
  }
  // q = 0: the half-edges, q = 1: the faces
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int bits = q == 0 ? eb : tb, k0 = q == 0 ? 1 : 0, nk = q == 0 ? 3 : 1;
    uint32_t* hist = q == 0 ? a.hist + a.cells_t + p.ecell : a.hist + p.tcell;
    if (bits == 0) continue;
    const bool lds = bits <= 14;
    uint32_t rank[R][3];
    if (lds) {
      for (int i = threadIdx.x; i < (1 << bits); i += 1024) s_cnt[i] = 0u;
      __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (c0 + r * 1024 + (int32_t)threadIdx.x >= p.n) continue;
#pragma unroll
      for (int k = 0; k < nk; ++k) {
        const uint32_t cell = key[r][k0 + k] >> (kMortonBits - bits);
        if (lds) {
          rank[r][k] = atomicAdd(&s_cnt[cell], 1u);
        } else if (__ballot(cell != (uint32_t)__builtin_amdgcn_readfirstlane((int)cell)) == 0ull) {
          const uint64_t all = __ballot(true);
          const int before = lanes_before(all);
          uint32_t base = 0;
          if (before == 0) base = atomicAdd(hist + cell, (uint32_t)__popcll(all));
          rank[r][k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + (uint32_t)before;
        } else {
          rank[r][k] = atomicAdd(hist + cell, 1u);
        }
      }
    }
    if (lds) {
      __syncthreads();
      uint32_t base[R][3];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (c0 + r * 1024 + (int32_t)threadIdx.x >= p.n) continue;
#pragma unroll
        for (int k = 0; k < nk; ++k) {
          const uint32_t cell = key[r][k0 + k] >> (kMortonBits - bits);
          if (rank[r][k] == 0u) base[r][k] = atomicAdd(hist + cell, s_cnt[cell]);
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (c0 + r * 1024 + (int32_t)threadIdx.x >= p.n) continue;
#pragma unroll
        for (int k = 0; k < nk; ++k)
          if (rank[r][k] == 0u) s_cnt[key[r][k0 + k] >> (kMortonBits - bits)] = base[r][k];
      }
      __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int32_t i = c0 + r * 1024 + (int32_t)threadIdx.x;
      if (i >= p.n) continue;
      const int64_t f = (int64_t)p.f0 + i;
#pragma unroll
      for (int k = 0; k < nk; ++k) {
        const uint32_t at = rank[r][k] + (lds ? s_cnt[key[r][k0 + k] >> (kMortonBits - bits)] : 0u);
        if (q == 0) a.erank[3 * f + k] = at;
        else a.rank[f] = at;
      }
    }
    __syncthreads();  // the counters are used again
  }
}

// First item of edge cell c of a mesh, from the mesh's first (the scan runs
// on through the triangle cells before).
__device__ __forceinline__ uint32_t ecell_start(const BuildArgs& a, const MeshPlan& p, uint32_t c) {
  return a.start[a.cells_t + p.ecell + c] - a.start[a.cells_t + p.ecell];
}

// Meshes of several cells: items to their cells.  A cell of more than kUnitCap
// items is listed by the one that takes place kUnitCap in it.  Meshes that are
// sorted in one cell: the codes.
__global__ __launch_bounds__(kBlock) void k_to_cells(BuildArgs a) {
  const int32_t block = block_id();
  if (*a.status != INT_MAX) return;
  if (block >= a.plan[a.n_meshes].tchunk) return;
  const int32_t m = a.tmap[block];
  const MeshPlan p = a.plan[m];
  const int tb = cell_bits(p.n), eb = cell_bits(3 * (int64_t)p.n);
  const int32_t c0 = (block - p.tchunk) * kTreeChunk, c1 = min(p.n, c0 + kTreeChunk);
  if (eb == 0) {
    float box[6];
    for (int k = 0; k < 6; ++k) box[k] = a.mesh[m].box[k];
    for (int32_t i = c0 + (int32_t)threadIdx.x; i < c1; i += kBlock) {
      const int64_t f = (int64_t)p.f0 + i;
      uint32_t key[4];
      face_codes(a, p, box, f, key);
      a.key[f] = key[0];
#pragma unroll
      for (int k = 0; k < 3; ++k) a.ekey[3 * f + k] = key[1 + k];
    }
    return;
  }
  const uint32_t t0 = a.start[p.tcell];
  for (int32_t i = c0 + (int32_t)threadIdx.x; i < c1; i += kBlock) {
    const int64_t f = (int64_t)p.f0 + i;
    if (tb) {
      const uint32_t key = a.key[f];
      const uint32_t cell = key >> (kMortonBits - tb), rank = a.rank[f];
      const int64_t at = (int64_t)p.f0 + (a.start[p.tcell + cell] - t0) + rank;
      a.tcells[at] = make_uint2(key, (uint32_t)f);
      if (rank == (uint32_t)kUnitCap) a.over[atomicAdd(a.ctr + 2, 1)] = make_int2(m, (int)cell);
    }
    if (eb) {
      const int32_t id[3] = {a.faces[3 * f], a.faces[3 * f + 1], a.faces[3 * f + 2]};
      for (int k = 0; k < 3; ++k) {
        const uint32_t key = a.ekey[3 * f + k], cell = key >> (kMortonBits - eb), rank = a.erank[3 * f + k];
        const int64_t at = 3 * (int64_t)p.f0 + ecell_start(a, p, cell) + rank;
        uint32_t lo, hi;
        half_edge(id, k, lo, hi);
        a.ecells[at] = Item{key, lo, hi};
        if (rank == (uint32_t)kUnitCap) a.over[atomicAdd(a.ctr + 2, 1)] = make_int2(m, (int)(cell | 0x80000000u));
      }
    }
  }
}

// Smallest cell start at or above `target` among the `cells` starts s (less
// s[0]); n when there is none.  Its cell goes to `at`.  One wave, 64 probes a
// round.
__device__ __forceinline__ int32_t first_start(const uint32_t* s, int64_t cells, int32_t target, int32_t n, int32_t& at) {
  const int lane = threadIdx.x & 63;
  const uint32_t s0 = s[0];
  int64_t lo = 0, hi = cells;  // the answer's cell lies in [lo, hi]
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) / 64;
    const int64_t c = lo + lane * step;
    const uint64_t ge = __ballot(c < hi && (int32_t)(s[c < hi ? c : lo] - s0) >= target);
    if (ge) {
      const int f = __builtin_ctzll(ge);
      hi = lo + f * step;
      if (f > 0) lo += (f - 1) * step + 1;
    } else {
      lo += (hi - lo - 1) / step * step + 1;
    }
  }
  at = (int32_t)hi;
  return hi < cells ? (int32_t)(s[hi] - s0) : n;
}

template <bool UNIQUE>
struct SortLds {
  using Low = std::conditional_t<UNIQUE, uint64_t, uint32_t>;
  uint32_t cnt[kBins + 1];       // bin counts, then first places
  uint32_t k[kUnitCap];
  Low low[kUnitCap];             // x, and y below it
  uint32_t keep[kUnitCap / 32];  // places of the sorted items that hold the first copy of one
  uint32_t before[kUnitCap / 32];
  uint32_t scan[kLdsBlock / 64];
  int full;                      // a bin holds more than kBinMax items
};

// (UNIQUE) fills in the kept items before each word of `keep`; returns their number.
__device__ __forceinline__ int32_t count_kept(SortLds<true>& s) {
  __syncthreads();
  if (threadIdx.x < 64) {
    const uint32_t c = (uint32_t)__popc(s.keep[threadIdx.x]);
    const uint32_t inc = wave_inclusive_sum(c);
    s.before[threadIdx.x] = inc - c;
    if (threadIdx.x == 63) s.scan[0] = inc;
  }
  __syncthreads();
  return (int32_t)s.scan[0];
}
__device__ __forceinline__ int32_t count_kept(SortLds<false>&) { return 0; }

template <bool UNIQUE>
__device__ __forceinline__ int32_t kept_place(const SortLds<UNIQUE>& s, uint32_t place) {
  return (int32_t)(UNIQUE ? s.before[place >> 5] + (uint32_t)__popc(s.keep[place >> 5] & ((1u << (place & 31u)) - 1u)) : place);
}

// Sorts the n <= kUnitCap items load(0) ... load(n - 1) and hands them to
// store(place, item), equal items once when UNIQUE; returns the number kept.
// One pass: the items go to bins bin(item) < kBins monotone in their order (any
// order within a bin), then each counts the items of its bin that come before
// it, few for codes as even as a surface's, and looks for a copy at a lower
// place.  Returns -1 with nothing stored when a bin has more than kBinMax
// items (k_sort_packed).  Bound by the instructions of the comparing loop: the
// edges of 2 x 35 M triangles take 2.34 ms with one loop without branches and
// took 5.07 ms with one for copies and one for places, each with early outs
// (2.74 ms with the splitting of overfull units in the same kernel: 79
// registers in place of 50).
// Every thread of the block calls it.
template <bool UNIQUE, typename Load, typename Bin, typename Store>
__device__ __forceinline__ int32_t lds_sort(SortLds<UNIQUE>& s, int32_t n, Load load, Bin bin, Store store) {
  constexpr int R = kUnitCap / kLdsBlock;
  using Low = typename SortLds<UNIQUE>::Low;
  static_assert(kUnitCap / 32 == 64, "one word of `keep` a lane");
  auto low_of = [](const Item& e) { return UNIQUE ? (Low)((uint64_t)e.x << 32 | e.y) : (Low)e.x; };
  const int t = threadIdx.x;
  for (int i = t; i <= kBins; i += kLdsBlock) s.cnt[i] = 0u;
  if (UNIQUE && t < kUnitCap / 32) s.keep[t] = 0u;
  if (t == 0) s.full = 0;
  __syncthreads();
  Item it[R];
  uint32_t b[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (t + r * kLdsBlock < n) it[r] = load(t + r * kLdsBlock);
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (t + r * kLdsBlock < n) b[r] = bin(it[r]);
  uint32_t rank[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (t + r * kLdsBlock < n) rank[r] = atomicAdd(&s.cnt[b[r]], 1u);
  __syncthreads();
  {
    constexpr int C = kBins / kLdsBlock;
    uint32_t v[C], sum = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) { v[c] = s.cnt[t * C + c]; sum += v[c]; }
    uint32_t total;
    uint32_t o = block_exclusive_sum<kLdsBlock>(sum, s.scan, total);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if (v[c] > (uint32_t)kBinMax) s.full = 1;
      s.cnt[t * C + c] = o;
      o += v[c];
    }
    if (t == 0) s.cnt[kBins] = total;
  }
  __syncthreads();
  if (s.full) return -1;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (t + r * kLdsBlock < n) {
      const uint32_t at = s.cnt[b[r]] + rank[r];
      s.k[at] = it[r].k;
      s.low[at] = low_of(it[r]);
    }
  __syncthreads();
  uint32_t place[R];  // ~0: a copy
#pragma unroll
  for (int r = 0; r < R; ++r) {
    place[r] = ~0u;
    if (t + r * kLdsBlock >= n) continue;
    const uint32_t j0 = s.cnt[b[r]], j1 = s.cnt[b[r] + 1], me = j0 + rank[r];
    const uint32_t k = it[r].k;
    const Low low = low_of(it[r]);
    uint32_t less = 0;
    bool copy = false;
    for (uint32_t j = j0; j < j1; ++j) {
      const uint32_t kj = s.k[j];
      const Low lj = s.low[j];
      less += (kj < k) | ((kj == k) & (lj < low)) ? 1u : 0u;
      if (UNIQUE) copy |= (j < me) & (kj == k) & (lj == low);
    }
    if (copy) continue;
    place[r] = j0 + less;
    if (UNIQUE) atomicOr(&s.keep[place[r] >> 5], 1u << (place[r] & 31u));
  }
  const int32_t kept = UNIQUE ? count_kept(s) : n;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (place[r] != ~0u) store(kept_place(s, place[r]), it[r]);
  return kept;
}

// The same for items whose codes are packed together, by a bitonic network.
template <bool UNIQUE, typename Load, typename Store>
__device__ __forceinline__ int32_t network_sort(SortLds<UNIQUE>& s, int32_t n, Load load, Store store) {
  using Low = typename SortLds<UNIQUE>::Low;
  const int t = threadIdx.x;
  if (UNIQUE && t < kUnitCap / 32) s.keep[t] = 0u;
  int size = 64;
  while (size < n) size <<= 1;
  for (int i = t; i < size; i += kLdsBlock) {
    const Item e = i < n ? load(i) : Item{~0u, ~0u, ~0u};
    s.k[i] = e.k;
    s.low[i] = UNIQUE ? (Low)((uint64_t)e.x << 32 | e.y) : (Low)e.x;
  }
  for (int g = 2; g <= size; g <<= 1)
    for (int d = g >> 1; d > 0; d >>= 1) {
      __syncthreads();
      for (int h = t; h < size / 2; h += kLdsBlock) {
        const int i = 2 * h - (h & (d - 1)), j = i + d;  // h's bits above d's, one place up
        const uint32_t ki = s.k[i], kj = s.k[j];
        const Low li = s.low[i], lj = s.low[j];
        const bool after = ki > kj || (ki == kj && li > lj);
        if (after == ((i & g) == 0)) {
          s.k[i] = kj; s.k[j] = ki;
          s.low[i] = lj; s.low[j] = li;
        }
      }
    }
  __syncthreads();
  auto copy = [&](int i) { return UNIQUE && i > 0 && s.k[i - 1] == s.k[i] && s.low[i - 1] == s.low[i]; };
  if (UNIQUE) {
    for (int i = t; i < n; i += kLdsBlock)
      if (!copy(i)) atomicOr(&s.keep[i >> 5], 1u << (i & 31));
  }
  const int32_t kept = UNIQUE ? count_kept(s) : n;
  for (int i = t; i < n; i += kLdsBlock)
    if (!copy(i)) {
      const uint64_t low = s.low[i];
      store(kept_place(s, (uint32_t)i), UNIQUE ? Item{s.k[i], (uint32_t)(low >> 32), (uint32_t)low} : Item{s.k[i], (uint32_t)low, 0u});
    }
  __syncthreads();  // s is reused by the next call
  return kept;
}

// The same for n <= 64 items, by one wave: each lane compares its item with all
// of them (a block's bins and barriers were 3.8 and 4.5 of 21 ms for a million
// meshes of one triangle; the other waves leave at once: 1.4 and 1.8 ms).
template <bool UNIQUE, typename Load, typename Store>
__device__ __forceinline__ int32_t wave_sort(int32_t n, Load load, Store store) {
  const int lane = threadIdx.x & 63;
  Item e{0, 0, 0};
  if (lane < n) e = load(lane);
  int32_t less = 0;  // items before this lane's, copies among them
  bool copy = false;
#pragma unroll 1
  for (int j = 0; j < n; ++j) {
    const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)e.k, j), x = (uint32_t)__builtin_amdgcn_readlane((int)e.x, j);
    const uint32_t y = UNIQUE ? (uint32_t)__builtin_amdgcn_readlane((int)e.y, j) : 0u;
    const bool same = k == e.k && x == e.x;
    less += k < e.k || (k == e.k && x < e.x) || (UNIQUE && same && y < e.y) ? 1 : 0;
    if (UNIQUE) copy |= same && y == e.y && j < lane;
  }
  if (!UNIQUE) {
    if (lane < n) store(less, e);
    return n;
  }
  // the places of the items that are kept, as a mask
  const bool keep = lane < n && !copy;
  uint64_t places = keep ? 1ull << less : 0ull;
  for (int o = 32; o > 0; o >>= 1) places |= __shfl_xor(places, o);
  if (keep) store(__popcll(places & ((1ull << less) - 1ull)), e);
  return __popcll(places);
}

// Overfull cells: a mesh whose detail is packed into a small part of its box
// (by one far vertex) has cells of far more items than LDS sorts.  One block
// takes such a cell and moves its items, in place, to bins of their order (up
// to 2^kSplitBits) below the highest bit of (k, x, y) in which any two of
// them differ, the bins of more than kUnitCap items again in turn, until every
// part holds at most kUnitCap items or copies of one.  The units then find the
// parts' starts as they find the cells'.  Bound by the passes of one block over
// its cell (differing bits, counts, scatter, copy back).  Build of a surface of
// 1 M triangles beside a triangle 3,000 times its size: 6.6 ms, of which 4.9
// here; splitting by one bit at a time in the sorts 1,376 ms.
template <bool EDGE>
__device__ __forceinline__ void split_cell(const BuildArgs& a, const MeshPlan& p, uint32_t cell, uint32_t* cnt, uint32_t* s_scan,
                           uint32_t* s_diff, int32_t* s_next) {
  const int t = threadIdx.x;
  const int32_t n = EDGE ? 3 * p.n : p.n;
  const int64_t base = EDGE ? 3 * (int64_t)p.f0 : (int64_t)p.f0;
  const uint32_t* start = a.start + (EDGE ? a.cells_t + p.ecell : (int64_t)p.tcell);
  const int64_t cells = (int64_t)1 << cell_bits(n);
  // the second buffer: arrays that are free after the scatter to cells and before the sorts
  uint32_t* const tk = EDGE ? a.ekey + base : a.key + base;
  uint32_t* const tx = EDGE ? a.erank + base : a.rank + base;
  uint32_t* const ty = EDGE ? a.uh + base : nullptr;
  int32_t* const first = EDGE ? a.efirst + p.eunit : a.tfirst + p.tunit;
  int32_t* const last = EDGE ? a.elast + p.eunit : a.tlast + p.tunit;
  auto get = [&](int32_t i) {
    if (EDGE) return a.ecells[base + i];
    const uint2 c = a.tcells[base + i];
    return Item{c.x, c.y, 0u};
  };
  auto part = [&](int32_t at) {  // one starts here
    atomicMin(first + at / kUnit, at);
    atomicMax(last + at / kUnit, at);
  };
  int32_t lo = (int32_t)(start[cell] - start[0]);
  int32_t hi = (int64_t)cell + 1 < cells ? (int32_t)(start[cell + 1] - start[0]) : n;
  if (t == 0) *s_next = -1;
  for (;;) {
    if (t < 3) s_diff[t] = 0u;
    __syncthreads();
    {
      const Item e0 = get(lo);
      uint32_t dk = 0, dx = 0, dy = 0;
#pragma unroll 4
      for (int32_t i = lo + t; i < hi; i += kSplitBlock) {
        const Item e = get(i);
        dk |= e.k ^ e0.k;
        dx |= e.x ^ e0.x;
        dy |= e.y ^ e0.y;
      }
      if (dk) atomicOr(s_diff, dk);
      if (dx) atomicOr(s_diff + 1, dx);
      if (dy) atomicOr(s_diff + 2, dy);
    }
    __syncthreads();
    const uint32_t dk = s_diff[0], dx = s_diff[1], dy = s_diff[2];
    if ((dk | dx | dy) == 0u) {  // copies of one item
      if (t == 0) part(lo);
    } else {
      const int top = dk ? 95 - __clz(dk) : (dx ? 63 - __clz(dx) : 31 - __clz(dy));
      const int want = 31 - __clz((uint32_t)(hi - lo)) - 4;  // 16 items a bin if they are spread evenly
      const int bits = min(top + 1, min(want, kSplitBits)), sh = top + 1 - bits;
      auto bin = [&](const Item& e) {
        const uint64_t kx = (uint64_t)e.k << 32 | e.x;
        const uint64_t v = sh >= 32 ? kx >> (sh - 32) : kx << (32 - sh) | e.y >> sh;
        return (uint32_t)v & ((1u << bits) - 1u);
      };
      const int per = (1 << bits) > kSplitBlock ? (1 << bits) / kSplitBlock : 1;
      for (int i = t; i < (1 << bits); i += kSplitBlock) cnt[i] = 0u;
      __syncthreads();
#pragma unroll 4
      for (int32_t i = lo + t; i < hi; i += kSplitBlock) atomicAdd(cnt + bin(get(i)), 1u);
      __syncthreads();
      uint32_t sum = 0, total;
      const bool mine = t * per < (1 << bits);
      if (mine)
        for (int c = 0; c < per; ++c) sum += cnt[t * per + c];
      uint32_t at = block_exclusive_sum<kSplitBlock>(sum, s_scan, total);
      if (mine)
        for (int c = 0; c < per; ++c) {
          const uint32_t v = cnt[t * per + c];
          cnt[t * per + c] = at;
          if (v > 0u && v <= (uint32_t)kUnitCap) part(lo + (int32_t)at);
          at += v;
        }
      __syncthreads();
#pragma unroll 4
      for (int32_t i = lo + t; i < hi; i += kSplitBlock) {
        const Item e = get(i);
        const int32_t to = lo + (int32_t)atomicAdd(cnt + bin(e), 1u);
        tk[to] = e.k;
        tx[to] = e.x;
        if (EDGE) ty[to] = e.y;
      }
      __syncthreads();
#pragma unroll 4
      for (int32_t i = lo + t; i < hi; i += kSplitBlock) {
        if (EDGE) a.ecells[base + i] = Item{tk[i], tx[i], ty[i]};
        else a.tcells[base + i] = make_uint2(tk[i], tx[i]);
      }
      __syncthreads();
      // the bins that are still too large, as a list through the second
      // buffer: at a bin's first item its end and the next bin's first item
      // (a bin's count is its end by now)
      for (int i = t; i < (1 << bits); i += kSplitBlock) {
        const uint32_t e = cnt[i], b = i > 0 ? cnt[i - 1] : 0u;
        if (e - b <= (uint32_t)kUnitCap) continue;
        tk[lo + (int32_t)b] = (uint32_t)(lo + (int32_t)e);
        tx[lo + (int32_t)b] = (uint32_t)atomicExch(s_next, lo + (int32_t)b);
      }
    }
    __syncthreads();
    lo = *s_next;
    if (lo < 0) return;
    hi = (int32_t)tk[lo];
    const int32_t next = (int32_t)tx[lo];
    __syncthreads();  // everyone has the bin
    if (t == 0) *s_next = next;
  }
}

__global__ __launch_bounds__(kSplitBlock) void k_split(BuildArgs a) {
  __shared__ uint32_t s_cnt[1 << kSplitBits], s_scan[kSplitBlock / 64], s_diff[3];
  __shared__ int32_t s_next;
  if (*a.status != INT_MAX) return;
  for (int32_t i = blockIdx.x; i < a.ctr[2]; i += gridDim.x) {
    const int2 o = a.over[i];
    if (o.y < 0) split_cell<true>(a, a.plan[o.x], (uint32_t)o.y & 0x7fffffffu, s_cnt, s_scan, s_diff, &s_next);
    else split_cell<false>(a, a.plan[o.x], (uint32_t)o.y, s_cnt, s_scan, s_diff, &s_next);
    __syncthreads();
  }
}

// The items of unit u of a mesh with n: the cells, and parts of overfull cells,
// that start in [kUnit u, kUnit (u + 1)).  All but the last of them hold less
// than kUnit items, the last kUnitCap at most or copies of one item.
struct UnitRange {
  int32_t b, e;  // first item, behind the last
  int32_t cut;   // where more than kUnitCap items are divided: the last cell or part
  bool parts;    // of overfull cells are among them
};

__device__ __forceinline__ UnitRange unit_range(const uint32_t* start, int bits, int32_t n, int32_t u, bool over,
                                                const int32_t* first, const int32_t* last, int32_t (*s)[3]) {
  if (bits == 0) return UnitRange{u == 0 ? 0 : n, n, n, false};
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (w < 2) {
    int32_t x = 0, cell = 0, part = 0;
    if (u + w > 0) x = first_start(start, (int64_t)1 << bits, kUnit * (u + w), n, cell);
    // the cell before that one holds the item before the target
    if (over && cell > 0 && x - (int32_t)(start[cell - 1] - start[0]) > kUnitCap) {
      part = 1;
      for (int32_t v = u + w; kUnit * v < x; v += 64) {
        const int32_t f = kUnit * (v + lane) < x ? first[v + lane] : INT_MAX;
        const uint64_t in = __ballot(f < x);  // a later cell's part may be the first of its unit
        if (in) {
          x = __builtin_amdgcn_readlane(f, __builtin_ctzll(in));
          break;
        }
      }
    }
    if (lane == 0) { s[w][0] = x; s[w][1] = cell; s[w][2] = part; }
  }
  __syncthreads();
  UnitRange r{s[0][0], s[1][0], 0, (s[0][2] | s[1][2]) != 0};
  r.cut = r.e;
  if (r.e - r.b > kUnitCap) r.cut = s[1][2] ? last[u] : (int32_t)(start[s[1][1] - 1] - start[0]);
  return r;
}

// Bin of a code in a unit: about the place it will take, from the place of its
// cell and the code's bits below the cell's (bins cut evenly from the unit's
// code range leave a whole cell in one bin where the range spans a gap).
__device__ __forceinline__ uint32_t place_bin(const uint32_t* start, int bits, int32_t n, int32_t b, uint32_t key) {
  if (bits == 0) return __umulhi(key << (32 - kMortonBits), (uint32_t)n);
  const uint32_t cell = key >> (kMortonBits - bits);
  const uint32_t c0 = start[cell];
  const uint32_t size = (int64_t)cell + 1 < ((int64_t)1 << bits) ? start[cell + 1] - c0 : (uint32_t)n - (c0 - start[0]);
  return c0 - start[0] - (uint32_t)b + __umulhi(key << (32 - kMortonBits + bits), size);
}

// Half-edge i of a mesh, in the faces' order (meshes that are sorted in one cell).
__device__ __forceinline__ Item half_edge_item(const BuildArgs& a, const MeshPlan& p, int32_t i) {
  const int64_t f = (int64_t)p.f0 + i / 3;
  const int k = i % 3;
  const uint32_t u = (uint32_t)a.faces[3 * f + k], v = (uint32_t)a.faces[3 * f + (k == 2 ? 0 : k + 1)];
  return Item{a.ekey[3 * (int64_t)p.f0 + i], u < v ? u : v, u < v ? v : u};
}

__device__ __forceinline__ void sort_tris(const BuildArgs& a, int32_t block, SortLds<false>& s, int32_t (*s_range)[3]) {
  const int32_t m = a.tumap[block];
  const MeshPlan p = a.plan[m];
  const int bits = cell_bits(p.n);
  if (p.n <= 64) {
    if (threadIdx.x < 64)
      wave_sort<false>(
          p.n, [&](int32_t i) { return Item{a.key[p.f0 + i], (uint32_t)(p.f0 + i), 0u}; },
          [&](int32_t i, const Item& e) { a.sk[p.f0 + i] = e.k; a.sv[p.f0 + i] = e.x; });
    return;
  }
  const UnitRange u = unit_range(a.start + p.tcell, bits, p.n, block - p.tunit, a.ctr[2] != 0, a.tfirst + p.tunit,
                                 a.tlast + p.tunit, s_range);
  const int32_t n = u.e - u.b;
  if (n <= 0) return;
  const int64_t g0 = (int64_t)p.f0 + u.b;
  auto item = [&](int32_t i) {
    if (bits == 0) return Item{a.key[g0 + i], (uint32_t)(g0 + i), 0u};
    const uint2 c = a.tcells[g0 + i];
    return Item{c.x, c.y, 0u};
  };
  auto bin = [&](const Item& x) { return place_bin(a.start + p.tcell, bits, p.n, u.b, x.k); };
  auto store = [&](int32_t i, const Item& x) {
    a.sk[g0 + i] = x.k;
    a.sv[g0 + i] = x.x;
  };
  if ((u.parts || n > kUnitCap || lds_sort<false>(s, n, item, bin, store) < 0) && threadIdx.x == 0)
    a.packed[atomicAdd(a.ctr + 3, 1)] = block;
}

__device__ __forceinline__ void sort_edges(const BuildArgs& a, int32_t block, SortLds<true>& s, int32_t (*s_range)[3]) {
  const int32_t m = a.emap[block];
  const MeshPlan p = a.plan[m];
  const int32_t n3 = 3 * p.n;
  const int bits = cell_bits(n3);
  auto face_item = [&](int32_t i) { return half_edge_item(a, p, i); };
  if (n3 <= 64) {
    if (threadIdx.x >= 64) return;
    const int32_t kept = wave_sort<true>(n3, face_item, [&](int32_t i, const Item& e) {
      a.ul[3 * (int64_t)p.f0 + i] = e.x;
      a.uh[3 * (int64_t)p.f0 + i] = e.y;
    });
    if (threadIdx.x == 0) {
      a.ustart[block] = 0;
      a.ucount[block] = kept;
    }
    return;
  }
  const UnitRange u = unit_range(a.start + a.cells_t + p.ecell, bits, n3, block - p.eunit, a.ctr[2] != 0,
                                 a.efirst + p.eunit, a.elast + p.eunit, s_range);
  const int32_t n = u.e - u.b;
  const int64_t g0 = 3 * (int64_t)p.f0 + u.b;
  int32_t kept = 0;
  if (n > 0) {
    auto item = [&](int32_t i) { return bits != 0 ? a.ecells[g0 + i] : face_item(i); };
    auto bin = [&](const Item& x) { return place_bin(a.start + a.cells_t + p.ecell, bits, n3, u.b, x.k); };
    auto store = [&](int32_t i, const Item& x) {
      a.ul[g0 + i] = x.x;
      a.uh[g0 + i] = x.y;
    };
    kept = u.parts || n > kUnitCap ? -1 : lds_sort<true>(s, n, item, bin, store);
  }
  if (threadIdx.x == 0) {
    a.ustart[block] = u.b;
    a.ucount[block] = kept;
    if (kept < 0) a.packed[atomicAdd(a.ctr + 3, 1)] = block | (int)0x80000000u;
  }
}

// The sort units: of triangles (KIND 0), of half-edges (1), or one after the
// other (2, half-edges from block `tris` on).
template <int KIND>
__global__ __launch_bounds__(kLdsBlock) void k_sort(BuildArgs a, int32_t tris) {
  __shared__ alignas(16) char s_mem[sizeof(SortLds<KIND != 0>)];
  __shared__ int32_t s_range[2][3];
  if (*a.status != INT_MAX) return;
  const int32_t block = block_id();
  if (KIND == 0 || (KIND == 2 && block < tris)) {
    if (block >= a.plan[a.n_meshes].tunit) return;
    sort_tris(a, block, *reinterpret_cast<SortLds<false>*>(s_mem), s_range);
  } else {
    const int32_t unit = KIND == 2 ? block - tris : block;
    if (unit >= a.plan[a.n_meshes].eunit) return;
    sort_edges(a, unit, *reinterpret_cast<SortLds<true>*>(s_mem), s_range);
  }
}

// The units that k_sort leaves: parts of overfull cells, more items
// than LDS holds, or codes packed together (a mesh that is small against its
// box).  Every bit of the code may be equal there, so bins do not help, and
// comparing all items of a unit takes 370 us where this network takes some 30
// (build of 1,500 triangles of one code: 544 us by comparing, so 248 us).
__global__ __launch_bounds__(kLdsBlock) void k_sort_packed(BuildArgs a) {
  __shared__ SortLds<true> s;
  __shared__ int32_t s_range[2][3];
  if (*a.status != INT_MAX) return;
  for (int32_t w = blockIdx.x; w < a.ctr[3]; w += gridDim.x) {
    const bool edges = a.packed[w] < 0;
    const int32_t unit = a.packed[w] & 0x7fffffff;
    const MeshPlan p = a.plan[edges ? a.emap[unit] : a.tumap[unit]];
    const int32_t n_all = edges ? 3 * p.n : p.n, bits = cell_bits(n_all);
    const UnitRange u =
        edges ? unit_range(a.start + a.cells_t + p.ecell, bits, n_all, unit - p.eunit, true, a.efirst + p.eunit,
                           a.elast + p.eunit, s_range)
              : unit_range(a.start + p.tcell, bits, n_all, unit - p.tunit, true, a.tfirst + p.tunit, a.tlast + p.tunit,
                           s_range);
    int32_t kept = 0;
    // at most two rounds: the unit, or what comes before its last cell and that
    for (int32_t b = u.b, e = u.cut; b < u.e; b = e, e = u.e) {
      if (b == e) continue;
      const int32_t n = e - b <= kUnitCap ? e - b : 1;  // (more than LDS holds: copies of one half-edge)
      const int64_t g0 = (edges ? 3 : 1) * (int64_t)p.f0 + b, o0 = (edges ? 3 : 1) * (int64_t)p.f0 + u.b + kept;
      kept += network_sort<true>(
          s, n,
          [&](int32_t i) {
            if (!edges) {
              if (bits == 0) return Item{a.key[g0 + i], (uint32_t)(g0 + i), 0u};
              const uint2 c = a.tcells[g0 + i];
              return Item{c.x, c.y, 0u};
            }
            return bits != 0 ? a.ecells[g0 + i] : half_edge_item(a, p, b + i);
          },
          [&](int32_t i, const Item& x) {
            if (edges) {
              a.ul[o0 + i] = x.x;
              a.uh[o0 + i] = x.y;
            } else {
              a.sk[o0 + i] = x.k;
              a.sv[o0 + i] = x.x;
            }
          });
    }
    if (edges && threadIdx.x == 0) a.ucount[unit] = kept;
    __syncthreads();  // s_range is written again
  }
}

// ---- step 4: radix tree and boxes --------------------------------------------------

// Length of the common prefix of the codes of positions i and i + 1 (equal
// codes are told apart by position).
__device__ __forceinline__ int prefix(uint32_t ki, uint32_t kj, int i) {
  return ki != kj ? __clz(ki ^ kj) : 32 + __clz((uint32_t)(i ^ (i + 1)));
}

__device__ __forceinline__ void grow_box(float* b, const float* c) {
#pragma unroll
  for (int k = 0; k < 3; ++k) { b[k] = fminf(b[k], c[k]); b[3 + k] = fmaxf(b[3 + k], c[3 + k]); }
}

// The radix tree over up to N consecutive units (positions, or subtrees that
// tile a range), bottom up in LDS.  A subtree over units [lo, hi] is the left
// child of its parent if the codes across hi share more bits than those across
// lo, so a climb needs the prefix lengths of neighbours only and no search for
// a node's range.  The parent is met at the boundary between its two
// children: the first to arrive leaves its box and its far end there and ends,
// the second goes on with both.
template <int N>
struct ClimbLds {
  float box[2][6][N + 1];  // by boundary: of the left child, of the right child
  uint32_t cnt[N + 1];     // arrivals << 16 | far end of the first (a sum once both are there)
  int32_t d[N + 1];        // prefix length across the boundary below unit u; -1 at the ends of a mesh
  uint32_t mark[N / 32];   // units that start a subtree left over
};

// Climbs from unit u of nu with box b; node(lo, split, hi, id of the node in
// units, left box, right box) takes each inner node.  A subtree whose parent
// reaches beyond the units stays at its boundary with one arrival.
template <int N, typename NodeOut>
__device__ __forceinline__ void climb(ClimbLds<N>& s, int u, float* b, NodeOut node) {
  int lo = u, hi = u;
  int dl = s.d[lo], dh = s.d[hi + 1];
  for (;;) {
    const bool left = dh > dl;
    const int at = left ? hi + 1 : lo;  // the boundary below unit `at`
#pragma unroll
    for (int k = 0; k < 6; ++k) s.box[left ? 0 : 1][k][at] = b[k];
    const uint32_t old = __hip_atomic_fetch_add(&s.cnt[at], 0x10000u + (uint32_t)(left ? lo : hi), __ATOMIC_ACQ_REL,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
    if (old == 0u) break;  // the sibling is not done yet, or lies beyond the units
    float o[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) o[k] = s.box[left ? 1 : 0][k][at];
    if (left) hi = (int)(old & 0xffffu);
    else lo = (int)(old & 0xffffu);
    dl = s.d[lo];
    dh = s.d[hi + 1];
    float lb[6], rb[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) { lb[k] = left ? b[k] : o[k]; rb[k] = left ? o[k] : b[k]; }
    node(lo, at - 1, hi, dh > dl, lb, rb);
    grow_box(b, o);
  }
}

// The subtrees left over, in order of position, to a root list: out(k, first
// unit, last unit, box) is called for the k-th.  Returns their number.
template <int N, int B, typename Out>
__device__ __forceinline__ int32_t leftover(ClimbLds<N>& s, int nu, Out out) {
  for (int i = threadIdx.x; i < N / 32; i += B) s.mark[i] = 0u;
  __syncthreads();
  for (int i = threadIdx.x; i <= nu; i += B) {
    if (s.cnt[i] >> 16 != 1u) continue;
    const int v = (int)(s.cnt[i] & 0xffffu), lo = v < i ? v : i;
    atomicOr(&s.mark[lo >> 5], 1u << (lo & 31));
  }
  __syncthreads();
  for (int i = threadIdx.x; i <= nu; i += B) {
    if (s.cnt[i] >> 16 != 1u) continue;
    const int v = (int)(s.cnt[i] & 0xffffu);
    const bool left = v < i;  // the left child [v, i - 1] or the right child [i, v]
    const int lo = left ? v : i;
    int32_t k = __popc(s.mark[lo >> 5] & ((1u << (lo & 31)) - 1u));
    for (int q = 0; q < lo >> 5; ++q) k += __popc(s.mark[q]);
    float b[6];
#pragma unroll
    for (int x = 0; x < 6; ++x) b[x] = s.box[left ? 0 : 1][x][i];
    out(k, lo, left ? i - 1 : v, b);
  }
  int32_t n = 0;
  for (int q = 0; q < N / 32; ++q) n += __popc(s.mark[q]);
  return n;
}

// A binary node, kept only where the collapse may open it.
__device__ __forceinline__ void put_node(const BuildArgs& a, const MeshPlan& p, int32_t lo, int32_t split, int32_t hi,
                                         bool left, const float* lb, const float* rb) {
  if (hi - lo < a.leaf) return;
  BinNode nd;
#pragma unroll
  for (int k = 0; k < 6; ++k) { nd.box[0][k] = lb[k]; nd.box[1][k] = rb[k]; }
  nd.lo = lo;
  nd.split = split;
  nd.hi = hi;
  nd.pad = 0;
  a.bin[(int64_t)p.f0 + (left ? hi : lo)] = nd;
}

// One chunk of kTreeChunk sorted positions: writes the triangles in leaf
// order (through LDS, whole lines at a time) and builds the nodes that lie
// inside the chunk.  The subtrees that tile the chunk go to its root list, and
// the nodes that reach beyond it are left to k_tree_top.  Most nodes of a mesh
// lie inside a chunk, where a level costs LDS latency instead of a round trip
// to memory.  Nodes of at most `leaf` triangles, more than half of them all at
// four, are not written.  Refit of 2 x 35 M triangles in 4,096 meshes: one
// block a mesh climbing in memory 11.1 ms, chunks with a search for each
// node's range and triangles written by their own lanes 4.6 ms, this 3.4 ms.
__global__ __launch_bounds__(kTreeBlock) void k_tree(BuildArgs a) {
  const int32_t block = block_id();
  static_assert(kTreeBlock == kTreeChunk, "one position a thread");
  __shared__ ClimbLds<kTreeChunk> s;
  if (*a.status != INT_MAX) return;
  if (block >= a.plan[a.n_meshes].tchunk) return;
  const int32_t m = a.tmap[block];
  const MeshPlan p = a.plan[m];
  const int32_t n = p.n, c0 = (block - p.tchunk) * kTreeChunk, nu = min(n - c0, kTreeChunk);
  const uint32_t* keys = a.sk + p.f0;
  const int t = threadIdx.x;
  float b[6];
  float* stage = &s.box[0][0][0];  // [9 * kTreeChunk] of its 12 * (kTreeChunk + 1)
  if (t < nu) {
    const int64_t g = (int64_t)p.f0 + c0 + t;
    const int64_t f = a.sv[g];
    float v[9];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const f3 x = load_v(a.verts, p.v0 + a.faces[3 * f + k]);
      v[3 * k] = x.x; v[3 * k + 1] = x.y; v[3 * k + 2] = x.z;
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) stage[9 * t + k] = v[k];
    a.triid[g] = (int32_t)(f - p.f0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      b[k] = fminf(fminf(v[k], v[3 + k]), v[6 + k]);
      b[3 + k] = fmaxf(fmaxf(v[k], v[3 + k]), v[6 + k]);
    }
  }
  s.cnt[t] = 0u;
  if (t == 0) s.cnt[nu] = 0u;
  for (int i = t; i <= nu; i += kTreeBlock) {
    const int32_t j = c0 + i;
    s.d[i] = j > 0 && j < n ? prefix(keys[j - 1], keys[j], j - 1) : -1;
  }
  __syncthreads();
  float* tr = a.tris + 9 * ((int64_t)p.f0 + c0);
  for (int i = t; i < 9 * nu; i += kTreeBlock) tr[i] = stage[i];
  __syncthreads();
  if (t < nu)
    climb(s, t, b, [&](int lo, int split, int hi, bool left, const float* lb, const float* rb) {
      put_node(a, p, c0 + lo, c0 + split, c0 + hi, left, lb, rb);
    });
  if (n <= kTreeChunk) return;
  const int32_t rc = p.rchunk + block - p.tchunk;  // the chunk's root list
  RootRec* out = a.roots + (int64_t)rc * kMaxRoots;
  const int32_t nr = leftover<kTreeChunk, kTreeBlock>(s, nu, [&](int32_t k, int, int hi, const float* x) {
    RootRec r;
#pragma unroll
    for (int q = 0; q < 6; ++q) r.box[q] = x[q];
    r.hi = c0 + hi;
    r.d = s.d[hi + 1];
    out[k] = r;
  });
  if (t == 0) a.nroots[rc] = nr;
}

// The nodes that span chunks, one block per mesh of several: the same climb
// with the chunks' subtrees as units, as many whole root lists at a time as
// LDS takes.  A mesh of more leaves shorter lists in place of its first ones
// and goes over them again, until one pass takes all (a pass takes at least
// kTopUnits / kMaxRoots lists and leaves one).  2 x 35 M triangles in 4,096
// meshes: climbing in memory 1.2 ms, this 0.31 ms.
__global__ __launch_bounds__(kTopUnits) void k_tree_top(BuildArgs a) {
  __shared__ ClimbLds<kTopUnits> s;
  __shared__ int32_t s_hi[kTopUnits];              // last position of each unit
  __shared__ int32_t s_off[kTopLists + 1], s_lists;  // first unit of each list of the pass
  if (*a.status != INT_MAX) return;
  const int t = threadIdx.x, lane = t & 63;
  for (int32_t k = blockIdx.x; k < a.ctr[0]; k += gridDim.x) {
    const int32_t m = a.big[k];
    const MeshPlan p = a.plan[m];
    int32_t lists = div_up(p.n, kTreeChunk), made = 0;
    do {
      made = 0;
      int32_t first = 0;  // first position of the next pass
      for (int32_t c = 0; c < lists; ++made) {
        __syncthreads();  // the last pass is read
        if (t < 64) {
          int32_t sum = 0, use = 0;
          for (; use < kTopLists; use += 64) {
            int32_t x = c + use + lane < lists ? a.nroots[p.rchunk + c + use + lane] : 0;
            for (int o = 1; o < 64; o <<= 1) {
              const int32_t y = __shfl_up(x, o);
              if (lane >= o) x += y;
            }
            s_off[use + lane + 1] = sum + x;
            const uint64_t fit = __ballot(c + use + lane < lists && sum + x <= kTopUnits);
            if (~fit) {
              use += __builtin_ctzll(~fit);
              break;
            }
            sum += __shfl(x, 63);
          }
          if (lane == 0) {
            s_off[0] = 0;
            s_lists = use;
          }
        }
        __syncthreads();
        const int32_t use = s_lists, nu = s_off[use];
        float b[6];
        s.cnt[t] = 0u;
        if (t == 0) s.cnt[nu] = 0u;
        if (t < nu) {
          int q = 0;  // the list that holds unit t
          for (int h = kTopLists >> 1; h > 0; h >>= 1)
            if (q + h < use && s_off[q + h] <= t) q += h;
          const RootRec r = a.roots[(int64_t)(p.rchunk + c + q) * kMaxRoots + t - s_off[q]];
#pragma unroll
          for (int x = 0; x < 6; ++x) b[x] = r.box[x];
          s_hi[t] = r.hi;
          s.d[t + 1] = r.d;
        }
        if (t == 0) s.d[0] = first > 0 ? prefix(a.sk[(int64_t)p.f0 + first - 1], a.sk[(int64_t)p.f0 + first], first - 1) : -1;
        __syncthreads();
        auto pos_lo = [&](int u) { return u == 0 ? first : s_hi[u - 1] + 1; };
        if (t < nu)
          climb(s, t, b, [&](int lo, int split, int hi, bool left, const float* lb, const float* rb) {
            put_node(a, p, pos_lo(lo), s_hi[split], s_hi[hi], left, lb, rb);
          });
        if (c > 0 || use < lists) {
          RootRec* out = a.roots + (int64_t)(p.rchunk + made) * kMaxRoots;
          const int32_t nr = leftover<kTopUnits, kTopUnits>(s, nu, [&](int32_t i, int, int hi, const float* x) {
            RootRec r;
#pragma unroll
            for (int q = 0; q < 6; ++q) r.box[q] = x[q];
            r.hi = s_hi[hi];
            r.d = s.d[hi + 1];
            out[i] = r;
          });
          if (t == 0) a.nroots[p.rchunk + made] = nr;
        }
        first = s_hi[nu - 1] + 1;
        c += use;
      }
      lists = made;
      __syncthreads();  // the lists are written before they are read again
    } while (made > 1);
  }
}

// ---- step 5: collapse to width W -------------------------------------------

__device__ __forceinline__ float half_area(const float* b) {
  float dx = b[3] - b[0], dy = b[4] - b[1], dz = b[5] - b[2];
  return dx * dy + dy * dz + dz * dx;
}

// What opening a child of more than L triangles is worth, at least -0.5.  A
// NaN (an overflowed extent times none) counts as the least: every such child
// can be opened, so a node of less than W children holds leaves only, which
// the capacity of nodes rests on.
__device__ __forceinline__ float score(const BuildArgs& a, const float* b, int32_t cn) {
  const float ar = half_area(b), s = a.builder == 1 ? ar * (float)cn : ar;
  return s >= 0.f ? s : -0.5f;
}

// One step of an argmax over a lane group: the better of the lane's candidate
// and that of the lane the DPP pattern names.
template <int DPP>
__device__ __forceinline__ void argmax_step(float& top, int& lane, int& node) {
  const float ot = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(top), DPP, 0xf, 0xf, true));
  const int ol = __builtin_amdgcn_mov_dpp(lane, DPP, 0xf, 0xf, true);
  const int on = __builtin_amdgcn_mov_dpp(node, DPP, 0xf, 0xf, true);
  if (ot > top || (ot == top && ol < lane)) { top = ot; lane = ol; node = on; }
}

// One wide node for each W lanes of the wave (lane c of the group holds child
// c): from the two children of binary node x, the group keeps opening the
// child of largest score (builder 0: surface area, builder 1: surface area
// x triangle count, its term of the surface-area cost) among those of more
// than L triangles until it has W or none can be opened; an opened child's two
// halves go to its own lane and to the next free one, each read straight from
// its binary node by get(node, side, box, lo, split, hi).  The node goes to the
// group's slot slot_of(), asked for (by the whole wave) when the children are
// known.  On return a lane whose child needs a wide node of its own has its
// binary node in cx, its triangles in cn and its first position in cf (f0 is
// that of position 0); its reference is still to be written (child_ref).
template <int W, typename Get, typename Slot>
__device__ __forceinline__ void collapse_group(const BuildArgs& a, int32_t node0, bool on, int32_t x, Get get,
                                               Slot slot_of, int32_t& cx, int32_t& cn, int32_t& cf, int32_t f0) {
  const int c = (int)(threadIdx.x & 63) % W;
  const int L = a.leaf;
  float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  int32_t node = -1;
  cf = 0;
  cn = 0;
  auto take = [&](int32_t y, int side) {
    int32_t lo, split, hi;
    get(y, side, b, lo, split, hi);
    cf = side == 0 ? lo : split + 1;
    cn = side == 0 ? split - lo + 1 : hi - split;
    node = side == 0 ? split : split + 1;
  };
  if (on && c < 2) take(x, c);
#pragma unroll 1
  for (int ns = 2; ns < W; ++ns) {
    // the best child: largest score, the lowest lane among equals
    float top = -1.f;
    if (cn > L) top = score(a, b, cn);
    int best = c, y = node;
    argmax_step<0xb1>(top, best, y);                // lanes 1 apart
    if (W >= 4) argmax_step<0x4e>(top, best, y);    // lanes 2 apart
    if (W >= 8) argmax_step<0x141>(top, best, y);   // the two halves of eight lanes, mirrored
    const bool open = on && top > -1.f;
    if (!__ballot(open)) break;
    // a group that opens none is done (its later rounds open none either)
    if (open && (c == best || c == ns)) take(y, c == best ? 0 : 1);
  }
  cx = -1;
  const int32_t slot = slot_of();
  if (on) {
    float* nd = reinterpret_cast<float*>(a.nodes + sizeof(Node<W>) * ((int64_t)node0 + slot));
#pragma unroll
    for (int k = 0; k < 6; ++k) nd[k * W + c] = b[k];
    int32_t* ch = reinterpret_cast<int32_t*>(nd) + 6 * W;
    ch[W + c] = 0;
    if (cn == 0) ch[c] = kEmpty;
    else if (cn <= L) ch[c] = leaf_ref(f0 + cf, cn);
    else cx = node;
  }
}

// Child c of the wide node at `slot` of a mesh is the one at slot `child`.
template <int W>
__device__ __forceinline__ void child_ref(const BuildArgs& a, int32_t node0, int32_t slot, int c, int32_t child) {
  reinterpret_cast<int32_t*>(a.nodes + sizeof(Node<W>) * ((int64_t)node0 + slot))[6 * W + c] = node0 + child;
}

// Top of the trees of meshes of more than kSubtree triangles, one block per
// mesh, one level of wide nodes a round: children of more than kSubtree
// triangles go on in the block, smaller ones to the list of subtrees.
// Slots are numbered in creation order (root 0, its inner children next).
template <int W>
__global__ __launch_bounds__(kBlock) void k_collapse_top(BuildArgs a) {
  constexpr int G = 64 / W, B = (kBlock / 64) * G;  // items of a wave, of a block
  __shared__ int32_t s_used, s_tail, s_depth;
  if (*a.status != INT_MAX) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int32_t k = blockIdx.x; k < a.ctr[0]; k += gridDim.x) {
    const int32_t m = a.big[k];
    const MeshPlan p = a.plan[m];
    int32_t* items = a.items + 3 * (int64_t)p.f0;
    if (threadIdx.x == 0) {
      items[0] = 0;
      items[1] = 0;
      items[2] = 1;
      s_used = 1;
      s_tail = 1;
      s_depth = 1;
    }
    __syncthreads();
    int32_t head = 0;
    for (;;) {
      const int32_t tail = s_tail;
      __syncthreads();  // every thread has the level's end before items are appended
      if (head >= tail) break;
      for (int32_t i0 = head; i0 < tail; i0 += B) {
        const int32_t i = i0 + w * G + lane / W;
        const bool on = i < tail;
        int32_t x = 0, slot = 0, dep = 0, cx, cn, cf;
        if (on) { x = items[3 * i]; slot = items[3 * i + 1]; dep = items[3 * i + 2]; }
        collapse_group<W>(a, p.node, on, x, [&](int32_t y, int side, float* bx, int32_t& lo, int32_t& split, int32_t& hi) {
          const BinNode& nd = a.bin[(int64_t)p.f0 + y];
#pragma unroll
          for (int q = 0; q < 6; ++q) bx[q] = nd.box[side][q];
          lo = nd.lo;
          split = nd.split;
          hi = nd.hi;
        }, [&] { return slot; }, cx, cn, cf, p.f0);
        const uint64_t inner = __ballot(cx >= 0), here = __ballot(cx >= 0 && cn > kSubtree), down = inner & ~here;
        int32_t s0 = 0, t0 = 0, l0 = 0;
        if (lane == 0) {
          if (inner) s0 = atomicAdd(&s_used, __popcll(inner));
          if (here) t0 = atomicAdd(&s_tail, __popcll(here));
          if (down) l0 = atomicAdd(a.ctr + 1, __popcll(down));
        }
        s0 = __shfl(s0, 0);
        t0 = __shfl(t0, 0);
        l0 = __shfl(l0, 0);
        if (cx >= 0) {
          const int32_t cs = s0 + lanes_before(inner);
          child_ref<W>(a, p.node, slot, lane % W, cs);
          if (cn > kSubtree) {
            int32_t* o = items + 3 * (t0 + lanes_before(here));
            o[0] = cx;
            o[1] = cs;
            o[2] = dep + 1;
          } else {
            const uint32_t last = cx != cf ? 0x80000000u : 0u;
            a.subs[l0 + lanes_before(down)] = SubItem{m, cf, cs, (uint32_t)(dep + 1) | (uint32_t)cn << 8 | last};
          }
        }
        if (on && lane % W == 0) atomicMax(&s_depth, dep);
      }
      head = tail;
      __syncthreads();  // the next level's items are written
    }
    if (threadIdx.x == 0) {
      a.used[m] = s_used;
      atomicMax(a.depth + m, s_depth);
    }
    __syncthreads();
  }
}

// The subtrees, packed: a block takes as many in a row as kPack positions
// hold.  Their binary nodes (those of their positions, one range of memory
// each) are read once, whole, into LDS, as ranges and the scores of the two
// children.  Then one thread collapses one wide node (rules and order of
// children as in collapse_group): it keeps its children's scores and names in
// registers, so an opened child costs one LDS round trip.  Wide nodes are
// queued breadth first, a round for each level; a node numbers its inner
// children when it is done, so the subtree's slots are reserved by one atomic
// at the end, and the nodes are written by W lanes each, lane by child, with
// the boxes read a second time.  Bound by those three passes over memory and,
// in small builds, by the chain of one pack.  2 x 35 M triangles at W = 8,
// L = 1 and 2 x 1 M at W = 4, L = 4: a wave for each subtree, W lanes for each
// node, reading binary nodes as they are opened 6.15 and 0.205 ms, with the
// boxes in LDS too (four packs a compute unit) 4.1 and 0.31 ms, this 3.35 and 0.156 ms.
template <int W>
__global__ __launch_bounds__(kPackBlock, 8) void k_collapse_sub(BuildArgs a) {
  // Wide nodes: those of less than W children hold leaves only, two triangles
  // or more, and each of the others adds W - 1 children to the tree.
  constexpr int Q = kPack / 2 + (kPack / 2) / (W - 1) + 1;
  constexpr uint32_t kNone = 0xffffu;
  __shared__ float s_score[2][kPack];  // of the children; -1: not to be opened
  __shared__ uint32_t s_at[kPack];     // lo | split << 10 | hi << 20, packed positions
  // binary node | subtree << 10 | number in the subtree << 16; once collapsed,
  // first inner child's number | subtree << 10 | number << 16
  __shared__ uint32_t s_q[Q];
  __shared__ uint16_t s_kid[Q * W];    // binary node | side << 10 of each child
  __shared__ int32_t s_mesh[64], s_node0[64], s_tri0[64];  // mesh, its first node, blob's triangle of packed position 0
  __shared__ int32_t s_slot[64], s_n[64];                  // root's slot, wide nodes
  __shared__ int32_t s_depth[64], s_deep[64];              // root's depth, levels below it
  __shared__ int32_t s_back[64];
  __shared__ uint8_t s_of[kPack];      // subtree of each position
  __shared__ int32_t s_off[65];        // first packed position of each subtree
  __shared__ int32_t s_push[3], s_use;
  static_assert(kSubtree <= kPack && kPack <= 1024, "ten bits a position");
  if (*a.status != INT_MAX) return;
  const int t = threadIdx.x, lane = t & 63, L = a.leaf;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int64_t total = a.ctr[1];
  const int32_t end = (int32_t)(total * (blockIdx.x + 1) / gridDim.x);
  for (int32_t e = (int32_t)(total * blockIdx.x / gridDim.x); e < end;) {
    __syncthreads();  // the last pack is done
    if (t < 64) {
      SubItem it{0, 0, 0, 0};
      if (e + lane < end) it = a.subs[e + lane];
      const int32_t n = (int32_t)(it.info >> 8 & 0x7fffffu);
      int32_t x = n;
      for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
      }
      const uint64_t full = ~__ballot(e + lane < end && x <= kPack);
      const int use = full ? __builtin_ctzll(full) : 64;
      if (lane < use) {
        const int32_t off = x - n;
        const MeshPlan& p = a.plan[it.mesh];
        s_mesh[lane] = it.mesh;
        s_node0[lane] = p.node;
        s_tri0[lane] = p.f0 + it.lo - off;
        s_back[lane] = off - it.lo;
        s_slot[lane] = it.slot;
        s_n[lane] = 1;
        s_depth[lane] = (int32_t)(it.info & 0xffu);
        s_deep[lane] = 0;
        s_off[lane + 1] = x;
        s_q[lane] = (uint32_t)(off + (it.info >> 31 ? n - 1 : 0)) | (uint32_t)lane << 10;
      }
      if (lane == 0) {
        s_off[0] = 0;
        s_use = use;
        s_push[0] = 0;
        s_push[1] = 0;
      }
    }
    __syncthreads();
    const int use = s_use;
    e += use;
    for (int q = w; q < use; q += kPackBlock / 64)
      for (int k = s_off[q] + lane; k < s_off[q + 1]; k += 64) s_of[k] = (uint8_t)q;
    __syncthreads();
    for (int k = t; k < s_off[use]; k += kPackBlock) {
      const BinNode nd = a.bin[(int64_t)s_tri0[s_of[k]] + k];
      const int back = s_back[s_of[k]], nl = nd.split - nd.lo + 1, nr = nd.hi - nd.split;
      s_at[k] = (uint32_t)(nd.lo + back) | (uint32_t)(nd.split + back) << 10 | (uint32_t)(nd.hi + back) << 20;
      s_score[0][k] = nl > L ? score(a, nd.box[0], nl) : -1.f;
      s_score[1][k] = nr > L ? score(a, nd.box[1], nr) : -1.f;
    }
    int32_t head = 0, tail = use;
    for (int r = 0; head < tail; ++r) {
      __syncthreads();  // the round's nodes and the scores are in place
      if (t == 0) s_push[(r + 1) % 3] = 0;
      for (int32_t i = head + t; i < tail; i += kPackBlock) {
        const uint32_t q = s_q[i];
        const uint32_t sub = q >> 10 & 63u;
        float sc[W];
        uint32_t kid[W];  // binary node | side << 10 | the child's own node << 16
        auto open = [&](uint32_t y, float& s0, uint32_t& k0, float& s1, uint32_t& k1) {
          const uint32_t split = s_at[y] >> 10 & 1023u;
          s0 = s_score[0][y];
          s1 = s_score[1][y];
          k0 = y | split << 16;
          k1 = y | 1024u | (split + 1) << 16;
        };
        open(q & 1023u, sc[0], kid[0], sc[1], kid[1]);
        int nk = 2;
        bool more = true;
#pragma unroll
        for (int ns = 2; ns < W; ++ns) {
          sc[ns] = -1.f;
          kid[ns] = kNone;
          // the best child: largest score, the first among equals
          float top = sc[0];
          uint32_t best = kid[0];
          int at = 0;
#pragma unroll
          for (int c = 1; c < ns; ++c)
            if (sc[c] > top) { top = sc[c]; best = kid[c]; at = c; }
          more = more && top > -1.f;
          if (more) {
            float s0;
            uint32_t k0;
            open(best >> 16, s0, k0, sc[ns], kid[ns]);
#pragma unroll
            for (int c = 0; c < ns; ++c)
              if (c == at) { sc[c] = s0; kid[c] = k0; }
            nk = ns + 1;
          }
        }
        uint32_t deeper = 0;  // children of more than L triangles
#pragma unroll
        for (int c = 0; c < W; ++c) {
          s_kid[i * W + c] = (uint16_t)(c < nk ? kid[c] & 2047u : kNone);
          if (c < nk && sc[c] > -1.f) deeper |= 1u << c;
        }
        uint32_t num = 0;
        if (deeper) {
          const int m = __popc(deeper);
          num = (uint32_t)atomicAdd(&s_n[sub], m);
          int32_t to = tail + atomicAdd(&s_push[r % 3], m);
          uint32_t nx = num;
#pragma unroll
          for (int c = 0; c < W; ++c)
            if (deeper >> c & 1u) s_q[to++] = kid[c] >> 16 | sub << 10 | nx++ << 16;
        }
        s_q[i] = num | (q & 0xfffffc00u);
        s_deep[sub] = r;  // every writer of a round has the same
      }
      __syncthreads();
      head = tail;
      tail += s_push[r % 3];
    }
    if (t < use) {
      const int32_t n = s_n[t];
      atomicMax(a.depth + s_mesh[t], s_depth[t] + s_deep[t]);
      s_n[t] = n > 1 ? atomicAdd(a.used + s_mesh[t], n - 1) - 1 : 0;
    }
    __syncthreads();
    for (int32_t i = t; i < tail * W; i += kPackBlock) {
      const uint32_t q = s_q[i / W], kid = s_kid[i];
      const uint32_t sub = q >> 10 & 63u, num = q >> 16;
      const int c = i % W, y = (int)(kid & 1023u), side = (int)(kid >> 10 & 1u);
      float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
      int32_t cn = 0, cf = 0;
      if (kid != kNone) {
        const uint32_t at = s_at[y];
        const int lo = (int)(at & 1023u), split = (int)(at >> 10 & 1023u), hi = (int)(at >> 20);
        cf = side == 0 ? lo : split + 1;
        cn = side == 0 ? split - lo + 1 : hi - split;
#pragma unroll
        for (int x = 0; x < 6; ++x) b[x] = a.bin[(int64_t)s_tri0[sub] + y].box[side][x];
      }
      const uint64_t inner = __ballot(cn > L) >> (lane - c) & ((1u << W) - 1u);
      const int32_t slot = num == 0 ? s_slot[sub] : s_n[sub] + (int32_t)num;
      const int32_t node0 = s_node0[sub];
      int32_t ref;
      if (cn == 0) ref = kEmpty;
      else if (cn <= L) ref = leaf_ref(s_tri0[sub] + cf, cn);
      else ref = node0 + s_n[sub] + (int32_t)(q & 1023u) + __popc((uint32_t)inner & ((1u << c) - 1u));
      float* nd = reinterpret_cast<float*>(a.nodes + sizeof(Node<W>) * ((int64_t)node0 + slot));
#pragma unroll
      for (int x = 0; x < 6; ++x) nd[x * W + c] = b[x];
      reinterpret_cast<int32_t*>(nd)[6 * W + c] = ref;
      reinterpret_cast<int32_t*>(nd)[7 * W + c] = 0;
    }
  }
}

// ---- step 6: groups of unique edges --------------------------------------------------

// Unique edges of each mesh, and of the mesh before each of its units; one wave per mesh.
__global__ __launch_bounds__(kBlock) void k_edge_mesh(BuildArgs a) {
  if (*a.status != INT_MAX) return;
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t m = (blockIdx.x * (int64_t)kBlock + threadIdx.x) >> 6; m < a.n_meshes; m += nw) {
    const int32_t u0 = a.plan[m].eunit, u1 = a.plan[m + 1].eunit;
    int32_t run = 0;
    for (int32_t u = u0; u < u1; u += 64) {
      const int32_t c = u + lane < u1 ? a.ucount[u + lane] : 0;
      const int32_t inc = wave_inclusive_sum(c);
      if (u + lane < u1) a.uoff[u + lane] = run + inc - c;
      run += __shfl(inc, 63);
    }
    if (lane == 0) {
      a.nedges[m] = run;
      a.groups[m] = (run + kChunk - 1) / kChunk;
    }
  }
}

// One block: groups before each mesh; the totals at [M].
__global__ __launch_bounds__(1024) void k_group_plan(BuildArgs a) {
  __shared__ int64_t s[16];
  if (*a.status != INT_MAX) return;
  int64_t run = 0, edges = 0;
  for (int64_t base = 0; base < a.n_meshes; base += 4096) {
    int64_t v[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t m = base + 4 * (int64_t)threadIdx.x + k;
      v[k] = m < a.n_meshes ? a.groups[m] : 0;
      edges += m < a.n_meshes ? a.nedges[m] : 0;
      sum += v[k];
    }
    int64_t total;
    int64_t o = run + block_exclusive_sum<1024>(sum, s, total);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t m = base + 4 * (int64_t)threadIdx.x + k;
      if (m < a.n_meshes) a.groups[m] = o;
      o += v[k];
    }
    run += total;
  }
  edges = block_sum<1024>(edges, s);
  if (threadIdx.x == 0) {
    a.groups[a.n_meshes] = run;
    *a.etotal = edges;
  }
}

// The descriptors' counts, and the mesh of every group; one wave per mesh.
__global__ __launch_bounds__(kBlock) void k_mesh_final(BuildArgs a) {
  if (*a.status != INT_MAX) return;
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t m = (blockIdx.x * (int64_t)kBlock + threadIdx.x) >> 6; m < a.n_meshes; m += nw) {
    const int64_t g0 = a.groups[m], g1 = a.groups[m + 1];
    const MeshPlan p = a.plan[m];
    if (lane == 0) {
      MeshDesc& d = a.mesh[m];
      d.chunk_base = (int32_t)g0;
      d.n_chunks = (int32_t)(g1 - g0);
      d.n_edges = a.nedges[m];
      if (p.n > a.leaf) {
        d.n_nodes = a.used[m];
        d.depth = a.depth[m];
        if (a.depth[m] > kMaxDepth || a.used[m] > a.plan[m + 1].node - p.node) atomicMin(a.status, p.f0);
      }
      if (g1 > a.chunk_cap) atomicMin(a.status, 0);
    }
    for (int64_t g = g0 + lane; g < g1 && g < a.chunk_cap; g += 64) a.cmesh[g] = (int32_t)m;
  }
}

// One wave per group of 64 unique edges: endpoints, vertex ids and the exact
// box of the group.
__global__ __launch_bounds__(kBlock) void k_groups(BuildArgs a) {
  if (*a.status != INT_MAX) return;
  const int lane = threadIdx.x & 63;
  const int64_t total = a.groups[a.n_meshes];
  const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t g = (blockIdx.x * (int64_t)kBlock + threadIdx.x) >> 6; g < total; g += nw) {
    const int32_t m = a.cmesh[g];
    const MeshPlan p = a.plan[m];
    const int32_t u1 = a.plan[m + 1].eunit, ne = a.nedges[m];
    const int32_t e0 = (int32_t)(g - a.groups[m]) * kChunk, e = e0 + lane;
    const bool live = e < ne;
    // the last unit that starts at or before e0, then on from there
    int32_t u = p.eunit;
    for (int32_t lo = p.eunit, n = u1 - p.eunit; n > 1;) {
      const int32_t step = (n + 63) / 64, probe = lo + lane * step;
      const uint64_t le = __ballot(probe < lo + n && a.uoff[min(probe, u1 - 1)] <= e0);
      lo += (63 - __builtin_clzll(le | 1ull)) * step;
      n = min(step, u1 - lo);
      u = lo;
    }
    if (live)
      while (u + 1 < u1 && a.uoff[u + 1] <= e) ++u;
    float v[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    uint32_t x = 0, y = 0;
    if (live) {
      const int64_t at = 3 * (int64_t)p.f0 + a.ustart[u] + (e - a.uoff[u]);
      x = a.ul[at];
      y = a.uh[at];
      const f3 s = load_v(a.verts, p.v0 + x), q = load_v(a.verts, p.v0 + y);
      v[0] = s.x; v[1] = s.y; v[2] = s.z; v[3] = q.x; v[4] = q.y; v[5] = q.z;
      float* o = a.seg + g * (6 * kChunk);
#pragma unroll
      for (int k = 0; k < 6; ++k) o[k * kChunk + lane] = v[k];
      int32_t* ed = a.edge + g * (2 * kChunk);
      ed[lane] = (int32_t)x;
      ed[kChunk + lane] = (int32_t)y;
    }
    float b[6];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      b[k] = live ? fminf(v[k], v[3 + k]) : INFINITY;
      b[3 + k] = live ? fmaxf(v[k], v[3 + k]) : -INFINITY;
    }
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        b[k] = fminf(b[k], __shfl_xor(b[k], o));
        b[3 + k] = fmaxf(b[3 + k], __shfl_xor(b[3 + k], o));
      }
    }
    if (lane < 8) {
      float w = 0.f;
#pragma unroll
      for (int k = 0; k < 6; ++k) w = lane == k ? b[k] : w;
      a.cbox[8 * g + lane] = w;
    }
  }
}

// Run boxes: the box of each run of 64 consecutive groups of a mesh, stored
// at the run's first group, so that the cull can skip 64 groups with one
// test; one wave per run, taken by the run's first group.
__global__ __launch_bounds__(kBlock) void k_run_box(BuildArgs a) {
  if (*a.status != INT_MAX) return;
  const int lane = threadIdx.x & 63;
  const int64_t total = a.groups[a.n_meshes];
  const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
  // a wave looks at 16 groups at a time for those that start a run (meshes of
  // a few groups start one every few groups)
  for (int64_t c0 = ((blockIdx.x * (int64_t)kBlock + threadIdx.x) >> 6) * 16; c0 < total; c0 += nw * 16) {
    int64_t base = 0, end = 0;
    const int64_t c = c0 + lane;
    if (c < total) {
      const int32_t m = a.cmesh[c];
      base = a.groups[m];
      end = a.groups[m + 1];
    }
    for (uint64_t starts = __ballot(lane < 16 && c < total && (c - base) % kChunk == 0); starts; starts &= starts - 1) {
      const int j = __builtin_ctzll(starts);
      const int64_t first = c0 + j, last = __shfl(end, j);
      const int64_t g = first + lane;
      float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
      if (g < last) {
#pragma unroll
        for (int k = 0; k < 6; ++k) b[k] = a.cbox[8 * g + k];
      }
      for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          b[k] = fminf(b[k], __shfl_xor(b[k], o));
          b[3 + k] = fmaxf(b[3 + k], __shfl_xor(b[3 + k], o));
        }
      }
      if (lane < 8) {
        float w = 0.f;
#pragma unroll
        for (int k = 0; k < 6; ++k) w = lane == k ? b[k] : w;
        a.rbox[8 * first + lane] = w;
      }
    }
  }
}

// The header and the status: the smallest bad face, or -1.
__global__ void k_header(BuildArgs a, BlobHeader h, int32_t* dev_status) {
  const int32_t st = *a.status;
  const bool ok = st == INT_MAX;
  h.n_chunks = ok ? a.groups[a.n_meshes] : 0;
  h.n_edges = ok ? *a.etotal : 0;
  h.exp_lo = a.exps[0];
  h.exp_hi = a.exps[1];
  *reinterpret_cast<BlobHeader*>(a.blob) = h;
  *dev_status = ok ? -1 : st;
}

// ---- sizes ------------------------------------------------------------------

struct Layout {
  int64_t node_cap, chunk_cap;
  int64_t off_mesh, off_node, off_tri, off_triid, off_seg, off_edge, off_cbox, off_cmesh, off_rep, off_rbox, total;
};

Layout blob_layout(int64_t M, int64_t F, int W, int L) {
  Layout y;
  y.node_cap = F / (W - 1) + F / (L + 1) + 2 * M + 1;
  y.chunk_cap = (3 * F) / kChunk + M + 1;
  int64_t o = align256(sizeof(BlobHeader));
  y.off_mesh = o; o = align256(o + M * (int64_t)sizeof(MeshDesc));
  y.off_node = o; o = align256(o + y.node_cap * node_bytes(W));
  // three triangles of slack after the last one: a leaf's triangles are
  // read four at a time as one contiguous block
  y.off_tri = o; o = align256(o + (F + 3) * 36);
  y.off_triid = o; o = align256(o + F * 4);
  y.off_seg = o; o = align256(o + y.chunk_cap * 6 * kChunk * 4);
  y.off_edge = o; o = align256(o + y.chunk_cap * 2 * kChunk * 4);
  y.off_cbox = o; o = align256(o + y.chunk_cap * 32);
  y.off_cmesh = o; o = align256(o + y.chunk_cap * 4);
  y.off_rep = o; o = align256(o + M * 16);
  y.off_rbox = o; o = align256(o + y.chunk_cap * 32);
  y.total = o;
  return y;
}

// Counting chunks: meshes of more than kUnitCap half-edges only.
int64_t code_chunks(int64_t F) { return F / (kUnitCap / 3) + 1; }

// Cells of more than kUnitCap triangles or half-edges, at most.
int64_t over_cells(int64_t F) { return F / (kUnitCap + 1) + 3 * F / (kUnitCap + 1); }

// Carves the workspace; with base == nullptr only measures.
void carve_ws(Carve& cv, BuildArgs& a, int64_t M, int64_t F) {
  const int64_t E3 = 3 * F;
  const int64_t tc = F / kTreeChunk + M + 1, tu = F / kUnit + M + 1, eu = E3 / kUnit + M + 1;
  a.cells_t = F / 8 + M;
  a.cells_all = a.cells_t + E3 / 8 + M;
  a.status = cv.take<int32_t>(4);
  a.exps = cv.take<int32_t>(4);
  a.ctr = cv.take<int32_t>(4);
  a.psum = cv.take<uint64_t>(M > kPlanOne ? 4 * kPlanBlocks : 0);
  a.plan = cv.take<MeshPlan>(M + 1);
  a.mm = cv.take<uint32_t>(8 * M);
  a.used = cv.take<int32_t>(M);
  a.depth = cv.take<int32_t>(M);
  a.nedges = cv.take<int32_t>(M);
  a.groups = cv.take<int64_t>(M + 1);
  a.etotal = cv.take<int64_t>(1);
  a.big = cv.take<int32_t>(M);
  a.tmap = cv.take<int32_t>(tc);
  a.tumap = cv.take<int32_t>(tu);
  a.emap = cv.take<int32_t>(eu);
  a.cmap = cv.take<int32_t>(code_chunks(F));
  a.hist = cv.take<uint32_t>(a.cells_all + 1);
  a.start = cv.take<uint32_t>(a.cells_all + 1);
  a.tsum = cv.take<int64_t>(scan_tiles_of(a.cells_all) + 1);
  a.key = cv.take<uint32_t>(F);
  a.rank = cv.take<uint32_t>(F);
  a.tcells = cv.take<uint2>(F);
  a.sk = cv.take<uint32_t>(F);
  a.sv = cv.take<uint32_t>(F);
  a.ekey = cv.take<uint32_t>(E3);
  a.erank = cv.take<uint32_t>(E3);
  a.ecells = cv.take<Item>(E3);
  a.ul = cv.take<uint32_t>(E3);
  a.uh = cv.take<uint32_t>(E3);
  a.over = cv.take<int2>(over_cells(F));
  a.packed = cv.take<int32_t>(tu + eu);
  a.tfirst = cv.take<int32_t>(tu);
  a.tlast = cv.take<int32_t>(tu);
  a.efirst = cv.take<int32_t>(eu);
  a.elast = cv.take<int32_t>(eu);
  a.ustart = cv.take<int32_t>(eu);
  a.ucount = cv.take<int32_t>(eu);
  a.uoff = cv.take<int32_t>(eu);
  a.bin = cv.take<BinNode>(F);
  const int64_t rc = 2 * F / kTreeChunk + 1;  // a mesh of several chunks has less than two per kTreeChunk faces
  a.roots = cv.take<RootRec>(rc * kMaxRoots);
  a.nroots = cv.take<int32_t>(rc);
  a.items = cv.take<int32_t>(3 * F);
  a.subs = cv.take<SubItem>(F / 2 + M + 1);
}

int check_params(int64_t M, int64_t F, int64_t V, const pr_bvh_params* p) {
  if (!p) { set_error("params is NULL"); return PR_E_ARG; }
  if (!(p->width == 2 || p->width == 4 || p->width == 8)) { set_error("width must be 2, 4 or 8"); return PR_E_ARG; }
  if (!(p->leaf_size == 1 || p->leaf_size == 2 || p->leaf_size == 4 || p->leaf_size == 8)) {
    set_error("leaf_size must be 1, 2, 4 or 8");
    return PR_E_ARG;
  }
  if (p->builder < 0 || p->builder > 1) { set_error("builder must be 0 or 1"); return PR_E_ARG; }
  if (p->reserved != 0) { set_error("reserved must be 0"); return PR_E_ARG; }
  if (M < 0 || F < 0 || V < 0) { set_error("negative size"); return PR_E_ARG; }
  if (M == 0 && (F > 0 || V > 0)) { set_error("faces or vertices without meshes"); return PR_E_ARG; }
  if (F >= ((int64_t)1 << 28) || V >= ((int64_t)1 << 31) || M >= ((int64_t)1 << 24)) {
    set_error("sizes beyond index ranges (f_total < 2^28, v_total < 2^31, n_meshes < 2^24)");
    return PR_E_UNSUPPORTED;
  }
  return PR_OK;
}

}  // namespace
}  // namespace pr

using namespace pr;

extern "C" int build_mesh_bvh_sizes(int64_t n_meshes, int64_t f_total, int64_t v_total,
                                    const pr_bvh_params* params, size_t* blob_bytes, size_t* ws_bytes) {
  int r = check_params(n_meshes, f_total, v_total, params);
  if (r) return r;
  if (!blob_bytes || !ws_bytes) { set_error("output pointer is NULL"); return PR_E_ARG; }
  *blob_bytes = (size_t)blob_layout(n_meshes, f_total, params->width, params->leaf_size).total;
  Carve cv{nullptr, 0};
  BuildArgs a{};
  carve_ws(cv, a, n_meshes, f_total);
  *ws_bytes = cv.used + 256;
  return PR_OK;
}

extern "C" size_t build_mesh_bvh_bytes(int64_t n_meshes, int64_t f_total, int64_t v_total,
                                       const pr_bvh_params* params) {
  if (check_params(n_meshes, f_total, v_total, params) != PR_OK) return 0;
  return (size_t)blob_layout(n_meshes, f_total, params->width, params->leaf_size).total;
}

extern "C" int build_mesh_bvh(const float* verts, const int64_t* vert_off, const int32_t* faces,
                              const int64_t* face_off, int64_t n_meshes, int64_t v_total, int64_t f_total,
                              const pr_bvh_params* params, void* blob, size_t blob_bytes, void* ws,
                              size_t ws_bytes, int32_t* dev_status, void* stream) {
  int r = check_params(n_meshes, f_total, v_total, params);
  if (r) return r;
  if (!blob || !ws || !dev_status || !vert_off || !face_off || (f_total > 0 && (!faces || !verts))) {
    set_error("null pointer argument");
    return PR_E_ARG;
  }
  const int W = params->width, L = params->leaf_size;
  Layout y = blob_layout(n_meshes, f_total, W, L);
  if (blob_bytes < (size_t)y.total) { set_error("blob_bytes %zu < required %lld", blob_bytes, (long long)y.total); return PR_E_CAPACITY; }
  hipStream_t s = (hipStream_t)stream;
  BuildArgs a{};
  Carve cv{(char*)ws, ws_bytes};
  carve_ws(cv, a, n_meshes, f_total);
  if (cv.used > ws_bytes) { set_error("ws_bytes %zu < required %zu", ws_bytes, cv.used); return PR_E_CAPACITY; }
  a.verts = verts; a.vert_off = vert_off; a.faces = faces; a.face_off = face_off;
  a.n_meshes = n_meshes; a.v_total = v_total; a.f_total = f_total; a.width = W; a.leaf = L;
  a.builder = params->builder;
  a.blob = (char*)blob;
  a.mesh = reinterpret_cast<MeshDesc*>(a.blob + y.off_mesh);
  a.nodes = a.blob + y.off_node;
  a.tris = reinterpret_cast<float*>(a.blob + y.off_tri);
  a.triid = reinterpret_cast<int32_t*>(a.blob + y.off_triid);
  a.seg = reinterpret_cast<float*>(a.blob + y.off_seg);
  a.edge = reinterpret_cast<int32_t*>(a.blob + y.off_edge);
  a.cbox = reinterpret_cast<float*>(a.blob + y.off_cbox);
  a.cmesh = reinterpret_cast<int32_t*>(a.blob + y.off_cmesh);
  a.rep = reinterpret_cast<float*>(a.blob + y.off_rep);
  a.rbox = reinterpret_cast<float*>(a.blob + y.off_rbox);
  a.node_cap = y.node_cap;
  a.chunk_cap = y.chunk_cap;

  const int64_t F = f_total, M = n_meshes;
  const int64_t tc = F / kTreeChunk + M, tu = F / kUnit + M, eu = 3 * F / kUnit + M;  // bounds of the tables
  const int gM = grid_for(M, kBlock), gMw = grid_for(M, kBlock / 64);
  const int64_t fill = a.cells_all > 8 * M ? a.cells_all : 8 * M;
  const int gI = grid_for(fill, kBlock) < 8192 ? grid_for(fill, kBlock) : 8192;
  // waves of the loops over groups, subtrees and large meshes
  const int kWide = 4096, kTops = 1024;
#define PR_W(kernel, grid, block)                                                                \
  do {                                                                                           \
    if (W == 2) hipLaunchKernelGGL(kernel<2>, dim3(grid), dim3(block), 0, s, a);                 \
    else if (W == 4) hipLaunchKernelGGL(kernel<4>, dim3(grid), dim3(block), 0, s, a);            \
    else hipLaunchKernelGGL(kernel<8>, dim3(grid), dim3(block), 0, s, a);                        \
  } while (0)
  hipLaunchKernelGGL(k_build_init, dim3(gI), dim3(kBlock), 0, s, a);
  int64_t span = M, plans = 1;
  if (M > kPlanOne) {
    span = ((M + kPlanBlocks - 1) / kPlanBlocks + 1023) / 1024 * 1024;
    plans = (M + span - 1) / span;
    hipLaunchKernelGGL(k_plan_sums, dim3((unsigned)plans), dim3(1024), 0, s, a, span);
  }
  hipLaunchKernelGGL(k_plan, dim3((unsigned)plans), dim3(1024), 0, s, a, span);
  if (F > 0) {
    hipLaunchKernelGGL(k_maps, dim3(gMw), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_prep, grid_of(tc), dim3(kBlock), 0, s, a);
  }
  if (M > 0) PR_W(k_desc, gM, kBlock);
  if (F > 0) {
    hipLaunchKernelGGL(k_codes_cells, dim3((unsigned)code_chunks(F)), dim3(1024), 0, s, a);
    PR_HIP(device_exclusive_scan((const uint32_t*)a.hist, a.start, a.cells_all, a.tsum, (int64_t*)nullptr, s));
    hipLaunchKernelGGL(k_to_cells, grid_of(tc), dim3(kBlock), 0, s, a);
    const int64_t splits = over_cells(F) < 512 ? over_cells(F) : 512;
    if (splits > 0) hipLaunchKernelGGL(k_split, dim3((unsigned)splits), dim3(kSplitBlock), 0, s, a);
    if (tu + eu <= kSortOne) {
      hipLaunchKernelGGL(k_sort<2>, grid_of(tu + eu), dim3(kLdsBlock), 0, s, a, (int32_t)tu);
    } else {
      hipLaunchKernelGGL(k_sort<0>, grid_of(tu), dim3(kLdsBlock), 0, s, a, 0);
      hipLaunchKernelGGL(k_sort<1>, grid_of(eu), dim3(kLdsBlock), 0, s, a, 0);
    }
    hipLaunchKernelGGL(k_sort_packed, dim3((unsigned)(tu + eu < 1024 ? tu + eu : 1024)), dim3(kLdsBlock), 0, s, a);
    hipLaunchKernelGGL(k_tree, grid_of(tc), dim3(kTreeBlock), 0, s, a);
    const int tops = (int)(M < kTops ? M : kTops);
    hipLaunchKernelGGL(k_tree_top, dim3(tops), dim3(kTopUnits), 0, s, a);
    PR_W(k_collapse_top, tops, kBlock);
    const int64_t sub = F / 2 + M;
    PR_W(k_collapse_sub, (int)(sub < kWide ? sub : kWide), kPackBlock);
  }
  if (M > 0) {
    hipLaunchKernelGGL(k_edge_mesh, dim3(gMw), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_group_plan, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(k_mesh_final, dim3(gMw), dim3(kBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_group_plan, dim3(1), dim3(1024), 0, s, a);
  }
  if (F > 0) {
    hipLaunchKernelGGL(k_groups, dim3(grid_for(a.chunk_cap, kBlock / 64)), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_run_box, dim3(grid_for(a.chunk_cap, kBlock / 4)), dim3(kBlock), 0, s, a);
  }
#undef PR_W
  BlobHeader h{};
  h.magic = kMagic;
  h.version = PR_ABI_VERSION;
  h.width = W;
  h.leaf_size = L;
  h.n_meshes = M;
  h.f_total = F;
  h.v_total = v_total;
  h.node_cap = y.node_cap;
  h.chunk_cap = y.chunk_cap;
  h.off_mesh = y.off_mesh;
  h.off_node = y.off_node;
  h.off_tri = y.off_tri;
  h.off_triid = y.off_triid;
  h.off_seg = y.off_seg;
  h.off_edge = y.off_edge;
  h.off_cbox = y.off_cbox;
  h.off_cmesh = y.off_cmesh;
  h.off_rep = y.off_rep;
  h.off_rbox = y.off_rbox;
  h.total_bytes = y.total;
  hipLaunchKernelGGL(k_header, dim3(1), dim3(1), 0, s, a, h, dev_status);
  PR_HIP(hipGetLastError());
  return PR_OK;
}
