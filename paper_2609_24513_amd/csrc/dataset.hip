// The paper's own dataset-level design (Sections 3.2 and 3.5), beside the
// per-pair refinement: one BVH over all triangles of the target dataset
// (a blob built from one mesh that holds every triangle), a
// triangle-to-object map, every unique source edge traced against that
// tree with all of its hits collected (the multi-hit loop: a traversal that
// does not stop at the first hit visits every leaf the segment's path
// reaches), and the (source object, target object) records materialised in
// one of the paper's ways:
//  * counting two-pass: a pass counts each source group's records, a scan
//    gives offsets, a second pass writes them, then sort + unique;
//  * single pass into a hashmap that drops duplicates on insert, sized by
//    the selectivity estimate (or a fixed capacity).
// The selectivity estimate (Section 3.5's grid statistics, interaction
// volume, shape factor and cap) runs here too.
//
// Work unit: one group of 64 segments (64 unique edges of one source mesh);
// a wave traces it with a packet traversal in batches of nodes, a stack of
// (node, lane mask) entries in VGPR lanes and LDS.  Leaf tests are the closed
// segment-triangle test, FP32 filter with the exact fallback in place.  A
// lane drops a record equal to its previous one (consecutive hits of one
// target object).
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include "scan.h"

#include <algorithm>
#include <climits>
#include <cmath>

#include "common.h"
#include "predicates.h"
#include "wave.h"

namespace pr {
namespace {

constexpr int kDB = 256;                       // threads per block
constexpr int kDWaves = kDB / 64;
constexpr int kGrab = 8;                       // groups taken per grab, at most
constexpr int kXcd = 8;
constexpr int kCtrWords = 512;                 // u64 words between counters
constexpr uint64_t kEmptyKey = ~0ull;

enum { D_GROUPS = 0, D_VISITS, D_TESTS, D_HITS, D_RECORDS, D_EXACT, D_OVER, D_NEW, D_N };
static_assert(sizeof(pr_dataset_stats) == D_N * 8, "stats layout");

// The headers and sections of the two blobs, through the scalar cache (no
// kernel here writes a blob).
using HeaderPtr = cptr_t<BlobHeader>;
__device__ __forceinline__ HeaderPtr header_of(const char* b) { return cview(reinterpret_cast<const BlobHeader*>(b)); }

__device__ __forceinline__ uint64_t mix64(uint64_t x) {  // splitmix64 finaliser
  x ^= x >> 30;
  x *= 0xbf58476d1ce4e5b9ull;
  x ^= x >> 27;
  x *= 0x94d049bb133111ebull;
  x ^= x >> 31;
  return x;
}

struct TraceArgs {
  const char* src;            // per-mesh blob of the source dataset (its edges)
  const char* dst;            // dataset-level blob of the target dataset (one mesh)
  const int32_t* tri_obj;     // target: object of each leaf-order triangle
  int64_t n_src_objects, n_dst_objects;
  int32_t op, flip;
  uint64_t* counts;           // [groups] op 0 out / op 1 in
  const uint64_t* offsets;    // [groups] op 1
  uint64_t* keys;
  int64_t key_cap;
  int64_t max_groups;         // entries of counts / offsets
  unsigned long long* grab;   // kXcd grab counters, kCtrWords apart
  unsigned long long* stats;  // D_N counters
  int32_t* status;
  uint32_t* xlist;            // [max_groups] groups for the exact pass
  uint32_t* xcount;           // [1]
};

// Leaf triangle test of one lane's segment: 1 hit, 0 miss, -1 when the FP32
// bound cannot decide and EXACT is off (the group is then traced again by the
// exact kernel); with EXACT, the FP64 filter and exact expansions decide.
template <bool EXACT>
__device__ __forceinline__ int dleaf(f3 p, f3 q, f3 a, f3 b, f3 c, bool safe, uint32_t& exact) {
  const int r = safe ? seg_tri_f32(p, q, a, b, c) : kAmbig;
  if (r != kAmbig) return r == kHit ? 1 : 0;
  if (!EXACT) return -1;
  ++exact;
  ExactCounters ec{0};
  return seg_tri_exact(p, q, a, b, c, ec) ? 1 : 0;
}

// Pending nodes from which a step takes one node only, so that the stack stays
// bounded: up to kBatchTop entries a batch adds at most (W - 1) 64 / W, beyond
// it single steps add W - 1 a level.
constexpr int kBatchTop = 32;
template <int W>
constexpr int dstack_cap() { return kBatchTop + (W - 1) * (64 / W) + (W - 1) * kMaxDepth; }
template <int W>
constexpr int dlds_cap() { return dstack_cap<W>() - kRegStack; }

// Traces group g and emits its records for op 0 (count), 1 (write at the
// group's offset) or 2 (hash insert).  Returns false when a test needs the
// exact tier and EXACT is off: the group is then appended to the exact list
// and traced again, whole, by the exact kernel (which rewrites its count,
// rewrites its records at the same offsets, or inserts them again).
//
// Every hit is wanted, so the order of the walk is free, and a step takes up
// to 64 / W pending nodes at once: lane j W + d loads the box and reference of
// child d of the j-th node, all of them are tested against the group's box
// together, and each child that meets it is broadcast and tested by the lanes
// whose segments met its parent.  The next step's loads are issued before the
// step's leaves are tested.  Bound by the chain of dependent loads, now a few
// steps long: one node at a time took 2.5 ms for 50,000 groups of 18 segments
// against 600,000 triangles (W = 8, L = 2).
template <int W, int OP, bool EXACT>
__device__ bool trace_group_ds(const TraceArgs& a, int64_t g, int32_t* s_ref, uint64_t* s_mask,
                               uint32_t (&cnt)[D_N]) {
  const int lane = threadIdx.x & 63;
  const HeaderPtr hs = header_of(a.src), ht = header_of(a.dst);
  const int32_t sm = cview(reinterpret_cast<const int32_t*>(a.src + hs->off_cmesh))[g];
  const cptr_t<MeshDesc> smd = cview(reinterpret_cast<const MeshDesc*>(a.src + hs->off_mesh)) + sm;
  const cptr_t<MeshDesc> tmd = cview(reinterpret_cast<const MeshDesc*>(a.dst + ht->off_mesh));
  const char* const tnodes = a.dst + ht->off_node;
  const float* const ttris = reinterpret_cast<const float*>(a.dst + ht->off_tri);
  const int32_t live = min((int32_t)kChunk, smd->n_edges - (int32_t)(g - smd->chunk_base) * kChunk);
  const bool safe = (smd->flags & tmd->flags & kMeshSafe) != 0;
  const int32_t root = tmd->root;
  const float* sp = reinterpret_cast<const float*>(a.src + hs->off_seg) + g * (6 * kChunk);
  const f3 p{sp[lane], sp[kChunk + lane], sp[2 * kChunk + lane]};
  const f3 q{sp[3 * kChunk + lane], sp[4 * kChunk + lane], sp[5 * kChunk + lane]};
  float cb[6];
  {
    const cptr_t<float> cbp = cview(reinterpret_cast<const float*>(a.src + hs->off_cbox)) + 8 * g;
#pragma unroll
    for (int k = 0; k < 6; ++k) cb[k] = cbp[k];
  }
  Ray r;
  r.px = p.x; r.py = p.y; r.pz = p.z;
  axis_rcp(q.x - p.x, safe, r.ix, r.bx);
  axis_rcp(q.y - p.y, safe, r.iy, r.by);
  axis_rcp(q.z - p.z, safe, r.iz, r.bz);
  cnt[D_GROUPS] += lane == 0 ? 1u : 0u;
  int32_t last = -1;         // per lane: target object of its previous record
  uint32_t mine = 0;         // per lane: records (op 0)
  uint32_t wrote = 0;        // op 1: records of the group written so far (uniform)
  uint64_t obase = 0, oend = 0;
  int32_t seen = -1;         // op 2: lane k < n_seen holds the k-th target object to insert
  int32_t n_seen = 0;
  if (OP == 1) {
    obase = a.offsets[g];
    oend = obase + a.counts[g];
  }
  auto key_of = [&](int32_t tobj) {
    return a.flip ? ((uint64_t)(uint32_t)tobj << 32) | (uint32_t)sm : ((uint64_t)(uint32_t)sm << 32) | (uint32_t)tobj;
  };
  // op 2: open addressing, linear probing; each lane inserts its own key, all
  // of a group in one round of atomics
  auto insert_seen = [&]() {
    if (lane < n_seen) {
      const uint64_t key = key_of(seen), capm = (uint64_t)a.key_cap - 1;
      uint64_t h = mix64(key) & capm;
      bool done = false;
      for (int64_t probe = 0; probe < a.key_cap; ++probe) {
        const uint64_t prev = atomicCAS(reinterpret_cast<unsigned long long*>(a.keys + h), kEmptyKey, key);
        if (prev == kEmptyKey) { ++cnt[D_NEW]; done = true; break; }
        if (prev == key) { done = true; break; }
        h = (h + 1) & capm;
      }
      if (!done) ++cnt[D_OVER];
    }
    n_seen = 0;
  };
  auto record = [&](bool hit, int32_t tobj) {
    const bool emit = hit && tobj != last;
    if (hit) last = tobj;
    if (OP == 0) {
      mine += emit ? 1u : 0u;
      return;
    }
    const uint64_t em = ballot(emit);
    if (!em) return;
    if (OP == 1) {
      const uint64_t pos = obase + wrote + (uint64_t)lanes_below(em);
      if (emit) {
        if (pos < oend && pos < (uint64_t)a.key_cap) a.keys[pos] = key_of(tobj);
        else ++cnt[D_OVER];
      }
      wrote = (uint32_t)uni((int32_t)wrote + __popcll(em));
      return;
    }
    // OP == 2: the records of a triangle all have one key (a group is of one
    // mesh), kept once in `seen` and inserted together
    cnt[D_RECORDS] += emit ? 1u : 0u;
    if (ballot(lane < n_seen && seen == tobj)) return;
    if (n_seen == 64) insert_seen();
    seen = lane_write(tobj, n_seen, seen);
    n_seen = uni(n_seen + 1);
  };
  const uint64_t m0 = ballot(lane < live);
  if (m0 && root != kEmpty && meet6(cb, tmd->box[0], tmd->box[1], tmd->box[2], tmd->box[3], tmd->box[4], tmd->box[5])) {
    WaveStack stk;
    stk.ref = 0; stk.mlo = 0; stk.mhi = 0;
    stk.lref = s_ref; stk.lmask = s_mask; stk.top = 0;
    const int grp = lane / W, d = lane % W;
    float bx[6];
    int32_t cref;
    auto load_children = [&](int32_t nref) {
      const float* nd = reinterpret_cast<const float*>(tnodes + sizeof(Node<W>) * (int64_t)nref);
#pragma unroll
      for (int k = 0; k < 6; ++k) bx[k] = nd[k * W + d];
      cref = reinterpret_cast<const int32_t*>(nd)[6 * W + d];
    };
    int32_t nb = 1;  // nodes of the batch
    int32_t pmlo = (int32_t)(uint32_t)m0, pmhi = (int32_t)(uint32_t)(m0 >> 32);  // lane mask of each lane's parent
    load_children(root);
    while (true) {
      nb = uni(nb);
      cnt[D_VISITS] += lane == 0 ? (uint32_t)nb : 0u;
      const uint64_t in = nb * W >= 64 ? ~0ull : (1ull << (nb * W)) - 1ull;
      uint64_t f = ballot(cref != kEmpty && meet6(cb, bx[0], bx[1], bx[2], bx[3], bx[4], bx[5])) & in;
      int32_t lref = 0, lmlo = 0, lmhi = 0;  // leaves hit: entry i in lane i
      int32_t nl = 0;
      while (f) {
        nl = uni(nl);
        stk.top = uni(stk.top);
        const int c = __builtin_ctzll(f);
        f = uni64(f & (f - 1));
        const uint64_t nm = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(pmhi, c) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane(pmlo, c);
        const float lx = lane_f(bx[0], c), ly = lane_f(bx[1], c), lz = lane_f(bx[2], c);
        const float hx = lane_f(bx[3], c), hy = lane_f(bx[4], c), hz = lane_f(bx[5], c);
        bool hit = slab(r, lx, ly, lz, hx, hy, hz);
        if (!safe)
          hit = hit && fminf(p.x, q.x) <= hx && fmaxf(p.x, q.x) >= lx && fminf(p.y, q.y) <= hy &&
                fmaxf(p.y, q.y) >= ly && fminf(p.z, q.z) <= hz && fmaxf(p.z, q.z) >= lz;
        const uint64_t m = ballot(hit) & nm;
        if (!m) continue;
        const int32_t ref = __builtin_amdgcn_readlane(cref, c);
        if (ref < 0) {
          lref = lane_write(ref, nl, lref);
          lmlo = lane_write((int32_t)(uint32_t)m, nl, lmlo);
          lmhi = lane_write((int32_t)(uint32_t)(m >> 32), nl, lmhi);
          ++nl;
        } else {
          push_node(stk, ref, m);
        }
      }
      nl = uni(nl);
      stk.top = uni(stk.top);
      if (stk.top > dstack_cap<W>() - W) {  // not for a valid blob (depth <= kMaxDepth)
        if (lane == 0) atomicMin(a.status, (int32_t)PR_E_UNSUPPORTED);
        return true;
      }
      // the first leaves' loads, then the next batch's
      auto load_leaf = [&](int i) {
        const int32_t lr = ~__builtin_amdgcn_readlane(lref, i);
        return ttris[9 * (int64_t)(lr >> 3) + min(lane, 9 * ((lr & 7) + 1) - 1)];
      };
      auto load_objs = [&](int i) {
        const int32_t lr = ~__builtin_amdgcn_readlane(lref, i);
        return a.tri_obj[(lr >> 3) + min(lane, lr & 7)];
      };
      float t0 = 0.f, t1 = 0.f;
      int32_t o0 = 0, o1 = 0;
      if (nl > 0) { t0 = load_leaf(0); o0 = load_objs(0); }
      if (nl > 1) { t1 = load_leaf(1); o1 = load_objs(1); }
      nb = uni(stk.top > kBatchTop ? 1 : min(stk.top, 64 / W));
      if (nb > 0) {
        int32_t nref;
        if (stk.top > kRegStack) {  // one entry, from LDS
          nref = uni(stk.lref[stk.top - 1 - kRegStack]);
          const uint64_t m = uni64(stk.lmask[stk.top - 1 - kRegStack]);
          pmlo = (int32_t)(uint32_t)m;
          pmhi = (int32_t)(uint32_t)(m >> 32);
        } else {
          const int src = stk.top - 1 - min(grp, nb - 1);
          nref = __shfl(stk.ref, src);
          pmlo = __shfl(stk.mlo, src);
          pmhi = __shfl(stk.mhi, src);
        }
        stk.top = uni(stk.top - nb);
        load_children(nref);
      }
#pragma unroll 1
      for (int i = 0; i < nl; i = uni(i + 1)) {
        const float tv = t0;
        const int32_t to = o0;
        t0 = t1;
        o0 = o1;
        if (i + 2 < nl) { t1 = load_leaf(i + 2); o1 = load_objs(i + 2); }
        const int32_t lr = ~__builtin_amdgcn_readlane(lref, i);
        const uint64_t nm = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(lmhi, i) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane(lmlo, i);
        const int32_t first = lr >> 3;
        const int n = (lr & 7) + 1;
        const bool on = (nm >> lane) & 1ull;
#pragma unroll 1
        for (int t = 0; t < n; t = uni(t + 1)) {
          // triangle t's nine coordinates sit in lanes 9 t ... 9 t + 8 (the
          // eighth triangle's do not fit and are loaded for it)
          float v = tv;
          int at = 9 * t;
          if (t == 7) {
            v = ttris[9 * (int64_t)(first + 7) + min(lane, 8)];
            at = 0;
          }
          const f3 ta{lane_f(v, at), lane_f(v, at + 1), lane_f(v, at + 2)};
          const f3 tb{lane_f(v, at + 3), lane_f(v, at + 4), lane_f(v, at + 5)};
          const f3 tc{lane_f(v, at + 6), lane_f(v, at + 7), lane_f(v, at + 8)};
          uint32_t ex = 0;
          const int res = on ? dleaf<EXACT>(p, q, ta, tb, tc, safe, ex) : 0;
          if (!EXACT && ballot(res < 0)) return false;
          const bool hit = res > 0;
          cnt[D_EXACT] += ex;
          cnt[D_TESTS] += on ? 1u : 0u;
          cnt[D_HITS] += hit ? 1u : 0u;
          if (ballot(hit)) record(hit, __builtin_amdgcn_readlane(to, t));
        }
      }
      if (nb == 0) break;
    }
  }
  if (OP == 0) {
    const uint32_t n = wave_sum(mine);
    if (lane == 0) a.counts[g] = n;
    cnt[D_RECORDS] += lane == 0 ? n : 0u;
  } else if (OP == 1) {
    cnt[D_RECORDS] += lane == 0 ? wrote : 0u;
  } else {
    insert_seen();
  }
  return true;
}

__device__ __forceinline__ void flush_counts(const TraceArgs& a, const uint32_t (&cnt)[D_N]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < D_N; ++k) {
    uint32_t s = cnt[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0 && s) atomicAdd(a.stats + k, (unsigned long long)s);
  }
}

__device__ __forceinline__ bool dblobs_ok(const TraceArgs& a, int W) {
  const HeaderPtr hs = header_of(a.src), ht = header_of(a.dst);
  return hs->magic == kMagic && ht->magic == kMagic && ht->n_meshes == 1 && ht->width == W &&
         a.n_src_objects <= hs->n_meshes && hs->n_chunks <= a.max_groups;
}

// Persistent waves over the source groups: one contiguous share per XCD
// (blocks are dealt to the XCDs round-robin), taken up to kGrab groups at a
// time, fewer where a wave has only a few to trace.
template <int W, int OP>
__global__ __launch_bounds__(kDB, 5) void k_dtrace(TraceArgs a) {
  __shared__ int32_t s_ref[kDWaves][dlds_cap<W>()];
  __shared__ uint64_t s_mask[kDWaves][dlds_cap<W>()];
  const int wv = uni((int32_t)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  uint32_t cnt[D_N] = {};
  if (!dblobs_ok(a, W)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicMin(a.status, (int32_t)PR_E_UNSUPPORTED);
    return;
  }
  const int64_t G = header_of(a.src)->n_chunks;
  const int xs = (int)(blockIdx.x % kXcd);
  const int64_t lo = G * xs / kXcd, hi = G * (xs + 1) / kXcd;
  const int64_t per_wave = G / ((int64_t)gridDim.x * kDWaves * 4);
  const int grab = (int)(per_wave < 1 ? 1 : (per_wave < kGrab ? per_wave : kGrab));
  unsigned long long* ctr = a.grab + kCtrWords * xs;
  while (true) {
    unsigned long long b = 0;
    if (lane == 0) b = atomicAdd(ctr, (unsigned long long)grab);
    const int64_t g0 = lo + (int64_t)uni64(b);
    if (g0 >= hi) break;
    const int64_t g1 = g0 + grab < hi ? g0 + grab : hi;
    for (int64_t g = g0; g < g1; g = (int64_t)uni64((uint64_t)(g + 1)))
      if (!trace_group_ds<W, OP, false>(a, g, s_ref[wv], s_mask[wv], cnt)) {
        if (lane == 0) a.xlist[atomicAdd(a.xcount, 1u)] = (uint32_t)g;  // at most one entry per group
      }
  }
  flush_counts(a, cnt);
}

// The groups that met a test the FP32 bound could not decide, traced again
// with the exact tier (one wave per group).
template <int W, int OP>
__global__ __launch_bounds__(kDB) void k_dtrace_exact(TraceArgs a) {
  __shared__ int32_t s_ref[kDWaves][dlds_cap<W>()];
  __shared__ uint64_t s_mask[kDWaves][dlds_cap<W>()];
  const int wv = uni((int32_t)(threadIdx.x >> 6));
  uint32_t cnt[D_N] = {};
  if (!dblobs_ok(a, W)) return;
  const uint32_t n = *a.xcount;
  for (uint32_t k = blockIdx.x * kDWaves + wv; k < n; k += gridDim.x * kDWaves)
    trace_group_ds<W, OP, true>(a, (int64_t)(uint32_t)uni((int32_t)a.xlist[k]), s_ref[wv], s_mask[wv], cnt);
  flush_counts(a, cnt);
}

__global__ void k_dclear(uint64_t* keys, int64_t n, uint64_t* counts, int64_t n_counts, unsigned long long* grab,
                         unsigned long long* stats, int32_t* status, uint64_t* dev_n, int zero_n,
                         uint32_t* xcount = nullptr) {
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t i = i0; i < n; i += (int64_t)gridDim.x * blockDim.x) keys[i] = kEmptyKey;
  for (int64_t i = i0; i < n_counts; i += (int64_t)gridDim.x * blockDim.x) counts[i] = 0ull;
  if (grab && i0 < kXcd) grab[kCtrWords * i0] = 0ull;
  if (stats && i0 < D_N) stats[i0] = 0ull;
  if (i0 == 0) {
    *status = PR_OK;
    if (zero_n && dev_n) *dev_n = 0ull;
    if (xcount) *xcount = 0u;
  }
}

__global__ void k_dreport(const unsigned long long* stats, const int32_t* status, const uint64_t* offsets,
                          int64_t groups, pr_dataset_stats* out, int32_t* dev_status, uint64_t* dev_n, int op) {
  const int t = threadIdx.x;
  if (t < D_N && out) reinterpret_cast<uint64_t*>(out)[t] = stats[t];
  if (t == 0) {
    if (dev_status) *dev_status = *status;
    if (dev_n) {
      if (op == 0) *dev_n = offsets[groups];
      else if (op == 2) *dev_n = stats[D_NEW];
    }
  }
}

// ---- triangle -> object --------------------------------------------------

__global__ void k_tri_obj(const char* blob, const int64_t* face_off, int64_t n_obj, int32_t* tri_obj,
                          int64_t f_cap, int32_t* status) {
  const BlobHeader* h = reinterpret_cast<const BlobHeader*>(blob);
  const int32_t* triid = reinterpret_cast<const int32_t*>(blob + h->off_triid);
  if (h->magic != kMagic || h->n_meshes != 1 || h->f_total != f_cap) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicMin(status, (int32_t)PR_E_UNSUPPORTED);
    return;
  }
  const int64_t F = f_cap;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < F; k += (int64_t)gridDim.x * blockDim.x) {
    const int64_t f = triid[k];
    // last object o with face_off[o] <= f
    int64_t lo = 0, hi = n_obj;  // face_off[lo] <= f < face_off[hi]
    if (f < face_off[0] || f >= face_off[n_obj]) {
      atomicMin(status, (int32_t)PR_E_ARG);
      tri_obj[k] = -1;
      continue;
    }
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (face_off[mid] <= f) lo = mid; else hi = mid;
    }
    tri_obj[k] = (int32_t)lo;
  }
}

// ---- selectivity estimate ------------------------------------------------

constexpr double kEstEps = 1e-3;
constexpr double kEstGamma = 0.8;

struct EstArgs {
  const char* blob[2];
  int64_t n[2];
  int32_t cells;
  double* side[2];    // [n] mean box side
  double* ratio[2];   // [n] volume ratio
  double* ext;        // [6] union box lo xyz, hi xyz (as ordered ints for the reduction)
  double* grid;       // [2][3][cells^3]: count, sum of sides, sum of ratios
  double* out;
};

__device__ __forceinline__ void amin_d(double* p, double v) {
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  unsigned long long old = *q;
  while (__longlong_as_double((long long)old) > v) {
    const unsigned long long prev = atomicCAS(q, old, (unsigned long long)__double_as_longlong(v));
    if (prev == old) break;
    old = prev;
  }
}
__device__ __forceinline__ void amax_d(double* p, double v) {
  unsigned long long* q = reinterpret_cast<unsigned long long*>(p);
  unsigned long long old = *q;
  while (__longlong_as_double((long long)old) < v) {
    const unsigned long long prev = atomicCAS(q, old, (unsigned long long)__double_as_longlong(v));
    if (prev == old) break;
    old = prev;
  }
}

__global__ void k_est_init(EstArgs e, int64_t grid_words) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < grid_words;
       i += (int64_t)gridDim.x * blockDim.x)
    e.grid[i] = 0.0;
  if (blockIdx.x == 0 && threadIdx.x < 6) e.ext[threadIdx.x] = threadIdx.x < 3 ? INFINITY : -INFINITY;
  if (blockIdx.x == 0 && threadIdx.x == 0) *e.out = 0.0;
}

// Volume of a mesh by the divergence theorem over its triangles (FP64), mean
// box side and volume ratio; the union box.  One wave per mesh where the mean
// mesh has at most kEstWave triangles (a block's other waves and its barriers
// were most of 0.18 ms for 50,000 meshes of 12), else one block.  Among small
// meshes the waves leave those of more than kEstBig triangles to their whole
// block, up to kEstList of them (beside 50,000 cubes one mesh of 2 M triangles
// takes a wave 19.4 ms, a block 5.1).  The union
// box is kept in registers and joined once a block.  (The host checks nothing
// on the device blobs: a count above the blob's is cut to it.)
constexpr int kEstWave = 512;
constexpr int kEstBig = 4096;
constexpr int kEstList = 16;

__global__ __launch_bounds__(kDB) void k_est_objects(EstArgs e, int d) {
  __shared__ double s_red[kDWaves], s_ext[6][kDWaves];
  __shared__ int64_t s_big[kEstList];
  __shared__ int s_nbig;
  const BlobHeader* h = reinterpret_cast<const BlobHeader*>(e.blob[d]);
  if (h->magic != kMagic) return;
  const int64_t nm = e.n[d] < h->n_meshes ? e.n[d] : h->n_meshes;
  const MeshDesc* md = reinterpret_cast<const MeshDesc*>(e.blob[d] + h->off_mesh);
  const float* tris = reinterpret_cast<const float*>(e.blob[d] + h->off_tri);
  const bool by_wave = h->f_total <= kEstWave * h->n_meshes;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_nbig = 0;
  __syncthreads();
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  // one mesh by a wave, or (every thread of the block calls it) by the block
  auto object = [&](int64_t m, const MeshDesc& D, bool wave) {
    const int t0 = wave ? lane : (int)threadIdx.x, step = wave ? 64 : kDB;
    double acc = 0.0;
    for (int32_t t = t0; t < D.n_tris; t += step) {
      const float* p = tris + 9 * ((int64_t)D.tri_base + t);
      const double ax = p[0], ay = p[1], az = p[2], bx = p[3], by = p[4], bz = p[5];
      const double cx = p[6], cy = p[7], cz = p[8];
      acc += ax * (by * cz - bz * cy) + ay * (bz * cx - bx * cz) + az * (bx * cy - by * cx);
    }
    acc = wave_sum(acc);
    if (!wave) {
      if (lane == 0) s_red[w] = acc;
      __syncthreads();
      acc = 0.0;
      for (int k = 0; k < kDWaves; ++k) acc += s_red[k];
      __syncthreads();
    }
    if (t0 == 0) {
      const double v = fabs(acc / 6.0);
      if (D.n_tris > 0) {
        const double ex = (double)D.box[3] - D.box[0], ey = (double)D.box[4] - D.box[1],
                     ez = (double)D.box[5] - D.box[2];
        e.side[d][m] = (ex + ey + ez) / 3.0;
        const double bv = ex * ey * ez;
        e.ratio[d][m] = bv > 0.0 ? fmin(fmax(v / bv, 0.0), 1.0) : 1.0;
      } else {
        e.side[d][m] = 0.0;
        e.ratio[d][m] = 0.0;
      }
    }
    if (D.n_tris > 0) {
      for (int k = 0; k < 3; ++k) {
        lo[k] = fmin(lo[k], (double)D.box[k]);
        hi[k] = fmax(hi[k], (double)D.box[3 + k]);
      }
    }
  };
  if (by_wave) {
    for (int64_t m = (int64_t)blockIdx.x * kDWaves + w; m < nm; m += (int64_t)gridDim.x * kDWaves) {
      const MeshDesc D = md[m];
      int at = kEstList;
      if (D.n_tris > kEstBig) {
        if (lane == 0) at = atomicAdd(&s_nbig, 1);
        at = __shfl(at, 0);
      }
      if (at < kEstList) {
        if (lane == 0) s_big[at] = m;
      } else {
        object(m, D, true);
      }
    }
    __syncthreads();
    for (int k = 0; k < min(s_nbig, kEstList); ++k) object(s_big[k], md[s_big[k]], false);
  } else {
    for (int64_t m = blockIdx.x; m < nm; m += gridDim.x) object(m, md[m], false);
  }
  if (lane == 0)
    for (int k = 0; k < 3; ++k) { s_ext[k][w] = lo[k]; s_ext[3 + k][w] = hi[k]; }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int k = threadIdx.x;
    double v = s_ext[k][0];
    for (int q = 1; q < kDWaves; ++q) v = k < 3 ? fmin(v, s_ext[k][q]) : fmax(v, s_ext[k][q]);
    if (k < 3) amin_d(e.ext + k, v);
    else amax_d(e.ext + k, v);
  }
}

__device__ __forceinline__ void grid_frame(const EstArgs& e, double* lo, double* size) {
  for (int k = 0; k < 3; ++k) {
    lo[k] = e.ext[k];
    const double hi = e.ext[3 + k];
    size[k] = hi > lo[k] ? (hi - lo[k]) / e.cells : 1.0;
  }
}

// One thread per object: adds it to every cell its closed box touches.
__global__ void k_est_cells(EstArgs e, int d) {
  const BlobHeader* h = reinterpret_cast<const BlobHeader*>(e.blob[d]);
  if (h->magic != kMagic) return;
  const int64_t nm = e.n[d] < h->n_meshes ? e.n[d] : h->n_meshes;
  const MeshDesc* md = reinterpret_cast<const MeshDesc*>(e.blob[d] + h->off_mesh);
  double lo[3], size[3];
  grid_frame(e, lo, size);
  const int G = e.cells;
  const int64_t C = (int64_t)G * G * G;
  double* cnt = e.grid + (int64_t)d * 3 * C;
  double* sid = cnt + C;
  double* rat = sid + C;
  for (int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; m < nm; m += (int64_t)gridDim.x * blockDim.x) {
    const MeshDesc D = md[m];
    if (D.n_tris <= 0) continue;
    int c0[3], c1[3];
    for (int k = 0; k < 3; ++k) {
      double a = ceil(((double)D.box[k] - lo[k]) / size[k] - 1.0);
      double b = floor(((double)D.box[3 + k] - lo[k]) / size[k]);
      a = fmin(fmax(a, 0.0), (double)(G - 1));
      b = fmin(fmax(b, 0.0), (double)(G - 1));
      c0[k] = (int)a;
      c1[k] = (int)b;
    }
    const double s = e.side[d][m], r = e.ratio[d][m];
    for (int x = c0[0]; x <= c1[0]; ++x)
      for (int y = c0[1]; y <= c1[1]; ++y)
        for (int z = c0[2]; z <= c1[2]; ++z) {
          const int64_t c = ((int64_t)x * G + y) * G + z;
          atomicAdd(cnt + c, 1.0);
          atomicAdd(sid + c, s);
          atomicAdd(rat + c, r);
        }
  }
}

__global__ void k_est_sum(EstArgs e) {
  __shared__ double s_red[kDB / 64];
  double lo[3], size[3];
  grid_frame(e, lo, size);
  const double vcell = size[0] * size[1] * size[2];
  const int64_t C = (int64_t)e.cells * e.cells * e.cells;
  const double* n1 = e.grid;
  const double* s1 = n1 + C;
  const double* r1 = s1 + C;
  const double* n2 = e.grid + 3 * C;
  const double* s2 = n2 + C;
  const double* r2 = s2 + C;
  double acc = 0.0;
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < C; c += (int64_t)gridDim.x * blockDim.x) {
    if (n1[c] > 0.0 && n2[c] > 0.0) {
      const double S1 = s1[c] / n1[c], S2 = s2[c] / n2[c];
      const double R1 = r1[c] / n1[c], R2 = r2[c] / n2[c];
      const double w = S1 + S2 + kEstEps;
      const double pb = w * w * w / vcell;
      const double fs = pow(sqrt(R1 * R2), kEstGamma);
      acc += n1[c] * n2[c] * fmin(pb * fs, 1.0);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double v = 0.0;
    for (int k = 0; k < kDB / 64; ++k) v += s_red[k];
    atomicAdd(e.out, v);
  }
}

// ---- sort + unique ---------------------------------------------------------

__global__ void k_unique_flags(const uint64_t* keys, int64_t n, uint32_t* flags) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    flags[i] = (keys[i] != kEmptyKey && (i == 0 || keys[i] != keys[i - 1])) ? 1u : 0u;
}

__global__ void k_unique_write(const uint64_t* keys, int64_t n, const uint32_t* flags, const uint64_t* pos,
                               int32_t* out, int64_t cap, int64_t* count) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    if (flags[i] && (int64_t)pos[i] < cap) {
      out[2 * pos[i]] = (int32_t)(keys[i] >> 32);
      out[2 * pos[i] + 1] = (int32_t)(uint32_t)keys[i];
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *count = n > 0 ? (int64_t)(pos[n - 1] + flags[n - 1]) : 0;
}

template <typename T>
T* take(char*& p, size_t& left, int64_t n) {
  const size_t need = (size_t)align256((int64_t)(sizeof(T) * (size_t)(n > 0 ? n : 1)));
  if (need > left) return nullptr;
  T* r = reinterpret_cast<T*>(p);
  p += need;
  left -= need;
  return r;
}

int unique_ws(int64_t n, size_t* bytes) {
  size_t sort_tmp = 0;
  const hipError_t e =
      hipcub::DeviceRadixSort::SortKeys(nullptr, sort_tmp, (const uint64_t*)nullptr, (uint64_t*)nullptr, (int)n, 0, 64);
  if (e != hipSuccess) return hip_fail(e, "hipcub SortKeys size");
  const size_t scan_tmp = (size_t)(8 * (scan_tiles_of(n) + 1));
  *bytes = (size_t)align256(8 * n) + (size_t)align256(4 * n) + (size_t)align256(8 * n) +
           (size_t)align256((int64_t)std::max(sort_tmp, scan_tmp)) + 1024;
  return PR_OK;
}

size_t trace_ws(int64_t groups) {
  const size_t scan_tmp = (size_t)(8 * (scan_tiles_of(groups + 1) + 1));
  return (size_t)align256(8 * (groups + 1)) + (size_t)align256(8 * kXcd * kCtrWords) + (size_t)align256(8 * D_N) +
         256 + 256 + (size_t)align256(4 * (groups > 0 ? groups : 1)) + (size_t)align256((int64_t)scan_tmp) + 1024;
}

size_t est_ws(int64_t na, int64_t nb, int32_t cells) {
  const int64_t C = (int64_t)cells * cells * cells;
  return (size_t)align256(16 * (na > 0 ? na : 1)) + (size_t)align256(16 * (nb > 0 ? nb : 1)) + 256 +
         (size_t)align256(8 * 6 * C) + 1024;
}

}  // namespace
}  // namespace pr

using namespace pr;

extern "C" int dataset_tri_objects(const void* dblob, const int64_t* face_off, int64_t n_objects, int32_t* tri_obj,
                                   int64_t f_total, int32_t* dev_status, void* stream) {
  if (!dblob || !face_off || !tri_obj || !dev_status || n_objects <= 0 || f_total < 0) {
    set_error("null pointer or bad size");
    return PR_E_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_dclear, dim3(1), dim3(64), 0, s, (uint64_t*)nullptr, (int64_t)0, (uint64_t*)nullptr,
                     (int64_t)0, (unsigned long long*)nullptr, (unsigned long long*)nullptr, dev_status,
                     (uint64_t*)nullptr, 0);
  hipLaunchKernelGGL(k_tri_obj, dim3(grid_for(f_total, 256)), dim3(256), 0, s, (const char*)dblob, face_off,
                     n_objects, tri_obj, f_total, dev_status);
  PR_HIP(hipGetLastError());
  return PR_OK;
}

extern "C" int dataset_trace_ws_bytes(int64_t max_groups, size_t* ws_bytes) {
  if (max_groups < 0 || !ws_bytes) { set_error("bad argument"); return PR_E_ARG; }
  if (max_groups >= INT_MAX) { set_error("too many groups"); return PR_E_UNSUPPORTED; }
  *ws_bytes = trace_ws(max_groups);
  return PR_OK;
}

extern "C" int dataset_trace(const void* src_blob, int64_t n_src_objects, const void* dst_blob,
                             const int32_t* tri_obj, int64_t n_dst_objects, const pr_dataset_params* params,
                             uint64_t* counts, int64_t max_groups, uint64_t* keys, uint64_t* dev_n,
                             pr_dataset_stats* dev_stats, int32_t* dev_status, void* ws, size_t ws_bytes,
                             void* stream) {
  if (!src_blob || !dst_blob || !params || !dev_status || !ws || n_src_objects < 0 || n_dst_objects < 0 ||
      max_groups < 0) {
    set_error("null pointer or negative size");
    return PR_E_ARG;
  }
  const int op = params->op;
  if (op < 0 || op > 3 || (params->flip != 0 && params->flip != 1) || params->width < 2 || params->width > 8 ||
      (params->width & (params->width - 1))) {
    set_error("bad params (op %d, flip %d, width %d)", op, params->flip, params->width);
    return PR_E_ARG;
  }
  if ((op == 0 || op == 1) && !counts) { set_error("counts is NULL"); return PR_E_ARG; }
  if (op != 0 && (!keys || params->key_cap <= 0)) { set_error("keys / key_cap"); return PR_E_ARG; }
  if (op == 2 && (params->key_cap & (params->key_cap - 1))) { set_error("key_cap must be a power of two"); return PR_E_ARG; }
  if (op != 3 && !tri_obj) { set_error("tri_obj is NULL"); return PR_E_ARG; }
  if (max_groups >= INT_MAX) { set_error("too many groups"); return PR_E_UNSUPPORTED; }
  if (ws_bytes < trace_ws(max_groups)) { set_error("ws_bytes %zu < required %zu", ws_bytes, trace_ws(max_groups)); return PR_E_CAPACITY; }
  hipStream_t s = (hipStream_t)stream;
  char* p = (char*)ws;
  size_t left = ws_bytes;
  uint64_t* offsets = take<uint64_t>(p, left, max_groups + 1);
  unsigned long long* grab = take<unsigned long long>(p, left, kXcd * kCtrWords);
  unsigned long long* stats = take<unsigned long long>(p, left, D_N);
  int32_t* status = take<int32_t>(p, left, 64);
  uint32_t* xcount = take<uint32_t>(p, left, 64);
  uint32_t* xlist = take<uint32_t>(p, left, max_groups);
  void* scan_tmp = p;
  TraceArgs a{};
  a.src = (const char*)src_blob;
  a.dst = (const char*)dst_blob;
  a.tri_obj = tri_obj;
  a.n_src_objects = n_src_objects;
  a.n_dst_objects = n_dst_objects;
  a.op = op;
  a.flip = params->flip;
  a.counts = counts;
  a.offsets = offsets;
  a.keys = keys;
  a.key_cap = params->key_cap;
  a.max_groups = max_groups;
  a.grab = grab;
  a.stats = stats;
  a.status = status;
  a.xlist = xlist;
  a.xcount = xcount;
  // op 3 clears the table (and the key count), op 0 the per-group counts
  // (every one of max_groups + 1 entries: the scan reads them all); every op
  // clears the grab counters, statistics and status
  const int64_t nclear = op == 3 ? params->key_cap : 0;
  const int64_t ncounts = op == 0 ? max_groups + 1 : 0;
  const int64_t nmax = std::max<int64_t>(std::max<int64_t>(nclear, ncounts), 64);
  hipLaunchKernelGGL(k_dclear, dim3(grid_for(nmax, 256)), dim3(256), 0, s, keys, nclear, counts, ncounts, grab,
                     stats, status, dev_n, op == 3 ? 1 : 0, xcount);
  if (op == 3) {
    hipLaunchKernelGGL(k_dreport, dim3(1), dim3(64), 0, s, (const unsigned long long*)stats, (const int32_t*)status,
                       (const uint64_t*)offsets, (int64_t)0, dev_stats, dev_status, (uint64_t*)nullptr, op);
    PR_HIP(hipGetLastError());
    return PR_OK;
  }
  if (op == 1) {
    PR_HIP(device_exclusive_scan((const uint64_t*)counts, offsets, max_groups, (int64_t*)scan_tmp, (int64_t*)nullptr, s));
  }
  int dev = 0;
  PR_HIP(hipGetDevice(&dev));
  int cus = 0;
  PR_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int blocks = cus * 5;  // five waves a SIMD (the traces' registers)
  const int W = params->width;
#define PR_DT(w, o)                                                                     \
  if (W == w && op == o) {                                                              \
    hipLaunchKernelGGL((k_dtrace<w, o>), dim3(blocks), dim3(kDB), 0, s, a);             \
    hipLaunchKernelGGL((k_dtrace_exact<w, o>), dim3(256), dim3(kDB), 0, s, a);          \
  }
  PR_DT(2, 0); PR_DT(2, 1); PR_DT(2, 2);
  PR_DT(4, 0); PR_DT(4, 1); PR_DT(4, 2);
  PR_DT(8, 0); PR_DT(8, 1); PR_DT(8, 2);
#undef PR_DT
  if (op == 0) {
    // offsets of every group and, at [max_groups], the total
    PR_HIP(device_exclusive_scan((const uint64_t*)counts, offsets, max_groups + 1, (int64_t*)scan_tmp, (int64_t*)nullptr, s));
  }
  hipLaunchKernelGGL(k_dreport, dim3(1), dim3(64), 0, s, (const unsigned long long*)stats, (const int32_t*)status,
                     (const uint64_t*)offsets, max_groups, dev_stats, dev_status, dev_n, op);
  PR_HIP(hipGetLastError());
  return PR_OK;
}

extern "C" int pairs_unique_ws_bytes(int64_t n_keys, size_t* ws_bytes) {
  if (n_keys < 0 || !ws_bytes) { set_error("bad argument"); return PR_E_ARG; }
  if (n_keys >= INT_MAX) { set_error("n_keys %lld beyond 2^31", (long long)n_keys); return PR_E_UNSUPPORTED; }
  return unique_ws(n_keys, ws_bytes);
}

extern "C" int pairs_unique(const uint64_t* keys, int64_t n_keys, int32_t* out_pairs, int64_t out_cap,
                            int64_t* dev_count, void* ws, size_t ws_bytes, void* stream) {
  if (n_keys < 0 || out_cap < 0 || !dev_count || !ws || (n_keys > 0 && !keys) || (out_cap > 0 && !out_pairs)) {
    set_error("null pointer or negative size");
    return PR_E_ARG;
  }
  if (n_keys >= INT_MAX) { set_error("n_keys beyond 2^31"); return PR_E_UNSUPPORTED; }
  size_t need = 0;
  const int r = unique_ws(n_keys, &need);
  if (r != PR_OK) return r;
  if (ws_bytes < need) { set_error("ws_bytes %zu < required %zu", ws_bytes, need); return PR_E_CAPACITY; }
  hipStream_t s = (hipStream_t)stream;
  char* p = (char*)ws;
  size_t left = ws_bytes;
  uint64_t* sorted = take<uint64_t>(p, left, n_keys);
  uint32_t* flags = take<uint32_t>(p, left, n_keys);
  uint64_t* pos = take<uint64_t>(p, left, n_keys);
  void* tmp = p;
  size_t tmp_bytes = left;
  if (n_keys == 0) {
    hipLaunchKernelGGL(k_unique_write, dim3(1), dim3(64), 0, s, (const uint64_t*)sorted, (int64_t)0,
                       (const uint32_t*)flags, (const uint64_t*)pos, out_pairs, out_cap, dev_count);
    PR_HIP(hipGetLastError());
    return PR_OK;
  }
  PR_HIP(hipcub::DeviceRadixSort::SortKeys(tmp, tmp_bytes, keys, sorted, (int)n_keys, 0, 64, s));
  hipLaunchKernelGGL(k_unique_flags, dim3(grid_for(n_keys, 256)), dim3(256), 0, s, (const uint64_t*)sorted, n_keys,
                     flags);
  PR_HIP(device_exclusive_scan((const uint32_t*)flags, pos, n_keys, (int64_t*)tmp, (int64_t*)nullptr, s));
  hipLaunchKernelGGL(k_unique_write, dim3(grid_for(n_keys, 256)), dim3(256), 0, s, (const uint64_t*)sorted, n_keys,
                     (const uint32_t*)flags, (const uint64_t*)pos, out_pairs, out_cap, dev_count);
  PR_HIP(hipGetLastError());
  return PR_OK;
}

extern "C" int estimate_pairs_ws_bytes(int64_t n_meshes_a, int64_t n_meshes_b, int32_t cells, size_t* ws_bytes) {
  if (n_meshes_a < 0 || n_meshes_b < 0 || cells < 1 || cells > 256 || !ws_bytes) {
    set_error("bad argument");
    return PR_E_ARG;
  }
  *ws_bytes = est_ws(n_meshes_a, n_meshes_b, cells);
  return PR_OK;
}

extern "C" int estimate_pairs(const void* blob_a, int64_t n_meshes_a, const void* blob_b, int64_t n_meshes_b,
                              int32_t cells, double* dev_estimate, void* ws, size_t ws_bytes, void* stream) {
  if (!blob_a || !blob_b || !dev_estimate || !ws || n_meshes_a < 0 || n_meshes_b < 0 || cells < 1 || cells > 256) {
    set_error("null pointer or bad size");
    return PR_E_ARG;
  }
  if (ws_bytes < est_ws(n_meshes_a, n_meshes_b, cells)) { set_error("ws_bytes too small"); return PR_E_CAPACITY; }
  hipStream_t s = (hipStream_t)stream;
  char* p = (char*)ws;
  size_t left = ws_bytes;
  EstArgs e{};
  e.blob[0] = (const char*)blob_a;
  e.blob[1] = (const char*)blob_b;
  e.n[0] = n_meshes_a;
  e.n[1] = n_meshes_b;
  e.cells = cells;
  e.side[0] = take<double>(p, left, n_meshes_a);
  e.ratio[0] = take<double>(p, left, n_meshes_a);
  e.side[1] = take<double>(p, left, n_meshes_b);
  e.ratio[1] = take<double>(p, left, n_meshes_b);
  e.ext = take<double>(p, left, 8);
  const int64_t C = (int64_t)cells * cells * cells;
  e.grid = take<double>(p, left, 6 * C);
  e.out = dev_estimate;
  if (!e.grid) { set_error("ws_bytes too small"); return PR_E_CAPACITY; }
  hipLaunchKernelGGL(k_est_init, dim3(grid_for(6 * C, 256)), dim3(256), 0, s, e, 6 * C);
  for (int d = 0; d < 2; ++d)
    if (e.n[d] > 0)
      hipLaunchKernelGGL(k_est_objects, dim3((int)std::min<int64_t>(e.n[d], 2048)), dim3(kDB), 0, s, e, d);
  for (int d = 0; d < 2; ++d)
    if (e.n[d] > 0) hipLaunchKernelGGL(k_est_cells, dim3(grid_for(e.n[d], 256)), dim3(256), 0, s, e, d);
  hipLaunchKernelGGL(k_est_sum, dim3(grid_for(C, kDB)), dim3(kDB), 0, s, e);
  PR_HIP(hipGetLastError());
  return PR_OK;
}
