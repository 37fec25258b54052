// k_bin.hip -- stage 2a of Alg. 1: tile assignment (QueryDisc) and pair
// emission.  Tile t is assigned to Gaussian i when the angle between t's cap
// centre and i's direction is at most r_s,i + R_t + guard; the NESTED
// quadtree of caps (each containing its children's) is walked from the 12
// faces, pruning subtrees whose cap misses the disc or that hold no active
// pixel.  Gaussians are processed in order of radial depth so that every list
// is depth-ordered.
#include "hp_cone.h"
#include "hp_sort_impl.h"
#include <type_traits>

// Work is split in two so that no lane walks a large Gaussian alone:
//  coarse: the Gaussians' nodes at the split level Ls = kt - 3 ("tasks");
//  fine:   the (at most 64) tiles below a task's node.
// hp_bin_sorted (k_bin_cols, k_bin_emit_sorted) takes its tasks in node order,
// depth order inside a node: up to kListNodes nodes straight from one walk
// whose waves share a stack (k_task_walk, k_task_place), beyond them from a walk
// per Gaussian and a stable sort by node.  hp_bin writes (tile, Gaussian) pairs
// in depth order for a stable tile sort: it walks per Gaussian too, and both
// its stages run twice, to count and to write at scanned offsets.
constexpr int kSplitDepth = 3;

struct BinWs {
  uint32_t* dkey;    // [P] depth bits, then sorted
  uint32_t* order;   // [P] Gaussian ids in depth order
  uint32_t* tcount;  // [P] tasks per Gaussian (depth order)
  uint64_t* toff;    // [P] exclusive scan of tcount (64-bit: the total may pass 2^32)
  uint32_t* task_g;  // [cap_t] Gaussian of each task
  uint32_t* task_n;  // [cap_t] node index at the split level
  uint32_t* pcount;  // [cap_t] pairs per task
  uint64_t* pmask;   // [cap_t] tiles hit below the task's node (bit per leaf)
  uint64_t* poff;    // [cap_t] exclusive scan of pcount
  // device scalars
  uint64_t* t_total;  // tasks wanted (scan total)
  uint64_t* nt;       // tasks kept: min(t_total, cap_t)
  uint64_t* p_total;  // pairs
  uint64_t* ncol;     // (chunk, leaf) count entries to scan (sorted emission)
  uint32_t* over;     // 1 when the tasks exceeded cap_t
  uint64_t* n_live;   // Gaussians in depth order (those that can reach an active tile)
  uint64_t* n_over;   // tasks in the walk's overflow part (zeroed by the depth sort's first kernel)
  void* sort_ws;
  void* scan_ws;
  int64_t cap_t;
};

static int64_t task_capacity(int64_t P) { return 16 * P + (1 << 20); }

static size_t bin_ws_size(int64_t P) {
  const int64_t ct = task_capacity(P);
  return 3 * hp_align256(P * 4) + hp_align256(P * 8) + 3 * hp_align256(ct * 4) + 2 * hp_align256(ct * 8) + 256 +
         hpsort::radix_ws_bytes(P) + hpsort::scan_ws_bytes<uint64_t>(ct > P ? ct : P);
}

static BinWs bin_ws(void* base, int64_t P) {
  BinWs w;
  const int64_t ct = task_capacity(P);
  char* p = (char*)base;
  w.dkey = (uint32_t*)p; p += hp_align256(P * 4);
  w.order = (uint32_t*)p; p += hp_align256(P * 4);
  w.tcount = (uint32_t*)p; p += hp_align256(P * 4);
  w.toff = (uint64_t*)p; p += hp_align256(P * 8);
  w.task_g = (uint32_t*)p; p += hp_align256(ct * 4);
  w.task_n = (uint32_t*)p; p += hp_align256(ct * 4);
  w.pcount = (uint32_t*)p; p += hp_align256(ct * 4);
  w.pmask = (uint64_t*)p; p += hp_align256(ct * 8);
  w.poff = (uint64_t*)p; p += hp_align256(ct * 8);
  w.t_total = (uint64_t*)p;
  w.nt = (uint64_t*)(p + 8);
  w.p_total = (uint64_t*)(p + 16);
  w.ncol = (uint64_t*)(p + 24);
  w.over = (uint32_t*)(p + 32);
  w.n_live = (uint64_t*)(p + 40);
  w.n_over = (uint64_t*)(p + 48);
  p += 256;
  w.sort_ws = p; p += hpsort::radix_ws_bytes(P);
  w.scan_ws = p;
  w.cap_t = ct;
  return w;
}

// pmask holds 8 B for each of the 16 P + 2^20 tasks; the sorted emission uses it
// for counts of its COUNT phase only
void* hp_bin_spare(void* ws, int64_t P) { return bin_ws(ws, P).pmask; }

// tasks kept and the overflow flag, from the scanned task total
__global__ void k_task_clamp(const uint64_t* __restrict__ t_total, int64_t cap_t, uint64_t* __restrict__ nt,
                             uint32_t* __restrict__ over) {
  const uint64_t t = *t_total;
  *over = t > (uint64_t)cap_t ? 1u : 0u;
  *nt = t > (uint64_t)cap_t ? (uint64_t)cap_t : t;
}

struct BinTables {
  const float4* cap;
  const float2* sc;
  const uint8_t* node_active;  // null: every node holds active pixels (full sphere)
  const uint8_t* leaf_active;  // never null: active flags of every node (all set for the full sphere)
  const int32_t* tile_compact;
  int kt, ls;
  // (sin, cos) of half an angle added to every Gaussian's test angle: (0, 1)
  // for the binning itself, a margin when the pairs are candidates for a
  // narrower query that filters them afterwards
  float wsin, wcos;
};

// Cap test: angle(cap centre c, u) <= R + theta as a chord comparison,
// |c - u|^2 <= (2 sin((R + theta) / 2))^2, always true once R + theta >= pi
// (cos((R + theta) / 2) <= 0).  (sR, cR) = (sin R/2, cos R/2) of the cap,
// (sg, cg) = (sin theta/2, cos theta/2) of the Gaussian (theta = r_s + guard).
// Every binning kernel tests through this one function with explicit FMAs,
// so the sorted and the unsorted emission take identical decisions.
__device__ __forceinline__ bool hp_cap_test(float cx, float cy, float cz, float sR, float cR, float ux, float uy,
                                            float uz, float sg, float cg) {
  const float dx = cx - ux, dy = cy - uy, dz = cz - uz;
  const float chord2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
  const float sh2 = fmaf(2.f * sR, cg, (2.f * cR) * sg);  // 2 sin((R + theta) / 2)
  const float ch = fmaf(cR, cg, -(sR * sg));               // cos((R + theta) / 2)
  return (ch <= 0.f) | (chord2 <= sh2 * sh2);
}

// The same test without the cos((R + theta) / 2) <= 0 branch, for callers
// that know R + theta < pi: when cos(theta / 2) > sin(R / 2) + 1e-5 the
// half-angle sum is below pi / 2 by a margin far beyond the rounding of ch,
// so the branch cannot fire and both forms decide alike.
__device__ __forceinline__ bool hp_cap_test_near(float cx, float cy, float cz, float sR, float cR, float ux, float uy,
                                                 float uz, float sg, float cg) {
  const float dx = cx - ux, dy = cy - uy, dz = cz - uz;
  const float chord2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
  const float sh2 = fmaf(2.f * sR, cg, (2.f * cR) * sg);
  return chord2 <= sh2 * sh2;
}
constexpr float kNearMargin = 1e-5f;

// largest value of v over the wave (all lanes active)
__device__ __forceinline__ float hp_wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// cap test of node `node` (inactive nodes fail)
__device__ __forceinline__ bool node_pass(const BinTables& T, int64_t node, float ux, float uy, float uz, float sg,
                                          float cg) {
  if (T.node_active && !T.node_active[node]) return false;
  const float4 c = T.cap[node];
  const float2 h = T.sc[node];
  return hp_cap_test(c.x, c.y, c.z, h.x, h.y, ux, uy, uz, sg, cg);
}

// Stackless depth-first walk of the implicit quadtree (node (l, i) has
// children 4i..4i+3 at level l+1; level 0 holds the 12 faces) from root
// (l0, i0) -- or from all 12 faces when l0 < 0 -- down to level `stop`; calls
// f(i) for every passing node at `stop`.
template <class Pass, class F>
__device__ __forceinline__ void quad_walk(int l0, int64_t i0, int stop, Pass&& pass, F&& f) {
  const bool forest = l0 < 0;
  const int lroot = forest ? 0 : l0;
  int l = lroot;
  int64_t i = forest ? 0 : i0;
  int64_t loff = hp_level_offset(l);
  while (true) {
    if (pass(loff + i)) {
      if (l == stop) {
        f(i);
      } else {
        loff += 12ll << (2 * l);
        ++l;
        i *= 4;
        continue;
      }
    }
    while (l > lroot && (i & 3) == 3) {
      --l;
      loff -= 12ll << (2 * l);
      i >>= 2;
    }
    if (l == lroot) {
      if (forest && i < 11) {
        ++i;
        continue;
      }
      break;
    }
    ++i;
  }
}

// (sin, cos) of half the test angle widened by the table's margin: the sum
// of half-angles, exact (bit for bit) when the margin is zero
__device__ __forceinline__ void widen_half(float wsin, float wcos, float* sg, float* cg) {
  const float s0 = *sg, c0 = *cg;
  *sg = fmaf(s0, wcos, c0 * wsin);
  *cg = fmaf(c0, wcos, -(s0 * wsin));
}

// direction and (sin, cos) of half the test angle r_s + guard (the sine is
// precomputed in the Gaussian's disc entry; the half angle is at most pi/2,
// so the cosine is the non-negative root), widened by the table's margin.
// A culled Gaussian (r_s = 0) has an all-zero disc entry, so the sine alone
// tells it apart (a kept one has r_s > 0 and a positive sine): one gather
// per Gaussian, not two.
__device__ __forceinline__ void gauss_dir(const float4* disc, const float* radius, uint32_t gid, const BinTables& T,
                                          float* u, float* sg, float* cg, bool* ok) {
  (void)radius;
  const hp_cfloatp r = (hp_cfloatp)disc + 4 * (int64_t)gid;
  *ok = r[3] > 0.f;
  if (!*ok) return;
  u[0] = r[0]; u[1] = r[1]; u[2] = r[2];
  *sg = r[3];
  *cg = sqrtf(fmaxf(0.f, 1.f - *sg * *sg));
  widen_half(T.wsin, T.wcos, sg, cg);
}

// coarse walk: tasks of Gaussian order[k].  With `slots` (slot-major
// [kSlots][P]) the count walk also keeps the first kSlots task nodes, and the
// emit pass copies them instead of walking again when they are all there.
constexpr int kSlots = 16;
constexpr int kTopNodes = 252;  // quadtree levels 0..2

// The quadtree's top levels (faces and two more: 252 nodes) in LDS, where
// every walk starts.  Returns how many are there.  The caller synchronises.
struct TopNodes {
  float4 cap[kTopNodes];
  float2 sc[kTopNodes];
  uint8_t act[kTopNodes];
};
__device__ __forceinline__ int load_top_nodes(const BinTables& T, TopNodes& S) {
  const int64_t nlev = hp_level_offset(T.ls + 1);  // nodes of levels 0..ls
  const int ntop = (int)(nlev < kTopNodes ? nlev : kTopNodes);
  for (int t = threadIdx.x; t < ntop; t += blockDim.x) {
    S.cap[t] = T.cap[t];
    S.sc[t] = T.sc[t];
    S.act[t] = T.node_active ? T.node_active[t] : (uint8_t)1;
  }
  return ntop;
}

// largest sin(R/2) over the LDS copy's nodes below the faces (levels 1-2), for
// the near-test guard; called by every lane after the copy is synchronised
__device__ __forceinline__ float top_srmax(const TopNodes& S, int ntop) {
  float m = 0.f;
  for (int t = 12 + hp_lane(); t < ntop; t += 64) m = fmaxf(m, S.sc[t].x);
  return hp_wave_max(m);
}

// Calls emit(i) for the passing nodes i at level T.ls, in increasing order,
// of the Gaussian with direction u and half test angle (sg, cg): the top
// levels are tested from the LDS copy, deeper ones from memory.  Level 1 (48
// nodes) is tested by every lane in the same order, which keeps the wave
// converged where a walk from the 12 faces would diverge at once; below a
// passing level-1 node the children are tested in order (level 2) and deeper
// levels are walked depth-first.
// srmax: top_srmax of the LDS copy.  When every walking lane of the wave has
// cos(theta / 2) > srmax + margin, the LDS nodes take the near test.
template <class Emit>
__device__ __forceinline__ void coarse_nodes(const BinTables& T, const TopNodes& S, int ntop, float srmax,
                                             const float* u, float sg, float cg, Emit&& emit) {
  const bool near = __builtin_amdgcn_ballot_w64(!(cg > srmax + kNearMargin)) == 0;
  auto pass = [&](int64_t node) -> bool {
    if (node < ntop) {
      if (!S.act[node]) return false;
      const float4 c = S.cap[node];
      const float2 h = S.sc[node];
      return near && node >= 12 ? hp_cap_test_near(c.x, c.y, c.z, h.x, h.y, u[0], u[1], u[2], sg, cg)
                                : hp_cap_test(c.x, c.y, c.z, h.x, h.y, u[0], u[1], u[2], sg, cg);
    }
    return node_pass(T, node, u[0], u[1], u[2], sg, cg);
  };
  if (T.ls == 0) {
    for (int f = 0; f < 12; ++f)
      if (pass(f)) emit(f);
    return;
  }
  uint64_t m1 = 0;
#pragma unroll 4
  for (int j = 0; j < 48; ++j) m1 |= pass(12 + j) ? (1ull << j) : 0ull;
  while (m1 != 0) {
    const int j = __builtin_ctzll(m1);
    m1 &= m1 - 1;
    if (T.ls == 1) {
      emit(j);
      continue;
    }
    for (int c = 0; c < 4; ++c) {
      const int64_t i2 = 4 * (int64_t)j + c;
      if (T.ls == 2) {
        if (pass(60 + i2)) emit(i2);
      } else {
        quad_walk(2, i2, T.ls, pass, emit);
      }
    }
  }
}

template <bool EMIT>
__global__ __launch_bounds__(256) void k_bin_coarse(int64_t P, const uint64_t* __restrict__ n_live,
                                                    const uint32_t* __restrict__ order,
                                                    const float4* __restrict__ disc, const float* __restrict__ radius,
                                                    BinTables T, float guard, uint32_t* __restrict__ tcount,
                                                    const uint64_t* __restrict__ toff, int64_t cap_t,
                                                    uint32_t* __restrict__ task_g, uint32_t* __restrict__ task_n,
                                                    uint32_t* __restrict__ slots) {
  __shared__ TopNodes S;
  const int ntop = load_top_nodes(T, S);
  __syncthreads();
  const float srmax = top_srmax(S, ntop);
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (int64_t)*n_live) return;
  const uint32_t gid = order[k];
  // the emit pass writes a Gaussian's tasks at its scanned offset, and none
  // past the task capacity (the count pass then flagged the overflow)
  const uint64_t base = EMIT ? toff[k] : 0ull;
  const uint32_t room = EMIT ? (base >= (uint64_t)cap_t ? 0u
                                : (uint32_t)min((uint64_t)tcount[k], (uint64_t)cap_t - base))
                             : 0u;
  if (EMIT && slots) {
    const uint32_t cnt = tcount[k];
    if (cnt <= (uint32_t)kSlots) {
      for (uint32_t j = 0; j < room; ++j) {
        task_g[base + j] = gid;
        task_n[base + j] = slots[(int64_t)j * P + k];
      }
      return;
    }
  }
  float u[3], sg, cg;
  bool ok;
  gauss_dir(disc, radius, gid, T, u, &sg, &cg, &ok);
  if (!ok) {
    if (!EMIT) tcount[k] = 0;
    return;
  }
  uint32_t cnt = 0;
  coarse_nodes(T, S, ntop, srmax, u, sg, cg, [&](int64_t i) {
    if (EMIT && cnt < room) {
      task_g[base + cnt] = gid;
      task_n[base + cnt] = (uint32_t)i;
    }
    if (!EMIT && slots && cnt < (uint32_t)kSlots) slots[(int64_t)cnt * P + k] = (uint32_t)i;
    ++cnt;
  });
  if (!EMIT) tcount[k] = cnt;
}

// ---- task list in node order without a sort --------------------------------
// For split levels of at most kListNodes nodes.  A workgroup walks the tree for
// 256 Gaussians (in depth order) over one group of kWalkGroup split-level
// nodes, and leaves their tasks in node order, depth order inside a node, in
// a run of its own, with its task count per node in a node-major histogram
// [nn][G] (G workgroups of Gaussians).  An exclusive scan of every histogram
// row and of the node totals then gives each (node, workgroup) its first
// slot, and k_task_place moves the runs there: the order that a stable sort
// of the depth-ordered tasks by node gives.
constexpr int kWalkGroup = 768;
constexpr int kListNodes = 4 * kWalkGroup;
constexpr int kWalkSmall = 192;  // nodes of the split levels up to 2: LDS for these alone (k_task_walk)
constexpr int kStageFixed = 4096;  // staged tasks per 256 Gaussians; the rest overflow
static_assert(kListNodes <= 12 * 256, "k_task_segments takes twelve nodes per thread");

// Where k_task_walk leaves its runs: block v's first `fixed` tasks at
// [v * fixed], the others at obase[v] of the shared overflow part, allocated
// by one atomic (only workgroups of wide Gaussians have any).  Tasks past the
// overflow part are not written: the total then exceeds the task capacity
// (ocap is that capacity) and nothing is emitted.
struct TaskStage {
  uint32_t* g;      // Gaussian of each task
  uint16_t* n;      // its node within the group
  uint32_t* og;
  uint16_t* on;
  uint32_t* cnt;    // [blocks]
  uint64_t* obase;  // [blocks]
  uint64_t* ocount; // overflow tasks so far
  int64_t ocap;
  int fixed;
};

// The 256-Gaussian blocks b of a workgroup: first, first + step, ... below
// the live ones.  XCD h mod 8 takes runs of 32 consecutive numbers, whose
// 4-byte entries of a histogram row share a cache line, and the workgroups of a
// bounded grid (what is resident at once) loop: a launch of one workgroup per 256 Gaussians of
// the scene spent tens of microseconds on starting idle ones when a narrow
// view keeps an eighth of the scene.
constexpr unsigned kWalkGrid = 768, kWalkGridSmall = 1024, kPlaceGrid = 1024;
static unsigned walk_grid(unsigned G, unsigned most) { return G < most ? (G + 255u) & ~255u : most; }
__device__ __forceinline__ int64_t walk_first(uint32_t h) {
  const uint32_t x = h & 7u, k = h >> 3;
  return (int64_t)(((k >> 5) * 8u + x) * 32u + (k & 31u));
}

// Balanced tree walk.  The lanes of a wave share a stack of (Gaussian, node)
// entries that passed: up to 64 at a time leave it, each lane tests one child
// of sixteen of them in turn, and the children that pass go back on it, or,
// at the split level, set the Gaussian's bit in the node's row of a bit matrix
// in LDS.  A Gaussian next to the camera reaches hundreds of nodes, and a lane
// that walked them alone held up its wave: 250K Gaussians seen by a 75-degree
// pinhole at Nside 1024 took 105 us to count and 219 us to place, one lane's
// chain of dependent tests; the shared stack makes that 38 and 11 us (1M
// Gaussians on the full sphere at Nside 512: 72 + 122 us became 77 + 21 us).
// Four lanes to a parent read its four children's caps as one 64-byte line.
// The same nodes pass as in coarse_nodes: the faces, which that walk does not
// test, are tested with a margin (a face's cap contains its descendants'), so
// they only save work.
//
// A task's place in its node's row is the number of set bits before its own.
// The waves also list their tasks: a workgroup whose lists hold them all
// takes the tasks from there.  The others (wide Gaussians) read the matrix
// back with a lane per 32-bit word, the eight words of a node side by side, so
// that a few nodes that every Gaussian reaches are spread over the workgroup
// (with a thread per three nodes one thread wrote hundreds of tasks one by one).
//
// Stack bound: entries leave 64 at a time and push at most 256 of the next
// deeper levels, so going up the stack each batch holds deeper levels only, and
// at most 192 entries remain of each of the levels 1 to ls - 1 above at most 63
// faces: 63 + 192 + 192 + 256 = 703 at ls = 4.
// Bound by vector issue (1,690 instructions per 64 Gaussians, 45 us of the case
// above) and latency: 52 KB of LDS for 768 nodes, three workgroups per CU, 94 us;
// with LDS for the 192 nodes that split levels up to 2 have, 31 KB and four
// workgroups (118 registers), 77 us; five, held to 96 registers, the same.
constexpr int kWalkStack = 704;  // entries per wave: Gaussian of the wave << 10 | heap index
constexpr int kWalkList = 1024;  // tasks listed per wave: node << 6 | Gaussian of the wave
template <int GROUP>
struct WalkLds {
  static constexpr int kRow = GROUP + 8;  // pitch of the bit matrix: its eight words of a node in different banks
  float4 cap[kTopNodes];  // levels 0..2: centre and sin(R/2)
  float cr[kTopNodes];    // cos(R/2); NaN for inactive nodes, which then pass no test
  uint32_t bits[8][kRow];
  uint32_t cnt[GROUP];  // tasks per node
  uint16_t list[4][kWalkList];
  uint16_t stack[4][kWalkStack];
  union {
    struct {
      float4 disc[256];
      float cg[256];
    };
    struct {  // after the walk
      uint32_t start[GROUP];  // the node's first place in the run
      uint32_t gid[256];
    };
  };
};
template <int GROUP>
__global__ __launch_bounds__(256) void k_task_walk(const uint64_t* __restrict__ n_live,
                                                   const uint32_t* __restrict__ order,
                                                   const float4* __restrict__ disc, BinTables T, int nn, int64_t G,
                                                   uint32_t* __restrict__ hist, TaskStage st) {
  constexpr int kRow = WalkLds<GROUP>::kRow, kPer = (GROUP + 255) / 256;
  __shared__ WalkLds<GROUP> s;
  __shared__ uint32_t s_w[4], s_listed[4];
  __shared__ uint64_t s_ob;
  const int64_t n_in = (int64_t)*n_live;
  const int64_t bfirst = walk_first(blockIdx.x);
  if (bfirst * 256 >= n_in) return;
  const int tid = threadIdx.x, wv = tid >> 6, lane = hp_lane();
  const int n0 = (int)blockIdx.y * GROUP;
  const int ng = nn - n0 < GROUP ? nn - n0 : GROUP;
  const int nroot = 12 / (int)gridDim.y, root0 = (int)blockIdx.y * nroot;  // the group's faces
  bool any = !T.node_active;
  if (T.node_active)
    for (int r = 0; r < nroot; ++r) any |= T.node_active[root0 + r] != 0;
  if (!any) {  // k_hist_rows leaves out the rows of inactive nodes
    for (int64_t b = bfirst; b * 256 < n_in; b += gridDim.x)
      if (tid == 0) st.cnt[(int64_t)blockIdx.y * G + b] = 0u;
    return;
  }
  const int64_t nlev = hp_level_offset(T.ls + 1);  // nodes of levels 0..ls
  const int ntop = (int)(nlev < kTopNodes ? nlev : kTopNodes);
  for (int t = tid; t < ntop; t += 256) {
    const float4 c = T.cap[t];
    const float2 h = T.sc[t];
    const bool act = !T.node_active || T.node_active[t] != 0;
    const float nan = __int_as_float(0x7fc00000);
    s.cap[t] = act ? make_float4(c.x, c.y, c.z, h.x) : make_float4(nan, nan, nan, nan);
    s.cr[t] = act ? h.y : nan;
  }
  const int leaf0 = (int)hp_level_offset(T.ls);  // heap index of the split level's first node
  const uint64_t below = (1ull << lane) - 1ull;
  uint16_t* stack = s.stack[wv];
  uint16_t* list = s.list[wv];
  const float4* wdisc = s.disc + 64 * wv;
  const float* wcg = s.cg + 64 * wv;
  const int w8 = tid & 7;
  const int rounds = (ng + 31) / 32;

  // this block's Gaussian; the next block's is fetched during the walk
  auto fetch = [&](int64_t b, uint32_t* id, float4* d) {
    const int64_t k = b * 256 + tid;
    *id = k < n_in ? order[k] : 0u;
    *d = k < n_in ? disc[*id] : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  uint32_t gid_next;
  float4 dg_next;
  fetch(bfirst, &gid_next, &dg_next);

  for (int64_t b = bfirst; b * 256 < n_in; b += gridDim.x) {
    const int64_t vb = (int64_t)blockIdx.y * G + b;
    __syncthreads();  // the previous block's reads are done
    for (int i = tid; i < 8 * kRow / 4; i += 256) reinterpret_cast<uint4*>(&s.bits[0][0])[i] = make_uint4(0, 0, 0, 0);
    for (int i = tid; i < GROUP; i += 256) s.cnt[i] = 0u;
    const uint32_t gid = gid_next;
    const float4 dg = dg_next;
    const bool live = dg.w > 0.f;
    float sg = dg.w, cg = sqrtf(fmaxf(0.f, 1.f - dg.w * dg.w));
    widen_half(T.wsin, T.wcos, &sg, &cg);
    s.disc[tid] = make_float4(dg.x, dg.y, dg.z, sg);
    s.cg[tid] = cg;
    fetch(b + gridDim.x, &gid_next, &dg_next);
    __syncthreads();
    // the faces the Gaussian may reach: the angle to the face's centre at most
    // R + theta, by cosines (their rounding, 1e-6, is far below the margin)
    uint32_t faces = 0;
#pragma unroll
    for (int r = 0; r < 12; ++r) {
      const int n = r < nroot ? root0 + r : root0;
      const float4 c = s.cap[n];
      const float cr = s.cr[n];
      const float sh = fmaf(c.w, cg, cr * sg), ch = fmaf(cr, cg, -(c.w * sg));  // (R + theta) / 2
      const float dot = fmaf(c.z, dg.z, fmaf(c.y, dg.y, c.x * dg.x));
      faces |= live && (ch <= 1e-4f || dot >= fmaf(-2.f * sh, sh, 1.f - 1e-4f)) ? 1u << r : 0u;
    }
    int top = 0, f = 0, nlist = 0;
    // a task of this lane: its bit, its node's count and the wave's list
    auto emit = [&](bool in, int node, uint32_t g) {
      const uint64_t em = __ballot(in);
      if (em == 0) return;
      if (in) {
        atomicOr(&s.bits[2 * wv + (int)(g >> 5)][node], 1u << (g & 31u));
        atomicAdd(&s.cnt[node], 1u);
        const int at = nlist + (int)__popcll(em & below);
        if (at < kWalkList) list[at] = (uint16_t)((node << 6) | (int)g);
      }
      nlist += (int)__popcll(em);
    };
    if (T.ls == 0) {
      for (; f < 12; ++f) {
        const float4 c = s.cap[f];
        emit(live && hp_cap_test(c.x, c.y, c.z, c.w, s.cr[f], dg.x, dg.y, dg.z, sg, cg), f, (uint32_t)lane);
      }
    }
    while (true) {
      while (f < nroot && top < 64) {
        const bool in = ((faces >> f) & 1u) != 0u;
        const uint64_t m = __ballot(in);
        if (in) stack[top + __popcll(m & below)] = (uint16_t)((lane << 10) | (root0 + f));
        top += (int)__popcll(m);
        ++f;
      }
      if (top == 0) break;
      const int m = top < 64 ? top : 64;
      top -= m;
      // entry 16 r + lane / 4 of the popped ones: its child lane % 4
      uint32_t it[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int e = 16 * r + (lane >> 2);
        it[r] = stack[top + (e < m ? e : 0)];
      }
      float4 c[4], d[4];
      float cr[4], dcg[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // children of heap node X: 4 (X + 3) .. 4 (X + 3) + 3
        const int child = 4 * (int)((it[r] & 1023u) + 3u) + (lane & 3);
        d[r] = wdisc[it[r] >> 10];
        dcg[r] = wcg[it[r] >> 10];
        if (child < kTopNodes) {
          c[r] = s.cap[child];
          cr[r] = s.cr[child];
        } else {
          c[r] = T.cap[child];
          const float2 h = T.sc[child];
          c[r].w = h.x;
          cr[r] = T.node_active && !T.node_active[child] ? __int_as_float(0x7fc00000) : h.y;
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (16 * r >= m) break;
        const int child = 4 * (int)((it[r] & 1023u) + 3u) + (lane & 3);
        const uint32_t g = it[r] >> 10;
        // an inactive node's NaN fails both comparisons
        const bool in = 16 * r + (lane >> 2) < m &&
                        hp_cap_test(c[r].x, c[r].y, c[r].z, c[r].w, cr[r], d[r].x, d[r].y, d[r].z, d[r].w, dcg[r]);
        const bool leaf = child >= leaf0;
        const uint64_t pm = __ballot(in && !leaf);
        if (in && !leaf) stack[top + __popcll(pm & below)] = (uint16_t)((g << 10) | (uint32_t)child);
        top += (int)__popcll(pm);
        emit(in && leaf, child - leaf0 - n0, g);
      }
    }
    if (lane == 0) s_listed[wv] = nlist <= kWalkList;
    __syncthreads();
    // the node counts to the histogram, and scanned (thread t: kPer nodes from kPer t)
    s.gid[tid] = gid;
    uint32_t cnt[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int n = kPer * tid + q;
      cnt[q] = n < ng ? s.cnt[n] : 0u;
      if (n < ng) hist[(int64_t)(n0 + n) * G + b] = cnt[q];
      sum += cnt[q];
    }
    uint32_t total;
    uint32_t pos = hpsort::block_exclusive<uint32_t>(sum, &total, s_w);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (kPer * tid + q < ng) s.start[kPer * tid + q] = pos;
      pos += cnt[q];
    }
    const uint32_t fixed = (uint32_t)st.fixed;
    if (tid == 0) {
      st.cnt[vb] = total;
      if (total > fixed) {
        const uint64_t o = atomicAdd((unsigned long long*)st.ocount, (unsigned long long)(total - fixed));
        st.obase[vb] = o;
        s_ob = o;
      }
    }
    __syncthreads();
    const uint64_t ob = total > fixed ? s_ob : 0ull;
    auto put = [&](uint32_t at, uint32_t g, uint32_t n) {
      if (at < fixed) {
        st.g[vb * fixed + at] = g;
        st.n[vb * fixed + at] = (uint16_t)n;
      } else if (ob + (at - fixed) < (uint64_t)st.ocap) {
        st.og[ob + (at - fixed)] = g;
        st.on[ob + (at - fixed)] = (uint16_t)n;
      }
    };
    if (s_listed[0] & s_listed[1] & s_listed[2] & s_listed[3]) {
      for (int t = lane; t < nlist; t += 64) {
        const uint32_t e = list[t], n = e >> 6, g = e & 63u;
        const int w = 2 * wv + (int)(g >> 5);
        uint32_t rank = (uint32_t)__popc(s.bits[w][n] & ((1u << (g & 31u)) - 1u));
#pragma unroll
        for (int v = 0; v < 7; ++v) rank += v < w ? (uint32_t)__popc(s.bits[v][n]) : 0u;
        put(s.start[n] + rank, s.gid[64 * wv + (int)g], n);
      }
    } else {
      // word w8 of node 32 r + tid / 8: its tasks after those of the words before
      for (int r = 0; r < rounds; ++r) {
        const int n = 32 * r + (tid >> 3);
        uint32_t bits = s.bits[w8][n];
        uint32_t x = (uint32_t)__popc(bits);
        const uint32_t own = x;
        const uint32_t y1 = hpsort::dpp_u32<0x111, 0xf, true>(x);
        x += w8 >= 1 ? y1 : 0u;
        const uint32_t y2 = hpsort::dpp_u32<0x112, 0xf, true>(x);
        x += w8 >= 2 ? y2 : 0u;
        const uint32_t y4 = hpsort::dpp_u32<0x114, 0xf, true>(x);
        x += w8 >= 4 ? y4 : 0u;
        uint32_t at = (n < ng ? s.start[n] : 0u) + x - own;
        while (bits != 0) {
          put(at++, s.gid[32 * w8 + __builtin_ctz(bits)], (uint32_t)n);
          bits &= bits - 1;
        }
      }
    }
  }
}

// One workgroup per node n: the histogram row hist[n][0..G) becomes its
// exclusive scan hoff[n][0..G) (where workgroup b's tasks at node n start
// among the node's tasks) and rowtot[n] the node's task count (a Gaussian has
// at most one task per node, so 32 bits hold a row).  The node offsets (an
// exclusive scan of rowtot) follow in k_task_segments.  Rows have room for G
// workgroups; those of the *n_live Gaussians are filled, and none where the
// node (active: the split level's flags, or null) is inactive.
__global__ __launch_bounds__(256) void k_hist_rows(const uint32_t* __restrict__ hist, int64_t G,
                                                   const uint64_t* __restrict__ n_live,
                                                   const uint8_t* __restrict__ active, uint32_t* __restrict__ hoff,
                                                   uint64_t* __restrict__ rowtot) {
  __shared__ uint32_t s_w[4];
  constexpr int kItems = 16;
  if (active && !active[blockIdx.x]) {
    if (threadIdx.x == 0) rowtot[blockIdx.x] = 0ull;
    return;
  }
  const int64_t g_live = (int64_t)((*n_live + 255) / 256);
  const uint32_t* row = hist + (int64_t)blockIdx.x * G;
  uint32_t* out = hoff + (int64_t)blockIdx.x * G;
  uint32_t carry = 0;
  for (int64_t t0 = 0; t0 < g_live; t0 += 256 * kItems) {
    const int64_t j0 = t0 + (int64_t)kItems * threadIdx.x;
    uint32_t v[kItems], acc = 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      v[k] = j0 + k < g_live ? row[j0 + k] : 0u;
      acc += v[k];
    }
    uint32_t tot;
    uint32_t ex = hpsort::block_exclusive<uint32_t>(acc, &tot, s_w) + carry;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      if (j0 + k < g_live) out[j0 + k] = ex;
      ex += v[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) rowtot[blockIdx.x] = carry;
}

// Every staged run to its nodes' places in the task list (the blocks of
// k_task_walk, in the same order); also the node of every chunk of 64 tasks,
// nodes strided over the workgroups.  6 B read and 4 B written per task, bound
// by the chain of loads before a run's writes: a task's node and Gaussian are
// read once and together (31 -> 21 us for 4.8M tasks of 1M Gaussians on the full
// sphere at Nside 512; with a pass for the nodes' places before one that read
// the tasks again it waited for memory once more).
constexpr int kPlaceThreads = 512, kPlaceIlp = 4;
__global__ __launch_bounds__(kPlaceThreads) void k_task_place(const uint64_t* __restrict__ n_live, int nn, int64_t G,
                                                              TaskStage st, const uint32_t* __restrict__ hoff,
                                                              const uint64_t* __restrict__ node_off, int64_t cap_t,
                                                              uint32_t* __restrict__ task_g,
                                                              const uint32_t* __restrict__ choff,
                                                              uint32_t* __restrict__ cnode) {
  __shared__ uint64_t s_first[kWalkGroup];
  for (int64_t n = (int64_t)blockIdx.y * gridDim.x + blockIdx.x; n < nn; n += (int64_t)gridDim.x * gridDim.y) {
    const uint32_t c1 = choff[n + 1];
    for (uint32_t c = choff[n] + threadIdx.x; c < c1; c += blockDim.x) cnode[c] = (uint32_t)n;
  }
  const int64_t n_in = (int64_t)*n_live;
  const int n0 = (int)blockIdx.y * kWalkGroup;
  for (int64_t b = walk_first(blockIdx.x); b * 256 < n_in; b += gridDim.x) {
    const int64_t vb = (int64_t)blockIdx.y * G + b;
    const uint32_t total = st.cnt[vb], fixed = (uint32_t)st.fixed;
    if (total == 0) continue;
    const uint64_t ob = total > fixed ? st.obase[vb] : 0ull;
    // task t of the run; tasks that the overflow part did not hold are past tmax
    const uint64_t room = ob < (uint64_t)st.ocap ? (uint64_t)st.ocap - ob : 0ull;
    const uint32_t tmax = total > fixed && total - fixed > room ? fixed + (uint32_t)room : total;
    auto node = [&](uint32_t t) { return (uint32_t)(t < fixed ? st.n[vb * fixed + t] : st.on[ob + (t - fixed)]); };
    __syncthreads();  // the previous run's reads are done
    // kPlaceIlp tasks of a thread at a time, their loads all in flight: the
    // runs of the widest Gaussians are tens of times the others' length.  A
    // node's first place is set in the step that holds its first task, so later
    // steps, whose nodes are others, need no barrier before they set theirs.
    constexpr uint32_t kStep = kPlaceThreads * kPlaceIlp;
    for (uint32_t b0 = 0; b0 < tmax; b0 += kStep) {
      uint32_t n[kPlaceIlp], before[kPlaceIlp], g[kPlaceIlp];
#pragma unroll
      for (int j = 0; j < kPlaceIlp; ++j) {
        const uint32_t t = b0 + threadIdx.x + j * kPlaceThreads;
        n[j] = t < tmax ? node(t) : 0u;
        before[j] = t > 0 && t < tmax ? node(t - 1) : ~0u;
        g[j] = t >= tmax ? 0u : (t < fixed ? st.g[vb * fixed + t] : st.og[ob + (t - fixed)]);
      }
#pragma unroll
      for (int j = 0; j < kPlaceIlp; ++j) {
        const uint32_t t = b0 + threadIdx.x + j * kPlaceThreads;
        if (t < tmax && n[j] != before[j]) s_first[n[j]] = node_off[n0 + n[j]] + hoff[(int64_t)(n0 + n[j]) * G + b] - t;
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kPlaceIlp; ++j) {
        const uint32_t t = b0 + threadIdx.x + j * kPlaceThreads;
        const uint64_t pos = t < tmax ? s_first[n[j]] + t : (uint64_t)cap_t;
        if (pos < (uint64_t)cap_t) task_g[pos] = g[j];
      }
    }
  }
}

// One workgroup: every node's first task (an exclusive scan of the node task
// counts, into node_off), the task total and overflow flag, every node's task
// segment (clamped to the capacity), its chunks of 64 tasks and their
// offsets, and the number of (chunk, leaf) columns.  After an overflow no
// chunk is made.
__global__ __launch_bounds__(256) void k_task_segments(int nn, const uint64_t* __restrict__ rowtot,
                                                       uint64_t* __restrict__ node_off, int64_t cap_t, int depth,
                                                       uint64_t* __restrict__ t_total, uint64_t* __restrict__ nt,
                                                       uint32_t* __restrict__ over, uint32_t* __restrict__ seg,
                                                       uint32_t* __restrict__ choff, uint64_t* __restrict__ ncol) {
  __shared__ uint64_t s_w64[4];
  __shared__ uint32_t s_w[4];
  // thread t takes the `per` consecutive nodes from per * t (at most kPer)
  constexpr int kPer = kListNodes / 256;
  const int per = (nn + 255) / 256;
  uint64_t cnt[kPer], sum = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int n = per * (int)threadIdx.x + q;
    cnt[q] = q < per && n < nn ? rowtot[n] : 0ull;
    sum += cnt[q];
  }
  uint64_t tot;
  uint64_t pre = hpsort::block_exclusive<uint64_t>(sum, &tot, s_w64);
  const bool ov = tot > (uint64_t)cap_t;
  const uint64_t lim = ov ? (uint64_t)cap_t : tot;
  uint32_t nch[kPer], csum = 0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int n = per * (int)threadIdx.x + q;
    nch[q] = 0u;
    if (q < per && n < nn) {
      node_off[n] = pre;
      uint64_t s0 = pre, s1 = pre + cnt[q];
      s0 = s0 < lim ? s0 : lim;
      s1 = s1 < lim ? s1 : lim;
      seg[2 * n] = (uint32_t)s0;
      seg[2 * n + 1] = (uint32_t)s1;
      nch[q] = ov ? 0u : (uint32_t)((s1 - s0 + 63) / 64);
    }
    pre += cnt[q];
    csum += nch[q];
  }
  uint32_t total;
  uint32_t ex = hpsort::block_exclusive<uint32_t>(csum, &total, s_w);
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int n = per * (int)threadIdx.x + q;
    if (q < per && n < nn) choff[n] = ex;
    ex += nch[q];
  }
  if (threadIdx.x == 0) {
    choff[nn] = total;
    *ncol = (uint64_t)total << (2 * depth);
    *t_total = tot;
    *nt = lim;
    *over = ov ? 1u : 0u;
  }
}

// fine stage: one lane per tile below a task's node (64 tiles three levels
// down).  A wave takes 64 consecutive tasks at a time (their Gaussian and
// node ids in one coalesced load, then read out lane by lane) and issues the
// loads of kFineGroup tasks before testing any of them, so that many memory
// requests are in flight per wave.  The count pass keeps each task's 64-bit
// hit mask; the emit pass only turns masks into pairs, each hit written at
// its rank among the task's hits so that the pairs of a task are contiguous
// and tasks stay in depth order.
constexpr int kFineGroup = 8;

__device__ __forceinline__ uint64_t hp_readlane64(uint64_t v, int i) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, i);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), i);
  return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(256) void k_bin_fine_count(const uint64_t* __restrict__ n_tasks, int64_t cap_t,
                                                        const uint32_t* __restrict__ task_g,
                                                        const uint32_t* __restrict__ task_n,
                                                        const float4* __restrict__ disc, BinTables T,
                                                        uint64_t* __restrict__ pmask, uint32_t* __restrict__ pcount) {
  int64_t nt = (int64_t)*n_tasks;
  if (nt > cap_t) nt = cap_t;
  const int lane = hp_lane();
  const int depth = T.kt - T.ls;  // 0..3 levels below the task node
  const bool leaf_lane = lane < (1 << (2 * depth));
  const int leaf_mask = (1 << (2 * depth)) - 1;
  const int64_t leaf_off = hp_level_offset(T.kt);
  const int64_t nch = (nt + 63) >> 6;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  // the 64 tasks' discs, one gather per lane, read back as LDS broadcasts
  __shared__ float4 s_disc[4][64];
  const int wv = threadIdx.x >> 6;
  for (int64_t c = (int64_t)blockIdx.x * (blockDim.x >> 6) + hp_uniform(threadIdx.x >> 6); c < nch; c += waves) {
    const int64_t t0 = c << 6;
    const int nin = nt - t0 < 64 ? (int)(nt - t0) : 64;
    const uint32_t tg = lane < nin ? task_g[t0 + lane] : 0u;
    const uint32_t tn = lane < nin ? task_n[t0 + lane] : 0u;
    __builtin_amdgcn_wave_barrier();  // the previous chunk's reads are done
    s_disc[wv][lane] = lane < nin ? disc[tg] : make_float4(0.f, 0.f, 0.f, 0.f);
    __builtin_amdgcn_wave_barrier();
    uint64_t mine = 0;
    for (int i0 = 0; i0 < nin; i0 += kFineGroup) {
      float3 cap[kFineGroup];  // cap centre (the radius enters through sc)
      float2 sc[kFineGroup];
      uint32_t act[kFineGroup];
      float ux[kFineGroup], uy[kFineGroup], uz[kFineGroup], sg[kFineGroup];
#pragma unroll
      for (int q = 0; q < kFineGroup; ++q) {
        // past the chunk's end the last task is loaded again; its result is dropped
        const int i = i0 + q < nin ? i0 + q : nin - 1;
        // lanes past the node's leaves (depth < 3) load a valid leaf and drop it
        const int64_t node = leaf_off + ((int64_t)(uint32_t)__builtin_amdgcn_readlane((int)tn, i) << (2 * depth)) +
                             (lane & leaf_mask);
        const float4 d = s_disc[wv][i];  // same address on every lane: a broadcast
        ux[q] = d.x; uy[q] = d.y; uz[q] = d.z; sg[q] = d.w;
        const float* cp = (const float*)(T.cap + node);
        cap[q] = make_float3(cp[0], cp[1], cp[2]);
        sc[q] = T.sc[node];
        act[q] = (uint32_t)T.leaf_active[node];
      }
#pragma unroll
      for (int q = 0; q < kFineGroup; ++q) {
        const float cg = sqrtf(fmaxf(0.f, 1.f - sg[q] * sg[q]));
        const bool hit = leaf_lane && (act[q] != 0u) &&
                         hp_cap_test(cap[q].x, cap[q].y, cap[q].z, sc[q].x, sc[q].y, ux[q], uy[q], uz[q], sg[q], cg);
        const uint64_t m = __ballot(hit);
        if (lane == i0 + q) mine = m;
      }
    }
    if (lane < nin) {
      pmask[t0 + lane] = mine;
      pcount[t0 + lane] = (uint32_t)__popcll(mine);
    }
  }
}

__global__ __launch_bounds__(256) void k_bin_fine_emit(const uint64_t* __restrict__ n_tasks, int64_t cap_t,
                                                       const uint32_t* __restrict__ task_g,
                                                       const uint32_t* __restrict__ task_n, BinTables T,
                                                       const uint64_t* __restrict__ pmask,
                                                       const uint64_t* __restrict__ poff,
                                                       const int64_t* __restrict__ n_pairs, int64_t capacity,
                                                       uint32_t* __restrict__ keys, uint32_t* __restrict__ vals) {
  int64_t nt = (int64_t)*n_tasks;
  if (nt > cap_t) nt = cap_t;
  if (*n_pairs > capacity) return;
  const int lane = hp_lane();
  const int depth = T.kt - T.ls;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int64_t nch = (nt + 63) >> 6;
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  for (int64_t c = (int64_t)blockIdx.x * (blockDim.x >> 6) + hp_uniform(threadIdx.x >> 6); c < nch; c += waves) {
    const int64_t t0 = c << 6;
    const int nin = nt - t0 < 64 ? (int)(nt - t0) : 64;
    const uint32_t tg = lane < nin ? task_g[t0 + lane] : 0u;
    const uint32_t tn = lane < nin ? task_n[t0 + lane] : 0u;
    const uint64_t mk = lane < nin ? pmask[t0 + lane] : 0ull;
    const uint64_t of = lane < nin ? poff[t0 + lane] : 0ull;
    for (int i0 = 0; i0 < nin; i0 += kFineGroup) {
      // all addresses and values of the group first, then only stores: no
      // register that an in-flight store reads is written before it drains
      int32_t comp[kFineGroup];
      uint32_t gv[kFineGroup];
      uint32_t* kp[kFineGroup];
      uint32_t* vp[kFineGroup];
      bool hit[kFineGroup];
#pragma unroll
      for (int q = 0; q < kFineGroup; ++q) {
        const int i = i0 + q < nin ? i0 + q : nin - 1;
        const uint64_t m = i0 + q < nin ? hp_readlane64(mk, i) : 0ull;
        const int64_t leaf = ((int64_t)(uint32_t)__builtin_amdgcn_readlane((int)tn, i) << (2 * depth)) + lane;
        hit[q] = ((m >> lane) & 1ull) != 0;
        comp[q] = hit[q] ? T.tile_compact[leaf] : 0;
        const uint64_t at = hp_readlane64(of, i) + (uint64_t)__popcll(m & below);
        kp[q] = keys + at;
        vp[q] = vals + at;
        gv[q] = (uint32_t)__builtin_amdgcn_readlane((int)tg, i);
      }
      // wait once for the group's gathers (vmcnt 0; expcnt and lgkmcnt left
      // at their maxima), so that the masked stores below need no waits
      __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
      for (int q = 0; q < kFineGroup; ++q) {
        if (hit[q]) {
          *kp[q] = (uint32_t)comp[q];
          *vp[q] = gv[q];
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Pairs straight into per-tile depth order (no sort of the pairs).  Every
// task names one node at the split level and one Gaussian.  After a stable
// sort of the tasks by node, the pairs of tile t = (node n, leaf b) are the
// tasks of n's segment whose test on leaf b passes, in depth order.  Each
// segment is cut into chunks of 64 tasks; a wave per chunk keeps one leaf per
// lane and tests the chunk's tasks one after the other, collecting for leaf b
// the 64-bit column W_b of hits.  popcount(W_b) per (chunk, leaf), laid out
// tile-major -- for each node, for each leaf, its chunks in order -- and
// scanned, gives every (chunk, leaf) its first output slot; inside a chunk
// the task at bit j writes at popcount(W_b below j).
// ---------------------------------------------------------------------------
__global__ void k_seg_ranges(const uint32_t* __restrict__ keys, const uint64_t* __restrict__ n_dev, uint32_t nn,
                             uint32_t* __restrict__ seg) {
  const int64_t n = (int64_t)*n_dev;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t k = keys[i];
    if (k >= nn) continue;
    if (i == 0 || keys[i - 1] != k) seg[2 * (int64_t)k] = (uint32_t)i;
    if (i == n - 1 || keys[i + 1] != k) seg[2 * (int64_t)k + 1] = (uint32_t)(i + 1);
  }
}

__global__ void k_seg_chunks(const uint32_t* __restrict__ seg, uint32_t nn, uint32_t* __restrict__ nch) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nn) nch[i] = (seg[2 * i + 1] - seg[2 * i] + 63) / 64;
}

__global__ void k_fill_zero_u32(uint32_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// node of every chunk: workgroup n fills the chunks [choff[n], choff[n+1])
__global__ void k_chunk_nodes(const uint32_t* __restrict__ choff, uint32_t* __restrict__ cnode) {
  const uint32_t n = blockIdx.x, c1 = choff[n + 1];
  for (uint32_t c = choff[n] + threadIdx.x; c < c1; c += blockDim.x) cnode[c] = n;
}

struct ChunkInfo {
  uint32_t node, local, nchn, t0, ntask;
};
__device__ __forceinline__ ChunkInfo chunk_info(const uint32_t* choff, const uint32_t* seg, const uint32_t* cnode,
                                                uint32_t c) {
  ChunkInfo ci;
  ci.node = hp_uniform(((hp_cu32p)cnode)[c]);
  const uint32_t c0 = hp_uniform(((hp_cu32p)choff)[ci.node]);
  ci.nchn = hp_uniform(((hp_cu32p)choff)[ci.node + 1]) - c0;
  ci.local = c - c0;
  const uint32_t s0 = hp_uniform(((hp_cu32p)seg)[2 * ci.node]), s1 = hp_uniform(((hp_cu32p)seg)[2 * ci.node + 1]);
  ci.t0 = s0 + 64 * ci.local;
  ci.ntask = s1 - ci.t0 < 64 ? s1 - ci.t0 : 64;
  return ci;
}

// The chunks of the calling wave.  Workgroup b runs on XCD b mod 8, so XCD
// x takes the contiguous range [x n / 8, (x + 1) n / 8), shared by the waves
// of its workgroups.  Neighbouring chunks belong to the same or neighbouring
// quadtree nodes, whose tasks gather the same Gaussians' records and write
// the same tiles' lists: within one XCD they meet in one L2.  With fewer than
// 8 workgroups every wave strides over all chunks.
struct ChunkRange {
  uint32_t first, end, stride;
};
__device__ __forceinline__ ChunkRange xcd_chunks(uint32_t n) {
  // the wave index is uniform, which the compiler cannot see: without the
  // readfirstlane every chunk index (and the node search below) would live
  // in vector registers, with a vector load per search step
  const uint32_t nb = gridDim.x, wpb = blockDim.x >> 6, w = hp_uniform(threadIdx.x >> 6);
  ChunkRange r;
  if (nb < 8u) {
    r.first = blockIdx.x * wpb + w;
    r.end = n;
    r.stride = nb * wpb;
    return r;
  }
  const uint32_t x = blockIdx.x & 7u, k = blockIdx.x >> 3;
  const uint32_t nbx = (nb - x + 7u) / 8u;  // workgroups b < nb with b mod 8 = x
  r.first = (uint32_t)((uint64_t)n * x / 8u) + k * wpb + w;
  r.end = (uint32_t)((uint64_t)n * (x + 1u) / 8u);
  r.stride = nbx * wpb;
  return r;
}

// w = 2 w + (the lane's bit of in[q]) for q = 0, 1, ...: one instruction each,
// with the mask as carry-in; the compiler makes a select and an or of it. The
// s_nop keeps the two wait states between a compare and its mask's use.
static_assert(kFineGroup == 8, "shift_in_bits takes eight masks");
__device__ __forceinline__ void shift_in_bits(uint32_t* w, const uint64_t* in) {
#define HP_SHIFT_IN(n) "v_addc_co_u32_e64 %0, vcc, %0, %0, %" n "\n\t"
  asm("s_nop 1\n\t" HP_SHIFT_IN("1") HP_SHIFT_IN("2") HP_SHIFT_IN("3") HP_SHIFT_IN("4") HP_SHIFT_IN("5")
      HP_SHIFT_IN("6") HP_SHIFT_IN("7") HP_SHIFT_IN("8")
      : "+v"(*w)
      : "s"(in[0]), "s"(in[1]), "s"(in[2]), "s"(in[3]), "s"(in[4]), "s"(in[5]), "s"(in[6]), "s"(in[7])
      : "vcc");
#undef HP_SHIFT_IN
}

// per chunk: the hit columns W_b (kept) and their popcounts, tile-major
// Bound by vector instruction issue, 11 per (task, 64 leaves): 107 -> 76 us (1M
// Gaussians on the full sphere at Nside 512), 68 -> 48 us (3M, pinhole of 60
// degrees at Nside 2048) since the bits are shifted in.
__global__ __launch_bounds__(256) void k_bin_cols(const uint32_t* __restrict__ choff, uint32_t nn,
                                                  const uint32_t* __restrict__ seg, const uint32_t* __restrict__ cnode,
                                                  const uint32_t* __restrict__ tgid,
                                                  const float4* __restrict__ disc, BinTables T,
                                                  uint64_t* __restrict__ wcol, uint32_t* __restrict__ cnt) {
  const uint32_t nchunks = hp_uniform(((hp_cu32p)choff)[nn]);
  const int lane = hp_lane();
  const int depth = T.kt - T.ls;
  const int nleaf = 1 << (2 * depth);
  const bool leaf_lane = lane < nleaf;
  const int64_t leaf_off = hp_level_offset(T.kt);
  // the chunk's 64 tasks' discs, one per lane, published for the whole wave:
  // (direction, sin) and cos of half the widened test angle
  __shared__ float4 s_disc[4][64];
  __shared__ float s_cg[4][64];
  const int wv = threadIdx.x >> 6;
  const ChunkRange cr = xcd_chunks(nchunks);
  for (uint32_t c = cr.first; c < cr.end; c += cr.stride) {
    const ChunkInfo ci = chunk_info(choff, seg, cnode, c);
    const uint32_t ntask = hp_uniform(ci.ntask);
    // this lane's leaf below the chunk's node (lanes past the leaves test a
    // valid leaf and drop the result)
    const int64_t leaf = leaf_off + ((int64_t)ci.node << (2 * depth)) + (lane & (nleaf - 1));
    const float* cp = (const float*)(T.cap + leaf);
    const float cx = cp[0], cy = cp[1], cz = cp[2];
    const float2 h = T.sc[leaf];
    const bool act = leaf_lane && T.leaf_active[leaf] != 0;
    const uint32_t tg = (uint32_t)lane < ntask ? tgid[ci.t0 + lane] : 0u;
    // every task's disc in one gather (lane j: task j); (sin, cos) of
    // (r_s + guard) / 2 by the same expressions as the rest of the binning
    // (identical decisions)
    const float4 dl = (uint32_t)lane < ntask ? disc[tg] : make_float4(0.f, 0.f, 0.f, 0.f);
    float sgl = dl.w;
    float cgl = sqrtf(fmaxf(0.f, 1.f - sgl * sgl));
    widen_half(T.wsin, T.wcos, &sgl, &cgl);
    __builtin_amdgcn_wave_barrier();  // the previous chunk's reads are done
    s_disc[wv][lane] = make_float4(dl.x, dl.y, dl.z, sgl);
    s_cg[wv][lane] = cgl;
    __builtin_amdgcn_wave_barrier();
    // tasks far from the antipodal case for every leaf of the node, as a wave
    // mask: groups of such tasks take the near test (hp_cap_test_near),
    // which decides alike; a Gaussian whose disc covers nearly the whole
    // sphere keeps the full test
    const float srl = hp_wave_max(h.x);
    const uint64_t nearmask = __builtin_amdgcn_ballot_w64(!((uint32_t)lane < ntask) || cgl > srl + kNearMargin);
    // A task's decisions are a wave mask (one lane per leaf); every lane shifts its
    // bit into its column with one add-with-carry, W = 2 W + bit (as a select and an
    // or it took two and a half instructions a task, of 12.5). After r groups
    // the last task of a half stands at bit 0 and the first at bit 8 r - 1.
    uint32_t Wh[2] = {0u, 0u};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const uint32_t jend = ntask < 32u * (half + 1) ? ntask : 32u * (half + 1);
      uint32_t w = 0u, j0 = 32u * half;
      for (; j0 < jend; j0 += kFineGroup) {
        // entries past the chunk's end are read too (stale or zero LDS, in
        // bounds) and their bits dropped, so the reads take fixed offsets
        auto group = [&](auto near_tag) {
          constexpr bool NEAR = decltype(near_tag)::value;
          float ux[kFineGroup], uy[kFineGroup], uz[kFineGroup], sg[kFineGroup], cg[kFineGroup];
#pragma unroll
          for (int q = 0; q < kFineGroup; ++q) {
            const float4 d = s_disc[wv][j0 + q];  // same address on every lane: a broadcast
            ux[q] = d.x; uy[q] = d.y; uz[q] = d.z; sg[q] = d.w;
            cg[q] = s_cg[wv][j0 + q];
          }
          uint64_t in[kFineGroup];
#pragma unroll
          for (int q = 0; q < kFineGroup; ++q)
            in[q] = __builtin_amdgcn_ballot_w64(
                NEAR ? hp_cap_test_near(cx, cy, cz, h.x, h.y, ux[q], uy[q], uz[q], sg[q], cg[q])
                     : hp_cap_test(cx, cy, cz, h.x, h.y, ux[q], uy[q], uz[q], sg[q], cg[q]));
          shift_in_bits(&w, in);
        };
        if (((nearmask >> j0) & 0xffull) == 0xffull)
          group(std::true_type{});
        else
          group(std::false_type{});
      }
      // task 32 half + j to bit j, bits past the chunk's end dropped
      const uint32_t done = j0 - 32u * half, cnt_h = jend - 32u * half;
      if (done != 0u) Wh[half] = (__builtin_bitreverse32(w) >> (32u - done)) & (~0u >> (32u - cnt_h));
    }
    const uint64_t W = act ? ((uint64_t)Wh[1] << 32) | Wh[0] : 0ull;
    if (leaf_lane) {
      wcol[(int64_t)c * 64 + lane] = W;
      const int64_t flat = (int64_t)(c - ci.local) * nleaf + (int64_t)lane * ci.nchn + ci.local;
      cnt[flat] = (uint32_t)__popcll(W);
    }
  }
}

// Per chunk: every hit of leaf b's column goes to its slot in tile (node, b).
// The chunk's hits are numbered in (leaf, task) order: column lane b lists
// its hits (column and task, lowest task first) in LDS at their numbers,
// and the wave then writes 64 of them per store, lane k taking hit o + k,
// whose rank in its column gives the slot.  So each store instruction is
// full (the slots of one column are consecutive), where a store per column
// would carry ~10 lanes.
// Bound by LDS round trips and, on long lists, by the 4 B written per pair:
// 73 -> 68 us (full sphere, order 9, 1M Gaussians) and 100 -> 95 us (pinhole of 60
// degrees, order 11, 3M, some 75M pairs) with 32-bit slots; listing the hits in
// windows of 1,024, for twice the workgroups per CU, measured 76 and 124 us.
constexpr int kMaxChunkHits = 64 * 64;

// (start, end) of every active tile from the scanned column counts; the end
// of the last tile of the last node is the total.  When nothing is emitted
// (the pairs exceed the capacity, or the count has not completed) every
// range is empty, so that a render over them reads no list entry.  Written
// by the emission kernel's threads, strided over its grid.
struct TileRanges {
  int32_t n_tiles;
  const int32_t* active_tiles;
  const uint64_t* ncol;   // (chunk, leaf) count entries
  const uint64_t* total;  // pairs
  uint32_t* ranges;
};
__device__ __forceinline__ void write_tile_ranges(const TileRanges& R, int depth, const uint32_t* __restrict__ choff,
                                                  const uint32_t* __restrict__ start, bool none) {
  const int nleaf = 1 << (2 * depth);
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < R.n_tiles;
       k += (int64_t)gridDim.x * blockDim.x) {
    if (none) {
      R.ranges[2 * k] = 0u;
      R.ranges[2 * k + 1] = 0u;
      continue;
    }
    const int t = R.active_tiles[k];
    const uint32_t n = (uint32_t)t >> (2 * depth), b = (uint32_t)t & (uint32_t)(nleaf - 1);
    const int64_t c0 = choff[n], nchn = (int64_t)choff[n + 1] - c0;
    const uint64_t nc = *R.ncol;
    const uint64_t i0 = (uint64_t)(c0 * nleaf + b * nchn), i1 = (uint64_t)(c0 * nleaf + (b + 1) * nchn);
    R.ranges[2 * k] = i0 < nc ? start[i0] : (uint32_t)*R.total;
    R.ranges[2 * k + 1] = i1 < nc ? start[i1] : (uint32_t)*R.total;
  }
}

__global__ __launch_bounds__(256) void k_bin_emit_sorted(const uint32_t* __restrict__ choff, uint32_t nn,
                                                         const uint32_t* __restrict__ seg,
                                                         const uint32_t* __restrict__ cnode,
                                                         const uint32_t* __restrict__ tgid, int depth,
                                                         const uint64_t* __restrict__ wcol,
                                                         const uint32_t* __restrict__ start,
                                                         const int64_t* __restrict__ n_pairs, int64_t capacity,
                                                         uint32_t* __restrict__ vals, TileRanges tr) {
  const bool none = *n_pairs > capacity;
  write_tile_ranges(tr, depth, choff, start, none);
  if (none) return;
  __shared__ uint32_t s_g[4][64], s_slot[4][64];  // slot of column b's hit number k: s_slot[b] + k
  __shared__ uint16_t s_hit[4][kMaxChunkHits];    // column << 8 | task of every hit number
  const uint32_t nchunks = hp_uniform(((hp_cu32p)choff)[nn]);
  const int lane = hp_lane();
  const int wv = threadIdx.x >> 6;
  const int nleaf = 1 << (2 * depth);
  const bool leaf_lane = lane < nleaf;
  const ChunkRange cr = xcd_chunks(nchunks);
  // a chunk's columns, output slots and Gaussian ids
  auto fetch = [&](uint32_t c, uint64_t* W, uint32_t* base, uint32_t* g) {
    const ChunkInfo ci = chunk_info(choff, seg, cnode, c);
    *W = leaf_lane ? wcol[(int64_t)c * 64 + lane] : 0ull;
    *base = leaf_lane ? start[(int64_t)(c - ci.local) * nleaf + (int64_t)lane * ci.nchn + ci.local] : 0u;
    *g = (uint32_t)lane < ci.ntask ? tgid[ci.t0 + lane] : 0u;
  };
  uint32_t c = cr.first;
  if (c >= cr.end) return;
  uint64_t W;
  uint32_t base, g;
  fetch(c, &W, &base, &g);
  while (true) {
    // the next chunk's loads go out before this chunk's stores
    const uint32_t cn = c + cr.stride;
    const bool more = cn < cr.end;
    uint64_t Wn = 0ull;
    uint32_t basen = 0u, gn = 0u;
    if (more) fetch(cn, &Wn, &basen, &gn);
    const uint32_t cnt = (uint32_t)__popcll(W);
    const uint32_t incl = hpsort::wave_inclusive<uint32_t>(cnt);
    const uint32_t off = incl - cnt;
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    s_g[wv][lane] = g;
    s_slot[wv][lane] = base - off;
    // column lane b: its hits at numbers off, off + 1, ... (every number
    // below tot written once)
    {
      uint64_t w = W;
      const uint32_t col = (uint32_t)lane << 8;
      for (uint32_t r = off; w != 0; ++r) {
        s_hit[wv][r] = (uint16_t)(col | (uint32_t)__builtin_ctzll(w));
        w &= w - 1;
      }
    }
    __builtin_amdgcn_wave_barrier();
    for (uint32_t k = (uint32_t)lane; k < tot; k += 64) {
      const uint32_t e = s_hit[wv][k];
      vals[s_slot[wv][e >> 8] + k] = s_g[wv][e & 0xffu];
    }
    __builtin_amdgcn_wave_barrier();  // this chunk's LDS reads are done
    if (!more) break;
    c = cn;
    W = Wn;
    base = basen;
    g = gn;
  }
}

// number of (chunk, leaf) count entries: chunks x leaves per node
__global__ void k_col_count(const uint32_t* __restrict__ choff, uint32_t nn, int depth, uint64_t* __restrict__ ncol) {
  *ncol = (uint64_t)choff[nn] << (2 * depth);
}

__global__ void k_store_zero(int64_t* n_pairs) { *n_pairs = 0; }

// one wave per 64 tasks, at most 8192 blocks of 4 waves that loop over them
static unsigned fine_grid(int64_t nt) {
  const int64_t blocks = ((nt + 63) / 64 + 3) / 4;
  return (unsigned)(blocks < 8192 ? (blocks > 0 ? blocks : 1) : 8192);
}

// First pass of the depth sort: the digit histogram of the depths' bits
// (positive floats order as unsigned ints).  Culled Gaussians (depth +inf)
// and, with the mask's cone (hp_cone.h, widened like every test angle), those
// whose disc stays clear of it have no task and are left out of the order: a 60-degree pinhole keeps an eighth of a scene
// around it, and the later passes and the walk see only those (3M Gaussians
// seen by a 60-degree pinhole at Nside 2048: the forward view 1516 us, 1963 us
// when every Gaussian was sorted and walked).  A full-sphere camera has no
// cone, since every Gaussian would pass.  The cone's pass also writes the
// keys, so that the scatter drops the same Gaussians.  Bound by HBM: 4 B read
// per Gaussian, 24 B read and written with a cone.
// Also marks the count unfinished (see depth_order) and empties the walk's
// overflow part.
constexpr uint32_t kNoDepth = 0x7f800000u;  // +inf
// (sin, cos) of half the mask's cone, widened; (1, 0), which every disc
// passes, for a mask without one
__device__ __forceinline__ void read_cone(const float* __restrict__ cone, float wsin, float wcos, float* sr,
                                          float* cr) {
  if (__float_as_uint(cone[2]) != kConeMark) return;
  *sr = cone[0];
  *cr = cone[1];
  widen_half(wsin, wcos, sr, cr);
}
template <bool CONE>
__global__ __launch_bounds__(256) void k_depth_hist(const uint32_t* depth, const float4* __restrict__ disc, int64_t P,
                                                    const float* __restrict__ cone, float wsin, float wcos,
                                                    uint32_t* keys, uint32_t* __restrict__ hist,
                                                    int64_t* __restrict__ n_pairs, uint64_t* __restrict__ n_over) {
  __shared__ uint32_t s_h[256];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *n_pairs = INT64_MAX;
    *n_over = 0ull;
  }
  s_h[threadIdx.x] = 0u;
  __syncthreads();
  float sr = 1.f, cr = 0.f;
  if (CONE) read_cone(cone, wsin, wcos, &sr, &cr);
  int64_t t0, t1;
  hpsort::block_tiles(P, &t0, &t1, hpsort::kRadixTile);
  constexpr int kPer = hpsort::kRadixTile / 256;
  for (int64_t t = t0; t < t1; ++t) {
    uint32_t key[kPer];
    float4 d[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const int64_t i = t * hpsort::kRadixTile + r * 256 + threadIdx.x;
      key[r] = i < P ? depth[i] : kNoDepth;
      if (CONE) d[r] = i < P ? disc[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      if (CONE) {
        const int64_t i = t * hpsort::kRadixTile + r * 256 + threadIdx.x;
        const float cg = sqrtf(fmaxf(0.f, 1.f - d[r].w * d[r].w));
        if (!hp_cap_test(0.f, 0.f, 1.f, sr, cr, d[r].x, d[r].y, d[r].z, d[r].w, cg)) key[r] = kNoDepth;
        if (i < P) keys[i] = key[r];
      }
      if (key[r] < kNoDepth) atomicAdd(&s_h[key[r] & 255u], 1u);
    }
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = s_h[threadIdx.x];
}

// Depth order of at most kSmallSort Gaussians in one workgroup: the same keys,
// the same ones left out and, digit by digit and stable like the passes of
// radix_sort, the same order.  Twelve launches become one, which is what a
// small scene waits for: 2,000 Gaussians took 48 us of kernels, with a gap of
// some microseconds after each, and take 11.6 us; at 8,192 it is 31 us against
// 52, and one compute unit gains nothing on the whole chip beyond about that.
// Bound by one workgroup's chain of LDS round trips.
// Wave w holds the items [w 64 ipt, (w + 1) 64 ipt), lane l its items l, l + 64, ...:
// an item's place is that of its digit, of the waves before, of the rounds before
// and of the lanes before with the same digit.
constexpr int kSmallIpt = 8, kSmallSort = 1024 * kSmallIpt;
template <bool CONE>
__global__ __launch_bounds__(1024) void k_depth_sort_small(const uint32_t* __restrict__ depth,
                                                           const float4* __restrict__ disc, int P,
                                                           const float* __restrict__ cone, float wsin, float wcos,
                                                           uint32_t* __restrict__ order, uint64_t* __restrict__ n_live,
                                                           int64_t* __restrict__ n_pairs,
                                                           uint64_t* __restrict__ n_over) {
  __shared__ uint32_t s_key[kSmallSort];
  __shared__ uint16_t s_id[kSmallSort];
  __shared__ uint32_t s_cnt[16][256];  // per wave and digit
  __shared__ uint32_t s_base[256], s_w[4], s_live;
  const int tid = threadIdx.x, lane = hp_lane(), wv = (int)hp_uniform((uint32_t)tid >> 6);
  const int ipt = (P + 1023) / 1024, at0 = wv * 64 * ipt + lane;
  const uint64_t below = (1ull << lane) - 1ull;
  if (tid == 0) {
    *n_pairs = INT64_MAX;
    *n_over = 0ull;
    s_live = 0u;
  }
  float sr = 1.f, cr = 0.f;
  if (CONE) read_cone(cone, wsin, wcos, &sr, &cr);
  __syncthreads();
  uint32_t key[kSmallIpt], id[kSmallIpt];
#pragma unroll
  for (int r = 0; r < kSmallIpt; ++r) {
    if (r >= ipt) break;
    const int i = at0 + 64 * r;
    uint32_t k = i < P ? depth[i] : kNoDepth;
    if (CONE && i < P) {
      const float4 d = disc[i];
      const float cg = sqrtf(fmaxf(0.f, 1.f - d.w * d.w));
      if (!hp_cap_test(0.f, 0.f, 1.f, sr, cr, d.x, d.y, d.z, d.w, cg)) k = kNoDepth;
    }
    const bool live = k < kNoDepth;
    key[r] = live ? k : ~0u;  // behind every live one after the last digit
    id[r] = (uint32_t)i;
    const uint64_t m = __builtin_amdgcn_ballot_w64(live);
    if (lane == 0) atomicAdd(&s_live, (uint32_t)__builtin_popcountll(m));
  }
#pragma unroll 1
  for (int shift = 0; shift < 32; shift += 8) {
    for (int i = tid; i < 16 * 256; i += 1024) (&s_cnt[0][0])[i] = 0u;
    __syncthreads();
    uint32_t rank[kSmallIpt];
#pragma unroll
    for (int r = 0; r < kSmallIpt; ++r) {
      if (r >= ipt) break;
      const uint32_t dg = key[r] >> shift & 255u;
      uint64_t same = ~0ull;
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const bool on = (dg >> b & 1u) != 0u;
        const uint64_t m = __builtin_amdgcn_ballot_w64(on);
        same &= on ? m : ~m;
      }
      const uint32_t before = s_cnt[wv][dg];
      rank[r] = before + (uint32_t)__builtin_popcountll(same & below);
      __builtin_amdgcn_wave_barrier();  // every lane has read the count
      if ((same & below) == 0) s_cnt[wv][dg] = before + (uint32_t)__builtin_popcountll(same);
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (tid < 256) {  // digit tid: its counts of the waves before, and of the digits before
      uint32_t sum = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        const uint32_t c = s_cnt[w][tid];
        s_cnt[w][tid] = sum;
        sum += c;
      }
      const uint32_t incl = hpsort::wave_inclusive<uint32_t>(sum);
      s_base[tid] = incl - sum;
      if (lane == 63) s_w[wv] = incl;
    }
    __syncthreads();
    const uint32_t w0 = s_w[0], w1 = w0 + s_w[1], w2 = w1 + s_w[2];
#pragma unroll
    for (int r = 0; r < kSmallIpt; ++r) {
      if (r >= ipt) break;
      const uint32_t dg = key[r] >> shift & 255u, q = dg >> 6;
      const uint32_t pos = rank[r] + s_cnt[wv][dg] + s_base[dg] + (q == 0u ? 0u : (q == 1u ? w0 : (q == 2u ? w1 : w2)));
      s_key[pos] = key[r];
      s_id[pos] = (uint16_t)id[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSmallIpt; ++r) {
      if (r >= ipt) break;
      key[r] = s_key[at0 + 64 * r];
      id[r] = s_id[at0 + 64 * r];
    }
  }
  const int n = (int)s_live;
#pragma unroll
  for (int r = 0; r < kSmallIpt; ++r)
    if (r < ipt && at0 + 64 * r < n) order[at0 + 64 * r] = id[r];
  if (tid == 0) *n_live = (uint64_t)n;
}

// Depth order (shared by both emissions): w.order holds the ids of the
// *w.n_live Gaussians that can have a task, by increasing radial depth.  Its
// first kernel also sets *n_pairs = INT64_MAX: until the count completes, the
// count says that nothing may be emitted.
// cone: the mask's, or null to keep every Gaussian that was not culled.
static hp_status depth_order(const HpProjView& pv, int64_t P, const float* cone, const BinTables& T, BinWs& w,
                             int64_t* n_pairs, hipStream_t s) {
  const uint32_t* depth = reinterpret_cast<const uint32_t*>(pv.depth);
  if (P <= kSmallSort) {
    if (cone)
      hipLaunchKernelGGL(k_depth_sort_small<true>, dim3(1), dim3(1024), 0, s, depth, pv.disc, (int)P, cone, T.wsin,
                         T.wcos, w.order, w.n_live, n_pairs, w.n_over);
    else
      hipLaunchKernelGGL(k_depth_sort_small<false>, dim3(1), dim3(1024), 0, s, depth, pv.disc, (int)P, cone, T.wsin,
                         T.wcos, w.order, w.n_live, n_pairs, w.n_over);
    HP_CHECK_LAUNCH();
    return HP_OK;
  }
  uint32_t* hist = hpsort::radix_hist_ptr(w.sort_ws, P);
  const dim3 grid(hpsort::radix_grid(P));
  if (cone)
    hipLaunchKernelGGL(k_depth_hist<true>, grid, dim3(256), 0, s, depth, pv.disc, P, cone, T.wsin, T.wcos, w.dkey, hist,
                       n_pairs, w.n_over);
  else
    hipLaunchKernelGGL(k_depth_hist<false>, grid, dim3(256), 0, s, depth, pv.disc, P, cone, T.wsin, T.wcos, w.dkey, hist,
                       n_pairs, w.n_over);
  HP_CHECK_LAUNCH();
  const hpsort::RadixFirst first{cone ? w.dkey : depth, kNoDepth, w.n_live};
  return hpsort::radix_sort(w.dkey, w.order, nullptr, P, 32, w.sort_ws, s, nullptr, nullptr, &first);
}

// Depth order, coarse walk and task list: tasks (Gaussian, node at the split
// level) in order of radial depth; *w.nt holds their number and *w.over
// whether they exceeded the workspace's capacity.
static hp_status bin_tasks(const HpProjView& pv, int64_t P, const float* cone, const BinTables& T, float guard,
                           BinWs& w, uint32_t* slots, int64_t* n_pairs, hipStream_t s) {
  HP_TRY(depth_order(pv, P, cone, T, w, n_pairs, s));
  hipLaunchKernelGGL((k_bin_coarse<false>), dim3(hp_blocks(P, 256)), dim3(256), 0, s, P, (const uint64_t*)w.n_live,
                     (const uint32_t*)w.order, pv.disc, pv.radius,
                     T, guard, w.tcount, (const uint64_t*)nullptr, w.cap_t, (uint32_t*)nullptr, (uint32_t*)nullptr,
                     slots);
  HP_CHECK_LAUNCH();
  HP_TRY((hpsort::scan_exclusive<uint64_t, uint32_t>(w.tcount, w.toff, w.n_live, P, w.t_total, w.scan_ws, s)));
  hipLaunchKernelGGL(k_task_clamp, dim3(1), dim3(1), 0, s, (const uint64_t*)w.t_total, w.cap_t, w.nt, w.over);
  HP_CHECK_LAUNCH();
  hipLaunchKernelGGL((k_bin_coarse<true>), dim3(hp_blocks(P, 256)), dim3(256), 0, s, P, (const uint64_t*)w.n_live,
                     (const uint32_t*)w.order, pv.disc, pv.radius,
                     T, guard, w.tcount, (const uint64_t*)w.toff, w.cap_t, w.task_g, w.task_n, slots);
  HP_CHECK_LAUNCH();
  return HP_OK;
}

extern "C" size_t hp_bin_workspace_bytes(int64_t P) { return P < 0 ? 0 : bin_ws_size(P) + 256; }

extern "C" hp_status hp_bin(int32_t phase, const void* projected, int64_t P, const hp_view* view, const hp_params* prm,
                            const void* grid, const void* mask, uint32_t* keys, uint32_t* vals, int64_t capacity,
                            int64_t* n_pairs, void* ws, size_t ws_bytes, void* stream) {
  if (phase < HP_BIN_COUNT || phase > HP_BIN_ALL) return HP_ERR_INVALID_ARG;
  HP_TRY(hp_check_view(view, prm));
  if (P < 0 || P > ((int64_t)1 << 31) - 1 || capacity < 0) return HP_ERR_INVALID_ARG;
  if (!projected || !grid || !mask || !n_pairs || !ws) return HP_ERR_INVALID_ARG;
  if ((phase & HP_BIN_EMIT) && capacity > 0 && (!keys || !vals)) return HP_ERR_INVALID_ARG;
  if (ws_bytes < bin_ws_size(P)) return HP_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  const HpGeom g = hp_geom(view->order, prm->tile_log2);
  const HpProjView pv = hp_proj_view((const char*)projected, P);
  const HpGridView gv = hp_grid_view((void*)grid, g);
  const HpMaskView mv = hp_mask_view((const char*)mask, g);
  BinWs w = bin_ws(ws, P);
  const int ls = g.kt > kSplitDepth ? g.kt - kSplitDepth : 0;
  BinTables T{gv.cap, gv.sc, view->cam_type == HP_CAM_FULL ? nullptr : mv.node_active, mv.node_active,
              mv.tile_compact, g.kt, ls, 0.f, 1.f};
  if (phase & HP_BIN_COUNT) {
    if (P == 0) {
      hipLaunchKernelGGL(k_store_zero, dim3(1), dim3(1), 0, s, n_pairs);
      HP_CHECK_LAUNCH();
      return HP_OK;
    }
    HP_TRY(bin_tasks(pv, P, nullptr, T, prm->bin_guard, w, nullptr, n_pairs, s));
    // per task: its 64-bit hit mask and count; the counts scanned into offsets
    hipLaunchKernelGGL(k_bin_fine_count, dim3(fine_grid(w.cap_t)), dim3(256), 0, s, (const uint64_t*)w.nt, w.cap_t,
                       w.task_g, w.task_n, pv.disc, T, w.pmask, w.pcount);
    HP_CHECK_LAUNCH();
    // the pair total goes to *n_pairs with the scan (a count no buffer holds
    // when the tasks overflowed: the emission kernels then write nothing)
    HP_TRY((hpsort::scan_exclusive<uint64_t, uint32_t>(w.pcount, w.poff, w.nt, w.cap_t, w.p_total, w.scan_ws, s,
                                                       n_pairs, (const uint32_t*)w.over)));
  }
  if ((phase & HP_BIN_EMIT) && P > 0) {
    // the task count is read on the device; the grid covers the capacity bound
    hipLaunchKernelGGL(k_bin_fine_emit, dim3(fine_grid(w.cap_t)), dim3(256), 0, s, (const uint64_t*)w.nt, w.cap_t,
                       w.task_g, w.task_n, T, (const uint64_t*)w.pmask, (const uint64_t*)w.poff, n_pairs, capacity,
                       keys, vals);
    HP_CHECK_LAUNCH();
  }
  return HP_OK;
}

// ---- sorted emission: workspace and entry point -----------------------------
struct SortedWs {
  void* tsort_ws;    // radix sort of the tasks by node
  uint32_t* seg;     // [nn][2] task segment of every node
  uint32_t* nch;     // [nn] chunks per node
  uint32_t* choff;   // [nn + 1] first chunk of every node, total last
  uint32_t* cnt;     // [L] hits per (chunk, leaf), tile-major
  uint32_t* start;   // [L] exclusive scan of cnt: first output slot, modulo 2^32 (a list that long is not emitted)
  uint64_t* wcol;    // [nchunk_max][64] hit columns
  uint32_t* slots;   // [kSlots][P] first task nodes of every Gaussian (coarse walk)
  uint32_t* cnode;   // [nchunk_max] node of every chunk
  void* scan_ws;
  int64_t nn, nchunk_max, L;
};

static void sorted_dims(int64_t P, const HpGeom& g, int64_t* nn, int64_t* nchunk_max, int64_t* L) {
  const int ls = g.kt > kSplitDepth ? g.kt - kSplitDepth : 0;
  const int depth = g.kt - ls;
  *nn = 12ll << (2 * ls);
  *nchunk_max = task_capacity(P) / 64 + *nn + 1;
  *L = *nchunk_max * (1ll << (2 * depth));
}

static size_t sorted_ws_size(int64_t P, const HpGeom& g) {
  int64_t nn, ncm, L;
  sorted_dims(P, g, &nn, &ncm, &L);
  return hpsort::radix_ws_bytes(task_capacity(P)) + hp_align256(nn * 8) + hp_align256(nn * 4) +
         hp_align256((nn + 1) * 4) + hp_align256(L * 4) + hp_align256(L * 4) + hp_align256(ncm * 64 * 8) +
         hp_align256((size_t)kSlots * P * 4) + hp_align256((size_t)ncm * 4) +
         hpsort::scan_ws_bytes<uint64_t>(L > nn ? L : nn);
}

static SortedWs sorted_ws(void* base, int64_t P, const HpGeom& g) {
  SortedWs w;
  sorted_dims(P, g, &w.nn, &w.nchunk_max, &w.L);
  char* p = (char*)base;
  w.tsort_ws = p; p += hpsort::radix_ws_bytes(task_capacity(P));
  w.seg = (uint32_t*)p; p += hp_align256(w.nn * 8);
  w.nch = (uint32_t*)p; p += hp_align256(w.nn * 4);
  w.choff = (uint32_t*)p; p += hp_align256((w.nn + 1) * 4);
  w.cnt = (uint32_t*)p; p += hp_align256(w.L * 4);
  w.start = (uint32_t*)p; p += hp_align256(w.L * 4);
  w.wcol = (uint64_t*)p; p += hp_align256(w.nchunk_max * 64 * 8);
  w.slots = (uint32_t*)p; p += hp_align256((size_t)kSlots * P * 4);
  w.cnode = (uint32_t*)p; p += hp_align256((size_t)w.nchunk_max * 4);
  w.scan_ws = p;
  return w;
}

extern "C" size_t hp_bin_sorted_workspace_bytes(int64_t P, int32_t order, int32_t tile_log2) {
  if (P < 0 || order < 0 || order > HP_MAX_ORDER || tile_log2 < 0 || tile_log2 > 4) return 0;
  const HpGeom g = hp_geom(order, tile_log2);
  return bin_ws_size(P) + sorted_ws_size(P, g) + 512;
}

// one wave per chunk, at most kChunkBlocks blocks of 4 waves looping over the
// chunks (measured on config 2: 8192 blocks beat one resident round of 2048)
constexpr int64_t kChunkBlocks = 8192;
static unsigned chunk_grid(int64_t nchunks) {
  const int64_t blocks = (nchunks + 3) / 4;
  return (unsigned)(blocks < kChunkBlocks ? (blocks > 0 ? blocks : 1) : kChunkBlocks);
}

// The sorted emission with every Gaussian's test angle widened by `widen`
// radians (0: the binning of hp_bin_sorted).  No step waits for the host:
// every count that sizes a later step is read on the device, and the grids
// are sized from the workspace's bounds.
hp_status hp_bin_sorted_widened(int32_t phase, const void* projected, int64_t P, const hp_view* view,
                                const hp_params* prm, const void* grid, const void* mask, uint32_t* vals,
                                uint32_t* tile_ranges, int32_t n_tiles, int64_t capacity, int64_t* n_pairs, void* ws,
                                size_t ws_bytes, void* stream, double widen) {
  if (phase < HP_BIN_COUNT || phase > HP_BIN_ALL) return HP_ERR_INVALID_ARG;
  HP_TRY(hp_check_view(view, prm));
  if (P < 0 || P > ((int64_t)1 << 31) - 1 || capacity < 0 || capacity > ((int64_t)1 << 32) - 1 || n_tiles < 0)
    return HP_ERR_INVALID_ARG;
  if (!projected || !grid || !mask || !n_pairs || !ws) return HP_ERR_INVALID_ARG;
  if ((phase & HP_BIN_EMIT) && ((capacity > 0 && !vals) || (n_tiles > 0 && !tile_ranges))) return HP_ERR_INVALID_ARG;
  const HpGeom g = hp_geom(view->order, prm->tile_log2);
  if (n_tiles > g.ntile) return HP_ERR_INVALID_ARG;
  if (ws_bytes < hp_bin_sorted_workspace_bytes(P, view->order, prm->tile_log2)) return HP_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  const HpProjView pv = hp_proj_view((const char*)projected, P);
  const HpGridView gv = hp_grid_view((void*)grid, g);
  const HpMaskView mv = hp_mask_view((const char*)mask, g);
  BinWs w = bin_ws(ws, P);
  SortedWs sw = sorted_ws((char*)ws + hp_align256(bin_ws_size(P)), P, g);
  const int ls = g.kt > kSplitDepth ? g.kt - kSplitDepth : 0;
  const int depth = g.kt - ls;
  BinTables T{gv.cap, gv.sc, view->cam_type == HP_CAM_FULL ? nullptr : mv.node_active, mv.node_active,
              mv.tile_compact, g.kt, ls, (float)sin(0.5 * widen), (float)cos(0.5 * widen)};
  const uint32_t nn = (uint32_t)sw.nn;
  const float* cone = view->cam_type == HP_CAM_FULL ? nullptr : mv.cone;
  if (phase & HP_BIN_COUNT) {
    if (P == 0) {
      hipLaunchKernelGGL(k_store_zero, dim3(1), dim3(1), 0, s, n_pairs);
      HP_CHECK_LAUNCH();
      return HP_OK;
    }
    // until the count below completes, *n_pairs says that nothing may be
    // emitted (set by the depth sort's first kernel)
    if (sw.nn <= kListNodes) {
      // tasks written in node order straight from the walk (no task sort).
      // Buffers that this path does not otherwise use hold its tables: the
      // histogram in task_n (nn x G <= 12 (P + 255) <= task capacity), its row
      // scans, the node totals and offsets in poff, the staged runs in the
      // task sort's workspace (4096 tasks per 256 Gaussians, 16 P + 4080 <=
      // task capacity), their overflow in wcol (6 of its 8 B per task) and
      // their counts in pmask.
      HP_TRY(depth_order(pv, P, cone, T, w, n_pairs, s));
      const unsigned G = hp_blocks(P, 256);
      const int nni = (int)sw.nn;
      const unsigned groups = (unsigned)((nni + kWalkGroup - 1) / kWalkGroup);
      uint32_t* hist = w.task_n;
      uint32_t* hoff = (uint32_t*)w.poff;
      uint64_t* rowtot = w.poff + ((int64_t)nni * G + 1) / 2;
      uint64_t* node_off = rowtot + nni;
      TaskStage st;
      st.g = (uint32_t*)sw.tsort_ws;
      st.n = (uint16_t*)(st.g + w.cap_t);
      st.og = (uint32_t*)sw.wcol;
      st.on = (uint16_t*)(st.og + w.cap_t);
      st.obase = w.pmask;
      st.cnt = (uint32_t*)(w.pmask + (int64_t)G * groups);
      st.ocount = w.n_over;
      st.ocap = w.cap_t;
      st.fixed = kStageFixed / (int)groups;
      const dim3 wg(walk_grid(G, nni <= kWalkSmall ? kWalkGridSmall : kWalkGrid), groups), pg(walk_grid(G, kPlaceGrid), groups);
      if (nni <= kWalkSmall)
        hipLaunchKernelGGL(k_task_walk<kWalkSmall>, wg, dim3(256), 0, s, (const uint64_t*)w.n_live,
                           (const uint32_t*)w.order, pv.disc, T, nni, (int64_t)G, hist, st);
      else
        hipLaunchKernelGGL(k_task_walk<kWalkGroup>, wg, dim3(256), 0, s, (const uint64_t*)w.n_live,
                           (const uint32_t*)w.order, pv.disc, T, nni, (int64_t)G, hist, st);
      HP_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_hist_rows, dim3(nni), dim3(256), 0, s, (const uint32_t*)hist, (int64_t)G,
                         (const uint64_t*)w.n_live, T.node_active ? T.node_active + hp_level_offset(ls) : nullptr, hoff,
                         rowtot);
      HP_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_task_segments, dim3(1), dim3(256), 0, s, nni, (const uint64_t*)rowtot, node_off, w.cap_t,
                         depth, w.t_total, w.nt, w.over, sw.seg, sw.choff, w.ncol);
      HP_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_task_place, pg, dim3(kPlaceThreads), 0, s, (const uint64_t*)w.n_live, nni, (int64_t)G, st, (const uint32_t*)hoff,
                         (const uint64_t*)node_off, w.cap_t, w.task_g, (const uint32_t*)sw.choff, sw.cnode);
      HP_CHECK_LAUNCH();
    } else {
      HP_TRY(bin_tasks(pv, P, cone, T, prm->bin_guard, w, sw.slots, n_pairs, s));
      // stable sort of the tasks by node; segments and chunk offsets per node
      int nbits = 0;
      while (((int64_t)1 << nbits) < sw.nn) ++nbits;
      // the sorted node keys are only needed here: read them where the last
      // pass left them; the Gaussian ids go back to task_g for the emit phase
      uint32_t *snode = w.task_n, *sgid = w.task_g;
      HP_TRY(hpsort::radix_sort(w.task_n, w.task_g, w.nt, w.cap_t, nbits, sw.tsort_ws, s, &snode, &sgid));
      if (sgid != w.task_g) {
        hipLaunchKernelGGL(hpsort::k_copy_u32, dim3(hpsort::copy_grid(w.cap_t)), dim3(256), 0, s, (const uint32_t*)sgid,
                           w.task_g, (const uint64_t*)w.nt, w.cap_t);
        HP_CHECK_LAUNCH();
      }
      hipLaunchKernelGGL(k_fill_zero_u32, dim3(hp_blocks(2 * sw.nn, 256)), dim3(256), 0, s, sw.seg, 2 * sw.nn);
      HP_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_seg_ranges, dim3(hpsort::copy_grid(w.cap_t)), dim3(256), 0, s, (const uint32_t*)snode,
                         (const uint64_t*)w.nt, nn, sw.seg);
      HP_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_seg_chunks, dim3(hp_blocks(sw.nn, 256)), dim3(256), 0, s, sw.seg, nn, sw.nch);
      HP_CHECK_LAUNCH();
      HP_TRY((hpsort::scan_exclusive<uint32_t, uint32_t>(sw.nch, sw.choff, nullptr, sw.nn, sw.choff + sw.nn, sw.scan_ws,
                                                         s)));
      // hit columns and their counts (every count entry of the chunks present
      // is written), scanned in tile-major order into output slots
      hipLaunchKernelGGL(k_col_count, dim3(1), dim3(1), 0, s, (const uint32_t*)sw.choff, nn, depth, w.ncol);
      HP_CHECK_LAUNCH();
      hipLaunchKernelGGL(k_chunk_nodes, dim3(nn), dim3(256), 0, s, (const uint32_t*)sw.choff, sw.cnode);
      HP_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(k_bin_cols, dim3(chunk_grid(sw.nchunk_max)), dim3(256), 0, s, (const uint32_t*)sw.choff, nn,
                       (const uint32_t*)sw.seg, (const uint32_t*)sw.cnode, (const uint32_t*)w.task_g, pv.disc, T,
                       sw.wcol, sw.cnt);
    HP_CHECK_LAUNCH();
    // the pair total goes to *n_pairs with the scan (a count no buffer holds
    // when the tasks overflowed: the emission kernels then write nothing)
    HP_TRY((hpsort::scan_exclusive<uint64_t, uint32_t, uint32_t>(sw.cnt, sw.start, w.ncol, sw.L, w.p_total, sw.scan_ws, s,
                                                       n_pairs, (const uint32_t*)w.over)));
  }
  if ((phase & HP_BIN_EMIT) && P > 0) {
    // the chunk count is read on the device: launch for the workspace's bound
    // the emission also writes the tile ranges
    const TileRanges tr{n_tiles, mv.active_tiles, (const uint64_t*)w.ncol, (const uint64_t*)w.p_total, tile_ranges};
    hipLaunchKernelGGL(k_bin_emit_sorted, dim3(chunk_grid(sw.nchunk_max)), dim3(256), 0, s, (const uint32_t*)sw.choff,
                       nn, (const uint32_t*)sw.seg, (const uint32_t*)sw.cnode, (const uint32_t*)w.task_g, depth,
                       (const uint64_t*)sw.wcol, (const uint32_t*)sw.start, (const int64_t*)n_pairs, capacity, vals, tr);
    HP_CHECK_LAUNCH();
  } else if ((phase & HP_BIN_EMIT) && n_tiles > 0) {
    hipLaunchKernelGGL(k_fill_zero_u32, dim3(hp_blocks(2 * (int64_t)n_tiles, 256)), dim3(256), 0, s, tile_ranges,
                       2 * (int64_t)n_tiles);
    HP_CHECK_LAUNCH();
  }
  return HP_OK;
}

extern "C" hp_status hp_bin_sorted(int32_t phase, const void* projected, int64_t P, const hp_view* view,
                                   const hp_params* prm, const void* grid, const void* mask, uint32_t* vals,
                                   uint32_t* tile_ranges, int32_t n_tiles, int64_t capacity, int64_t* n_pairs,
                                   void* ws, size_t ws_bytes, void* stream) {
  return hp_bin_sorted_widened(phase, projected, P, view, prm, grid, mask, vals, tile_ranges, n_tiles, capacity,
                               n_pairs, ws, ws_bytes, stream, 0.0);
}
