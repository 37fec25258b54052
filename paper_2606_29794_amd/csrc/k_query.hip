// k_query.hip -- the paper's own tile queries (Sec. 3.3; Alg. 2 NESTED
// quadtree traversal, Alg. 3 RING sequential scan) at search depth f, as
// per-tile lists for the renderer.
//
// Both queries decide on centres at the query order kq = kt + log2 f, so their
// tile sets are narrower than the binning of hp_bin_sorted and can leave out
// tiles a Gaussian reaches (the aliasing of coarse queries in the ablation).
// Instead of a ring walk or a stack per Gaussian, membership is evaluated tile
// by tile: Gaussian i's set holds tile t exactly when one of t's query points
// passes the test the query applies to it --
//   RING:   a pixel of order kq on a ring whose latitude lies within r_s of
//           the disc centre's, at a position inside the ring's window
//           [floor, ceil] of Eq. ring_phi_range (whole ring when the ring lies
//           inside the disc);
//   NESTED: a node of order kt .. kq whose centre lies within r_s (what the
//           traversal reports when PixRad bounds the distance from a node
//           centre to its descendants' centres at order kq).
// Candidates are the pairs of hp_bin_sorted with every test angle widened by a
// margin that contains both sets (one ring step for RING, plus the distance
// from a query point to the nearest pixel centre of its tile); they arrive in
// per-tile depth order, and one wave or workgroup per tile keeps the entries
// that pass, compacting the tile's list in place, so the order is preserved.
#include "hp_common.h"

namespace {

constexpr int kMaxPts = 341;    // nodes of orders kt .. kt + 4 below one tile
constexpr int kMaxRings = 31;   // rings crossing one tile at f = 16

struct QueryArgs {
  int mode, kq, fl, order_t;
  const int32_t* active_tiles;
  const float4* gauss;  // per Gaussian what the test reads (k_query_gauss)
  uint32_t* vals;
  uint32_t* ranges;
  const int64_t* n_pairs;
  int64_t capacity;
  unsigned long long* n_kept;
};

// ring ir (1 .. 4N-1 from the north pole) at order kq: latitude, its cosine,
// number of pixels and the offset (in pixels) of pixel 0's centre from
// longitude 0
__device__ void ring_geom(int64_t N, int64_t ir, double* lat, double* clat, int* nring, float* off) {
  const double s6 = 2.449489742783178;  // sqrt(6)
  if (ir < N || ir > 3 * N) {
    const int64_t i = ir < N ? ir : 4 * N - ir;
    const double th = 2.0 * asin((double)i / ((double)N * s6));  // 1 - |z| = 2 sin^2(theta / 2)
    *lat = ir < N ? 0.5 * M_PI - th : th - 0.5 * M_PI;
    *clat = sin(th);
    *nring = (int)(4 * i);
    *off = 0.5f;
  } else {
    const double z = (double)(2 * N - ir) * (2.0 / (3.0 * (double)N));
    *lat = asin(z);
    *clat = sqrt((1.0 - z) * (1.0 + z));
    *nring = (int)(4 * N);
    *off = ((ir - N) & 1) ? 0.f : 0.5f;
  }
}

// ring and 0-based position along it of nested pixel p at order kq
__device__ void pix_ring(int kq, int64_t p, int64_t* ring, int* pos, int* x_minus_y) {
  int x, y, f;
  hp_nest_xyf(kq, p, &x, &y, &f);
  const int64_t N = (int64_t)1 << kq;
  const int row = f >> 2, col = f & 3;
  const int64_t ir = (int64_t)(row + 2) * N - x - y - 1;
  const int64_t lon = (row == 1) ? 2 * col : 2 * col + 1;
  int64_t jp, nring;
  if (ir < N || ir > 3 * N) {
    const int64_t nr = ir < N ? ir : 4 * N - ir;
    jp = (lon * nr + x - y + 1) / 2;
    nring = 4 * nr;
  } else {
    const int64_t s = (ir - N) & 1;
    jp = (lon * N + x - y + 1 + s) / 2;
    nring = 4 * N;
  }
  if (jp > nring) jp -= nring;
  if (jp < 1) jp += nring;
  *ring = ir;
  *pos = (int)(jp - 1);
  *x_minus_y = x - y;
}

// One ring crossing a tile at the query order, for the RING test.  The
// tile's pixels on it are a run of positions; the window of Eq. ring_phi_range
// ([floor, ceil] of its ends in pixel units) holds pixel ip exactly when
// |omega - lambda_ip| < d_omega + step (lambda_ip its centre longitude, step
// = 2 pi / nring), so it meets the run exactly when the longitude distance
// from omega to the run's interval widened by one step on both sides,
// [lambda_first - step, lambda_last + step], is below d_omega.
struct RingSlot {
  float sh, ch;    // sin, cos of half the ring's latitude; (4, 0), outside every
                   // disc's z range, when the tile has no pixel on the ring
  float clat;      // cos of its latitude
  float sm, cm;    // sin, cos of half the widened interval's middle longitude
  float shw, chw;  // sin, cos of half its half-width; shw = 2, which holds every
                   // longitude, when it covers the ring
};

// RING membership of the tile for a Gaussian with direction u and
// hrs = sin^2(r_s / 2).  With hav x = sin^2(x / 2):
//   num = hav r_s - hav(lat_r - lat_c),  den = cos lat_c cos lat_r,
//   hav d_omega = num / den  (Eq. ring_phi_range in haversine form),
// so the ring lies in the disc's z range when |sin((lat_r - lat_c) / 2)| <=
// sin(r_s / 2), wholly inside the disc when num >= den, meets it nowhere when
// num <= 0, and otherwise the run is hit when den hav(distance) < num.  Every
// small angle enters as the sine of its half, formed as a difference of
// products of half-angle sines and cosines: no cancellation for small discs,
// and no transcendental per ring.
// The Gaussian's part of the test: cos(lat_c), (cos, sin) of half the latitude
// and of half the longitude of its centre, sin(r_s / 2) and its square.
struct RingGauss {
  float cc, sc, sw, cw, clat, srs, hrs;
};
__device__ __forceinline__ RingGauss ring_gauss(float4 disc, float rs) {
  RingGauss G;
  const float hs = sinf(0.5f * rs);
  G.hrs = hs * hs;
  G.srs = sqrtf(G.hrs);
  G.clat = sqrtf(fmaf(disc.x, disc.x, disc.z * disc.z));
  // half of the centre's latitude: its cosine is at least 1/sqrt(2)
  G.cc = sqrtf(fmaf(0.5f, G.clat, 0.5f));
  G.sc = disc.y / (2.f * G.cc);
  sincosf(0.5f * atan2f(disc.x, disc.z), &G.sw, &G.cw);
  return G;
}
// The lanes of the wave whose Gaussian hits the ring.  Predicates are combined
// as wave masks (single compares, scalar logic): as lane booleans they were
// materialised in registers, twice the vector instructions.
__device__ __forceinline__ uint64_t ring_hit(const RingSlot& r, const RingGauss& G) {
  const float sd = fmaf(r.sh, G.cc, -(r.ch * G.sc));  // sin((lat_r - lat_c) / 2)
  const float num = fmaf(-sd, sd, G.hrs);
  const float den = G.clat * r.clat;
  // y = |omega - middle| reduced to [0, pi]: sin(y / 2), cos(y / 2)
  const float a = fabsf(fmaf(G.sw, r.cm, -(G.cw * r.sm)));
  const float b = fabsf(fmaf(G.cw, r.cm, G.sw * r.sm));
  const float sdist = fmaf(a, r.chw, -(b * r.shw));  // sin((y - half-width) / 2)
  // in the disc's z range, and: the whole ring lies in the disc (also at the
  // poles), or the disc reaches it and the centre's longitude lies in the
  // widened interval or near enough to it
  return __builtin_amdgcn_ballot_w64(fabsf(sd) <= G.srs) &
         (__builtin_amdgcn_ballot_w64(num >= den) |
          (__builtin_amdgcn_ballot_w64(num > 0.f) &
           (__builtin_amdgcn_ballot_w64(a <= r.shw) | __builtin_amdgcn_ballot_w64(den * (sdist * sdist) < num))));
}

// What the filter reads of a Gaussian, once per Gaussian instead of once per
// (tile, Gaussian) candidate, of which there are some 49 to one: RING 32 B
// (RingGauss), NESTED 16 B (direction and squared chord of r_s).
template <int MODE>
__global__ __launch_bounds__(256) void k_query_gauss(int64_t P, const float4* __restrict__ disc,
                                                     const float* __restrict__ radius, float4* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  const float4 d = disc[i];
  const float rs = radius[i];
  if (MODE == HP_QUERY_NESTED) {
    const float c = 2.f * sinf(0.5f * rs);
    out[i] = make_float4(d.x, d.y, d.z, c * c);
  } else {
    const RingGauss G = ring_gauss(d, rs);
    out[2 * i] = make_float4(G.cc, G.sc, G.sw, G.cw);
    out[2 * i + 1] = make_float4(G.clat, G.srs, G.hrs, 0.f);
  }
}

// A wave filters a tile's list, kQueryIlp x 64 entries at a time (their gathers
// in flight together); the four waves of a workgroup take four neighbouring
// tiles, whose lists hold mostly the same Gaussians in the same order, so
// that part of the gathers meet in the CU's cache and no barrier orders the
// waves, or share one tile (SHARED, below).  1M Gaussians on the full sphere at Nside 512, RING x 4, 49M
// candidates: 619 us with a workgroup per tile and the trigonometry per
// candidate, 446 us with that done once per Gaussian, 351 us with predicates as
// wave masks and two lanes to a record.  Bound by the vector instructions of
// the ring tests (225 us of issue) and by the gathers.
constexpr int kQueryIlp = 4;
constexpr int kRingShared = 1024;  // RING: tiles up to which a workgroup takes one

// The 32-byte records of 64 list entries: two lanes fetch a record together,
// one 16-byte half each (a lane per record spent two cache accesses on it, and
// the accesses bound the kernel), and exchange halves with their neighbour.
// Even lanes end with entry lane / 2, odd lanes with entry 32 + lane / 2.
__device__ __forceinline__ float swap_pair(float v) { return hp_dpp<0xB1>(v); }  // lane ^ 1
__device__ __forceinline__ RingGauss pair_load(const float4* __restrict__ gauss, uint32_t ga, uint32_t gb, bool odd) {
  const float4 ha = gauss[2 * (int64_t)ga + (odd ? 1 : 0)], hb = gauss[2 * (int64_t)gb + (odd ? 1 : 0)];
  const float4 t = odd ? ha : hb;
  const float4 r = make_float4(swap_pair(t.x), swap_pair(t.y), swap_pair(t.z), 0.f);
  const float rw = swap_pair(t.w);
  RingGauss G;
  G.cc = odd ? r.x : ha.x;
  G.sc = odd ? r.y : ha.y;
  G.sw = odd ? r.z : ha.z;
  G.cw = odd ? rw : ha.w;
  G.clat = odd ? hb.x : r.x;
  G.srs = odd ? hb.y : r.y;
  G.hrs = odd ? hb.z : r.z;
  return G;
}

// SHARED: the four waves of a workgroup take one tile's list together, a batch
// of kQueryIlp x 64 entries each at a time.  A wave each leaves the chip idle
// where tiles are few, and waits for its gathers alone.  Views of 3M Gaussians
// with a wave and with a workgroup per tile: RING x 4 and 192 tiles 3617 and
// 1868 us, 768 tiles 1902 and 1328, 3,072 tiles 1679 and 1726 (RING x 1: 2453 and
// 2562); NESTED x 4, whose tests are short beside the gathers, 2768 and 1531 us
// at 192 tiles, 1521 and 1443 at 3,072, 2610 and 2492 at 12,288.
template <int MODE, bool SHARED>
__global__ __launch_bounds__(256) void k_query_filter(QueryArgs A, int n_tiles) {
  if (*A.n_pairs > A.capacity) return;  // the candidates were not written
  __shared__ float4 s_pts[4][MODE == HP_QUERY_NESTED ? kMaxPts : 1];
  __shared__ RingSlot s_rings[4][MODE == HP_QUERY_RING ? kMaxRings : 1];
  __shared__ uint32_t s_keys[4][kMaxRings], s_lens[4][kMaxRings];
  const int lane = hp_lane();
  const int wv = (int)hp_uniform(threadIdx.x >> 6);
  __shared__ uint32_t s_kept[2][4];  // SHARED: entries kept per wave, by step parity
  const int wg = hp_xcd_tile((int)blockIdx.x, (int)gridDim.x);
  const int k = SHARED ? wg : 4 * wg + wv;
  if (k >= n_tiles) return;  // (SHARED: none; else the waves are independent, with no barrier below)
  float4* s_pt = s_pts[wv];
  RingSlot* s_ring = s_rings[wv];
  uint32_t *s_key = s_keys[wv], *s_len = s_lens[wv];
  const int t = A.active_tiles[k];
  const int f = 1 << A.fl, nsub = f * f;
  int npts = 0, nslot = 0;
  if (MODE == HP_QUERY_NESTED) {
    // centres of the nodes of orders kt .. kq below t, coarsest first
    npts = (4 * nsub - 1) / 3;
    for (int j = lane; j < npts; j += 64) {
      int o = 0, base = 0;
      while (j >= base + (1 << (2 * o))) { base += 1 << (2 * o); ++o; }
      double v[3];
      hp_pix_dir(A.order_t + o, ((int64_t)t << (2 * o)) + (j - base), v);
      s_pt[j] = make_float4((float)v[0], (float)v[1], (float)v[2], 0.f);
    }
  } else {
    // rings crossing t at order kq: ring_min is that of the tile's south
    // corner pixel; each ring holds a run of the tile's pixels
    nslot = 2 * f - 1;
    int xt, yt, ft;
    hp_nest_xyf(A.order_t, t, &xt, &yt, &ft);
    const int64_t N = (int64_t)1 << A.kq;
    const int64_t ring_min = (int64_t)((ft >> 2) + 2) * N - ((int64_t)xt * f + f - 1) - ((int64_t)yt * f + f - 1) - 1;
    if (lane < nslot) { s_key[lane] = 0xffffffffu; s_len[lane] = 0u; }
    __builtin_amdgcn_wave_barrier();
    for (int j = lane; j < nsub; j += 64) {
      int64_t ir;
      int pos, xmy;
      pix_ring(A.kq, ((int64_t)t << (2 * A.fl)) + j, &ir, &pos, &xmy);
      const int o = (int)(ir - ring_min);
      // first pixel of the run: the smallest x - y (positions grow with it)
      atomicMin(&s_key[o], ((uint32_t)(xmy + 16384) << 17) | (uint32_t)pos);
      atomicAdd(&s_len[o], 1u);
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < nslot) {
      double lat, clat;
      int nring;
      float off;
      ring_geom(N, ring_min + lane, &lat, &clat, &nring, &off);
      const int len = (int)s_len[lane];
      const int start = len ? (int)(s_key[lane] & 0x1ffffu) : 0;
      const double step = 2.0 * M_PI / (double)nring;
      const double mid = ((double)start + 0.5 * (double)(len - 1) + (double)off) * step;
      const double hw = 0.5 * (double)(len + 1) * step;
      RingSlot r;
      r.sh = (float)sin(0.5 * lat);
      r.ch = (float)cos(0.5 * lat);
      r.clat = (float)clat;
      r.sm = (float)sin(0.5 * mid);
      r.cm = (float)cos(0.5 * mid);
      r.shw = (float)sin(0.5 * (hw < M_PI ? hw : M_PI));
      r.chw = (float)cos(0.5 * (hw < M_PI ? hw : M_PI));
      if (hw >= M_PI) r.shw = 2.f;
      if (len == 0) { r.sh = 4.f; r.ch = 0.f; }
      // the middle ring first, then outwards: most candidates are decided by the
      // first rings, and a wave stops when all of its are
      const int out = lane - (f - 1);
      s_ring[out > 0 ? 2 * out - 1 : -2 * out] = r;
    }
  }
  __builtin_amdgcn_wave_barrier();

  // the tile's list; entries are numbered from its start, so that a list at the end
  // of 2^32 entries does not wrap
  const uint32_t s = hp_uniform(A.ranges[2 * k]), n = hp_uniform(A.ranges[2 * k + 1]) - s;
  uint32_t* list = A.vals + s;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  constexpr uint64_t kEven = 0x5555555555555555ull, kOdd = ~kEven;
  const bool odd = (lane & 1) != 0;
  uint32_t kept = 0;
  constexpr uint32_t kStep = (SHARED ? 4 : 1) * kQueryIlp * 64;
  int par = 0;
  for (uint32_t step = 0; step < n; step += kStep, par ^= 1) {
    const uint32_t base = SHARED ? step + (uint32_t)wv * (kQueryIlp * 64) : step;
    // RING: entry lane / 2 for the even lanes, 32 + lane / 2 for the odd ones
    // (pair_load); NESTED: entry `lane`
    uint32_t g[kQueryIlp], ga[kQueryIlp], gb[kQueryIlp];
    uint64_t m[kQueryIlp], have[kQueryIlp];  // lanes kept, lanes with an entry
#pragma unroll
    for (int q = 0; q < kQueryIlp; ++q) {
      if (MODE == HP_QUERY_RING) {
        const uint32_t ia = base + 64u * q + (uint32_t)(lane >> 1), ib = ia + 32u;
        ga[q] = ia < n ? list[ia] : 0u;
        gb[q] = ib < n ? list[ib] : 0u;
        g[q] = odd ? gb[q] : ga[q];
        have[q] = __builtin_amdgcn_ballot_w64((odd ? ib : ia) < n);
      } else {
        const uint32_t idx = base + 64u * q + (uint32_t)lane;
        have[q] = __builtin_amdgcn_ballot_w64(idx < n);
        g[q] = idx < n ? list[idx] : 0u;
      }
      m[q] = 0;
    }
    if (MODE == HP_QUERY_NESTED) {
      float4 d[kQueryIlp];
#pragma unroll
      for (int q = 0; q < kQueryIlp; ++q) d[q] = A.gauss[g[q]];
      for (int j = 0; j < npts; ++j) {
        const float4 p = s_pt[j];
        uint64_t open = 0;
#pragma unroll
        for (int q = 0; q < kQueryIlp; ++q) {
          const float dx = p.x - d[q].x, dy = p.y - d[q].y, dz = p.z - d[q].z;
          m[q] |= __builtin_amdgcn_ballot_w64(fmaf(dz, dz, fmaf(dy, dy, dx * dx)) <= d[q].w);
          open |= have[q] & ~m[q];
        }
        if (open == 0) break;
      }
    } else {
      RingGauss G[kQueryIlp];
#pragma unroll
      for (int q = 0; q < kQueryIlp; ++q) G[q] = pair_load(A.gauss, ga[q], gb[q], odd);
      for (int j = 0; j < nslot; ++j) {
        const RingSlot r = s_ring[j];
        uint64_t open = 0;
#pragma unroll
        for (int q = 0; q < kQueryIlp; ++q) {
          m[q] |= ring_hit(r, G[q]);
          open |= have[q] & ~m[q];
        }
        if (open == 0) break;
      }
    }
    // the kept ones of these entries move down to the tile's next free slots, in
    // order: every one of them has been read (the tests used them; SHARED: the
    // barrier is behind all four waves' reads), and the next ones lie behind them
    uint32_t at = kept;
    if constexpr (SHARED) {
      uint32_t mine = 0;
#pragma unroll
      for (int q = 0; q < kQueryIlp; ++q) mine += (uint32_t)__popcll(m[q] & have[q]);
      if (lane == 0) s_kept[par][wv] = mine;
      __syncthreads();  // (the other set is written in the next step, past every read of it)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        at += w < wv ? s_kept[par][w] : 0u;
        kept += s_kept[par][w];
      }
    }
#pragma unroll
    for (int q = 0; q < kQueryIlp; ++q) {
      m[q] &= have[q];
      // kept entries before this lane's
      const uint64_t before = MODE == HP_QUERY_RING ? (odd ? kEven | (kOdd & below) : kEven & below) : below;
      if ((m[q] >> lane) & 1ull) list[at + (uint32_t)__popcll(m[q] & before)] = g[q];
      at += (uint32_t)__popcll(m[q]);
    }
    if (!SHARED) kept = at;
  }
  if (SHARED ? threadIdx.x == 0 : lane == 0) {
    A.ranges[2 * k + 1] = s + kept;
    if (A.n_kept) atomicAdd(A.n_kept, (unsigned long long)kept);
  }
}

__global__ void k_zero_i64(int64_t* p) { *p = 0; }

}  // namespace

extern "C" size_t hp_bin_query_workspace_bytes(int64_t P, int32_t order, int32_t tile_log2) {
  return hp_bin_sorted_workspace_bytes(P, order, tile_log2);
}

extern "C" hp_status hp_bin_query(int32_t phase, int32_t mode, int32_t f, const void* projected, int64_t P,
                                  const hp_view* view, const hp_params* prm, const void* grid, const void* mask,
                                  uint32_t* vals, uint32_t* tile_ranges, int32_t n_tiles, int64_t capacity,
                                  int64_t* n_pairs, int64_t* n_kept, void* ws, size_t ws_bytes, void* stream) {
  if (mode != HP_QUERY_RING && mode != HP_QUERY_NESTED) return HP_ERR_INVALID_ARG;
  HP_TRY(hp_check_view(view, prm));
  const HpGeom g = hp_geom(view->order, prm->tile_log2);
  int fl = 0;
  while (fl < 5 && (1 << fl) < f) ++fl;
  if (f < 1 || (1 << fl) != f || fl > g.b) return HP_ERR_INVALID_ARG;  // query order at most the pixel order
  const int kq = g.kt + fl;
  // margin: one ring step at the query order (RING), plus the distance from a
  // query point to the nearest pixel centre of its tile (at most a pixel
  // radius, below 1.2 / Nside), plus float slack
  const double step = mode == HP_QUERY_RING ? M_PI / (2.0 * (double)((int64_t)1 << kq)) : 0.0;
  const double widen = step + 1.2 / (double)((int64_t)1 << view->order) + 1e-4;
  HP_TRY(hp_bin_sorted_widened(phase, projected, P, view, prm, grid, mask, vals, tile_ranges, n_tiles, capacity,
                               n_pairs, ws, ws_bytes, stream, widen));
  if (!(phase & HP_BIN_EMIT)) return HP_OK;
  hipStream_t s = (hipStream_t)stream;
  if (n_kept) {
    hipLaunchKernelGGL(k_zero_i64, dim3(1), dim3(1), 0, s, n_kept);
    HP_CHECK_LAUNCH();
  }
  if (P == 0 || n_tiles == 0) return HP_OK;
  const HpProjView pv = hp_proj_view((const char*)projected, P);
  const HpMaskView mv = hp_mask_view((const char*)mask, g);
  // in a part of the workspace that a repeated emission does not read
  float4* gauss = (float4*)hp_bin_spare(ws, P);
  const dim3 gg(hp_blocks(P, 256));
  if (mode == HP_QUERY_RING)
    hipLaunchKernelGGL(k_query_gauss<HP_QUERY_RING>, gg, dim3(256), 0, s, P, pv.disc, pv.radius, gauss);
  else
    hipLaunchKernelGGL(k_query_gauss<HP_QUERY_NESTED>, gg, dim3(256), 0, s, P, pv.disc, pv.radius, gauss);
  HP_CHECK_LAUNCH();
  QueryArgs A{mode, kq, fl, g.kt, mv.active_tiles, gauss, vals, tile_ranges, n_pairs, capacity,
              (unsigned long long*)n_kept};
  const dim3 per_tile((unsigned)n_tiles), per_four(hp_blocks(n_tiles, 4));
  if (mode == HP_QUERY_NESTED)
    hipLaunchKernelGGL((k_query_filter<HP_QUERY_NESTED, true>), per_tile, dim3(256), 0, s, A, (int)n_tiles);
  else if (n_tiles <= kRingShared)
    hipLaunchKernelGGL((k_query_filter<HP_QUERY_RING, true>), per_tile, dim3(256), 0, s, A, (int)n_tiles);
  else
    hipLaunchKernelGGL((k_query_filter<HP_QUERY_RING, false>), per_four, dim3(256), 0, s, A, (int)n_tiles);
  HP_CHECK_LAUNCH();
  return HP_OK;
}
