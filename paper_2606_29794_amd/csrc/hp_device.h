// hp_device.h -- device-side building blocks of the HEALPix rasterizer:
// buffer layouts shared by the kernels of this library, HEALPix geometry in
// double precision (Gorski et al. 2005, the grid of Sec. 3.1), the
// face-extended chart used by HEALPix-SSIM (Sec. 4.1) and wave64 helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/hp.h"

#define HP_HD __host__ __device__ __forceinline__

// ---------------------------------------------------------------------------
// Sizes and layouts
// ---------------------------------------------------------------------------
HP_HD size_t hp_align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct HpGeom {
  int order, b, kt;       // pixel order, log2 tile side, tile order
  int64_t npix, ntile;    // full-sphere pixels and tiles
  int per_tile;           // pixels per tile = 4^b
  int64_t nodes;          // quadtree nodes, levels 0..kt
};

HP_HD HpGeom hp_geom(int order, int tile_log2) {
  HpGeom g;
  g.order = order;
  g.b = tile_log2 < order ? tile_log2 : order;
  g.kt = order - g.b;
  g.npix = 12ll << (2 * order);
  g.ntile = 12ll << (2 * g.kt);
  g.per_tile = 1 << (2 * g.b);
  g.nodes = 12ll * (((int64_t)1 << (2 * (g.kt + 1))) - 1) / 3;
  return g;
}
HP_HD int64_t hp_level_offset(int level) { return 12ll * (((int64_t)1 << (2 * level)) - 1) / 3; }

// grid buffer: node caps (float4: centre xyz, radius) then (sin, cos) of half radius
struct HpGridView {
  float4* cap;
  float2* sc;
};
HP_HD size_t hp_grid_size(const HpGeom& g) { return hp_align256(g.nodes * sizeof(float4)) + hp_align256(g.nodes * sizeof(float2)); }
HP_HD HpGridView hp_grid_view(void* base, const HpGeom& g) {
  HpGridView v;
  char* p = (char*)base;
  v.cap = (float4*)p;
  v.sc = (float2*)(p + hp_align256(g.nodes * sizeof(float4)));
  return v;
}

// mask buffer
struct HpMaskView {
  int64_t* n_active;
  int32_t* n_tiles;
  float* cone;            // (sin, cos) of half the bounding cone's angle, then kConeMark (hp_cone.h)
  int32_t* tile_start;    // [ntile] first compact pixel slot of the tile
  int32_t* tile_count;    // [ntile] active pixels in the tile
  int32_t* tile_compact;  // [ntile] compact active tile id or -1
  uint32_t* tile_bits;    // [ntile][8] membership of the tile's pixels (nested order)
  int32_t* active_tiles;  // [ntile] compact id -> tile
  uint8_t* node_active;   // [nodes]
  int32_t* active_pix;    // [npix]
};
HP_HD size_t hp_mask_size(const HpGeom& g) {
  size_t s = 256;
  s += 4 * hp_align256(g.ntile * 4);
  s += hp_align256(g.ntile * 32);
  s += hp_align256(g.nodes);
  s += hp_align256(g.npix * 4);
  return s;
}
template <class P>
HP_HD HpMaskView hp_mask_view(P* base, const HpGeom& g) {
  HpMaskView v;
  char* p = (char*)base;
  v.n_active = (int64_t*)p;
  v.n_tiles = (int32_t*)(p + 8);
  v.cone = (float*)(p + 16);
  p += 256;
  size_t t4 = hp_align256(g.ntile * 4);
  v.tile_start = (int32_t*)p; p += t4;
  v.tile_count = (int32_t*)p; p += t4;
  v.tile_compact = (int32_t*)p; p += t4;
  v.active_tiles = (int32_t*)p; p += t4;
  v.tile_bits = (uint32_t*)p; p += hp_align256(g.ntile * 32);
  v.node_active = (uint8_t*)p; p += hp_align256(g.nodes);
  v.active_pix = (int32_t*)p;
  return v;
}

// projected buffer: 64-byte record per Gaussian, then depth and radius
//   r0 = (u_x, u_y, u_z, opacity)    unit camera-frame direction
//   r1 = (eo_x, eo_z, ep_x, ep_y)    tangent frame: e_omega = (eo_x, 0, eo_z)
//   r2 = (ep_z, A, B, C)             e_phi = (ep_x, ep_y, ep_z); q = A a^2 + 2 B a b + C b^2
//   r3 = (red, green, blue, sin((r_s + bin_guard) / 2))   the last entry drives the binning
// projected buffer: the 64-byte records, depth [P], radius [P], and disc [P]
// (unit direction, sin of half the tile-test angle r_s + guard: the 16 bytes
// the binning reads, apart from the records so that its gathers share lines)
struct HpProjView {
  float4* rec;
  float* depth;
  float* radius;
  float4* disc;
};
HP_HD size_t hp_proj_size(int64_t P) { return hp_align256(P * 64) + 2 * hp_align256(P * 4) + hp_align256(P * 16); }
template <class T>
HP_HD HpProjView hp_proj_view(T* base, int64_t P) {
  HpProjView v;
  char* p = (char*)base;
  v.rec = (float4*)p;
  v.depth = (float*)(p + hp_align256(P * 64));
  v.radius = (float*)(p + hp_align256(P * 64) + hp_align256(P * 4));
  v.disc = (float4*)(p + hp_align256(P * 64) + 2 * hp_align256(P * 4));
  return v;
}

// ---------------------------------------------------------------------------
// HEALPix NESTED geometry (double precision)
// ---------------------------------------------------------------------------
// bits of x at even positions, bits of y at odd positions
HP_HD uint32_t hp_compact_bits(uint32_t v) {
  v &= 0x55555555u;
  v = (v | (v >> 1)) & 0x33333333u;
  v = (v | (v >> 2)) & 0x0f0f0f0fu;
  v = (v | (v >> 4)) & 0x00ff00ffu;
  v = (v | (v >> 8)) & 0x0000ffffu;
  return v;
}
HP_HD uint32_t hp_spread_bits(uint32_t v) {
  v &= 0x0000ffffu;
  v = (v | (v << 8)) & 0x00ff00ffu;
  v = (v | (v << 4)) & 0x0f0f0f0fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}
HP_HD void hp_nest_xyf(int order, int64_t p, int* x, int* y, int* f) {
  *f = (int)(p >> (2 * order));
  const uint32_t q = (uint32_t)p & ((1u << (2 * order)) - 1u);
  *x = (int)hp_compact_bits(q);
  *y = (int)hp_compact_bits(q >> 1);
}
HP_HD int64_t hp_xyf_nest(int order, int x, int y, int f) {
  return ((int64_t)f << (2 * order)) + (int64_t)(hp_spread_bits((uint32_t)x) | (hp_spread_bits((uint32_t)y) << 1));
}

// Pixel-centre position: z, sin(theta) and the longitude phi (not wrapped).
// Face f: row f/4 sets the ring of the face's southern corner (rows 2, 3, 4
// in units of Nside); column f%4 sets its longitude (odd multiples of pi/4 for
// the polar rows, multiples of pi/2 for the equatorial row).
// Orders up to HP_MAX_ORDER: N^2 and 8 N fit 32 bits.
__device__ __forceinline__ void hp_pix_pos(int order, int64_t p, double* pz, double* psth, double* pphi) {
  int x, y, f;
  hp_nest_xyf(order, p, &x, &y, &f);
  const int N = 1 << order;
  const int row = f >> 2, col = f & 3;
  const int ring = (row + 2) * N - x - y - 1;               // 1 .. 4N-1 from the north pole
  const int lon_units = (row == 1) ? 2 * col : 2 * col + 1; // face centre longitude in pi/4
  double z, sth, phi;
  if (ring < N || ring > 3 * N) {
    const int nr = ring < N ? ring : 4 * N - ring;          // ring index counted from its pole
    const double tmp = (double)(nr * nr) / (3.0 * (double)(N * N));
    z = ring < N ? 1.0 - tmp : tmp - 1.0;
    sth = sqrt(tmp * (2.0 - tmp));
    // position along the ring: nr pixels per face, centred on the face longitude
    const int jp = (lon_units * nr + x - y + 1) / 2;        // 1-based within ring (may wrap)
    phi = ((double)jp - 0.5) * (M_PI / 2.0) / (double)nr;
  } else {
    z = (double)(2 * N - ring) * (2.0 / (3.0 * (double)N));
    sth = sqrt((1.0 - z) * (1.0 + z));
    const int s = (ring - N) & 1;
    const int jp = (lon_units * N + x - y + 1 + s) / 2;
    phi = ((double)jp - 0.5 * (1 + s)) * (M_PI / 2.0) / (double)N;
  }
  *pz = z;
  *psth = sth;
  *pphi = phi;
}

// Pixel-centre direction in the camera frame (pole = camera +y, longitude
// omega = atan2(t_x, t_z)): t = (sin(theta) sin(phi), z, sin(theta) cos(phi)).
__device__ __forceinline__ void hp_pix_dir(int order, int64_t p, double* t) {
  double z, sth, phi, sp, cp;
  hp_pix_pos(order, p, &z, &sth, &phi);
  sincos(phi, &sp, &cp);
  t[0] = sth * sp;
  t[1] = z;
  t[2] = sth * cp;
}

// ---------------------------------------------------------------------------
// Face-extended chart (HEALPix-SSIM neighbourhoods, Sec. 4.1).
// A face-local offset that leaves face f across one edge lands in the
// neighbouring face with its axes turned to line up; across a corner it lands
// in the diagonally opposite face only at four-face vertices (the poles and
// the equatorial corners); at the eight three-face vertices the diagonal
// quadrant does not exist.  Each case is an affine map
//   X = ax x + bx y + kx N + lx,  Y = ay x + by y + ky N + ly
// into face  base + (col + dcol) % 4  (dcol < 0: missing).
// ---------------------------------------------------------------------------
struct HpChartXf {
  int8_t base, dcol, ax, bx, kx, lx, ay, by, ky, ly;
};
// index: row*8 + dir, dir over (sx, sy) in order
// (+1,0) (-1,0) (0,+1) (0,-1) (+1,+1) (-1,-1) (+1,-1) (-1,+1)
__constant__ static const HpChartXf kHpChart[24] = {
    // north row
    {0, 1, 0, 1, 0, 0, -1, 0, 2, -1},   // +x: next polar face, turned
    {4, 0, 1, 0, 1, 0, 0, 1, 0, 0},     // -x: equatorial face below-west
    {0, 3, 0, -1, 2, -1, 1, 0, 0, 0},   // +y: previous polar face, turned
    {4, 1, 1, 0, 0, 0, 0, 1, 1, 0},     // -y: equatorial face below-east
    {0, 2, -1, 0, 2, -1, 0, -1, 2, -1}, // +x+y: across the pole
    {8, 0, 1, 0, 1, 0, 0, 1, 1, 0},     // -x-y: south face across the equatorial vertex
    {0, -1, 0, 0, 0, 0, 0, 0, 0, 0},    // three-face vertex
    {0, -1, 0, 0, 0, 0, 0, 0, 0, 0},
    // equatorial row
    {0, 0, 1, 0, -1, 0, 0, 1, 0, 0},    // +x: polar face above-east
    {8, 3, 1, 0, 1, 0, 0, 1, 0, 0},     // -x: south face below-west
    {0, 3, 1, 0, 0, 0, 0, 1, -1, 0},    // +y: polar face above-west
    {8, 0, 1, 0, 0, 0, 0, 1, 1, 0},     // -y: south face below-east
    {0, -1, 0, 0, 0, 0, 0, 0, 0, 0},    // +x+y: three-face vertex (north)
    {0, -1, 0, 0, 0, 0, 0, 0, 0, 0},    // -x-y: three-face vertex (south)
    {4, 1, 1, 0, -1, 0, 0, 1, 1, 0},    // +x-y: next equatorial face
    {4, 3, 1, 0, 1, 0, 0, 1, -1, 0},    // -x+y: previous equatorial face
    // south row
    {4, 1, 1, 0, -1, 0, 0, 1, 0, 0},    // +x: equatorial face above-east
    {8, 3, 0, 1, 0, 0, -1, 0, 0, -1},   // -x: previous polar face, turned
    {4, 0, 1, 0, 0, 0, 0, 1, -1, 0},    // +y: equatorial face above-west
    {8, 1, 0, -1, 0, -1, 1, 0, 0, 0},   // -y: next polar face, turned
    {0, 0, 1, 0, -1, 0, 0, 1, -1, 0},   // +x+y: north face across the equatorial vertex
    {8, 2, -1, 0, 0, -1, 0, -1, 0, -1}, // -x-y: across the south pole
    {0, -1, 0, 0, 0, 0, 0, 0, 0, 0},
    {0, -1, 0, 0, 0, 0, 0, 0, 0, 0},
};

// Nested pixel at face-local (x, y) of face f (x, y may be outside [0, N) by
// less than N), or -1 where the chart has no pixel.
__device__ __forceinline__ int64_t hp_chart_pixel(int order, int f, int x, int y) {
  const int N = 1 << order;
  const int sx = x < 0 ? -1 : (x >= N ? 1 : 0);
  const int sy = y < 0 ? -1 : (y >= N ? 1 : 0);
  if (sx == 0 && sy == 0) return hp_xyf_nest(order, x, y, f);
  int dir;
  if (sy == 0) dir = sx > 0 ? 0 : 1;
  else if (sx == 0) dir = sy > 0 ? 2 : 3;
  else if (sx == sy) dir = sx > 0 ? 4 : 5;
  else dir = sx > 0 ? 6 : 7;
  const HpChartXf m = kHpChart[(f >> 2) * 8 + dir];
  if (m.dcol < 0) return -1;
  const int g = m.base + (((f & 3) + m.dcol) & 3);
  const int X = m.ax * x + m.bx * y + m.kx * N + m.lx;
  const int Y = m.ay * x + m.by * y + m.ky * N + m.ly;
  if (X < 0 || X >= N || Y < 0 || Y >= N) return -1;
  return hp_xyf_nest(order, X, Y, g);
}

// ---------------------------------------------------------------------------
// wave64 helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ int hp_lane() { return (int)__lane_id(); }

// Read-only data addressed by a wave-uniform index: reading through the
// constant address space lets the compiler use scalar loads into SGPRs.
typedef const __attribute__((address_space(4))) float* hp_cfloatp;
typedef const __attribute__((address_space(4))) uint32_t* hp_cu32p;
__device__ __forceinline__ uint32_t hp_uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Workgroups go to the 8 XCDs round-robin by index.  Giving each XCD a
// contiguous range of tiles keeps neighbouring tiles, which share most of
// their data, in the same L2.  A bijection of [0, nb).
__device__ __forceinline__ int hp_xcd_tile(int b, int nb) {
  const int per = nb >> 3, rem = nb & 7;
  const int x = b & 7, k = b >> 3;
  return x * per + (x < rem ? x : rem) + k;
}

// The same for tiles of unequal work that only read what they share: XCD x
// takes groups x, x + 8, ... of kXcdGroup neighbouring tiles, the tiles past the
// last full round one by one.  A contiguous eighth of the sphere can hold 14 %
// more work than the mean eighth, groups of 16 tiles hold within 1 % of it: forward
// render 368 -> 352 us (full sphere, order 9), 376 -> 346 us (pinhole of 60
// degrees, order 11), 119 -> 112 us (order 10), loss with zone windows, whose polar
// tiles cost several others, 360 -> 331 us; groups of 4 and single tiles measured
// the same within 2 %.  A backward whose tiles add to value-major
// accumulators stays contiguous: with groups 144 -> 155 us on a fisheye of order 8.
constexpr int kXcdGroup = 16;
__device__ __forceinline__ int hp_xcd_group_tile(int b, int nb) {
  constexpr int G = kXcdGroup;
  if (b >= nb / (8 * G) * (8 * G)) return b;
  const int x = b & 7, k = b >> 3;
  return (k / G * 8 + x) * G + k % G;
}

template <int CTRL>
__device__ __forceinline__ float hp_dpp(float v) {
  // every source lane of the patterns used here is inside the row, so the
  // bound control setting never applies; it allows fusing into the add
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
// Sums over the 64 lanes of N values at once (all lanes active), wave-uniform
// results: quad butterflies and row mirrors give each 16-lane row its sum,
// then the four row sums are read out and added.  The N reductions advance
// step by step so that independent DPP operations interleave.
template <int N>
__device__ __forceinline__ void hp_wave_totals(float* v) {
#pragma unroll
  for (int m = 0; m < N; ++m) v[m] += hp_dpp<0xB1>(v[m]);   // quad_perm [1,0,3,2]: lane ^ 1
#pragma unroll
  for (int m = 0; m < N; ++m) v[m] += hp_dpp<0x4E>(v[m]);   // quad_perm [2,3,0,1]: lane ^ 2
#pragma unroll
  for (int m = 0; m < N; ++m) v[m] += hp_dpp<0x141>(v[m]);  // row_half_mirror: quads of a half-row
#pragma unroll
  for (int m = 0; m < N; ++m) v[m] += hp_dpp<0x140>(v[m]);  // row_mirror: half-rows of a row
#pragma unroll
  for (int m = 0; m < N; ++m) {
    const int x = __float_as_int(v[m]);
    v[m] = (__int_as_float(__builtin_amdgcn_readlane(x, 0)) + __int_as_float(__builtin_amdgcn_readlane(x, 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(x, 32)) + __int_as_float(__builtin_amdgcn_readlane(x, 48)));
  }
}

// Nine sums over the 64 lanes (all active) at once by recursive halving.  Inside
// a row of 16 lanes DPP adds whose bank mask writes only half of the lanes merge
// two values into one register, two instructions per pair and step; the rows
// are joined last, when two registers are left (a permlane swap takes two
// issue slots: joining the rows first, as gfx950's swaps also allow, took 36
// slots, this takes 25).  Returns, in lane L < 32, the total of value
// 4 (L bit 3) + 2 (L bit 2) + (L bit 4), and in every lane of the last row that
// of the ninth value.  The adds are in asm because the compiler does not form
// masked DPP adds; every register is written at least two instructions before
// a DPP operand reads it, as the hardware asks, and the s_nop cover the
// neighbours.
__device__ __forceinline__ float hp_wave_totals9(float* v) {
#define HP_RS_LO(x) "v_add_f32_dpp " x ", " x ", " x " row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
#define HP_RS_HI(x, y) "v_add_f32_dpp " x ", " y ", " y " row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
#define HP_RS_EVEN(x) "v_add_f32_dpp " x ", " x ", " x " row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
#define HP_RS_ODD(x, y) "v_add_f32_dpp " x ", " y ", " y " row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
#define HP_RS_ALL(x, ctrl) "v_add_f32_dpp " x ", " x ", " x " " ctrl " row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t"
      // lanes with bit 3 clear keep values 0..3, the others take 4..7
      HP_RS_LO("%0") HP_RS_LO("%1") HP_RS_LO("%2") HP_RS_LO("%3") HP_RS_ALL("%4", "row_ror:8")
      HP_RS_HI("%0", "%5") HP_RS_HI("%1", "%6") HP_RS_HI("%2", "%7") HP_RS_HI("%3", "%8")
      // lanes with bit 2 clear keep %0 and %1, the others take %2 and %3
      HP_RS_ALL("%4", "row_half_mirror") HP_RS_EVEN("%0") HP_RS_EVEN("%1")
      HP_RS_ALL("%4", "quad_perm:[1,0,3,2]") HP_RS_ODD("%0", "%2") HP_RS_ODD("%1", "%3")
      HP_RS_ALL("%4", "quad_perm:[2,3,0,1]") "s_nop 1"
      : "+&v"(v[0]), "+&v"(v[1]), "+&v"(v[2]), "+&v"(v[3]), "+&v"(v[8])
      : "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
#undef HP_RS_LO
#undef HP_RS_HI
#undef HP_RS_EVEN
#undef HP_RS_ODD
#undef HP_RS_ALL
  // even rows keep %0, odd rows take %1
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
  float x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  x += hp_dpp<0xB1>(x);
  x += hp_dpp<0x4E>(x);
  // the halves of x in lanes 0..31, those of the ninth value in lanes 32..63
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(v[8]), false, false);
  float w = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  asm("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0x8 bank_mask:0xf" : "+v"(w));
  return w;
}

// The sum over the 64 lanes in every lane (each swap pairs the value with itself).
__device__ __forceinline__ float hp_wave_sum_dpp(float z) {
  {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    z = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    z = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  z += hp_dpp<0x128>(z);  // row_ror:8
  z += hp_dpp<0xB1>(z);
  z += hp_dpp<0x4E>(z);
  z += hp_dpp<0x141>(z);
  return z;
}

// The same for the largest of 64 values; fmaxf passes over a NaN.
__device__ __forceinline__ float hp_wave_max_dpp(float z) {
  {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    z = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(z), __float_as_uint(z), false, false);
    z = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  z = fmaxf(z, hp_dpp<0x128>(z));
  z = fmaxf(z, hp_dpp<0xB1>(z));
  z = fmaxf(z, hp_dpp<0x4E>(z));
  return fmaxf(z, hp_dpp<0x141>(z));
}
