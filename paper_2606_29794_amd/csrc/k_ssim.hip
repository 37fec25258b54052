// k_ssim.hip -- HEALPix-SSIM and the training loss of Sec. 4.1.
//
// One workgroup per active tile.  The tile's B x B pixels plus a 5-pixel halo
// are gathered into LDS through the face-extended chart (neighbouring faces
// with their axes turned to line up; the missing quadrant of a three-face
// vertex and inactive pixels carry weight 0).  Dividing the window sums by
// the summed weight renormalises where neighbours are missing.
//
// Windows.  The isotropic chart window exp(-(a^2 + b^2) / (2 sigma^2)) is
// separable on the patch: two 11-tap passes, each thread sliding the window
// along a strip held in registers (one LDS read per input value, four or
// eight outputs per strip).  With zone-specific windows, a pixel of a polar
// cap weighs its neighbours by great-circle distance instead,
// exp(-d^2 / (2 sigma^2 Omega)), Omega = 4 pi / Npix, which is not separable:
// tiles holding such pixels take a direct 121-tap path with the pixel-centre
// directions in LDS (from order 8 on two pixels per thread, ss_pair_rows).
//
// The backward pass is the transposed window: the chart neighbourhood
// relation is symmetric with equal offset lengths, so the adjoint gathers the
// per-pixel SSIM partials over the same window, each neighbour's partials
// weighted by that neighbour's own window at the pixel.
#include "hp_common.h"

#define SS_R 5
#define SS_W 11

// patch table entries: compact slot, bit 30 set for a polar-cap pixel, -1
// for a missing or inactive neighbour
constexpr int32_t kSsPolarBit = 1 << 30;
constexpr int32_t kSsSlotMask = kSsPolarBit - 1;
// the backward's per-pixel partials: 9 floats at a 12-float (48-byte) stride
constexpr int kSsG = 12;

struct SsimArgs {
  int order, b, kt;
  const int32_t* active_tiles;
  const int32_t* tile_start;
  const int32_t* tile_count;
  const uint32_t* tile_bits;
  int64_t n_active;
  float C1, C2, lam;
  float g[SS_W];   // chart window taps exp(-a^2 / (2 sigma^2)), a = -5..5
  float gsum;      // their sum, accumulated in the order of the passes
  double wscale;   // 1 / (2 sigma^2 Omega): polar windows are exp(-d^2 wscale)
  double w2[3];    // the same in base 2 as a series in s^2 = |u - v|^2 / 4 (ss_polar_weight)
  bool fine;       // small windows: the polar weights are ss_polar_weight
  const int32_t* tables;  // [n_tiles][H*H] patch slots (see k_ssim_tables)
};

// compact slot of nested pixel q, or -1 when inactive / absent
__device__ __forceinline__ int64_t ss_slot(const SsimArgs& A, int64_t q) {
  if (q < 0) return -1;
  const int per_b = 2 * A.b;
  const int64_t t = q >> per_b;
  const int loc = (int)(q - (t << per_b));
  // a fully active tile holds its pixels in nested order: no rank to count
  if (A.tile_count[t] == (1 << per_b)) return (int64_t)A.tile_start[t] + loc;
  const uint32_t* bits = A.tile_bits + 8 * t;
  const uint32_t word = bits[loc >> 5];
  if (!((word >> (loc & 31)) & 1u)) return -1;
  int rank = __popc(word & ((1u << (loc & 31)) - 1u));
  for (int k = 0; k < (loc >> 5); ++k) rank += __popc(bits[k]);
  return (int64_t)A.tile_start[t] + rank;
}

// polar cap pixel: ring jr = jrll(f) N - x - y - 1 outside [N, 3N]
__device__ __forceinline__ bool ss_polar(int order, int64_t q) {
  int x, y, f;
  hp_nest_xyf(order, q, &x, &y, &f);
  const int N = 1 << order;
  return f < 4 ? (x + y >= N) : (f >= 8 ? (x + y <= N - 2) : false);
}

// Patch cell (x, y) of gather index i (a bijection of [0, H*H)): the first
// B*B indices are the tile's own pixels in NESTED order, which a fully
// active tile stores contiguously (coalesced loads), the rest the halo row by
// row.
template <int B>
__device__ __forceinline__ void ss_cell(int i, int* cx, int* cy) {
  constexpr int H = B + 2 * SS_R;
  if (i < B * B) {
    *cx = (int)hp_compact_bits((uint32_t)i) + SS_R;
    *cy = (int)hp_compact_bits((uint32_t)i >> 1) + SS_R;
    return;
  }
  int h = i - B * B;
  if (h < SS_R * H) { *cy = h / H; *cx = h % H; return; }  // rows above the tile
  h -= SS_R * H;
  if (h < 2 * SS_R * B) {  // left and right of the tile's rows
    *cy = SS_R + h / (2 * SS_R);
    const int c = h % (2 * SS_R);
    *cx = c < SS_R ? c : c + B;
    return;
  }
  h -= 2 * SS_R * B;
  *cy = SS_R + B + h / H;  // rows below
  *cx = h % H;
}

__device__ __forceinline__ void ss_tile_origin(const SsimArgs& A, int ct, int* f, int* x0, int* y0) {
  const int t = A.active_tiles[ct];
  int tx, ty;
  hp_nest_xyf(A.kt, t, &tx, &ty, f);
  *x0 = tx << A.b;
  *y0 = ty << A.b;
}

// squared great-circle distance between unit vectors u, v (double):
// d = 2 asin(s), s = |u - v| / 2; d^2 = 4 s^2 (asin s / s)^2, the factor as
// its series in s^2 below s^2 = 1/16 (truncation < 1e-9), asin beyond
__device__ __forceinline__ double ss_dist2(const double* u, const double* v) {
  const double dx = u[0] - v[0], dy = u[1] - v[1], dz = u[2] - v[2];
  const double c2 = dx * dx + dy * dy + dz * dz;
  const double s2 = 0.25 * c2;
  if (s2 < 0.0625) {
    const double k = 1.0 + s2 * (1.0 / 3.0 + s2 * (8.0 / 45.0 + s2 * (4.0 / 35.0 + s2 * (128.0 / 1575.0 +
                     s2 * (128.0 / 2079.0 + s2 * (1024.0 / 21021.0))))));
    return c2 * k;
  }
  const double d = 2.0 * asin(fmin(1.0, sqrt(s2)));
  return d * d;
}

// Polar window weight exp(-d^2 wscale) of a cell in direction v at the pixel in
// direction u, h = -u / 2, where A.fine: s^2 = |u - v|^2 / 4 = 1/2 - u.v / 2 as three
// fused multiply-adds, then the exponent to base 2 with the series of ss_dist2
// cut after s^4; 11 vector instructions instead of 27.  From order 8 on a window
// reaches ten steps between neighbouring centres, each under 1.6 / nside: s^2 <
// 1e-3, where the terms left out are under 1.2e-10 of the sum.  The rounding of s^2,
// under 5e-16, has to move the exponent by less than half a float ulp of 1: true
// of sigma = 1.5 at every order (4.5e-9 at order 12), not of a window far
// narrower than a pixel, which takes the general path.
constexpr int kSsFineOrder = 8;
__device__ __forceinline__ float ss_polar_weight(const SsimArgs& A, const double* h, double vx, double vy, double vz) {
  const double s2 = fma(h[0], vx, fma(h[1], vy, fma(h[2], vz, 0.5)));
  return __builtin_amdgcn_exp2f((float)(s2 * fma(s2, fma(s2, A.w2[2], A.w2[1]), A.w2[0])));
}

// Items of the direct path on tiles of 16 x 16: thread t of each half of the
// workgroup has the pixels (t % 16, 2 (t / 16)) and the one below, so a cell of
// their windows is read from LDS once for both.  The first half takes the first
// six of the twelve cell rows, the second half the others; of them the first
// row belongs to the upper pixel alone, the last one to the lower.  Bound by
// vector instructions (about 37 per pixel and tap forward, 25 backward), the
// columns as a real loop: unrolled, the loads gathered in front took 168
// registers (245 and 195 us).  Fisheye of 200 degrees at order 9, 1.8 M pixels:
// forward 335 -> 188 us, backward 391 -> 175 us against one thread per pixel
// with the general distance (172 and 153 us with the tiles interleaved over the
// XCDs).
//   row(b, up, low): cell row b with the upper (window row b) and the lower
//   pixel (window row b - 1) as the compile-time flags say
template <bool B>
struct SsBool {
  static constexpr bool value = B;
};
template <class Row>
__device__ __forceinline__ void ss_pair_rows(int half, Row row) {
  if (half == 0) row(0, SsBool<true>{}, SsBool<false>{});
#pragma unroll 1
  for (int b = half == 0 ? 1 : 6, e = b + 5; b < e; ++b) row(b, SsBool<true>{}, SsBool<true>{});
  if (half != 0) row(SS_W, SsBool<false>{}, SsBool<true>{});
}

// SSIM of one pixel and channel from its normalised window moments, and the
// partials of the backward: d SSIM / d (sum x, sum x^2, sum xy) / Z
__device__ __forceinline__ float ss_index(float C1, float C2, float iZ, float Sx, float Sy, float Sxx, float Syy,
                                          float Sxy, float* G0, float* G1, float* G2) {
  const float mx = Sx * iZ, my = Sy * iZ;
  const float vx = Sxx * iZ - mx * mx, vy = Syy * iZ - my * my;
  const float cxy = Sxy * iZ - mx * my;
  const float An = 2.f * mx * my + C1, Bn = 2.f * cxy + C2;
  const float Ad = mx * mx + my * my + C1, Bd = vx + vy + C2;
  // reciprocals to 1 ulp (v_rcp_f32) instead of IEEE divisions
  const float iAd = __builtin_amdgcn_rcpf(Ad), iBd = __builtin_amdgcn_rcpf(Bd);
  const float iden = iAd * iBd;
  const float s = An * Bn * iden;
  // s(sx, sxx, sxy) with the y sums fixed; sx = mx etc. (normalised)
  const float ds_dmx = (2.f * my * Bn - An * 2.f * my) * iden - s * (2.f * mx * iAd - 2.f * mx * iBd);
  *G0 = ds_dmx * iZ;
  *G1 = (-s * iBd) * iZ;
  *G2 = (2.f * An * iden) * iZ;
  return s;
}

// nested index of patch-interior pixel (x, y) of a tile: x bits at even
// positions, y bits at odd ones
__device__ __forceinline__ int ss_nest_local(int x, int y) {
  auto spread = [](uint32_t v) {
    v = (v | (v << 8)) & 0x00FF00FFu;
    v = (v | (v << 4)) & 0x0F0F0F0Fu;
    v = (v | (v << 2)) & 0x33333333u;
    v = (v | (v << 1)) & 0x55555555u;
    return v;
  };
  return (int)(spread((uint32_t)x) | (spread((uint32_t)y) << 1));
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
// LDS: the gathered patch (mask, x[3], y[3]); the first pass's output [16][H][B]
// goes over it and the second pass's output [16][B*B] over that, each kept in
// registers until the reads are done.  The cells' directions are only needed
// with zone windows.
template <int B, bool ZONES>
struct SsFwdLds {
  // row pitch HP: 16-byte aligned rows for the strip loads; P1S: the pass-1
  // output's quantity stride, 16 mod 32 words so that the two quantities a
  // half-wave reads in the second pass fall in different banks
  static constexpr int H = B + 2 * SS_R, HP = (H + 3) & ~3, P1S = H * B + ((48 - (H * B) % 32) % 32);
  union {
    float in[7][H][HP];
    float p1[16][P1S];
  };
  double dir[3][ZONES ? H * H : 1];
};

// A workgroup per tile.  Its phases (gather, two passes, the pixel's index,
// output) wait for each other, so what counts is how many workgroups a CU has
// in different ones: 27 KB of LDS and 96 registers let five run.  Three per CU
// that kept 48 KB and fetched the next tile's cells meanwhile in registers
// took 127 us, five take 112 us, at 3.1 M pixels; its instructions alone take 73 us,
// its bytes 51 us.
// Forward: SSIM per active pixel and channel; per-block partial sums of SSIM
// and |img - ref|; optionally the per-pixel partials needed by the backward,
// G[m][n] = (d SSIM / d S_m) / Z for m in (sum x, sum x^2, sum xy) x channel.
template <int B, bool ZONES>
__global__ __launch_bounds__(256, ZONES ? 3 : 5) void k_ssim_fwd(SsimArgs A, const float* __restrict__ img,
                                                  const float* __restrict__ ref, float* __restrict__ smap,
                                                  float* __restrict__ G, float2* __restrict__ part, int n_tiles) {
  using L = SsFwdLds<B, ZONES>;
  constexpr int H = L::H;
  __shared__ L s;
  __shared__ float s_red[2][4];
  float(*S)[B * B] = reinterpret_cast<float(*)[B * B]>(&s.in[0][0][0]);  // after pass 2
  const int tid = threadIdx.x;
  constexpr int NG = (H * H + 255) / 256;
  const int ct = ZONES ? hp_xcd_group_tile(blockIdx.x, n_tiles) : hp_xcd_tile(blockIdx.x, n_tiles);
  const int32_t* tab = A.tables + (int64_t)ct * (H * H);
  int32_t e[NG];
  float v[NG][6];
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    const int i = tid + 256 * gi;
    e[gi] = i < H * H ? tab[i] : -1;
  }
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    const int64_t slot = e[gi] & kSsSlotMask;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      v[gi][ch] = e[gi] >= 0 ? img[ch * A.n_active + slot] : 0.f;
      v[gi][3 + ch] = e[gi] >= 0 ? ref[ch * A.n_active + slot] : 0.f;
    }
  }
  float ssum = 0.f, lsum = 0.f;  // this thread's SSIM and L1 sums
  int f, x0, y0;
  ss_tile_origin(A, ct, &f, &x0, &y0);
  // zone windows: the tile takes the direct path when it holds a polar pixel
  const int N = 1 << A.order;
  // tiles narrower than 8 pixels (orders 0-2) always take the direct path
  constexpr bool kSmall = B < 8;
  const bool direct =
      kSmall || (ZONES && (f < 4 ? (x0 + y0 + 2 * B - 2 >= N) : (f >= 8 ? (x0 + y0 <= N - 2) : false)));
  bool mine_full = true;
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    const int i = tid + 256 * gi;
    if (i < H * H) {
      int cx, cy;
      ss_cell<B>(i, &cx, &cy);
      mine_full &= e[gi] >= 0;
      s.in[0][cy][cx] = e[gi] >= 0 ? 1.f : 0.f;
#pragma unroll
      for (int k = 0; k < 6; ++k) s.in[1 + k][cy][cx] = v[gi][k];
      if (ZONES && direct) {
        const int64_t q = hp_chart_pixel(A.order, f, x0 + cx - SS_R, y0 + cy - SS_R);
        double d[3] = {0.0, 0.0, 0.0};
        if (q >= 0) hp_pix_dir(A.order, q, d);
        s.dir[0][cy * H + cx] = d[0];
        s.dir[1][cy * H + cx] = d[1];
        s.dir[2][cy * H + cx] = d[2];
      }
    }
  }
  // every cell of the patch active: the window weights need no mask and sum
  // to (sum of taps)^2 everywhere
  const bool full = __syncthreads_and(mine_full);
  // this thread's pixel: nested local index tid (slot order of a full tile)
  const int px = (int)hp_compact_bits((uint32_t)tid), py = (int)hp_compact_bits((uint32_t)tid >> 1);
  const bool own = tid < B * B;
  float xc[3] = {0.f, 0.f, 0.f}, yc[3] = {0.f, 0.f, 0.f};
  if (own) {
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      xc[ch] = s.in[1 + ch][py + SS_R][px + SS_R];
      yc[ch] = s.in[4 + ch][py + SS_R][px + SS_R];
    }
  }
  float Sm[16];
  if constexpr (!kSmall) if (!direct) {
    // pass 1 along x: item (row r, channel ch, third k) slides the window over
    // the cells behind its kOut outputs; the items of a tile fit one round of the workgroup
    constexpr int kOut = B == 16 ? 6 : 4, Q = (B + kOut - 1) / kOut, NI1 = H * 3 * Q, kIn = kOut + 2 * SS_R;
    static_assert(NI1 <= 256 && kIn % 2 == 0, "one item per thread, cells read in pairs");
    float o[6][kOut];
    const int r1 = tid / (3 * Q), rem1 = tid % (3 * Q), ch1 = rem1 / Q, c1 = kOut * (rem1 % Q);
    if (tid < NI1) {
      // (cells past the row's end, read by the last item of a row, go to outputs past it)
      float m[kIn], x[kIn], y[kIn];
      const float2* pm = reinterpret_cast<const float2*>(&s.in[0][r1][c1]);
      const float2* px2 = reinterpret_cast<const float2*>(&s.in[1 + ch1][r1][c1]);
      const float2* py2 = reinterpret_cast<const float2*>(&s.in[4 + ch1][r1][c1]);
#pragma unroll
      for (int j = 0; j < kIn; j += 2) {
        const float2 a = pm[j / 2], bx = px2[j / 2], by = py2[j / 2];
        m[j] = a.x; m[j + 1] = a.y;
        x[j] = bx.x; x[j + 1] = bx.y;
        y[j] = by.x; y[j + 1] = by.y;
      }
#pragma unroll
      for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int u = 0; u < kOut; ++u) o[k][u] = 0.f;
      if (full) {
        // m = 1 everywhere: no mask products, no weight sums
#pragma unroll
        for (int j = 0; j < kIn; ++j) {
          const float q5[5] = {x[j], y[j], x[j] * x[j], y[j] * y[j], x[j] * y[j]};
#pragma unroll
          for (int u = 0; u < kOut; ++u) {
            const int a = j - u;
            if (a >= 0 && a < SS_W) {
#pragma unroll
              for (int k = 0; k < 5; ++k) o[1 + k][u] = fmaf(A.g[a], q5[k], o[1 + k][u]);
            }
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < kIn; ++j) {
          const float wx = m[j] * x[j], wy = m[j] * y[j];
          const float q5[6] = {m[j], wx, wy, wx * x[j], wy * y[j], wx * y[j]};
#pragma unroll
          for (int u = 0; u < kOut; ++u) {
            const int a = j - u;
            if (a >= 0 && a < SS_W) {
#pragma unroll
              for (int k = 0; k < 6; ++k) o[k][u] = fmaf(A.g[a], q5[k], o[k][u]);
            }
          }
        }
      }
    }
    __syncthreads();  // every read of the patch is done
    if (tid < NI1) {
      // quantity index: 0 weight, 1+ch x, 4+ch y, 7+ch xx, 10+ch yy, 13+ch xy
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        if (k == 0 && (ch1 != 0 || full)) continue;
        float2* out = reinterpret_cast<float2*>(&s.p1[k == 0 ? 0 : 1 + 3 * (k - 1) + ch1][r1 * B + c1]);
#pragma unroll
        for (int u = 0; u < kOut; u += 2)
          if (c1 + u < B) out[u / 2] = make_float2(o[k][u], o[k][u + 1]);
      }
    }
    __syncthreads();
    // pass 2 along y: item (column c, quantity k, half hh) slides over the
    // B/2 + 10 rows behind its B/2 outputs
    constexpr int RO = B / 2, NI2 = B * 16 * 2, T2 = NI2 / 256;
    float o2[T2][RO];
#pragma unroll
    for (int t = 0; t < T2; ++t) {
      const int it = tid + 256 * t;
      const int c = it % B, k = (it / B) % 16, hh = it / (16 * B);
      float w[RO + 2 * SS_R];
#pragma unroll
      for (int j = 0; j < RO + 2 * SS_R; ++j) w[j] = s.p1[k][(hh * RO + j) * B + c];
#pragma unroll
      for (int u = 0; u < RO; ++u) {
        float acc = 0.f;
#pragma unroll
        for (int a = 0; a < SS_W; ++a) acc = fmaf(A.g[a], w[u + a], acc);
        o2[t][u] = acc;
      }
    }
    __syncthreads();  // every read of the first pass's output is done
#pragma unroll
    for (int t = 0; t < T2; ++t) {
      const int it = tid + 256 * t;
      const int c = it % B, k = (it / B) % 16, hh = it / (16 * B);
#pragma unroll
      for (int u = 0; u < RO; ++u) S[k][ss_nest_local(c, hh * RO + u)] = o2[t][u];  // nested order: read back by pixel tid
    }
    __syncthreads();
    if (own) {
#pragma unroll
      for (int k = 0; k < 16; ++k) Sm[k] = S[k][tid];
      if (full) Sm[0] = A.gsum * A.gsum;
    }
  }
  const bool paired = B == 16 && ZONES && direct && A.fine;
  if constexpr (B == 16 && ZONES) if (paired) {
    const int half = (int)hp_uniform((uint32_t)tid >> 7);
    const int x = tid & 15, yp = 2 * ((tid & 127) >> 4);
    const bool pol[2] = {ss_polar(A.order, hp_xyf_nest(A.order, x0 + x, y0 + yp, f)),
                         ss_polar(A.order, hp_xyf_nest(A.order, x0 + x, y0 + yp + 1, f))};
    const bool pure = __builtin_amdgcn_ballot_w64(!pol[0] || !pol[1]) == 0;
    double h[2][3];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int c = 0; c < 3; ++c) h[j][c] = -0.5 * s.dir[c][(yp + j + SS_R) * H + x + SS_R];
    float P[2][16];
#pragma unroll
    for (int k = 0; k < 16; ++k) P[0][k] = P[1][k] = 0.f;
    auto rows = [&](auto pure_tag) {
      ss_pair_rows(half, [&](int b, auto up, auto low) {
        constexpr bool on[2] = {decltype(up)::value, decltype(low)::value};
        const int cell = (yp + b) * H + x, at = (yp + b) * L::HP + x;
        const float* in = &s.in[0][0][0] + at;
#pragma unroll 1
        for (int a = 0; a < SS_W; ++a) {
          const double vx = s.dir[0][cell + a], vy = s.dir[1][cell + a], vz = s.dir[2][cell + a];
          float m, xv[3], yv[3], xx[3], yy[3], xy[3];
          m = in[a];
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) {
            xv[ch] = in[(1 + ch) * H * L::HP + a];
            yv[ch] = in[(4 + ch) * H * L::HP + a];
            xx[ch] = xv[ch] * xv[ch];
            yy[ch] = yv[ch] * yv[ch];
            xy[ch] = xv[ch] * yv[ch];
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            if (!on[j]) continue;
            float w = ss_polar_weight(A, h[j], vx, vy, vz);
            if constexpr (!decltype(pure_tag)::value) w = pol[j] ? w : A.g[a] * A.g[b - j];
            P[j][0] = fmaf(w, m, P[j][0]);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) {
              P[j][1 + ch] = fmaf(w, xv[ch], P[j][1 + ch]);
              P[j][4 + ch] = fmaf(w, yv[ch], P[j][4 + ch]);
              P[j][7 + ch] = fmaf(w, xx[ch], P[j][7 + ch]);
              P[j][10 + ch] = fmaf(w, yy[ch], P[j][10 + ch]);
              P[j][13 + ch] = fmaf(w, xy[ch], P[j][13 + ch]);
            }
          }
        }
      });
    };
    if (pure) rows(SsBool<true>{});
    else rows(SsBool<false>{});
    // the halves' sums meet in LDS, over the patch
    const int n0 = ss_nest_local(x, yp), n1 = ss_nest_local(x, yp + 1);
    __syncthreads();
    if (half == 0) {
#pragma unroll
      for (int k = 0; k < 16; ++k) { S[k][n0] = P[0][k]; S[k][n1] = P[1][k]; }
    }
    __syncthreads();
    if (half != 0) {
#pragma unroll
      for (int k = 0; k < 16; ++k) { S[k][n0] += P[0][k]; S[k][n1] += P[1][k]; }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) Sm[k] = S[k][tid];
  }
  if (direct && !paired) {
    // direct 121-tap sums: polar pixels (zone windows) weigh by great-circle
    // distance, the others by the chart window
#pragma unroll
    for (int k = 0; k < 16; ++k) Sm[k] = 0.f;
    if (own) {
      const bool polar = ZONES && ss_polar(A.order, hp_xyf_nest(A.order, x0 + px, y0 + py, f));
      const int cp = ZONES ? (py + SS_R) * H + px + SS_R : 0;
      const double up[3] = {s.dir[0][cp], s.dir[1][cp], s.dir[2][cp]};
      for (int b = 0; b < SS_W; ++b) {
        for (int a = 0; a < SS_W; ++a) {
          const int cy = py + b, cx = px + a;
          const float m = s.in[0][cy][cx];
          if (m == 0.f) continue;
          float xs[3], ys[3];  // read before the weight, whose chain is long
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) {
            xs[ch] = s.in[1 + ch][cy][cx];
            ys[ch] = s.in[4 + ch][cy][cx];
          }
          float w = m * (A.g[a] * A.g[b]);
          if (polar) {
            const int cq = ZONES ? cy * H + cx : 0;
            const double uq[3] = {s.dir[0][cq], s.dir[1][cq], s.dir[2][cq]};
            w = m * __expf(-(float)(ss_dist2(up, uq) * A.wscale));
          }
          Sm[0] += w;
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) {
            const float x = xs[ch], y = ys[ch];
            const float wx = w * x, wy = w * y;
            Sm[1 + ch] += wx;
            Sm[4 + ch] += wy;
            Sm[7 + ch] = fmaf(wx, x, Sm[7 + ch]);
            Sm[10 + ch] = fmaf(wy, y, Sm[10 + ch]);
            Sm[13 + ch] = fmaf(wx, y, Sm[13 + ch]);
          }
        }
      }
    }
  }
  int64_t slot = -1;
  float gl[kSsG] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (own) {
    slot = ss_slot(A, hp_xyf_nest(A.order, x0 + px, y0 + py, f));
    if (slot >= 0) {
      const float iZ = __builtin_amdgcn_rcpf(Sm[0]);
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        const float sv = ss_index(A.C1, A.C2, iZ, Sm[1 + ch], Sm[4 + ch], Sm[7 + ch], Sm[10 + ch], Sm[13 + ch],
                                  &gl[ch], &gl[3 + ch], &gl[6 + ch]);
        ssum += sv;
        lsum += fabsf(xc[ch] - yc[ch]);
        if (smap) smap[ch * A.n_active + slot] = sv;
      }
    }
  }
  if (G) {
    // the tile's partials leave as one contiguous run: its active pixels
    // hold the slots [start, start + count) (staged in LDS over the first
    // pass's place, once every thread is done reading it)
    const int t = A.active_tiles[ct];
    const int64_t start = A.tile_start[t];
    const int cnt = A.tile_count[t];
    float4* stage = reinterpret_cast<float4*>(&s.p1[0][0]);
    __syncthreads();
    if (slot >= 0) {
      const int loc = (int)(slot - start);
      stage[3 * loc] = make_float4(gl[0], gl[1], gl[2], gl[3]);
      stage[3 * loc + 1] = make_float4(gl[4], gl[5], gl[6], gl[7]);
      stage[3 * loc + 2] = make_float4(gl[8], 0.f, 0.f, 0.f);
    }
    __syncthreads();
    float4* out = reinterpret_cast<float4*>(G + start * kSsG);
    for (int i = tid; i < 3 * cnt; i += 256) out[i] = stage[i];
  }
  // the tile's (sum of SSIM, sum of |img - ref|)
  float red[2] = {ssum, lsum};
  hp_wave_totals<2>(red);
  if (hp_lane() == 0) { s_red[0][tid >> 6] = red[0]; s_red[1][tid >> 6] = red[1]; }
  __syncthreads();
  if (tid == 0)
    part[blockIdx.x] = make_float2(s_red[0][0] + s_red[0][1] + s_red[0][2] + s_red[0][3],
                                   s_red[1][0] + s_red[1][1] + s_red[1][2] + s_red[1][3]);
}

// Sums over the n partials of the tiles.  Bound by how many cache lines one
// compute unit waits for at a time: a workgroup that reads them all, two partials
// a load, takes 4.7 us at 12,288 (one a load: 5.7), 13.1 at 49,152 and 48 at
// 196,608; from kSsReduce on each piece of 1,024 is summed by its own workgroup
// first (4.6 us, left in 64 bits over the piece's first entries), and
// k_ssim_reduce takes 4.6 us more.
constexpr int kSsReduce = 16384, kSsPiece = 1024;
__global__ __launch_bounds__(256) void k_ssim_pieces(float2* __restrict__ part, int n) {
  __shared__ double s[2][4];
  float2* mine = part + kSsPiece * (int64_t)blockIdx.x;
  const int m = min(n - kSsPiece * (int)blockIdx.x, kSsPiece);
  float2 p[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = (int)threadIdx.x + 256 * j;
    p[j] = i < m ? mine[i] : make_float2(0.f, 0.f);
  }
  double a = 0, b = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) { a += p[j].x; b += p[j].y; }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
  }
  if (hp_lane() == 0) { s[0][threadIdx.x >> 6] = a; s[1][threadIdx.x >> 6] = b; }
  __syncthreads();  // every read of the piece is done
  if (threadIdx.x == 0) {
    double* out = reinterpret_cast<double*>(mine);
    out[0] = s[0][0] + s[0][1] + s[0][2] + s[0][3];
    // (a last piece of one entry is not the last of the array, whose length, 12 4^k
    // of at least 49,152, is a multiple of the piece's)
    out[1] = s[1][0] + s[1][1] + s[1][2] + s[1][3];
  }
}

// single block: mean SSIM, mean L1, loss
template <bool PIECES>
__global__ __launch_bounds__(1024) void k_ssim_reduce(const float2* __restrict__ part, int n, int64_t n_active,
                                                      float lam, float* __restrict__ out) {
  __shared__ double s[2][16];
  double a = 0, b = 0;
  if (PIECES) {
    for (int i = threadIdx.x; i < (n + kSsPiece - 1) / kSsPiece; i += 1024) {
      const double* p = reinterpret_cast<const double*>(part + kSsPiece * (int64_t)i);
      a += p[0];
      b += p[1];
    }
  } else {
    const float4* p2 = reinterpret_cast<const float4*>(part);
    for (int i = threadIdx.x; i < n / 2; i += 1024) {
      const float4 p = p2[i];
      a += (double)p.x + p.z;
      b += (double)p.y + p.w;
    }
    if ((n & 1) != 0 && threadIdx.x == 0) {
      a += part[n - 1].x;
      b += part[n - 1].y;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
  }
  if (hp_lane() == 0) { s[0][threadIdx.x >> 6] = a; s[1][threadIdx.x >> 6] = b; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sa = 0, sb = 0;
    for (int k = 0; k < 16; ++k) { sa += s[0][k]; sb += s[1][k]; }
    const double nn = 3.0 * (double)n_active;
    const double ssim = sa / nn, l1 = sb / nn;
    out[0] = (float)ssim;
    out[1] = (float)l1;
    out[2] = (float)((1.0 - lam) * l1 + lam * (1.0 - ssim));
  }
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// The gathered patch; once the first pass has read it (the pass keeps its
// outputs in registers until then), its output [9][P1S] and after that the
// second pass's sums [9][B*B] overlay it.  The cells' directions and polar
// flags are only needed with zone windows.
template <int B, bool ZONES>
struct SsBwdLds {
  static constexpr int H = B + 2 * SS_R, HP = (H + 3) & ~3, P1S = H * B + ((48 - (H * B) % 32) % 32);
  static_assert(B < 8 || 9 * P1S + 9 * B * B <= 9 * H * HP, "first-pass output and sums fit over the patch");
  float in[9][H][HP];
  double dir[3][ZONES ? H * H : 1];
  uint8_t polar[ZONES ? H * H : 1];
};

// A workgroup per tile, six per CU (26 KB of LDS, 42 registers): 71 us at 3.1 M
// pixels, 83 us with four that fetched the next tile's partials meanwhile.
// dL/dimg_p = dL/dloss * [ (1 - lam) sign(img - ref) / (3n)
//   - lam / (3n) * sum_{q in W(p)} w_q(p) (G0_q + 2 x_p G1_q + y_p G2_q) ]
// with w_q(p) the raw weight of q's window at p
template <int B, bool ZONES>
__global__ __launch_bounds__(256, ZONES ? 3 : 6) void k_ssim_bwd(SsimArgs A, const float* __restrict__ img,
                                                  const float* __restrict__ ref, const float* __restrict__ G,
                                                  const float* __restrict__ dL_dloss, float* __restrict__ dimg,
                                                  int n_tiles) {
  using L = SsBwdLds<B, ZONES>;
  constexpr int H = L::H;
  __shared__ L s;
  // over the patch: the first pass's output, then the second pass's sums
  float(*P1)[L::P1S] = reinterpret_cast<float(*)[L::P1S]>(&s.in[0][0][0]);
  float(*S)[B * B] = reinterpret_cast<float(*)[B * B]>(&s.in[0][0][0] + 9 * L::P1S);
  const int tid = threadIdx.x;
  constexpr int NG = (H * H + 255) / 256;
  const int ct = ZONES ? hp_xcd_group_tile(blockIdx.x, n_tiles) : hp_xcd_tile(blockIdx.x, n_tiles);
  const int32_t* tab = A.tables + (int64_t)ct * (H * H);
  int32_t e[NG];
  float v[NG][9];
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    const int i = tid + 256 * gi;
    e[gi] = i < H * H ? tab[i] : -1;
  }
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    const int64_t slot = e[gi] & kSsSlotMask;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a, c = a;
    if (e[gi] >= 0) {
      const float4* gp = reinterpret_cast<const float4*>(G + slot * kSsG);
      a = gp[0]; b = gp[1]; c = gp[2];
    }
    v[gi][0] = a.x; v[gi][1] = a.y; v[gi][2] = a.z; v[gi][3] = a.w;
    v[gi][4] = b.x; v[gi][5] = b.y; v[gi][6] = b.z; v[gi][7] = b.w;
    v[gi][8] = c.x;
  }
  int f, x0, y0;
  ss_tile_origin(A, ct, &f, &x0, &y0);
  bool any_polar = false, all_polar = true;  // all_polar: of the active cells
#pragma unroll
  for (int gi = 0; gi < NG; ++gi) {
    const int i = tid + 256 * gi;
    if (i < H * H) {
      int cx, cy;
      ss_cell<B>(i, &cx, &cy);
#pragma unroll
      for (int k = 0; k < 9; ++k) s.in[k][cy][cx] = v[gi][k];
      if (ZONES) {
        const bool pq = e[gi] >= 0 && (e[gi] & kSsPolarBit) != 0;
        s.polar[cy * H + cx] = pq ? 1 : 0;
        any_polar |= pq;
        all_polar &= pq || e[gi] < 0;
      }
    }
  }
  // the separable pass needs every neighbour's window to be the chart one;
  // tiles narrower than 8 pixels always take the direct path
  constexpr bool kSmall = B < 8;
  bool direct = kSmall;
  bool pure = false;  // every window of the patch is a polar one
  if (ZONES) {
    pure = __syncthreads_and(all_polar);
    direct = __syncthreads_or(any_polar) || kSmall;
  } else {
    __syncthreads();
  }
  const int px = (int)hp_compact_bits((uint32_t)tid), py = (int)hp_compact_bits((uint32_t)tid >> 1);
  float Sm[9];
  if constexpr (!kSmall) if (!direct) {
    constexpr int Q = B / 4, NI1 = H * 9 * Q;
    float o[4][4];  // up to 4 items per thread, 4 outputs each
    int kk[4], rr[4], cc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int it = tid + 256 * t;
      kk[t] = -1;
      if (it < NI1) {
        const int r = it / (9 * Q), rem = it % (9 * Q), k = rem / Q, c0 = 4 * (rem % Q);
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; j += 4) {
          const float4 a = *reinterpret_cast<const float4*>(&s.in[k][r][c0 + j]);
          v[j] = a.x; v[j + 1] = a.y; v[j + 2] = a.z; v[j + 3] = a.w;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float acc = 0.f;
#pragma unroll
          for (int a = 0; a < SS_W; ++a) acc = fmaf(A.g[a], v[u + a], acc);
          o[t][u] = acc;
        }
        kk[t] = k; rr[t] = r; cc[t] = c0;
      }
    }
    __syncthreads();  // every read of the patch is done: the output goes over it
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (kk[t] >= 0)
        *reinterpret_cast<float4*>(&P1[kk[t]][rr[t] * B + cc[t]]) = make_float4(o[t][0], o[t][1], o[t][2], o[t][3]);
    __syncthreads();
    constexpr int RO = B / 2, NI2 = B * 9 * 2;
    for (int it = tid; it < NI2; it += 256) {
      const int c = it % B, k = (it / B) % 9, hh = it / (9 * B);
      float w[RO + 2 * SS_R];
#pragma unroll
      for (int j = 0; j < RO + 2 * SS_R; ++j) w[j] = P1[k][(hh * RO + j) * B + c];
#pragma unroll
      for (int u = 0; u < RO; ++u) {
        float acc = 0.f;
#pragma unroll
        for (int a = 0; a < SS_W; ++a) acc = fmaf(A.g[a], w[u + a], acc);
        S[k][ss_nest_local(c, hh * RO + u)] = acc;
      }
    }
    __syncthreads();
    if (tid < B * B) {
#pragma unroll
      for (int k = 0; k < 9; ++k) Sm[k] = S[k][tid];
    }
  }
  if (direct) {
    // directions of the patch cells, for the polar windows
    if (ZONES) {
      for (int i = tid; i < H * H; i += 256) {
        const int cx = i % H, cy = i / H;
        const int64_t q = hp_chart_pixel(A.order, f, x0 + cx - SS_R, y0 + cy - SS_R);
        double d[3] = {0.0, 0.0, 0.0};
        if (q >= 0) hp_pix_dir(A.order, q, d);
        s.dir[0][i] = d[0];
        s.dir[1][i] = d[1];
        s.dir[2][i] = d[2];
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) Sm[k] = 0.f;
    const bool paired = B == 16 && ZONES && A.fine;
    if constexpr (B == 16 && ZONES) if (paired) {
      const int half = (int)hp_uniform((uint32_t)tid >> 7);
      const int x = tid & 15, yp = 2 * ((tid & 127) >> 4);
      double h[2][3];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int c = 0; c < 3; ++c) h[j][c] = -0.5 * s.dir[c][(yp + j + SS_R) * H + x + SS_R];
      float P[2][9];
#pragma unroll
      for (int k = 0; k < 9; ++k) P[0][k] = P[1][k] = 0.f;
      auto rows = [&](auto pure_tag) {
        ss_pair_rows(half, [&](int b, auto up, auto low) {
          constexpr bool on[2] = {decltype(up)::value, decltype(low)::value};
          const int cell = (yp + b) * H + x, at = (yp + b) * L::HP + x;
          const float* in = &s.in[0][0][0] + at;
#pragma unroll 1
          for (int a = 0; a < SS_W; ++a) {
            const double vx = s.dir[0][cell + a], vy = s.dir[1][cell + a], vz = s.dir[2][cell + a];
            const bool pol = decltype(pure_tag)::value || s.polar[cell + a] != 0;
            float g[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) g[k] = in[k * H * L::HP + a];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              if (!on[j]) continue;
              float w = ss_polar_weight(A, h[j], vx, vy, vz);
              if constexpr (!decltype(pure_tag)::value) w = pol ? w : A.g[a] * A.g[b - j];
#pragma unroll
              for (int k = 0; k < 9; ++k) P[j][k] = fmaf(w, g[k], P[j][k]);
            }
          }
        });
      };
      if (pure) rows(SsBool<true>{});
      else rows(SsBool<false>{});
      const int n0 = ss_nest_local(x, yp), n1 = ss_nest_local(x, yp + 1);
      __syncthreads();
      if (half == 0) {
#pragma unroll
        for (int k = 0; k < 9; ++k) { S[k][n0] = P[0][k]; S[k][n1] = P[1][k]; }
      }
      __syncthreads();
      if (half != 0) {
#pragma unroll
        for (int k = 0; k < 9; ++k) { S[k][n0] += P[0][k]; S[k][n1] += P[1][k]; }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 9; ++k) Sm[k] = S[k][tid];
    }
    if (!paired && tid < B * B) {
      const int cp = ZONES ? (py + SS_R) * H + px + SS_R : 0;
      const double up[3] = {s.dir[0][cp], s.dir[1][cp], s.dir[2][cp]};
      for (int b = 0; b < SS_W; ++b) {
        for (int a = 0; a < SS_W; ++a) {
          const int cy = py + b, cx = px + a, cq = ZONES ? cy * H + cx : 0;
          // q's own window at p: the great-circle Gaussian for a polar q,
          // the (symmetric) chart taps otherwise
          float w = A.g[a] * A.g[b];
          if (ZONES && s.polar[cq]) {
            const double uq[3] = {s.dir[0][cq], s.dir[1][cq], s.dir[2][cq]};
            w = __expf(-(float)(ss_dist2(up, uq) * A.wscale));
          }
#pragma unroll
          for (int k = 0; k < 9; ++k) Sm[k] = fmaf(w, s.in[k][cy][cx], Sm[k]);
        }
      }
    }
  }
  const int64_t slot = tid < B * B ? ss_slot(A, hp_xyf_nest(A.order, x0 + px, y0 + py, f)) : -1;
  if (slot >= 0) {
    const float up = *dL_dloss;
    const float inv3n = 1.f / (3.f * (float)A.n_active);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float x = img[ch * A.n_active + slot], y = ref[ch * A.n_active + slot];
      const float dssim = Sm[0 * 3 + ch] + 2.f * x * Sm[1 * 3 + ch] + y * Sm[2 * 3 + ch];
      const float sgn = (float)((x > y) - (x < y));
      dimg[ch * A.n_active + slot] = up * inv3n * ((1.f - A.lam) * sgn - A.lam * dssim);
    }
  }
}

// Patch tables: for every active tile and patch cell (in gather order), the
// compact slot of the chart neighbour (-1: missing or inactive), with bit 30
// set when that neighbour lies in a polar cap.  Image independent: built once
// per mask and reused by every forward and backward.
template <int B>
__global__ __launch_bounds__(256) void k_ssim_tables(SsimArgs A, int32_t* __restrict__ tables) {
  constexpr int H = B + 2 * SS_R;
  const int ct = blockIdx.x;
  int f, x0, y0;
  ss_tile_origin(A, ct, &f, &x0, &y0);
  for (int i = threadIdx.x; i < H * H; i += 256) {
    int cx, cy;
    ss_cell<B>(i, &cx, &cy);
    const int64_t q = hp_chart_pixel(A.order, f, x0 + cx - SS_R, y0 + cy - SS_R);
    const int64_t slot = ss_slot(A, q);
    tables[(int64_t)ct * H * H + i] = slot < 0 ? -1 : ((int32_t)slot | (ss_polar(A.order, q) ? kSsPolarBit : 0));
  }
}

static int ss_patch(int b) { const int H = (1 << b) + 2 * SS_R; return H * H; }

static size_t ssim_ws_size(int64_t n_active, int64_t ntile) {
  return hp_align256((size_t)kSsG * n_active * 4) + hp_align256((size_t)ntile * sizeof(float2));
}

extern "C" size_t hp_ssim_workspace_bytes(int32_t order, int32_t tile_log2, int64_t n_active) {
  if (order < 0 || order > HP_MAX_ORDER || tile_log2 < 0 || tile_log2 > 4 || n_active < 0) return 0;
  return ssim_ws_size(n_active, hp_geom(order, tile_log2).ntile);
}

extern "C" size_t hp_ssim_tables_bytes(int32_t order, int32_t tile_log2, int32_t n_tiles) {
  if (order < 0 || order > HP_MAX_ORDER || tile_log2 < 0 || tile_log2 > 4 || n_tiles < 0) return 0;
  return hp_align256((size_t)n_tiles * ss_patch(hp_geom(order, tile_log2).b) * 4);
}

static hp_status ssim_mask_args(int32_t order, const hp_params* prm, const void* mask, int64_t n_active,
                                int32_t n_tiles, SsimArgs* A) {
  HP_TRY(hp_check_params(prm));
  if (!mask) return HP_ERR_INVALID_ARG;
  if (order < 0 || order > HP_MAX_ORDER) return HP_ERR_INVALID_ARG;
  const HpGeom g = hp_geom(order, prm->tile_log2);
  // tiles of 1 to 16 pixels a side (tiles under 8 pixels take the direct path)
  if (g.b < 0 || g.b > 4) return HP_ERR_UNSUPPORTED;
  if (n_tiles <= 0 || n_tiles > g.ntile || n_active <= 0 || n_active > g.npix) return HP_ERR_INVALID_ARG;
  const HpMaskView mv = hp_mask_view((const char*)mask, g);
  A->order = order; A->b = g.b; A->kt = g.kt;
  A->active_tiles = mv.active_tiles; A->tile_start = mv.tile_start; A->tile_count = mv.tile_count;
  A->tile_bits = mv.tile_bits; A->n_active = n_active;
  return HP_OK;
}

extern "C" hp_status hp_ssim_tables(const hp_params* prm, const void* mask, int32_t order, int64_t n_active,
                                    int32_t n_tiles, int32_t* tables, size_t tables_bytes, void* stream) {
  SsimArgs A;
  HP_TRY(ssim_mask_args(order, prm, mask, n_active, n_tiles, &A));
  if (!tables) return HP_ERR_INVALID_ARG;
  if (tables_bytes < hp_ssim_tables_bytes(order, prm->tile_log2, n_tiles)) return HP_ERR_CAPACITY;
  hipStream_t s = (hipStream_t)stream;
  switch (A.b) {
    case 4: hipLaunchKernelGGL(k_ssim_tables<16>, dim3((unsigned)n_tiles), dim3(256), 0, s, A, tables); break;
    case 3: hipLaunchKernelGGL(k_ssim_tables<8>, dim3((unsigned)n_tiles), dim3(256), 0, s, A, tables); break;
    case 2: hipLaunchKernelGGL(k_ssim_tables<4>, dim3((unsigned)n_tiles), dim3(256), 0, s, A, tables); break;
    case 1: hipLaunchKernelGGL(k_ssim_tables<2>, dim3((unsigned)n_tiles), dim3(256), 0, s, A, tables); break;
    default: hipLaunchKernelGGL(k_ssim_tables<1>, dim3((unsigned)n_tiles), dim3(256), 0, s, A, tables); break;
  }
  HP_CHECK_LAUNCH();
  return HP_OK;
}

// shared argument checks and set-up of the three entry points
static hp_status ssim_setup(const float* img, const float* ref, int64_t n_active, int32_t n_tiles, int32_t order,
                            const hp_params* prm, const hp_ssim_params* sp, const void* mask, const int32_t* tables,
                            const void* ws, size_t ws_bytes, SsimArgs* A, float** Gm, float2** part) {
  HP_TRY(ssim_mask_args(order, prm, mask, n_active, n_tiles, A));
  if (!sp || !ws || !tables || !img || !ref) return HP_ERR_INVALID_ARG;
  if (!(sp->sigma > 0) || !(sp->C1 > 0) || !(sp->C2 > 0) || !(sp->lambda >= 0 && sp->lambda <= 1) ||
      (sp->zones != 0 && sp->zones != 1))
    return HP_ERR_INVALID_ARG;
  const HpGeom g = hp_geom(order, prm->tile_log2);
  if (ws_bytes < ssim_ws_size(n_active, g.ntile)) return HP_ERR_CAPACITY;
  A->tables = tables;
  A->C1 = sp->C1; A->C2 = sp->C2; A->lam = sp->lambda;
  A->gsum = 0.f;
  for (int a = 0; a < SS_W; ++a) {
    const double d = a - SS_R;
    A->g[a] = (float)exp(-d * d / (2.0 * (double)sp->sigma * (double)sp->sigma));
    A->gsum += A->g[a];
  }
  const double omega = 4.0 * M_PI / (double)g.npix;
  A->wscale = 1.0 / (2.0 * (double)sp->sigma * (double)sp->sigma * omega);
  // exp(-d^2 wscale) = 2^(w2[0] s^2 + w2[1] s^4 + w2[2] s^6), d^2 = 4 s^2 (1 + s^2 / 3 + 8 s^4 / 45 ...)
  A->w2[0] = -4.0 * A->wscale * 1.44269504088896340736;
  A->w2[1] = A->w2[0] / 3.0;
  A->w2[2] = A->w2[0] * (8.0 / 45.0);
  A->fine = order >= kSsFineOrder && A->w2[0] * -5e-16 <= 6e-8;
  *Gm = (float*)ws;
  *part = (float2*)((char*)ws + hp_align256((size_t)kSsG * n_active * 4));
  return HP_OK;
}

template <int B>
static hp_status ssim_fwd_launch_b(const SsimArgs& A, bool zones, const float* img, const float* ref,
                                   int32_t n_tiles, float* ssim_map, float* Gm, float2* part, hipStream_t s) {
  const dim3 grid((unsigned)n_tiles);
  if (zones)
    hipLaunchKernelGGL((k_ssim_fwd<B, true>), grid, dim3(256), 0, s, A, img, ref, ssim_map, Gm, part, (int)n_tiles);
  else
    hipLaunchKernelGGL((k_ssim_fwd<B, false>), grid, dim3(256), 0, s, A, img, ref, ssim_map, Gm, part, (int)n_tiles);
  HP_CHECK_LAUNCH();
  return HP_OK;
}

static hp_status ssim_fwd_launch(const SsimArgs& A, bool zones, const float* img, const float* ref, int32_t n_tiles,
                                 float lam, float* out, float* ssim_map, float* Gm, float2* part, hipStream_t s) {
  switch (A.b) {
    case 4: HP_TRY(ssim_fwd_launch_b<16>(A, zones, img, ref, n_tiles, ssim_map, Gm, part, s)); break;
    case 3: HP_TRY(ssim_fwd_launch_b<8>(A, zones, img, ref, n_tiles, ssim_map, Gm, part, s)); break;
    case 2: HP_TRY(ssim_fwd_launch_b<4>(A, zones, img, ref, n_tiles, ssim_map, Gm, part, s)); break;
    case 1: HP_TRY(ssim_fwd_launch_b<2>(A, zones, img, ref, n_tiles, ssim_map, Gm, part, s)); break;
    default: HP_TRY(ssim_fwd_launch_b<1>(A, zones, img, ref, n_tiles, ssim_map, Gm, part, s)); break;
  }
  // one partial per forward workgroup
  if (n_tiles > kSsReduce) {
    hipLaunchKernelGGL(k_ssim_pieces, dim3(hp_blocks(n_tiles, kSsPiece)), dim3(256), 0, s, part, (int)n_tiles);
    HP_CHECK_LAUNCH();
    hipLaunchKernelGGL(k_ssim_reduce<true>, dim3(1), dim3(1024), 0, s, (const float2*)part, (int)n_tiles, A.n_active,
                       lam, out);
  } else {
    hipLaunchKernelGGL(k_ssim_reduce<false>, dim3(1), dim3(1024), 0, s, (const float2*)part, (int)n_tiles, A.n_active,
                       lam, out);
  }
  HP_CHECK_LAUNCH();
  return HP_OK;
}

template <int B>
static hp_status ssim_bwd_launch_b(const SsimArgs& A, bool zones, const float* img, const float* ref,
                                   int32_t n_tiles, const float* Gm, const float* dL_dloss, float* dL_dimg,
                                   hipStream_t s) {
  const dim3 grid((unsigned)n_tiles);
  if (zones)
    hipLaunchKernelGGL((k_ssim_bwd<B, true>), grid, dim3(256), 0, s, A, img, ref, Gm, dL_dloss, dL_dimg, (int)n_tiles);
  else
    hipLaunchKernelGGL((k_ssim_bwd<B, false>), grid, dim3(256), 0, s, A, img, ref, Gm, dL_dloss, dL_dimg,
                       (int)n_tiles);
  HP_CHECK_LAUNCH();
  return HP_OK;
}

static hp_status ssim_bwd_launch(const SsimArgs& A, bool zones, const float* img, const float* ref, int32_t n_tiles,
                                 const float* Gm, const float* dL_dloss, float* dL_dimg, hipStream_t s) {
  switch (A.b) {
    case 4: return ssim_bwd_launch_b<16>(A, zones, img, ref, n_tiles, Gm, dL_dloss, dL_dimg, s);
    case 3: return ssim_bwd_launch_b<8>(A, zones, img, ref, n_tiles, Gm, dL_dloss, dL_dimg, s);
    case 2: return ssim_bwd_launch_b<4>(A, zones, img, ref, n_tiles, Gm, dL_dloss, dL_dimg, s);
    case 1: return ssim_bwd_launch_b<2>(A, zones, img, ref, n_tiles, Gm, dL_dloss, dL_dimg, s);
    default: return ssim_bwd_launch_b<1>(A, zones, img, ref, n_tiles, Gm, dL_dloss, dL_dimg, s);
  }
}

extern "C" hp_status hp_ssim(const float* img, const float* ref, int64_t n_active, int32_t n_tiles, int32_t order,
                             const hp_params* prm, const hp_ssim_params* sp, const void* mask, const int32_t* tables,
                             float* out, float* ssim_map, const float* dL_dloss, float* dL_dimg, void* ws,
                             size_t ws_bytes, void* stream) {
  SsimArgs A;
  float* Gm;
  float2* part;
  HP_TRY(ssim_setup(img, ref, n_active, n_tiles, order, prm, sp, mask, tables, ws, ws_bytes, &A, &Gm, &part));
  if (!out || (dL_dloss && !dL_dimg)) return HP_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const bool zones = sp->zones != 0;
  HP_TRY(ssim_fwd_launch(A, zones, img, ref, n_tiles, sp->lambda, out, ssim_map, dL_dloss ? Gm : nullptr, part, s));
  if (dL_dloss) HP_TRY(ssim_bwd_launch(A, zones, img, ref, n_tiles, Gm, dL_dloss, dL_dimg, s));
  return HP_OK;
}

extern "C" hp_status hp_ssim_forward_saved(const float* img, const float* ref, int64_t n_active, int32_t n_tiles,
                                           int32_t order, const hp_params* prm, const hp_ssim_params* sp,
                                           const void* mask, const int32_t* tables, float* out, float* ssim_map,
                                           void* ws, size_t ws_bytes, void* stream) {
  SsimArgs A;
  float* Gm;
  float2* part;
  HP_TRY(ssim_setup(img, ref, n_active, n_tiles, order, prm, sp, mask, tables, ws, ws_bytes, &A, &Gm, &part));
  if (!out) return HP_ERR_INVALID_ARG;
  return ssim_fwd_launch(A, sp->zones != 0, img, ref, n_tiles, sp->lambda, out, ssim_map, Gm, part,
                         (hipStream_t)stream);
}

extern "C" hp_status hp_ssim_backward_saved(const float* img, const float* ref, int64_t n_active, int32_t n_tiles,
                                            int32_t order, const hp_params* prm, const hp_ssim_params* sp,
                                            const void* mask, const int32_t* tables, const void* ws, size_t ws_bytes,
                                            const float* dL_dloss, float* dL_dimg, void* stream) {
  SsimArgs A;
  float* Gm;
  float2* part;
  HP_TRY(ssim_setup(img, ref, n_active, n_tiles, order, prm, sp, mask, tables, ws, ws_bytes, &A, &Gm, &part));
  if (!dL_dloss || !dL_dimg) return HP_ERR_INVALID_ARG;
  return ssim_bwd_launch(A, sp->zones != 0, img, ref, n_tiles, Gm, dL_dloss, dL_dimg, (hipStream_t)stream);
}
