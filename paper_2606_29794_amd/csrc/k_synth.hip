// k_synth.hip -- image synthesis between the HEALPix grid and camera images:
// the final step of rendering, I_C(u, v) = Interp_H(I_H, P_C(u, v))
// (Eq. camera_synthesis), and the reverse sampling of a camera image at the
// HEALPix pixel centres used for ground truth (supp. Eq.
// supp_image_to_healpix), with the camera mappings of the supplementary
// section on camera models (pinhole; anisotropic equidistant fisheye,
// Eq. fish_weff; equirectangular panorama).
//
// Conventions shared with the rest of the library: one camera frame for all
// models with +z the optical axis, +x right and +y up (the image's v axis
// points down, so v is negated for pinhole and fisheye); pixel (i, j) of a
// W x H image is centred at (u, v) = (i + 1/2, j + 1/2); the HEALPix pole is
// camera +y and its longitude is atan2(t_x, t_z).
//
// Interp_H: the two rings that enclose the point's colatitude, in each the
// two pixels that enclose its longitude; linear in longitude along each ring,
// linear in colatitude between the rings.  Above the first ring (below the
// last) the pole value is the mean of that ring's four pixels.  Neighbours
// outside the camera's active set get weight zero and the others are
// renormalised.  Geometry runs in double precision (CDNA4 issues FP64 vector
// FMAs at the FP32 rate), the colours in float.
//
// Both kernels are gathers over small, L2-resident inputs with coalesced
// outputs: one thread per output sample.
#include "hp_common.h"

namespace {

enum { CAM_FULL = 0, CAM_FISHEYE = 1, CAM_PINHOLE = 2 };

struct SynthCam {
  int type, W, H;
  double fx, fy;        // focal lengths in pixels
  double wx, wy;        // fisheye FoV / pi
  double cx, cy;        // principal point (image centre)
  double pu, pv;        // panorama: pixels per radian of longitude and latitude
  double ru, rv;        // and radians per pixel
};

SynthCam synth_cam(const hp_view* v, int W, int H) {
  SynthCam c;
  c.type = v->cam_type;
  c.W = W;
  c.H = H;
  c.cx = 0.5 * W;
  c.cy = 0.5 * H;
  if (c.type == CAM_PINHOLE) {
    c.fx = W / (2.0 * tan(0.5 * (double)v->fov_x));
    c.fy = H / (2.0 * tan(0.5 * (double)v->fov_y));
  } else {
    c.fx = W / M_PI;
    c.fy = H / M_PI;
  }
  c.pu = W / (2.0 * M_PI);
  c.pv = H / M_PI;
  c.ru = 2.0 * M_PI / W;
  c.rv = M_PI / H;
  c.wx = (double)v->fov_x / M_PI;
  c.wy = (double)v->fov_y / M_PI;
  return c;
}

// Position on the sphere by colatitude and longitude: z = cos(theta),
// sin(theta), longitude phi.
struct SynthPos {
  double z, st, phi;
};

// position of the ray through image position (u, v); false outside the
// camera's domain.  A panorama's row fixes z and its column the longitude
// (synth_row, synth_col); the other models pass through a direction.
__device__ __forceinline__ void synth_row(const SynthCam& c, double v, SynthPos* p) {
  sincos(0.5 * M_PI - v * c.rv, &p->z, &p->st);
}
__device__ __forceinline__ void synth_col(const SynthCam& c, double u, SynthPos* p) {
  const double om = u * c.ru - M_PI;
  p->phi = om < 0.0 ? om + 2.0 * M_PI : om;
}
__device__ __forceinline__ bool synth_ray(const SynthCam& c, double u, double v, SynthPos* p) {
  const double mx = (u - c.cx) / c.fx, my = -(v - c.cy) / c.fy;
  double d[3];
  bool ok = true;
  if (c.type == CAM_PINHOLE) {
    const double n = rsqrt(mx * mx + my * my + 1.0);
    d[0] = mx * n;
    d[1] = my * n;
    d[2] = n;
  } else {
    // the azimuth enters by its sine and cosine only
    const double rm = sqrt(mx * mx + my * my);
    const double cg = rm > 0.0 ? mx / rm : 1.0, sg = rm > 0.0 ? my / rm : 0.0;
    const double weff = sqrt(c.wx * cg * c.wx * cg + c.wy * sg * c.wy * sg);
    double sps, cps;
    sincos(rm * weff, &sps, &cps);
    d[0] = sps * cg;
    d[1] = sps * sg;
    d[2] = cps;
    ok = rm <= 0.5 * M_PI;
  }
  p->z = d[1];
  p->st = sqrt(d[0] * d[0] + d[2] * d[2]);
  const double phi = atan2(d[0], d[2]);
  p->phi = phi < 0.0 ? phi + 2.0 * M_PI : phi;
  return ok;
}

// image position of pixel p of the grid; false outside the camera's domain
__device__ __forceinline__ bool synth_project(const SynthCam& c, int order, int64_t p, double* u, double* v) {
  double z, st, phi;
  hp_pix_pos(order, p, &z, &st, &phi);
  if (c.type == CAM_FULL) {
    const double om = phi > M_PI ? phi - 2.0 * M_PI : phi;
    *u = (om + M_PI) * c.pu;
    *v = (0.5 * M_PI - asin(z)) * c.pv;
    return true;
  }
  double so, co;
  sincos(phi, &so, &co);
  const double d[3] = {st * so, z, st * co};
  if (c.type == CAM_PINHOLE) {
    if (!(d[2] > 0.0)) return false;
    *u = c.cx + c.fx * (d[0] / d[2]);
    *v = c.cy - c.fy * (d[1] / d[2]);
    return *u >= 0.0 && *u <= c.W && *v >= 0.0 && *v <= c.H;
  }
  const double psi = acos(fmin(1.0, fmax(-1.0, d[2])));
  const double rho = sqrt(d[0] * d[0] + d[1] * d[1]);
  const double cg = rho > 0.0 ? d[0] / rho : 1.0, sg = rho > 0.0 ? d[1] / rho : 0.0;
  const double weff = sqrt(c.wx * cg * c.wx * cg + c.wy * sg * c.wy * sg);
  const double rm = psi / weff;
  *u = c.cx + c.fx * rm * cg;
  *v = c.cy - c.fy * rm * sg;
  return rm <= 0.5 * M_PI;
}

// ---- ring structure of the grid (Gorski et al. 2005) -----------------------
// ring i (1 .. 4N-1): z, sin(theta), pixels and the longitude offset (in
// pixels) of its pixel 0's centre.  In the caps 1 - |z| = i^2 / (3 N^2), from
// which sin(theta) comes without cancellation.
struct RingGeo {
  double z, st, off;
  int n;
};
__device__ __forceinline__ RingGeo ring_geo(int N, int i) {
  RingGeo r;
  if (i < N || i > 3 * N) {
    const int nr = i < N ? i : 4 * N - i;
    const double h = (double)(nr * nr) / (3.0 * (double)(N * N));
    r.z = i < N ? 1.0 - h : h - 1.0;
    r.st = sqrt(h * (2.0 - h));
    r.n = 4 * nr;
    r.off = 0.5;
  } else {
    r.z = (double)(2 * N - i) * (2.0 / (3.0 * (double)N));
    r.st = sqrt((1.0 - r.z) * (1.0 + r.z));
    r.n = 4 * N;
    r.off = ((i - N) & 1) ? 0.0 : 0.5;
  }
  return r;
}

// asin for the small angles between neighbouring rings: its series below
// 0.05 (truncation < 1e-18), the library's beyond
__device__ __forceinline__ double small_asin(double x) {
  const double q = x * x;
  if (q < 0.0025)
    return x * (1.0 + q * (1.0 / 6.0 + q * (3.0 / 40.0 + q * (5.0 / 112.0 + q * (35.0 / 1152.0 + q * (63.0 / 2816.0 +
           q * (231.0 / 13312.0)))))));
  return asin(fmin(1.0, fmax(-1.0, x)));
}

// NESTED index of pixel j (0-based) of ring i.  Polar caps: face column
// j / nr, then the face-local (x, y) from the ring's position on the face.
// Equatorial belt: with u = 2 j + 1 - ((i - N) & 1), the position along the
// ring in half pixels, x = (u - i - 1 + N) / 2 and y = (N - i - 1 - u) / 2 modulo
// N, and the two quotients qx, qy give the face: its row -1 - qx - qy, and its
// centre's longitude qx - qy (mod 8) in units of pi / 4.
__device__ __forceinline__ int ring_nest(int order, int i, int j) {
  const int N = 1 << order;
  if (i < N || i > 3 * N) {
    const bool north = i < N;
    const int nr = north ? i : 4 * N - i;
    const int col = (j >= nr) + (j >= 2 * nr) + (j >= 3 * nr), q = j - col * nr;
    const int x = north ? N - nr + q : q;
    const int y = north ? N - 1 - q : nr - 1 - q;
    return (int)hp_xyf_nest(order, x, y, (north ? 0 : 8) + col);
  }
  const int u = 2 * j + 1 - ((i - N) & 1);
  const int a = u - i - 1 + N, b = N - i - 1 - u;
  const int qx = a >> (order + 1), qy = b >> (order + 1);
  const int x = (a & (2 * N - 1)) >> 1, y = (b & (2 * N - 1)) >> 1;
  const int row = -1 - qx - qy, col = ((qx - qy) & 7) >> 1;
  return (int)hp_xyf_nest(order, x, y, 4 * row + col);
}

// The rings of Interp_H and their weights: i1 and i2 enclose the point, and
// their weights are linear in colatitude, w2 = (theta - theta_1) / (theta_2 -
// theta_1).  Both differences come from the sine of the difference,
// sin(theta - theta_1) = sin(theta) z_1 - z sin(theta_1), so no colatitude is
// formed.  Beyond the first or last ring, pole is set, i1 is that ring, and
// w2 the weight of the ring's interpolation against its mean.
struct InterpRings {
  bool pole;
  int i1;
  RingGeo r1, r2;
  double w2;
};
__device__ __forceinline__ InterpRings interp_rings(int order, const SynthPos& p) {
  const int N = 1 << order;
  const double r6 = 2.449489742783178098197284;  // sqrt(6)
  // the ring coordinate of the point; in the caps N sqrt(6) sin(theta / 2)
  double ic;
  if (p.z > 2.0 / 3.0) ic = (double)N * r6 * (p.st / sqrt(2.0 * (1.0 + p.z)));
  else if (p.z < -2.0 / 3.0) ic = 4.0 * N - (double)N * r6 * (p.st / sqrt(2.0 * (1.0 - p.z)));
  else ic = 2.0 * N - 1.5 * N * p.z;
  int i1 = (int)floor(ic);
  i1 = i1 < 0 ? 0 : (i1 > 4 * N - 1 ? 4 * N - 1 : i1);
  InterpRings R;
  R.pole = i1 < 1 || i1 > 4 * N - 2;
  if (R.pole) {
    R.i1 = i1 < 1 ? 1 : 4 * N - 1;
    R.r1 = R.r2 = ring_geo(N, R.i1);
    R.w2 = small_asin(p.st) / small_asin(R.r1.st);
  } else {
    R.i1 = i1;
    R.r1 = ring_geo(N, i1);
    R.r2 = ring_geo(N, i1 + 1);
    R.w2 = small_asin(p.st * R.r1.z - p.z * R.r1.st) / small_asin(R.r2.st * R.r1.z - R.r2.z * R.r1.st);
  }
  R.w2 = fmin(1.0, fmax(0.0, R.w2));
  return R;
}

// the two pixels of a ring that enclose longitude phi, and the weight of the second
__device__ __forceinline__ void ring_pair(const RingGeo& r, double phi, int* ja, int* jb, double* f) {
  const double t = phi * ((double)r.n * (0.5 / M_PI)) - r.off;
  const double j1 = floor(t);
  *f = t - j1;
  int a = (int)j1;
  a = a < 0 ? a + r.n : (a >= r.n ? a - r.n : a);
  *ja = a;
  *jb = a + 1 == r.n ? 0 : a + 1;
}

// the four (ring, position) samples of Interp_H and their weights
__device__ __forceinline__ void interp4(const InterpRings& R, double phi, int ring[4], int pos[4], double w[4]) {
  double f1, f2;
  if (!R.pole) {
    ring_pair(R.r1, phi, &pos[0], &pos[1], &f1);
    ring_pair(R.r2, phi, &pos[2], &pos[3], &f2);
    ring[0] = ring[1] = R.i1;
    ring[2] = ring[3] = R.i1 + 1;
    w[0] = (1.0 - R.w2) * (1.0 - f1);
    w[1] = (1.0 - R.w2) * f1;
    w[2] = R.w2 * (1.0 - f2);
    w[3] = R.w2 * f2;
    return;
  }
  int a, b;
  ring_pair(R.r1, phi, &a, &b, &f1);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    ring[k] = R.i1;
    pos[k] = k;
    w[k] = 0.25 * (1.0 - R.w2) + (k == a ? R.w2 * (1.0 - f1) : 0.0) + (k == b ? R.w2 * f1 : 0.0);
  }
}

// compact slot of nested pixel q in the mask, or -1 (inactive)
__device__ __forceinline__ int synth_slot(const HpMaskView& m, const HpGeom& g, int q) {
  const int per_b = 2 * g.b;
  const int t = q >> per_b;
  const int loc = q - (t << per_b);
  // a fully active tile holds its pixels in nested order: no rank to count
  if (m.tile_count[t] == (1 << per_b)) return m.tile_start[t] + loc;
  const uint32_t* bits = m.tile_bits + 8 * (int64_t)t;
  const uint32_t word = bits[loc >> 5];
  if (!((word >> (loc & 31)) & 1u)) return -1;
  int rank = __popc(word & ((1u << (loc & 31)) - 1u));
  for (int k = 0; k < (loc >> 5); ++k) rank += __popc(bits[k]);
  return m.tile_start[t] + rank;
}

// ALL: every pixel of the grid is active, so slots are nested indices.
// A wave takes a patch of 16 x 4 image pixels, whose samples lie in a few lines
// of the nested image; 64 pixels of one image row cross a line each, and their
// twelve gathers then bound the kernel (a 3040 x 1520 panorama from Nside 512:
// 85 us by rows, 56 us by patches; 258 us by rows with the rings'
// colatitudes from asin and acos and 64-bit modulo arithmetic).
constexpr int kPatchW = 16, kPatchH = 4;
template <bool ALL>
__device__ __forceinline__ void synth_sample(const HpGeom& g, const HpMaskView& m, int64_t n_active,
                                             const InterpRings& R, double phi, bool inside,
                                             const float* __restrict__ img, int64_t k, int64_t HW,
                                             float* __restrict__ out, uint8_t* __restrict__ valid) {
  float a0 = 0.f, a1 = 0.f, a2 = 0.f;
  double ws = 0.0;
  if (inside) {
    int ring[4], pos[4];
    double w[4];
    interp4(R, phi, ring, pos, w);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int p = ring_nest(g.order, ring[q], pos[q]);
      const int s = ALL ? p : synth_slot(m, g, p);
      if (s < 0 || s >= n_active) continue;
      const float wf = (float)w[q];
      a0 += wf * img[s];
      a1 += wf * img[n_active + s];
      a2 += wf * img[2 * n_active + s];
      ws += w[q];
    }
  }
  const bool ok = ws > 0.0;
  const float inv = ok ? (float)(1.0 / ws) : 0.f;
  out[k] = a0 * inv;
  out[HW + k] = a1 * inv;
  out[2 * HW + k] = a2 * inv;
  if (valid) valid[k] = ok ? 1 : 0;
}

// Patches of a wave: kPatches side by side, in whose rows a panorama's rings
// are the same and are worked out once.
constexpr int kPatches = 4;
template <bool ALL, bool PANO>
__global__ __launch_bounds__(256) void k_sphere_to_image(HpGeom g, HpMaskView m, int64_t n_active, SynthCam c,
                                                         const float* __restrict__ img, float* __restrict__ out,
                                                         uint8_t* __restrict__ valid) {
  const int64_t HW = (int64_t)c.W * c.H;  // at most 2^31
  const uint32_t segs = ((uint32_t)c.W + kPatchW * kPatches - 1) / (kPatchW * kPatches);
  const uint32_t seg = blockIdx.x * 4u + hp_uniform(threadIdx.x >> 6);
  const uint32_t band = seg / segs;
  const int lane = hp_lane();
  const int64_t j = (int64_t)band * kPatchH + lane / kPatchW;
  if (j >= c.H) return;
  const int i0 = (int)(seg - band * segs) * (kPatchW * kPatches) + lane % kPatchW;
  SynthPos p;
  InterpRings R;
  bool inside = true;
  if (PANO) {
    synth_row(c, j + 0.5, &p);
    R = interp_rings(g.order, p);
  }
  for (int i = i0; i < i0 + kPatchW * kPatches && i < c.W; i += kPatchW) {
    if (PANO) {
      synth_col(c, i + 0.5, &p);
    } else {
      inside = synth_ray(c, i + 0.5, j + 0.5, &p);
      R = interp_rings(g.order, p);
    }
    synth_sample<ALL>(g, m, n_active, R, p.phi, inside, img, j * c.W + i, HW, out, valid);
  }
}

__global__ __launch_bounds__(256) void k_image_to_sphere(HpGeom g, HpMaskView m, int64_t n_active, SynthCam c,
                                                         const float* __restrict__ img, float* __restrict__ out,
                                                         uint8_t* __restrict__ valid) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_active) return;
  double u = 0.5 * c.W, v = 0.5 * c.H;
  const bool ok = synth_project(c, g.order, m.active_pix[k], &u, &v);
  // a position outside the image (an invalid sample) stays within the integers
  const double x = fmin(fmax(u - 0.5, -1.0), (double)c.W), y = fmin(fmax(v - 0.5, -1.0), (double)c.H);
  const double x0 = floor(x), y0 = floor(y);
  const float fx = (float)(x - x0), fy = (float)(y - y0);
  int xs[2] = {(int)x0, (int)x0 + 1}, ys[2] = {(int)y0, (int)y0 + 1};
  for (int a = 0; a < 2; ++a) {
    if (c.type == CAM_FULL) xs[a] = xs[a] < 0 ? xs[a] + c.W : (xs[a] >= c.W ? xs[a] - c.W : xs[a]);
    xs[a] = xs[a] < 0 ? 0 : (xs[a] >= c.W ? c.W - 1 : xs[a]);
    ys[a] = ys[a] < 0 ? 0 : (ys[a] >= c.H ? c.H - 1 : ys[a]);
  }
  const int64_t HW = (int64_t)c.W * c.H;
  const int64_t o00 = (int64_t)ys[0] * c.W + xs[0], o01 = (int64_t)ys[0] * c.W + xs[1],
                o10 = (int64_t)ys[1] * c.W + xs[0], o11 = (int64_t)ys[1] * c.W + xs[1];
  const float w00 = (1.f - fx) * (1.f - fy), w01 = fx * (1.f - fy), w10 = (1.f - fx) * fy, w11 = fx * fy;
  for (int ch = 0; ch < 3; ++ch) {
    const float* p = img + ch * HW;
    const float s = w00 * p[o00] + w01 * p[o01] + w10 * p[o10] + w11 * p[o11];
    out[ch * n_active + k] = ok ? s : 0.f;
  }
  if (valid) valid[k] = ok ? 1 : 0;
}

hp_status synth_check(const hp_view* view, const hp_params* prm, const void* mask, int32_t W, int32_t H) {
  HP_TRY(hp_check_view(view, prm));
  if (!mask || W <= 0 || H <= 0 || (int64_t)W * H > ((int64_t)1 << 31)) return HP_ERR_INVALID_ARG;
  return HP_OK;
}

}  // namespace

extern "C" hp_status hp_sphere_to_image(const void* mask, const hp_view* view, const hp_params* prm, int64_t n_active,
                                        const float* img, int32_t W, int32_t H, float* out, uint8_t* valid,
                                        void* stream) {
  HP_TRY(synth_check(view, prm, mask, W, H));
  const HpGeom g = hp_geom(view->order, prm->tile_log2);
  if (n_active < 0 || n_active > g.npix || !out || (n_active > 0 && !img)) return HP_ERR_INVALID_ARG;
  const HpMaskView mv = hp_mask_view((char*)const_cast<void*>(mask), g);
  const SynthCam c = synth_cam(view, W, H);
  const bool all = n_active == g.npix;
  hipStream_t s = (hipStream_t)stream;
  const int64_t segs = (int64_t)((W + kPatchW * kPatches - 1) / (kPatchW * kPatches)) * ((H + kPatchH - 1) / kPatchH);
  const dim3 grid(hp_blocks(segs, 4));
#define HP_SYNTH(ALL, PANO) \
  hipLaunchKernelGGL((k_sphere_to_image<ALL, PANO>), grid, dim3(256), 0, s, g, mv, n_active, c, img, out, valid)
  if (c.type == CAM_FULL) {
    if (all) HP_SYNTH(true, true);
    else HP_SYNTH(false, true);
  } else {
    if (all) HP_SYNTH(true, false);
    else HP_SYNTH(false, false);
  }
#undef HP_SYNTH
  HP_CHECK_LAUNCH();
  return HP_OK;
}

extern "C" hp_status hp_image_to_sphere(const void* mask, const hp_view* view, const hp_params* prm, int64_t n_active,
                                        const float* img, int32_t W, int32_t H, float* out, uint8_t* valid,
                                        void* stream) {
  HP_TRY(synth_check(view, prm, mask, W, H));
  const HpGeom g = hp_geom(view->order, prm->tile_log2);
  if (n_active < 0 || n_active > g.npix || !img || (n_active > 0 && !out)) return HP_ERR_INVALID_ARG;
  if (n_active == 0) return HP_OK;
  hipLaunchKernelGGL(k_image_to_sphere, dim3(hp_blocks(n_active, 256)), dim3(256), 0, (hipStream_t)stream, g,
                     hp_mask_view((char*)const_cast<void*>(mask), g), n_active, synth_cam(view, W, H), img, out,
                     valid);
  HP_CHECK_LAUNCH();
  return HP_OK;
}
