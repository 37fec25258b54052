// hp_cone.h -- the cone around the optical axis outside which no Gaussian
// reaches an active tile of a camera's mask (host code, no device types).
#pragma once

#include <math.h>
#include <stdint.h>

#include "../../include/hp.h"

// Bounding cone of a mask's active tiles as a cap around the optical axis +z,
// as (sin, cos) of half its angle.  An active tile holds an active pixel,
// which lies within the half field of view `a` of the axis (FISHEYE: the
// larger of the two halves bounds w_eff pi / 2; PINHOLE: the corner of the
// frustum), and the tile's cap centre within the cap's radius R of that
// pixel.  A Gaussian of test angle theta reaches the tile only where its
// direction lies within theta + R of the cap centre, so within theta + a +
// 2 R of the axis.  R is below 1.25 / Nside_t, Nside_t = 2^kt (a HEALPix pixel
// reaches 1.1 / Nside_t from its centre); 1e-3 rad are added against the
// rounding of the test.  (1, 0), which every direction passes, where the cone
// would be the whole sphere.
struct HpCone {
  float sr, cr;
};
// Word behind the two in a mask that holds its cone.  A mask buffer written
// before masks had one (kept in a file, or by another build) has other bytes
// there, and its Gaussians are all kept.
constexpr uint32_t kConeMark = 0x656e6f43u;
static inline HpCone hp_view_cone(const hp_view* v, int kt) {
  double a = M_PI;
  if (v->cam_type == HP_CAM_FISHEYE) {
    a = 0.5 * (v->fov_x > v->fov_y ? (double)v->fov_x : (double)v->fov_y);
  } else if (v->cam_type == HP_CAM_PINHOLE) {
    const double tx = tan(0.5 * (double)v->fov_x), ty = tan(0.5 * (double)v->fov_y);
    a = atan(sqrt(tx * tx + ty * ty));
  }
  const double ang = a + 2.5 / (double)((int64_t)1 << kt) + 1e-3;
  if (!(ang < M_PI)) return HpCone{1.f, 0.f};
  return HpCone{(float)sin(0.5 * ang), (float)cos(0.5 * ang)};
}
