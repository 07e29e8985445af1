// x Phi(x), the exact GELU, in float32.  Plain C++: Math supplies rcp(x) and
// exp2(x) (one ulp each), so that the function can be checked off the device.
#pragma once
#include <cmath>

#ifdef __HIPCC__
#define NV_HD __host__ __device__
#else
#define NV_HD
#endif

namespace nv {

// |x| < sqrt 2: Phi = 1/2 + x (c + u R(u)), u = x^2, with c the float32 next to
// 1 / sqrt(2 pi) and R of degree 5 fitted against that c (4e-9 of Phi(-|x|)).
// Beyond: Phi(-a) = exp(-a^2 / 2) t P(t), a = |x|, t = 1 / (1 + a / 2), P of degree
// 5 (2.5e-8 relative up to a = 4; float16 results end at 6).  Both are weighted
// minimax fits of the functions themselves.
// Error against float64 on the device, relative in the 2-norm over N(0, s^2)
// inputs, beside that of 0.5 x (1 + erff(x / sqrt 2)): s = 0.1 3.7e-8 (3.8e-8), 0.5
// 3.6e-8 (4.2e-8), 1 3.4e-8 (3.9e-8), 2 3.1e-8 (3.5e-8), 4 2.0e-8 (2.3e-8); no
// interval of x is worse, and the erff form, which cancels for negative x, is off
// by 0.9 % of the value at -4 to -5 where this one is by 4e-7.
// One evaluation of the SD-1.5-shaped network on 16 rows, gates of spread 0.4 to
// 0.7: 19.2 ms, 19.5 with both parts computed for every gate.
constexpr float GELU_SPLIT = 2.0f;  // on u

NV_HD inline float gelu_near(float x, float u) {
  float r = 4.4080695715820184e-07f;
  r = fmaf(r, u, -8.909227290132549e-06f);
  r = fmaf(r, u, 0.00011484260176075622f);
  r = fmaf(r, u, -0.001187099376693368f);
  r = fmaf(r, u, 0.009973634034395218f);
  r = fmaf(r, u, -0.06649045646190643f);
  return x * fmaf(x, fmaf(u, r, 0.3989422804014327f), 0.5f);
}

template <typename Math>
NV_HD inline float gelu_far(float x, float u) {
  const float t = Math::rcp(fmaf(0.5f, fabsf(x), 1.0f));
  float p = 0.12087258696556091f;
  p = fmaf(p, t, -0.30572769045829773f);
  p = fmaf(p, t, 0.16226355731487274f);
  p = fmaf(p, t, 0.12169518321752548f);
  p = fmaf(p, t, 0.20310306549072266f);
  p = fmaf(p, t, 0.19927644729614258f);
  const float h = p * t * Math::exp2(-0.72134752044448170f * u);
  return x * (x >= 0.0f ? 1.0f - h : h);
}

// Four gates at a time: a wave whose gates are all near 0 skips the far part.
template <typename Math>
NV_HD inline void gelu_quad(const float (&x)[4], float (&y)[4]) {
  float u[4];
  bool near = true;  // a NaN goes the far way
  for (int i = 0; i < 4; ++i) {
    u[i] = x[i] * x[i];
    y[i] = gelu_near(x[i], u[i]);
    near = near && u[i] < GELU_SPLIT;
  }
  if (!near)
    for (int i = 0; i < 4; ++i) {
      const float f = gelu_far<Math>(x[i], u[i]);
      y[i] = u[i] < GELU_SPLIT ? y[i] : f;
    }
}

}  // namespace nv
