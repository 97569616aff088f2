// Discrete dynamics x_{t+1} = F(x_t, v_t) (arXiv 2409.07563, Eq. dynamics),
// evaluated per sample in registers: forward Euler (the paper's default) or
// classic RK4 with the control held over the step.
//
// Precision: the first Model::kComp state components (positions that grow to
// tens of metres while a step moves them by centimetres) are advanced with
// compensated (Kahan) summation; the running compensation term is kept in
// registers and also handed to the cost, which uses it where a cost is steep
// in position (the costmap).  Without it binary32 rounding of p + dp
// accumulates over the horizon.
#pragma once

#include "common.h"

namespace mppi {

// (px, py, vx, vy), control (ax, ay)
struct DoubleIntegrator {
  static constexpr int N = 4, M = 2, kComp = 0;
  __device__ __forceinline__ static void deriv(const float* x, const float* v, float* d,
                                               const DevParams&) {
    d[0] = x[2]; d[1] = x[3]; d[2] = v[0]; d[3] = v[1];
  }
  __device__ __forceinline__ static void post_step(float*, const DevParams&) {}
};

// Kinematic bicycle (px, py, yaw, speed, steer), control (accel, steer rate).
// FAST: the hardware sine/cosine units (v_sin_f32 / v_cos_f32), as the paper
// does with CUDA's trigonometric intrinsics (Sec. III-B); otherwise the
// correctly range-reduced library functions.
template <bool FAST>
struct Bicycle {
  static constexpr int N = 5, M = 2, kComp = 2;
  __device__ __forceinline__ static void deriv(const float* x, const float* v, float* d,
                                               const DevParams& p) {
    float sn, cs, tn;
    if constexpr (FAST) {
      sn = __sinf(x[2]);
      cs = __cosf(x[2]);
      tn = __sinf(x[4]) * __builtin_amdgcn_rcpf(__cosf(x[4]));
    } else {
      sincosf(x[2], &sn, &cs);
      tn = tanf(x[4]);
    }
    d[0] = x[3] * cs;
    d[1] = x[3] * sn;
    d[2] = x[3] * tn * p.inv_wheelbase;
    d[3] = v[0];
    d[4] = v[1];
  }
  __device__ __forceinline__ static void post_step(float*, const DevParams&) {}
};

// Rigid-body quadrotor: p(3), q = (w, x, y, z), v(3) world frame, omega(3) body
// frame; control (thrust, tau_x, tau_y, tau_z).  q is renormalised after each
// step.
struct Quadrotor {
  static constexpr int N = 13, M = 4, kComp = 0;
  __device__ __forceinline__ static void deriv(const float* x, const float* v, float* d,
                                               const DevParams& p) {
    const float qw = x[3], qx = x[4], qy = x[5], qz = x[6];
    const float wx = x[10], wy = x[11], wz = x[12];
    d[0] = x[7]; d[1] = x[8]; d[2] = x[9];
    d[3] = 0.5f * (-qx * wx - qy * wy - qz * wz);
    d[4] = 0.5f * (qw * wx + qy * wz - qz * wy);
    d[5] = 0.5f * (qw * wy + qz * wx - qx * wz);
    d[6] = 0.5f * (qw * wz + qx * wy - qy * wx);
    const float a = v[0] * p.inv_mass;
    d[7] = 2.0f * (qx * qz + qw * qy) * a;
    d[8] = 2.0f * (qy * qz - qw * qx) * a;
    d[9] = (1.0f - 2.0f * (qx * qx + qy * qy)) * a - p.gravity;
    const float h0 = p.inertia[0] * wx, h1 = p.inertia[1] * wy, h2 = p.inertia[2] * wz;
    d[10] = (v[1] - (wy * h2 - wz * h1)) * p.inv_inertia[0];
    d[11] = (v[2] - (wz * h0 - wx * h2)) * p.inv_inertia[1];
    d[12] = (v[3] - (wx * h1 - wy * h0)) * p.inv_inertia[2];
  }
  __device__ __forceinline__ static void post_step(float* x, const DevParams&) {
    const float inv = rsqrtf(x[3] * x[3] + x[4] * x[4] + x[5] * x[5] + x[6] * x[6]);
    x[3] *= inv; x[4] *= inv; x[5] *= inv; x[6] *= inv;
  }
};

enum { kEuler = MPPI_INT_EULER, kRK4 = MPPI_INT_RK4 };

// x <- x + inc, compensated for the first kComp components (comp[] carries the
// rounding error of the previous additions with its sign flipped).
template <class Model>
__device__ __forceinline__ void advance(float* x, const float* x0, const float* inc,
                                        float* comp) {
#pragma unroll
  for (int i = 0; i < Model::N; ++i) {
    if (i < Model::kComp) {
      const float y = inc[i] - comp[i];
      const float t = x0[i] + y;
      comp[i] = (t - x0[i]) - y;
      x[i] = t;
    } else {
      x[i] = x0[i] + inc[i];
    }
  }
}

// One step.
template <class Model, int INTEG>
__device__ __forceinline__ void step(float* x, const float* v, float* comp, const DevParams& p) {
  constexpr int N = Model::N;
  float x0[N], inc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) x0[i] = x[i];
  if constexpr (INTEG == kEuler) {
    float d[N];
    Model::deriv(x0, v, d, p);
#pragma unroll
    for (int i = 0; i < N; ++i) inc[i] = p.dt * d[i];
  } else {
    float k[N], acc[N], xs[N];
    Model::deriv(x0, v, k, p);
#pragma unroll
    for (int i = 0; i < N; ++i) { acc[i] = k[i]; xs[i] = x0[i] + p.half_dt * k[i]; }
    Model::deriv(xs, v, k, p);
#pragma unroll
    for (int i = 0; i < N; ++i) { acc[i] += 2.0f * k[i]; xs[i] = x0[i] + p.half_dt * k[i]; }
    Model::deriv(xs, v, k, p);
#pragma unroll
    for (int i = 0; i < N; ++i) { acc[i] += 2.0f * k[i]; xs[i] = x0[i] + p.dt * k[i]; }
    Model::deriv(xs, v, k, p);
#pragma unroll
    for (int i = 0; i < N; ++i) inc[i] = p.sixth_dt * (acc[i] + k[i]);
  }
  advance<Model>(x, x0, inc, comp);
  Model::post_step(x, p);
}

// The bicycle with a residual, x' = F(x, v) + dt g(x, v), in two parts that
// different waves may evaluate: bicycle_increment gives what the residual is
// added to, add_residual the new state.  Every operation is spelled out (no
// contraction is left to the compiler), so the parts round the same wherever
// they run.
//   q[0..2]  the increment of position and yaw (rounded)
//   q[3..4]  speed and steer: the increment before its last factor, inc_scale
template <bool FAST>
__device__ __forceinline__ float bicycle_tan(float d) {
  if constexpr (FAST) {
    return __sinf(d) * __builtin_amdgcn_rcpf(__cosf(d));
  } else {
    return tanf(d);
  }
}
template <bool FAST>
__device__ __forceinline__ void bicycle_sincos(float a, float& s, float& c) {
  if constexpr (FAST) {
    s = __sinf(a);
    c = __cosf(a);
  } else {
    sincosf(a, &s, &c);
  }
}
template <int INTEG>
__device__ __forceinline__ float inc_scale(const DevParams& p) {
  return INTEG == kEuler ? p.dt : p.sixth_dt;
}

template <bool FAST, int INTEG>
__device__ __forceinline__ void bicycle_increment(const float* x, const float* v,
                                                  const DevParams& p, float* q) {
#pragma clang fp contract(off)
  const float il = p.inv_wheelbase;
  const float s1 = x[3];
  if constexpr (INTEG == kEuler) {
    float sn, cs;
    bicycle_sincos<FAST>(x[2], sn, cs);
    q[0] = p.dt * (s1 * cs);
    q[1] = p.dt * (s1 * sn);
    q[2] = p.dt * (s1 * bicycle_tan<FAST>(x[4]) * il);
    q[3] = v[0];
    q[4] = v[1];
  } else {
    // speed and steer are linear over the step, so stages 2 and 3 share them
    // and their yaw rate
    const float s2 = __builtin_fmaf(p.half_dt, v[0], s1), s4 = __builtin_fmaf(p.dt, v[0], s1);
    const float d2 = __builtin_fmaf(p.half_dt, v[1], x[4]), d4 = __builtin_fmaf(p.dt, v[1], x[4]);
    const float k1 = s1 * bicycle_tan<FAST>(x[4]) * il;
    const float k2 = s2 * bicycle_tan<FAST>(d2) * il;
    const float r4 = s4 * bicycle_tan<FAST>(d4);  // times il: the fourth stage's yaw rate
    float sn1, cs1, sn2, cs2, sn3, cs3, sn4, cs4;
    bicycle_sincos<FAST>(x[2], sn1, cs1);
    bicycle_sincos<FAST>(__builtin_fmaf(p.half_dt, k1, x[2]), sn2, cs2);
    bicycle_sincos<FAST>(__builtin_fmaf(p.half_dt, k2, x[2]), sn3, cs3);
    bicycle_sincos<FAST>(__builtin_fmaf(p.dt, k2, x[2]), sn4, cs4);
    auto sum4 = [&](float t1, float t2, float t3, float t4) {
      float a = __builtin_fmaf(s1, t1, 2.0f * (s2 * t2));
      a = __builtin_fmaf(2.0f, s2 * t3, a);
      return __builtin_fmaf(s4, t4, a);
    };
    q[0] = p.sixth_dt * sum4(cs1, cs2, cs3, cs4);
    q[1] = p.sixth_dt * sum4(sn1, sn2, sn3, sn4);
    float a = __builtin_fmaf(2.0f, k2, k1);
    a = __builtin_fmaf(2.0f, k2, a);
    q[2] = p.sixth_dt * __builtin_fmaf(r4, il, a);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float b = __builtin_fmaf(2.0f, v[j], v[j]);
      b = __builtin_fmaf(2.0f, v[j], b);
      q[3 + j] = b + v[j];
    }
  }
}

// The values of v in the lanes n, 16 + n, 32 + n, 48 + n of the wave (n = lane
// mod 16), in every one of them.
__device__ __forceinline__ void rows_gather(float v, float (&out)[4]) {
  const uint32_t b = __float_as_uint(v);
  // the odd rows of the first operand trade places with the even rows of the second
  const auto r = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  const auto e = __builtin_amdgcn_permlane32_swap(r[0], r[0], false, false);
  const auto o = __builtin_amdgcn_permlane32_swap(r[1], r[1], false, false);
  out[0] = __uint_as_float(e[0]);
  out[1] = __uint_as_float(o[0]);
  out[2] = __uint_as_float(e[1]);
  out[3] = __uint_as_float(o[1]);
}

// bicycle_increment of RK4 where the four 16-lane rows of a wave hold the same
// sample in the same lane: row g takes stage g's tan, sin and cos (the stage
// yaw rates need only speed and steer, so the stages do not wait for each
// other), three gathers bring them together, and every row forms the same
// increment with the operations of bicycle_increment.  mid() is called half way.
template <bool FAST, class Mid>
__device__ __forceinline__ void bicycle_increment_rows(const float* x, const float* v, int g,
                                                       const DevParams& p, float* q, Mid&& mid) {
#pragma clang fp contract(off)
  const float il = p.inv_wheelbase;
  const float s1 = x[3];
  const float s2 = __builtin_fmaf(p.half_dt, v[0], s1), s4 = __builtin_fmaf(p.dt, v[0], s1);
  const float d2 = __builtin_fmaf(p.half_dt, v[1], x[4]), d4 = __builtin_fmaf(p.dt, v[1], x[4]);
  const float s = g == 0 ? s1 : g == 3 ? s4 : s2;
  float r[4], cs[4], sn[4], mysn, mycs;
  rows_gather(s * bicycle_tan<FAST>(g == 0 ? x[4] : g == 3 ? d4 : d2), r);
  const float k1 = r[0] * il, k2 = r[1] * il;
  mid();
  // stage 2 leaves from x along k1, stages 3 and 4 along k2 (k3 = k2)
  const float a1 = __builtin_fmaf(g == 3 ? p.dt : p.half_dt, g == 1 ? k1 : k2, x[2]);
  bicycle_sincos<FAST>(g == 0 ? x[2] : a1, mysn, mycs);
  rows_gather(mycs, cs);
  rows_gather(mysn, sn);
  auto sum4 = [&](const float (&t)[4]) {
    float a = __builtin_fmaf(s1, t[0], 2.0f * (s2 * t[1]));
    a = __builtin_fmaf(2.0f, s2 * t[2], a);
    return __builtin_fmaf(s4, t[3], a);
  };
  q[0] = p.sixth_dt * sum4(cs);
  q[1] = p.sixth_dt * sum4(sn);
  float a = __builtin_fmaf(2.0f, k2, k1);
  a = __builtin_fmaf(2.0f, k2, a);
  q[2] = p.sixth_dt * __builtin_fmaf(r[3], il, a);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float b = __builtin_fmaf(2.0f, v[j], v[j]);
    b = __builtin_fmaf(2.0f, v[j], b);
    q[3 + j] = b + v[j];
  }
}

template <int INTEG>
__device__ __forceinline__ void add_residual(float* x, float* comp, const float* q,
                                             const float* res, const DevParams& p) {
#pragma clang fp contract(off)
  const float h = inc_scale<INTEG>(p);
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // compensated, as advance() does
    const float y = __builtin_fmaf(p.dt, res[i], q[i]) - comp[i];
    const float t = x[i] + y;
    comp[i] = (t - x[i]) - y;
    x[i] = t;
  }
  x[2] = x[2] + __builtin_fmaf(p.dt, res[2], q[2]);
#pragma unroll
  for (int i = 3; i < 5; ++i) x[i] = x[i] + __builtin_fmaf(h, q[i], p.dt * res[i]);
}

template <bool FAST, int INTEG>
__device__ __forceinline__ void residual_step(float* x, const float* v, float* comp,
                                              const DevParams& p, const float* res) {
  float q[5];
  bicycle_increment<FAST, INTEG>(x, v, p, q);
  add_residual<INTEG>(x, comp, q, res, p);
}

}  // namespace mppi
