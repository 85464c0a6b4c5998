// Device-side FP64 helpers for the visual-inertial step: 3x3 algebra, the
// rotation exponential/logarithm and right Jacobians, and quaternions.
// Matrices are row-major double[9].  All functions are written for single
// lanes, without cross-lane communication, except the last ones, of one wave.
#pragma once
#include <hip/hip_runtime.h>

namespace vi {

__device__ __forceinline__ double rsqrt_refined(double v) {
  // hardware reciprocal square root (relative error about 2^-23), then one
  // third-order step: with e = 1 - v y^2, v^-1/2 = y (1 - e)^-1/2 =
  // y (1 + e/2 + 3 e^2/8 + 5 e^3/16 + ...); the dropped terms are below 2^-64
  // relative.  Four dependent operations after the estimate, where two
  // Newton steps take six (the pivot chain of the leaf factor runs through it).
  const double y = __builtin_amdgcn_rsq(v);
  const double e = __builtin_fma(-v, y * y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// Values that one workgroup hands to another inside a launch: stored and loaded
// at agent scope one by one, past the caches that the XCDs do not share.  (A
// release fence instead would write back a whole L2.)
__device__ __forceinline__ void agent_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool AG>
__device__ __forceinline__ double agent_load(const double* p) {
  return AG ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}

// A pointer that was itself loaded from memory, declared as one to global
// memory: through the generic type its loads are flat ones, which count as LDS
// operations too, so that every wait for LDS waits for them.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* as_global(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

__device__ __forceinline__ void m3_mul(const double* A, const double* B, double* C) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      C[r * 3 + c] = A[r * 3 + 0] * B[0 * 3 + c] + A[r * 3 + 1] * B[1 * 3 + c] + A[r * 3 + 2] * B[2 * 3 + c];
}

// C = A^T B
__device__ __forceinline__ void m3_tmul(const double* A, const double* B, double* C) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      C[r * 3 + c] = A[0 * 3 + r] * B[0 * 3 + c] + A[1 * 3 + r] * B[1 * 3 + c] + A[2 * 3 + r] * B[2 * 3 + c];
}

// y = A x
__device__ __forceinline__ void m3_vec(const double* A, const double* x, double* y) {
#pragma unroll
  for (int r = 0; r < 3; ++r) y[r] = A[r * 3 + 0] * x[0] + A[r * 3 + 1] * x[1] + A[r * 3 + 2] * x[2];
}

// y = A^T x
__device__ __forceinline__ void m3_tvec(const double* A, const double* x, double* y) {
#pragma unroll
  for (int r = 0; r < 3; ++r) y[r] = A[0 * 3 + r] * x[0] + A[1 * 3 + r] * x[1] + A[2 * 3 + r] * x[2];
}

__device__ __forceinline__ void skew(const double* w, double* S) {
  S[0] = 0.0;   S[1] = -w[2]; S[2] = w[1];
  S[3] = w[2];  S[4] = 0.0;   S[5] = -w[0];
  S[6] = -w[1]; S[7] = w[0];  S[8] = 0.0;
}

// Functions of the angle t = |w| by their power series in t^2.  Up to t^2 =
// kSeriesT2 (t = 0.5, where an increment, a residual or the rotation of one IMU
// sample lies) the dropped terms are below 2^-54 of the sum, without the
// cancellation of 1 - cos t and t - sin t, and 7 or 8 fused operations replace
// a square root, a sine, a cosine and divisions (some 200 instructions on the
// serial lanes that form the inertial factors).  The logarithm has the series of
// the arc sine instead, in sin t, up to sin t = 1/8: beyond it the terms fall
// too slowly.
constexpr double kSeriesT2 = 0.25;
__device__ __forceinline__ double series_sinc(double x) {           // sin t / t
  return 1.0 + x * (-1.0 / 6 + x * (1.0 / 120 + x * (-1.0 / 5040 + x * (1.0 / 362880 + x * (-1.0 / 39916800 +
         x * (1.0 / 6227020800.0))))));
}
__device__ __forceinline__ double series_cosc(double x) {           // (1 - cos t) / t^2
  return 0.5 + x * (-1.0 / 24 + x * (1.0 / 720 + x * (-1.0 / 40320 + x * (1.0 / 3628800 + x * (-1.0 / 479001600 +
         x * (1.0 / 87178291200.0))))));
}
__device__ __forceinline__ double series_sinc3(double x) {          // (t - sin t) / t^3
  return 1.0 / 6 + x * (-1.0 / 120 + x * (1.0 / 5040 + x * (-1.0 / 362880 + x * (1.0 / 39916800 + x * (-1.0 / 6227020800.0 +
         x * (1.0 / 1307674368000.0))))));
}
// (1 - t / 2 cot(t / 2)) / t^2 = sum |B_2n| t^(2n - 2) / (2n)!
__device__ __forceinline__ double series_cot(double x) {
  return 1.0 / 12 + x * (1.0 / 720 + x * (1.0 / 30240 + x * (1.0 / 1209600 + x * (1.0 / 47900160 +
         x * (691.0 / 1307674368000.0 + x * (1.0 / 74724249600.0 + x * (3617.0 / 10670622842880000.0)))))));
}
// asin(s) / s, x = s^2 up to 1 / 64
__device__ __forceinline__ double series_asinc(double x) {
  return 1.0 + x * (1.0 / 6 + x * (3.0 / 40 + x * (5.0 / 112 + x * (35.0 / 1152 + x * (63.0 / 2816 + x * (231.0 / 13312 +
         x * (143.0 / 10240 + x * (6435.0 / 557056))))))));
}

// Exp(w) by Rodrigues: I + a K + b K^2 with K = [w]x, a = sin t / t, b = (1 - cos t) / t^2.
__device__ inline void so3_exp(const double* w, double* R) {
  const double t2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
  double a, b;
  if (t2 < kSeriesT2) {
    a = series_sinc(t2);
    b = series_cosc(t2);
  } else {
    const double t = sqrt(t2);
    a = sin(t) / t;
    b = (1.0 - cos(t)) / t2;
  }
  // K^2 = w w^T - t2 I
  const double x = w[0], y = w[1], z = w[2];
  R[0] = 1.0 + b * (x * x - t2); R[1] = -a * z + b * x * y;     R[2] = a * y + b * x * z;
  R[3] = a * z + b * x * y;      R[4] = 1.0 + b * (y * y - t2); R[5] = -a * x + b * y * z;
  R[6] = -a * y + b * x * z;     R[7] = a * x + b * y * z;      R[8] = 1.0 + b * (z * z - t2);
}

// Log(R): angle from atan2(|vee(R - R^T)|/2, (tr R - 1)/2); near pi the axis
// comes from the symmetric part.
__device__ inline void so3_log(const double* R, double* w) {
  const double vx = R[7] - R[5], vy = R[2] - R[6], vz = R[3] - R[1];
  const double s2 = 0.25 * (vx * vx + vy * vy + vz * vz);
  const double c = 0.5 * (R[0] + R[4] + R[8] - 1.0);
  if (s2 < 1.0 / 64 && c > 0.0) {
    const double f = 0.5 * series_asinc(s2);     // t / (2 sin t)
    w[0] = f * vx; w[1] = f * vy; w[2] = f * vz;
    return;
  }
  const double t = atan2(sqrt(s2), c);
  if (M_PI - t > 1e-6) {
    const double f = 0.5 * t / sin(t);
    w[0] = f * vx; w[1] = f * vy; w[2] = f * vz;
    return;
  }
  // u u^T = (R + R^T - 2 c I) / (2 (1 - c))
  const double den = 2.0 * (1.0 - c);
  double M[9];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int q = 0; q < 3; ++q) M[r * 3 + q] = (R[r * 3 + q] + R[q * 3 + r] - (r == q ? 2.0 * c : 0.0)) / den;
  // column k of the largest diagonal entry, chosen by selects (an index into
  // M would put M in scratch memory)
  int k = 0;
  double mk = M[0];
  if (M[4] > mk) { k = 1; mk = M[4]; }
  if (M[8] > mk) { k = 2; mk = M[8]; }
  const double nk = sqrt(fmax(mk, 1e-300));
  double u[3] = {(k == 0 ? M[0] : k == 1 ? M[1] : M[2]) / nk, (k == 0 ? M[3] : k == 1 ? M[4] : M[5]) / nk,
                 (k == 0 ? M[6] : k == 1 ? M[7] : M[8]) / nk};
  if (u[0] * vx + u[1] * vy + u[2] * vz < 0.0) { u[0] = -u[0]; u[1] = -u[1]; u[2] = -u[2]; }
  w[0] = t * u[0]; w[1] = t * u[1]; w[2] = t * u[2];
}

// Right Jacobian: I - a K + b K^2, a = (1 - cos t)/t^2, b = (t - sin t)/t^3.
__device__ inline void so3_jr(const double* w, double* J) {
  const double t2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
  double a, b;
  if (t2 < kSeriesT2) {
    a = series_cosc(t2);
    b = series_sinc3(t2);
  } else {
    const double t = sqrt(t2);
    a = (1.0 - cos(t)) / t2;
    b = (t - sin(t)) / (t2 * t);
  }
  const double x = w[0], y = w[1], z = w[2];
  J[0] = 1.0 + b * (x * x - t2); J[1] = a * z + b * x * y;       J[2] = -a * y + b * x * z;
  J[3] = -a * z + b * x * y;     J[4] = 1.0 + b * (y * y - t2); J[5] = a * x + b * y * z;
  J[6] = a * y + b * x * z;      J[7] = -a * x + b * y * z;     J[8] = 1.0 + b * (z * z - t2);
}

// Inverse right Jacobian: I + K/2 + c K^2, c = 1/t^2 - (1 + cos t) / (2 t sin t).
__device__ inline void so3_jr_inv(const double* w, double* J) {
  const double t2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
  double c;
  if (t2 < kSeriesT2) {
    c = series_cot(t2);
  } else {
    const double t = sqrt(t2);
    c = 1.0 / t2 - (1.0 + cos(t)) / (2.0 * t * sin(t));
  }
  const double x = w[0], y = w[1], z = w[2];
  J[0] = 1.0 + c * (x * x - t2); J[1] = -0.5 * z + c * x * y;    J[2] = 0.5 * y + c * x * z;
  J[3] = 0.5 * z + c * x * y;    J[4] = 1.0 + c * (y * y - t2); J[5] = -0.5 * x + c * y * z;
  J[6] = -0.5 * y + c * x * z;   J[7] = 0.5 * x + c * y * z;    J[8] = 1.0 + c * (z * z - t2);
}

// Rotation matrix of the quaternion (x, y, z, w), normalised on the fly.
__device__ inline void quat_to_rot(const double* q, double* R) {
  const double n = q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3];
  const double s = 2.0 / n;
  const double x = q[0], y = q[1], z = q[2], w = q[3];
  R[0] = 1.0 - s * (y * y + z * z); R[1] = s * (x * y - z * w);       R[2] = s * (x * z + y * w);
  R[3] = s * (x * y + z * w);       R[4] = 1.0 - s * (x * x + z * z); R[5] = s * (y * z - x * w);
  R[6] = s * (x * z - y * w);       R[7] = s * (y * z + x * w);       R[8] = 1.0 - s * (x * x + y * y);
}

// Unit quaternion (x, y, z, w) of a rotation matrix, from the largest of
// 1 + tr R, 1 + 2 R_00 - tr R, 1 + 2 R_11 - tr R, 1 + 2 R_22 - tr R (the
// numerically safe pivot), normalised at the end.
__device__ inline void rot_to_quat(const double* R, double* q) {
  const double tr = R[0] + R[4] + R[8];
  const double c[4] = {1.0 + tr, 1.0 + 2.0 * R[0] - tr, 1.0 + 2.0 * R[4] - tr, 1.0 + 2.0 * R[8] - tr};
  int k = 0;
  double ck = c[0];                     // c[k], kept by value (an index into c would put c in scratch memory)
#pragma unroll
  for (int i = 1; i < 4; ++i)
    if (c[i] > ck) { k = i; ck = c[i]; }
  const double s = 0.5 / sqrt(ck);     // 4 * (the pivot component) = 2 sqrt(c[k])
  double x, y, z, w;
  if (k == 0) {
    w = 0.5 * sqrt(c[0]); x = (R[7] - R[5]) * s; y = (R[2] - R[6]) * s; z = (R[3] - R[1]) * s;
  } else if (k == 1) {
    x = 0.5 * sqrt(c[1]); w = (R[7] - R[5]) * s; y = (R[1] + R[3]) * s; z = (R[2] + R[6]) * s;
  } else if (k == 2) {
    y = 0.5 * sqrt(c[2]); w = (R[2] - R[6]) * s; x = (R[1] + R[3]) * s; z = (R[5] + R[7]) * s;
  } else {
    z = 0.5 * sqrt(c[3]); w = (R[3] - R[1]) * s; x = (R[2] + R[6]) * s; y = (R[5] + R[7]) * s;
  }
  const double n = 1.0 / sqrt(x * x + y * y + z * z + w * w);
  q[0] = x * n; q[1] = y * n; q[2] = z * n; q[3] = w * n;
}

// q <- normalise(q (x) exp_q(w)): the quaternion form of R <- R Exp(w).
__device__ inline void quat_retract(double* q, const double* w) {
  const double t2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
  double sh, ch;
  if (t2 < kSeriesT2) {
    const double x = 0.25 * t2;
    sh = 0.5 * series_sinc(x);         // sin(t/2)/t
    ch = 1.0 - x * series_cosc(x);     // cos(t/2)
  } else {
    const double t = sqrt(t2);
    sh = sin(0.5 * t) / t;
    ch = cos(0.5 * t);
  }
  const double bx = w[0] * sh, by = w[1] * sh, bz = w[2] * sh, bw = ch;
  const double ax = q[0], ay = q[1], az = q[2], aw = q[3];
  double nx = aw * bx + ax * bw + ay * bz - az * by;
  double ny = aw * by - ax * bz + ay * bw + az * bx;
  double nz = aw * bz + ax * by - ay * bx + az * bw;
  double nw = aw * bw - ax * bx - ay * by - az * bz;
  const double inv = 1.0 / sqrt(nx * nx + ny * ny + nz * nz + nw * nw);
  q[0] = nx * inv; q[1] = ny * inv; q[2] = nz * inv; q[3] = nw * inv;
}

// LDS operations of one wave complete in order: a compiler barrier is enough
// between a write of one lane and the read of another
__device__ __forceinline__ void wave_lds_sync() { asm volatile("" ::: "memory"); }

// Cholesky factor of a 9 x 9 SPD block by one wave, every lane in registers: L
// holds the lower part packed by rows, on return the factor below the diagonal
// and on it the pivots L_jj^2.  Along with it each lane solves L x = v for its
// own v.  Returns the first pivot that is not positive, or -1.
__device__ __forceinline__ constexpr int tri9c(int i, int j) { return i * (i + 1) / 2 + j; }

__device__ __forceinline__ int factor9_solve(double (&L)[46], double (&v)[9]) {
  int bad = -1;
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    const double piv = L[tri9c(j, j)];
    const bool ok = piv > 0.0;
    if (!ok && bad < 0) bad = j;
    const double r = ok ? rsqrt_refined(__builtin_fabs(piv)) : 1.0;
    v[j] *= r;
#pragma unroll
    for (int i = 1; i < 9; ++i)
      if (i > j) L[tri9c(i, j)] *= r;
#pragma unroll
    for (int i = 1; i < 9; ++i)
#pragma unroll
      for (int m = 1; m < 9; ++m)
        if (i > j && m > j && m <= i) L[tri9c(i, m)] -= L[tri9c(i, j)] * L[tri9c(m, j)];
#pragma unroll
    for (int i = 1; i < 9; ++i)
      if (i > j) v[i] -= L[tri9c(i, j)] * v[j];
  }
  return bad;
}

}  // namespace vi
