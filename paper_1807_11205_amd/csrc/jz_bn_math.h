// Batch normalization per channel and per element, for every kernel that finishes one.  Included inside a kernel file's anonymous
// namespace.
#pragma once

// One element of dx.  Written out where kernels share a formula: left to the compiler, products and sums are contracted one way here
// and another way there, and the bits differ.
__device__ __forceinline__ float bn_dx(float a, float g, float p, float x, float q) { return fmaf(a, g, fmaf(p, x, q)); }

// mean and 1 / sqrt(var + eps) of one channel (written where the pointers are not null) and y = a x + b
__device__ __forceinline__ void bn_fwd_coef(double s, double q, double inv_rows, float eps, float gamma, float beta, float* save_mean,
                                            float* save_invstd, float* coef, int pitch) {
  const double m = s * inv_rows;
  double var = fma(-m, m, q * inv_rows);
  if (var < 0.0) var = 0.0;
  const double is = 1.0 / sqrt(var + (double)eps);
  const float mf = (float)m, isf = (float)is;
  if (save_mean) *save_mean = mf;
  if (save_invstd) *save_invstd = isf;
  const float a = gamma * isf;
  coef[0] = a;
  coef[pitch] = fmaf(-mf, a, beta);
}

// the parameter gradients of one channel (written where the pointers are not null) and its dx = a (g - dbeta/M - x^ dgamma/M),
// x^ = (x - mean) invstd, as a g + P x + Q
__device__ __forceinline__ void bn_bwd_coef(double sb, double sg, double inv_rows, float gamma, float mean, float invstd,
                                            unsigned short* dgamma16, unsigned short* dbeta16, float* coef, int pitch) {
  _Float16 hg = (_Float16)(float)sg, hb = (_Float16)(float)sb;
  if (dgamma16) __builtin_memcpy(dgamma16, &hg, 2);
  if (dbeta16) __builtin_memcpy(dbeta16, &hb, 2);
  const double a = (double)gamma * (double)invstd;
  const double t = a * (sg * inv_rows) * (double)invstd;
  coef[0] = (float)a;
  coef[pitch] = (float)(-t);
  coef[2 * pitch] = (float)fma(t, (double)mean, -(a * (sb * inv_rows)));
}
