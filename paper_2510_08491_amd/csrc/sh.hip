// Spherical-harmonics colour of degree 3 (the colour the paper adopts for
// novel-view synthesis, Sec. 3.1; four bands as in 3DGS, Sec. 3.3): per
// (primitive, view), with d = normalize(x_B - o_v) and the 16 real
// orthonormal harmonics Y_k of degrees 0..3 in (l, m) order (0,0), (1,-1),
// (1,0), (1,1), (2,-2) ... (3,3),
//
//     colour_c = max(0, 1/2 + sum_k Y_k(d) sh[k][c])
//
// Coefficients are stored per primitive as sh[16][3] (basis, channel).  In
// the dynamic-scene application the zero-order coefficient is a function of
// the time xi_t: sh[0][c] + sum_k tb_k sh_t[k][c] with tb = (xi, xi^2, xi^3,
// xi^4, cos xi, ..., cos 4 xi, sin xi, ..., sin 4 xi) (a polynomial and a
// Fourier series of degree 4).
#include "snp_internal.h"

namespace snp {

// normalisation constants of the real harmonics: 1/2 sqrt(1/pi), sqrt(3/(4pi)),
// 1/2 sqrt(15/pi), 1/4 sqrt(5/pi), 1/4 sqrt(15/pi), 1/4 sqrt(35/(2pi)),
// 1/2 sqrt(105/pi), 1/4 sqrt(21/(2pi)), 1/4 sqrt(7/pi), 1/4 sqrt(105/pi)
constexpr float kSh0 = 0.28209479177387814f;
constexpr float kSh1 = 0.4886025119029199f;
constexpr float kSh2a = 1.0925484305920792f;
constexpr float kSh2b = 0.31539156525252005f;
constexpr float kSh2c = 0.5462742152960396f;
constexpr float kSh3a = 0.5900435899266435f;
constexpr float kSh3b = 2.890611442640554f;
constexpr float kSh3c = 0.4570457994644658f;
constexpr float kSh3d = 0.3731763325901154f;
constexpr float kSh3e = 1.445305721320277f;

__device__ __forceinline__ void sh_basis(float x, float y, float z, float (&Y)[16]) {
  const float xx = x * x, yy = y * y, zz = z * z;
  Y[0] = kSh0;
  Y[1] = kSh1 * y;
  Y[2] = kSh1 * z;
  Y[3] = kSh1 * x;
  Y[4] = kSh2a * x * y;
  Y[5] = kSh2a * y * z;
  Y[6] = kSh2b * (3.f * zz - 1.f);
  Y[7] = kSh2a * x * z;
  Y[8] = kSh2c * (xx - yy);
  Y[9] = kSh3a * y * (3.f * xx - yy);
  Y[10] = kSh3b * x * y * z;
  Y[11] = kSh3c * y * (5.f * zz - 1.f);
  Y[12] = kSh3d * z * (5.f * zz - 3.f);
  Y[13] = kSh3c * x * (5.f * zz - 1.f);
  Y[14] = kSh3e * z * (xx - yy);
  Y[15] = kSh3a * x * (xx - 3.f * yy);
}

// gradient with respect to (x, y, z) of sum_k w_k Y_k (the polynomials above)
__device__ __forceinline__ void sh_weighted_grad(float x, float y, float z, const float (&w)[16], float& gx, float& gy,
                                                 float& gz) {
  const float xx = x * x, yy = y * y, zz = z * z;
  gx = kSh1 * w[3] + kSh2a * (y * w[4] + z * w[7]) + 2.f * kSh2c * x * w[8] + 6.f * kSh3a * x * y * w[9] +
       kSh3b * y * z * w[10] + kSh3c * (5.f * zz - 1.f) * w[13] + 2.f * kSh3e * x * z * w[14] +
       3.f * kSh3a * (xx - yy) * w[15];
  gy = kSh1 * w[1] + kSh2a * (x * w[4] + z * w[5]) - 2.f * kSh2c * y * w[8] + 3.f * kSh3a * (xx - yy) * w[9] +
       kSh3b * x * z * w[10] + kSh3c * (5.f * zz - 1.f) * w[11] - 2.f * kSh3e * y * z * w[14] -
       6.f * kSh3a * x * y * w[15];
  gz = kSh1 * w[2] + kSh2a * (y * w[5] + x * w[7]) + 6.f * kSh2b * z * w[6] + kSh3b * x * y * w[10] +
       10.f * kSh3c * y * z * w[11] + kSh3d * (15.f * zz - 3.f) * w[12] + 10.f * kSh3c * x * z * w[13] +
       kSh3e * (xx - yy) * w[14];
}

__device__ __forceinline__ void view_dir(const ShArgs& a, int v, const float (&xb)[3], float& x, float& y, float& z) {
  const CamDev& cam = a.cams[v];
  const float dx = xb[0] - cam.o_f[0];
  const float dy = xb[1] - cam.o_f[1];
  const float dz = xb[2] - cam.o_f[2];
  const float il = 1.0f / sqrtf(dx * dx + dy * dy + dz * dz);
  x = dx * il;
  y = dy * il;
  z = dz * il;
}

// Four lanes per primitive (kGroup): lane q holds the coefficients 4 q .. 4 q
// + 3 and the time coefficients 3 q .. 3 q + 2, a quarter of a row each, so
// that a wave reads and writes whole runs of memory.  A channel's sum passes
// from lane to lane, so that its terms are added in the order of k.  Bound by that traffic (100k primitives; a thread per
// primitive before: forward of one view 18 -> 8.1 us, of two views with the
// time term 38 -> 16.4 us, adjoint 21 -> 18 us and 40 -> 23.6 us; adding the
// lanes' shares in a tree instead takes 1 us less and rounds differently).
static_assert(kGroup == 4 && kShTime == 12, "a quarter of the rows per lane");

// lane L's value of each group of four
template <int L>
__device__ __forceinline__ float group_lane(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x55 * L, 0xF, 0xF, false));  // quad_perm L,L,L,L
}

// the value of lane q's quarter.  (By value, in registers: an index or a
// select among the elements of an array would put it into scratch.)
__device__ __forceinline__ float pick4(float a0, float a1, float a2, float a3, int q) {
  asm("" : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3));
  const float lo = q == 0 ? a0 : a1, hi = q == 2 ? a2 : a3;
  return q < 2 ? lo : hi;
}

// this lane's four of the sixteen basis values
__device__ __forceinline__ void own_basis(const float (&Y)[16], int q, float (&Yq)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) Yq[i] = pick4(Y[i], Y[4 + i], Y[8 + i], Y[12 + i], q);
}

// this lane's k-th function of the time
__device__ __forceinline__ float own_time(const ShArgs& a, int q, int k) {
  return pick4(a.tb[k], a.tb[3 + k], a.tb[6 + k], a.tb[9 + k], q);
}

// x[ch] = fma(f[i], r[i][ch], x[ch]) for i = FROM .. n - 1 with lane L's f
// and r, the result in every lane
template <int L, int FROM, int n>
__device__ __forceinline__ void chain(const float (&f)[n], const float (&r)[n][3], float (&x)[3]) {
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    float y = x[ch];
#pragma unroll
    for (int i = FROM; i < n; ++i) y = __builtin_fmaf(f[i], r[i][ch], y);
    x[ch] = group_lane<L>(y);
  }
}

// this lane's coefficients and the zero-order coefficient of the primitive
// (time dependent with sh_t)
__device__ __forceinline__ void own_coeffs(const ShArgs& a, int64_t p, int q, float (&c)[4][3], float (&zo)[3]) {
  const float* r = a.sh + p * kShCoeffs + 12 * q;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) c[i][ch] = r[3 * i + ch];
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) zo[ch] = group_lane<0>(c[0][ch]);
  if (a.sh_t) {
    const float* t = a.sh_t + p * (kShTime * 3) + 9 * q;
    float f[3], tc[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      f[k] = own_time(a, q, k);
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) tc[k][ch] = t[3 * k + ch];
    }
    chain<0, 0>(f, tc, zo);
    chain<1, 0>(f, tc, zo);
    chain<2, 0>(f, tc, zo);
    chain<3, 0>(f, tc, zo);
  }
}

// one group per (view, primitive): colour into the record
__global__ void __launch_bounds__(256) sh_fwd_kernel(ShArgs a) {
  const int64_t i = (pair_block() * 256 + threadIdx.x) / kGroup;
  const int q = (int)(threadIdx.x % kGroup);
  if (i >= (int64_t)a.V * a.P || a.tile_counts[i] == 0) return;  // whole groups
  const int v = (int)(i / a.P);
  const int64_t p = i - (int64_t)v * a.P;
  float x, y, z, Y[16], Yq[4], c[4][3], zo[3], s[3] = {0.5f, 0.5f, 0.5f};
  const float xb[3] = {a.centers[3 * p], a.centers[3 * p + 1], a.centers[3 * p + 2]};
  own_coeffs(a, p, q, c, zo);
  view_dir(a, v, xb, x, y, z);
  sh_basis(x, y, z, Y);
  own_basis(Y, q, Yq);
  chain<0, 1>(Yq, c, s);
  chain<1, 0>(Yq, c, s);
  chain<2, 0>(Yq, c, s);
  chain<3, 0>(Yq, c, s);
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) s[ch] = __builtin_fmaf(Y[0], zo[ch], s[ch]);
  if (q < 3) a.records[i * kRecFloats + 11 + 4 * q] = fmaxf(q == 0 ? s[0] : q == 1 ? s[1] : s[2], 0.f);
}

// one group per primitive, its views in turn: coefficient gradients summed
// over the views (kept in registers), the direction gradient of each view
// written to the view's gradient record (slots 21..23) for the chain to the
// centre; a clamped channel passes no gradient
template <bool ADD>
__global__ void __launch_bounds__(256) sh_bwd_kernel(ShArgs a) {
  const int64_t p = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kGroup;
  const int q = (int)(threadIdx.x % kGroup);
  if (p >= a.P) return;
  float c[4][3], g[4][3], zo[3], g0[3] = {0.f, 0.f, 0.f};
  const float xb[3] = {a.centers[3 * p], a.centers[3 * p + 1], a.centers[3 * p + 2]};
  own_coeffs(a, p, q, c, zo);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) g[i][ch] = 0.f;
  for (int v = 0; v < a.V; ++v) {
    const int64_t i = (int64_t)v * a.P + p;
    float* gv = a.gview + i * kGViewFloats;
    float gc[3] = {gv[18], gv[19], gv[20]};  // in flight together with the count
    if (a.tile_counts[i] == 0) continue;
    float x, y, z, Y[16], Yq[4], s[3];
    view_dir(a, v, xb, x, y, z);
    sh_basis(x, y, z, Y);
    own_basis(Y, q, Yq);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) s[ch] = __builtin_fmaf(Y[0], zo[ch], 0.5f);
    chain<0, 1>(Yq, c, s);
    chain<1, 0>(Yq, c, s);
    chain<2, 0>(Yq, c, s);
    chain<3, 0>(Yq, c, s);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      if (!(s[ch] > 0.f)) gc[ch] = 0.f;
      g0[ch] = __builtin_fmaf(gc[ch], kSh0, g0[ch]);
    }
    float wq[4], w[16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) g[k][ch] = __builtin_fmaf(gc[ch], Yq[k], g[k][ch]);
      wq[k] = gc[0] * c[k][0] + gc[1] * c[k][1] + gc[2] * c[k][2];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // every lane gets all sixteen
      w[k] = group_lane<0>(wq[k]);
      w[4 + k] = group_lane<1>(wq[k]);
      w[8 + k] = group_lane<2>(wq[k]);
      w[12 + k] = group_lane<3>(wq[k]);
    }
    float gx, gy, gz;
    sh_weighted_grad(x, y, z, w, gx, gy, gz);
    if (q < 3) gv[21 + q] = q == 0 ? gx : q == 1 ? gy : gz;
  }
  if (a.g_sh) {
    float* r = a.g_sh + p * kShCoeffs + 12 * q;
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) put_grad<ADD>(r + 3 * k + ch, g[k][ch]);
  }
  // the time coefficients: d S0(xi) / d sh_t[k][c] = tb_k
  // (zero where the colour does not depend on the time)
  if (a.g_sh_t && (a.sh_t || !ADD)) {
    float* r = a.g_sh_t + p * (kShTime * 3) + 9 * q;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float tb = own_time(a, q, k);
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) put_grad<ADD>(r + 3 * k + ch, a.sh_t ? tb * g0[ch] : 0.f);
    }
  }
}

hipError_t launch_sh_fwd(const ShArgs& a, hipStream_t st) {
  const int64_t n = (int64_t)a.V * a.P * kGroup;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sh_fwd_kernel, pair_grid((n + 255) / 256), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_sh_bwd(const ShArgs& a, hipStream_t st) {
  if (a.P <= 0) return hipSuccess;
  const dim3 grid((unsigned)((a.P * kGroup + 255) / 256)), block(256);
  if (a.accumulate)
    hipLaunchKernelGGL(sh_bwd_kernel<true>, grid, block, 0, st, a);
  else
    hipLaunchKernelGGL(sh_bwd_kernel<false>, grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace snp
