// Per-ray relighting colour (colour mode 4), the preprocess side: the colour
// network in the ellipsoid's unit-sphere frame, and its adjoint back to the
// network's parameters, the rotation, the scales and the centres.
//
// The relighting application colours each view ray by a constant colour plus
// a per-primitive colour network of the 3D position, the ray direction and
// the light direction, the latter relative to the primitive's centre; the
// position is the ray's entry point into the bounding ellipsoid, normalised
// as the density network's input (Eq. 5).  The rasterizer evaluates it per
// (pixel, primitive) pair from the table built here (see RayColourLayout).
#include "snp_internal.h"

namespace snp {

__device__ __forceinline__ void rotation_f64(const float* qf, double Rp[3][3]) {
  const double q0 = qf[0], q1 = qf[1], q2 = qf[2], q3 = qf[3];
  const double qn = sqrt(((q0 * q0 + q1 * q1) + q2 * q2) + q3 * q3);
  const double w = q0 / qn, x = q1 / qn, y = q2 / qn, z = q3 / qn;
  Rp[0][0] = 1.0 - 2.0 * (y * y + z * z);
  Rp[0][1] = 2.0 * (x * y - w * z);
  Rp[0][2] = 2.0 * (x * z + w * y);
  Rp[1][0] = 2.0 * (x * y + w * z);
  Rp[1][1] = 1.0 - 2.0 * (x * x + z * z);
  Rp[1][2] = 2.0 * (y * z - w * x);
  Rp[2][0] = 2.0 * (x * z - w * y);
  Rp[2][1] = 2.0 * (y * z + w * x);
  Rp[2][2] = 1.0 - 2.0 * (x * x + y * y);
}

// kGroup lanes per primitive: Au, Ad and the copied hidden and output layers.
// The lanes take the units in turn, so that a row is read and written as
// whole runs of memory, whose traffic is the bound (200k primitives of 16
// units: 1.05 ms with a thread per primitive, now 0.26).
template <int W, int D>
__global__ void __launch_bounds__(256) ray_table_kernel(RayColourArgs a) {
  using Lt = RayColourLayout<W, D>;
  const int64_t p = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kGroup;
  const int q = (int)(threadIdx.x % kGroup);
  if (p >= a.P) return;
  constexpr int K = kRayIn * W + W + (D - 1) * (W * W + W) + 3 * W + 3;
  const float* c = a.cmlp + p * K;
  double Rp[3][3];
  rotation_f64(a.quats + 4 * p, Rp);
  const double s[3] = {a.scales[3 * p], a.scales[3 * p + 1], a.scales[3 * p + 2]};
  const double m = fmax(s[0], fmax(s[1], s[2]));
  float* row = a.ctab + p * Lt::CTS;
#pragma unroll
  for (int u = 0; u < W / kGroup; ++u) {
    const int k = u * kGroup + q;
    const float* w1 = c + k * kRayIn;
    for (int j = 0; j < 3; ++j) {
      const double rs = s[j];
      row[Lt::AU + 3 * k + j] = (float)(((w1[0] * Rp[0][j] + w1[1] * Rp[1][j]) + w1[2] * Rp[2][j]) * rs / m);
      row[Lt::AD + 3 * k + j] = (float)(((w1[3] * Rp[0][j] + w1[4] * Rp[1][j]) + w1[5] * Rp[2][j]) * rs);
    }
  }
  int pos = kRayIn * W + W;  // after W1 and b1
  if (D == 2) {
#pragma unroll 4
    for (int i = q; i < W * W + W; i += kGroup) row[Lt::WH + i] = c[pos + i];
    pos += W * W + W;
  }
#pragma unroll
  for (int i = q; i < 3 * W + 3; i += kGroup) row[Lt::WO + i] = c[pos + i];
  for (int i = Lt::CT + q; i < Lt::CTS; i += kGroup) row[i] = 0.f;
}

// one thread per (view, primitive): cb = b1 + W1[:, 6:9] normalize(l_v - x_B)
template <int W>
__global__ void __launch_bounds__(256) ray_bias_kernel(RayColourArgs a, int K) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.P * a.V) return;
  const int v = (int)(i / a.P);
  const int64_t p = i - (int64_t)v * a.P;
  float* cb = a.cbias + i * W;
  if (a.tile_counts[i] == 0) {
    for (int k = 0; k < W; ++k) cb[k] = 0.f;
    return;
  }
  const CamDev& cam = a.cams[v];
  const float lx = cam.light[0] - a.centers[3 * p];
  const float ly = cam.light[1] - a.centers[3 * p + 1];
  const float lz = cam.light[2] - a.centers[3 * p + 2];
  const float il = 1.0f / sqrtf(lx * lx + ly * ly + lz * lz);
  const float* c = a.cmlp + p * K;
  for (int k = 0; k < W; ++k) {
    const float* w1 = c + k * kRayIn;
    cb[k] = c[kRayIn * W + k] + (w1[6] * lx + w1[7] * ly + w1[8] * lz) * il;
  }
}

// Adjoint, kGroup lanes per primitive, each with the units k = lane (mod the
// group).  From the table gradients: the hidden and output layers directly,
// W1's position and direction columns, and the rotation and scales through
// Au = W1p R S / m, Ad = W1d R S (written to extra_rs for the preprocess
// adjoint, which chains them to the raw quaternion and the scales); from the
// bias gradients over the views: b1, W1's light columns and the centre
// through the light direction.  The rotation and the scales need only the sums
// P[i][j] = sum_k g_Au_k[j] W1p_k[i] and Q[i][j] = sum_k g_Ad_k[j] W1d_k[i].
// Bound by its traffic (200k primitives of 16 units: 1.32 ms with a thread
// per primitive, now 0.26).
template <int W, int D, bool ADD>
__global__ void __launch_bounds__(256) ray_colour_bwd_kernel(RayColourArgs a) {
  using Lt = RayColourLayout<W, D>;
  constexpr int UPL = W / kGroup;  // units per lane
  const int64_t p = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kGroup;
  const int q = (int)(threadIdx.x % kGroup);
  if (p >= a.P) return;
  constexpr int K = kRayIn * W + W + (D - 1) * (W * W + W) + 3 * W + 3;
  const float* c = a.cmlp + p * K;
  const float* gt = a.gctab + p * Lt::CTS;
  float* gc = a.g_cmlp ? a.g_cmlp + p * K : nullptr;
  double Rp[3][3];
  rotation_f64(a.quats + 4 * p, Rp);
  const double s[3] = {a.scales[3 * p], a.scales[3 * p + 1], a.scales[3 * p + 2]};
  const double m = fmax(s[0], fmax(s[1], s[2]));
  const int am = (s[0] >= s[1] && s[0] >= s[2]) ? 0 : (s[1] >= s[2] ? 1 : 2);
  // bias: b1 and the light columns per view, the light direction to x_B
  double gb1[UPL], gwl[UPL][3], gx[3] = {0, 0, 0};
#pragma unroll
  for (int u = 0; u < UPL; ++u) {
    gb1[u] = 0.0;
    for (int ii = 0; ii < 3; ++ii) gwl[u][ii] = 0.0;
  }
  for (int v = 0; v < a.V; ++v) {
    const int64_t i = (int64_t)v * a.P + p;
    if (a.tile_counts[i] == 0) continue;
    const float* gb = a.gcbias + i * W;
    const CamDev& cam = a.cams[v];
    const double lv[3] = {(double)cam.light[0] - a.centers[3 * p], (double)cam.light[1] - a.centers[3 * p + 1],
                          (double)cam.light[2] - a.centers[3 * p + 2]};
    const double len = sqrt(lv[0] * lv[0] + lv[1] * lv[1] + lv[2] * lv[2]);
    const double ld[3] = {lv[0] / len, lv[1] / len, lv[2] / len};
    double gld[3] = {0, 0, 0};
#pragma unroll
    for (int u = 0; u < UPL; ++u) {
      const int k = u * kGroup + q;
      const double g = gb[k];
      gb1[u] += g;
      for (int ii = 0; ii < 3; ++ii) {
        gwl[u][ii] += g * ld[ii];
        gld[ii] += g * c[k * kRayIn + 6 + ii];
      }
    }
    for (int ii = 0; ii < 3; ++ii) gld[ii] = group_sum(gld[ii]);
    // ld = (l - x_B) / |l - x_B|:  d ld / d x_B = -(I - ld ld^T) / |l - x_B|
    const double dd = ld[0] * gld[0] + ld[1] * gld[1] + ld[2] * gld[2];
    for (int ii = 0; ii < 3; ++ii) gx[ii] -= (gld[ii] - ld[ii] * dd) / len;
  }
  double Pu[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, Qu[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
#pragma unroll
  for (int u = 0; u < UPL; ++u) {
    const int k = u * kGroup + q;
    const float* w1 = c + k * kRayIn;
    double gau[3], gad[3];
    for (int j = 0; j < 3; ++j) {
      gau[j] = gt[Lt::AU + 3 * k + j];
      gad[j] = gt[Lt::AD + 3 * k + j];
    }
    for (int ii = 0; ii < 3; ++ii) {
      double gp = 0.0, gd = 0.0;
      for (int j = 0; j < 3; ++j) {
        Pu[ii][j] += gau[j] * w1[ii];
        Qu[ii][j] += gad[j] * w1[3 + ii];
        gp += gau[j] * Rp[ii][j] * s[j];
        gd += gad[j] * Rp[ii][j] * s[j];
      }
      if (gc) {
        put_grad<ADD>(gc + k * kRayIn + ii, (float)(gp / m));
        put_grad<ADD>(gc + k * kRayIn + 3 + ii, (float)gd);
        put_grad<ADD>(gc + k * kRayIn + 6 + ii, (float)gwl[u][ii]);
      }
    }
    if (gc) put_grad<ADD>(gc + kRayIn * W + k, (float)gb1[u]);
  }
  if (gc) {
    int pos = kRayIn * W + W;
    if (D == 2) {
#pragma unroll 4
      for (int i = q; i < W * W + W; i += kGroup) put_grad<ADD>(gc + pos + i, gt[Lt::WH + i]);
      pos += W * W + W;
    }
#pragma unroll
    for (int i = q; i < 3 * W + 3; i += kGroup) put_grad<ADD>(gc + pos + i, gt[Lt::WO + i]);
  }
  double gR[3][3], gs[3], gm = 0.0;
  for (int j = 0; j < 3; ++j) {
    double rp = 0.0, rq = 0.0;
    for (int ii = 0; ii < 3; ++ii) {
      const double pu = group_sum(Pu[ii][j]), qu = group_sum(Qu[ii][j]);
      gR[ii][j] = pu * s[j] / m + qu * s[j];
      rp += Rp[ii][j] * pu;
      rq += Rp[ii][j] * qu;
    }
    gs[j] = rp / m + rq;
    gm -= s[j] * rp / (m * m);
  }
  if (q != 0) return;
  if (a.g_centers)
    for (int ii = 0; ii < 3; ++ii) put_grad<ADD>(a.g_centers + 3 * p + ii, (float)gx[ii]);
  float* ex = a.extra_rs + p * 12;
  for (int ii = 0; ii < 3; ++ii)
    for (int j = 0; j < 3; ++j) ex[3 * ii + j] = (float)gR[ii][j];
  for (int j = 0; j < 3; ++j) ex[9 + j] = (float)(gs[j] + (j == am ? gm : 0.0));
}

// the rasterizers evaluate the network with one hidden layer of 16 units
bool ray_colour_supported(int width, int depth) { return width == 16 && depth == 1; }

int ray_colour_param_count(int width, int depth) {
  return kRayIn * width + width + (depth - 1) * (width * width + width) + 3 * width + 3;
}

hipError_t launch_ray_colour_fwd(const RayColourArgs& a, hipStream_t st) {
  const dim3 block(256);
  const dim3 gp((unsigned)((a.P * kGroup + 255) / 256)), gv((unsigned)((a.P * a.V + 255) / 256));
  const int K = ray_colour_param_count(a.W, a.D);
  if (a.W != 16) return hipErrorInvalidValue;
  if (a.D == 1)
    hipLaunchKernelGGL((ray_table_kernel<16, 1>), gp, block, 0, st, a);
  else if (a.D == 2)
    hipLaunchKernelGGL((ray_table_kernel<16, 2>), gp, block, 0, st, a);
  else
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(ray_bias_kernel<16>, gv, block, 0, st, a, K);
  return hipGetLastError();
}

template <int D>
static void ray_colour_bwd(const RayColourArgs& a, hipStream_t st) {
  const dim3 block(256), grid((unsigned)((a.P * kGroup + 255) / 256));
  if (a.accumulate)
    hipLaunchKernelGGL((ray_colour_bwd_kernel<16, D, true>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((ray_colour_bwd_kernel<16, D, false>), grid, block, 0, st, a);
}

hipError_t launch_ray_colour_bwd(const RayColourArgs& a, hipStream_t st) {
  if (a.W != 16) return hipErrorInvalidValue;
  if (a.D == 1)
    ray_colour_bwd<1>(a, st);
  else if (a.D == 2)
    ray_colour_bwd<2>(a, st);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace snp
