// Compositing of the primitives' colours into an image for one camera
// (Section 3.1: C = sum_i T_i alpha_i c_i, alpha_i = sigma_i rho_i,
// T_i = prod_{j<i} (1 - alpha_j)), with the gradients of a loss on the image
// with respect to the per-primitive colours (what the appearance backward
// consumes), opacities and, on request, the geometry (mean, scales,
// quaternion) through rho.
//
// The primitives are 3D Gaussians (mean, per-axis scale, quaternion
// rotation); rho on a pixel's ray is the Gaussian projected onto the image
// plane (the local affine approximation of the perspective map at the mean),
// evaluated at the pixel centre. A primitive reaches a pixel only inside its
// 3-sigma ellipse and only in front of the near plane Z = 0.2; alpha is
// clamped at 0.99; the background is black.
//
// Pipeline (all on the caller's stream, nothing allocated, no host sync):
//   project : per primitive, FP64 pixel mean, inverse 2D covariance, depth and
//             the 16 x 16-pixel tiles its ellipse's bounding box touches, kept
//             with the colour and opacity in a 64-byte render record; the same
//             launch clears the tile cursors;
//   bin     : each primitive's 64-bit depth key (float depth bits, index)
//             goes to the lists of those tiles (a cursor per tile, fixed
//             capacity per tile; entries beyond it are dropped and flagged);
//             blocks count their entries per tile in LDS and take one device
//             atomic per touched tile;
//   sort    : per tile, the list is sorted by (depth, primitive index), which
//             fixes the compositing order: a bucket sort on the depth bits in
//             LDS, a count of the smaller keys for short lists, or a bitonic
//             network on the 64-bit keys where depths crowd into few buckets;
//   render  : one block per tile, front to back over the list in chunks staged
//             through LDS; where the entry's q <= 9 ellipse reaches decides
//             which wavefronts look at it at all. The support
//             test and the quadratic form are FP64 (so both sides of a
//             parity check take the same support decisions), rho = exp(-q/2)
//             is FP32, and the transmittance (with an explicit power-of-two
//             exponent) and the colour sum are FP64: with no early
//             termination a pixel may composite thousands of layers;
//   backward: back to front over the same list, with dC/dc_i = alpha_i T_i
//             and dC/dalpha_i = T_i (c_i - R_{i+1}), R the colour seen from
//             the next layer on in units of its transmittance, built (as its
//             product with the upstream gradient) by a convex-combination
//             recursion (no cancellation at any depth), and T_i recovered from
//             the forward's final transmittance. Per primitive, a lane sums
//             its pixels' terms, the wavefront totals them over its lanes by
//             halving exchanges, and the lanes holding the totals add them to
//             FP64 per-primitive accumulators with one atomic instruction. With
//             geometry gradients the same pass also sums the moments that
//             dL/d(u, v, a, b, c) are made of;
//   finish  : per primitive, the accumulators rounded to the float32
//             outputs and, with geometry gradients, the FP64 chain from
//             dL/d(u, v, a, b, c) through the projection to the mean, scales
//             and quaternion.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "../../include/nasg.h"
#include "nasg_device.hpp"
#include "raster.hpp"

namespace nasg {

constexpr double kNear = 0.2;
constexpr double kClamp = 0.99;
constexpr double kSupport = 9.0;
constexpr int kBinParts = 8;  // most tile classes of the binning pass
constexpr int kBinLdsTiles = 8192;      // class tiles one LDS-counting block holds
constexpr int kBinThreads = 1024;       // of an LDS-counting block

// A primitive reaches a pixel with rho >= e^{-9/2} = 0.0111, so an opacity
// above 0.99 / 0.0111 = 89.2 is clamped on its whole support: any larger one
// (or a NaN, whose alpha is the clamp too) acts as kSigmaMax.
constexpr float kSigmaMax = 128.f;
__device__ inline double opacity(float sigma) {
  return static_cast<double>(fminf(sigma, kSigmaMax));
}

// Every thread of the grid (which covers the tiles and the primitives): the
// tile cursors, the overflow flag and the forward's stamp.
__device__ inline void begin_frame(const RasterArgs& a, int64_t t) {
  if (t < static_cast<int64_t>(a.tiles_x) * a.tiles_y) a.cursor[t] = 0;
  if (t == 0) {
    *a.overflow = 0;
    RasterStamp st;
    st.magic = kStampMagic;
    st.cap = a.cap;
    st.tiles_x = a.tiles_x;
    st.tiles_y = a.tiles_y;
    st.n = a.n;
    *a.stamp = st;
  }
}

__global__ void raster_zero_acc(double* acc, int64_t n, int32_t* stale) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i == 0) *stale = 0;
  if (i < n) {
#pragma unroll
    for (int k = 0; k < kAccStride; ++k) acc[kAccStride * i + k] = 0.0;
  }
}

// Gradients of the loss with respect to a primitive's mean, scales and
// quaternion from its sums g2 = (dL/du, dL/dv, dL/da, dL/db, dL/dc) over the
// image (b the conic's off-diagonal entry), in FP64, by the chain through the
// projection: K = Sigma_2^{-1} with dL/dSigma_2 = -K dL/dK K, Sigma_2 = M M^T
// (dL/dM = 2 dL/dSigma_2 M), M = J R_cw R(q/|q|) S, and u, v and J functions
// of the camera-space mean.
__device__ void geometry_chain(const RasterArgs& a, int64_t i, const double* g2, float* gm,
                               float* gs, float* gr) {
  double out_m[3] = {0.0, 0.0, 0.0}, out_s[3] = {0.0, 0.0, 0.0}, out_q[4] = {0.0, 0.0, 0.0, 0.0};
  const double* R = a.cam_rot;
  const double mx = a.means[3 * i], my = a.means[3 * i + 1], mz = a.means[3 * i + 2];
  const double X = R[0] * mx + R[1] * my + R[2] * mz + a.cam_t[0];
  const double Y = R[3] * mx + R[4] * my + R[5] * mz + a.cam_t[1];
  const double Z = R[6] * mx + R[7] * my + R[8] * mz + a.cam_t[2];
  const bool any = g2[0] != 0.0 || g2[1] != 0.0 || g2[2] != 0.0 || g2[3] != 0.0 || g2[4] != 0.0;
  if (any && Z > kNear) {
    const double iz = 1.0 / Z, iz2 = iz * iz;
    double qw = a.rots[4 * i], qx = a.rots[4 * i + 1], qy = a.rots[4 * i + 2], qz = a.rots[4 * i + 3];
    const double qn = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
    qw *= qn;
    qx *= qn;
    qy *= qn;
    qz *= qn;
    const double Rw[3][3] = {{1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy)},
                             {2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx)},
                             {2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)}};
    const double sc[3] = {a.scales[3 * i], a.scales[3 * i + 1], a.scales[3 * i + 2]};
    double A[3][3];  // R_cw R_w S
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c)
        A[r][c] = (R[3 * r] * Rw[0][c] + R[3 * r + 1] * Rw[1][c] + R[3 * r + 2] * Rw[2][c]) * sc[c];
    const double J[2][3] = {{a.fx * iz, 0.0, -a.fx * X * iz2}, {0.0, a.fy * iz, -a.fy * Y * iz2}};
    double M[2][3];
    for (int r = 0; r < 2; ++r)
      for (int c = 0; c < 3; ++c) M[r][c] = J[r][0] * A[0][c] + J[r][1] * A[1][c] + J[r][2] * A[2][c];
    const double sxx = M[0][0] * M[0][0] + M[0][1] * M[0][1] + M[0][2] * M[0][2];
    const double sxy = M[0][0] * M[1][0] + M[0][1] * M[1][1] + M[0][2] * M[1][2];
    const double syy = M[1][0] * M[1][0] + M[1][1] * M[1][1] + M[1][2] * M[1][2];
    const double id = 1.0 / (sxx * syy - sxy * sxy);
    const double K[2][2] = {{syy * id, -sxy * id}, {-sxy * id, sxx * id}};
    const double gK[2][2] = {{g2[2], 0.5 * g2[3]}, {0.5 * g2[3], g2[4]}};
    double T1[2][2], gS[2][2];
    for (int r = 0; r < 2; ++r)
      for (int c = 0; c < 2; ++c) T1[r][c] = K[r][0] * gK[0][c] + K[r][1] * gK[1][c];
    for (int r = 0; r < 2; ++r)
      for (int c = 0; c < 2; ++c) gS[r][c] = -(T1[r][0] * K[0][c] + T1[r][1] * K[1][c]);
    double gM[2][3];
    for (int r = 0; r < 2; ++r)
      for (int c = 0; c < 3; ++c) gM[r][c] = 2.0 * (gS[r][0] * M[0][c] + gS[r][1] * M[1][c]);
    double gJ[2][3];
    for (int r = 0; r < 2; ++r)
      for (int c = 0; c < 3; ++c) gJ[r][c] = gM[r][0] * A[c][0] + gM[r][1] * A[c][1] + gM[r][2] * A[c][2];
    double gA[3][3];
    for (int r = 0; r < 3; ++r)
      for (int c = 0; c < 3; ++c) gA[r][c] = J[0][r] * gM[0][c] + J[1][r] * gM[1][c];
    double gRw[3][3];
    for (int k = 0; k < 3; ++k) {
      for (int c = 0; c < 3; ++c) {
        const double grs = R[k] * gA[0][c] + R[3 + k] * gA[1][c] + R[6 + k] * gA[2][c];  // (R_cw^T gA)
        out_s[c] += grs * Rw[k][c];
        gRw[k][c] = grs * sc[c];
      }
    }
    // d R(u) / d(w, x, y, z) contracted with gRw, then the unit-norm projection
    const double gw = 2.0 * (-gRw[0][1] * qz + gRw[0][2] * qy + gRw[1][0] * qz - gRw[1][2] * qx -
                             gRw[2][0] * qy + gRw[2][1] * qx);
    const double gx = 2.0 * (gRw[0][1] * qy + gRw[0][2] * qz + gRw[1][0] * qy - 2.0 * gRw[1][1] * qx -
                             gRw[1][2] * qw + gRw[2][0] * qz + gRw[2][1] * qw - 2.0 * gRw[2][2] * qx);
    const double gy = 2.0 * (-2.0 * gRw[0][0] * qy + gRw[0][1] * qx + gRw[0][2] * qw + gRw[1][0] * qx +
                             gRw[1][2] * qz - gRw[2][0] * qw + gRw[2][1] * qz - 2.0 * gRw[2][2] * qy);
    const double gz = 2.0 * (-2.0 * gRw[0][0] * qz - gRw[0][1] * qw + gRw[0][2] * qx + gRw[1][0] * qw -
                             2.0 * gRw[1][1] * qz + gRw[1][2] * qy + gRw[2][0] * qx + gRw[2][1] * qy);
    const double dot = gw * qw + gx * qx + gy * qy + gz * qz;
    out_q[0] = (gw - qw * dot) * qn;
    out_q[1] = (gx - qx * dot) * qn;
    out_q[2] = (gy - qy * dot) * qn;
    out_q[3] = (gz - qz * dot) * qn;
    // camera-space mean through (u, v) and J
    const double gX = g2[0] * a.fx * iz - gJ[0][2] * a.fx * iz2;
    const double gY = g2[1] * a.fy * iz - gJ[1][2] * a.fy * iz2;
    const double gZ = -g2[0] * a.fx * X * iz2 - g2[1] * a.fy * Y * iz2 - gJ[0][0] * a.fx * iz2 +
                      gJ[0][2] * 2.0 * a.fx * X * iz2 * iz - gJ[1][1] * a.fy * iz2 +
                      gJ[1][2] * 2.0 * a.fy * Y * iz2 * iz;
    for (int k = 0; k < 3; ++k) out_m[k] = gX * R[k] + gY * R[3 + k] + gZ * R[6 + k];
  }
  if (gm != nullptr)
    for (int k = 0; k < 3; ++k) gm[3 * i + k] = static_cast<float>(out_m[k]);
  if (gs != nullptr)
    for (int k = 0; k < 3; ++k) gs[3 * i + k] = static_cast<float>(out_s[k]);
  if (gr != nullptr)
    for (int k = 0; k < 4; ++k) gr[4 * i + k] = static_cast<float>(out_q[k]);
}

template <bool GEOM>
__global__ void raster_finish_grads(RasterArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  // the render kernel's sums are in units of the opacity (see there)
  const double* acc = a.grad_acc + kAccStride * i;
  const double sg = opacity(a.opac[i]);
  if (a.grad_colors != nullptr) {
    a.grad_colors[3 * i + 0] = static_cast<float>(sg * acc[0]);
    a.grad_colors[3 * i + 1] = static_cast<float>(sg * acc[1]);
    a.grad_colors[3 * i + 2] = static_cast<float>(sg * acc[2]);
  }
  if (a.grad_opac != nullptr) a.grad_opac[i] = static_cast<float>(acc[3]);
  if constexpr (GEOM) {
    // dL/dq = -sigma s / 2 per pixel, q = a dx^2 + 2 b dx dy + c dy^2
    const double g2[5] = {sg * acc[4], sg * acc[5], -0.5 * sg * acc[6], -sg * acc[7],
                          -0.5 * sg * acc[8]};
    geometry_chain(a, i, g2, a.grad_means, a.grad_scales, a.grad_rots);
  }
}

__global__ void raster_project(RasterArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  begin_frame(a, i);
  if (i >= a.n) return;
  RenderRec rec{};
  BinRec bin{};
  bin.tx0 = 1;  // empty tile range unless the ellipse lands on the image
  bin.tx1 = 0;
  bin.ty0 = 1;
  bin.ty1 = 0;
  const double mx = a.means[3 * i], my = a.means[3 * i + 1], mz = a.means[3 * i + 2];
  const double* R = a.cam_rot;
  const double X = R[0] * mx + R[1] * my + R[2] * mz + a.cam_t[0];
  const double Y = R[3] * mx + R[4] * my + R[5] * mz + a.cam_t[1];
  const double Z = R[6] * mx + R[7] * my + R[8] * mz + a.cam_t[2];
  bin.z = Z;
  if (Z > kNear) {
    const double iz = 1.0 / Z;
    rec.u = a.fx * X * iz + a.cx;
    rec.v = a.fy * Y * iz + a.cy;
    // world rotation of the normalised quaternion
    double qw = a.rots[4 * i], qx = a.rots[4 * i + 1], qy = a.rots[4 * i + 2], qz = a.rots[4 * i + 3];
    const double qn = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
    qw *= qn;
    qx *= qn;
    qy *= qn;
    qz *= qn;
    const double Rw[9] = {1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy),
                          2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx),
                          2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)};
    const double s[3] = {a.scales[3 * i], a.scales[3 * i + 1], a.scales[3 * i + 2]};
    // M = J R_cw R_w S (2 x 3), projected covariance Sigma_2 = M M^T
    const double J0[3] = {a.fx * iz, 0.0, -a.fx * X * iz * iz};
    const double J1[3] = {0.0, a.fy * iz, -a.fy * Y * iz * iz};
    double A0[3], A1[3];
    for (int c = 0; c < 3; ++c) {
      A0[c] = J0[0] * R[c] + J0[1] * R[3 + c] + J0[2] * R[6 + c];
      A1[c] = J1[0] * R[c] + J1[1] * R[3 + c] + J1[2] * R[6 + c];
    }
    double m0[3], m1[3];
    for (int c = 0; c < 3; ++c) {
      m0[c] = (A0[0] * Rw[c] + A0[1] * Rw[3 + c] + A0[2] * Rw[6 + c]) * s[c];
      m1[c] = (A1[0] * Rw[c] + A1[1] * Rw[3 + c] + A1[2] * Rw[6 + c]) * s[c];
    }
    const double sxx = m0[0] * m0[0] + m0[1] * m0[1] + m0[2] * m0[2];
    const double sxy = m0[0] * m1[0] + m0[1] * m1[1] + m0[2] * m1[2];
    const double syy = m1[0] * m1[0] + m1[1] * m1[1] + m1[2] * m1[2];
    const double det = sxx * syy - sxy * sxy;
    if (det > 0.0) {
      const double id = 1.0 / det;
      rec.a = syy * id;
      rec.b2 = -2.0 * sxy * id;
      rec.c = sxx * id;
      // q <= 9 implies |dx| <= 3 sqrt(sxx) and |dy| <= 3 sqrt(syy). The
      // float half-extents are rounded outward (relative 1e-5 plus 1e-2
      // pixel, far above the rounding of the inverse), and binning adds a
      // pixel more; pixel px has its centre at px + 1/2
      const double ex = 3.0 * sqrt(sxx), ey = 3.0 * sqrt(syy);
      rec.ex = static_cast<float>(ex * (1.0 + 1e-5) + 1e-2);
      rec.ey = static_cast<float>(ey * (1.0 + 1e-5) + 1e-2);
      const double px0 = fmax(rec.u - ex - 1.5, 0.0), px1 = fmin(rec.u + ex + 0.5, a.width - 1.0);
      const double py0 = fmax(rec.v - ey - 1.5, 0.0), py1 = fmin(rec.v + ey + 0.5, a.height - 1.0);
      if (px0 <= px1 && py0 <= py1) {
        bin.tx0 = static_cast<int16_t>(static_cast<int32_t>(px0) / kTile);
        bin.tx1 = static_cast<int16_t>(static_cast<int32_t>(px1) / kTile);
        bin.ty0 = static_cast<int16_t>(static_cast<int32_t>(py0) / kTile);
        bin.ty1 = static_cast<int16_t>(static_cast<int32_t>(py1) / kTile);
      }
    }
  }
  rec.c0 = a.colors[3 * i];
  rec.c1 = a.colors[3 * i + 1];
  rec.c2 = a.colors[3 * i + 2];
  rec.sigma = a.opac[i];
  a.rec[i] = rec;
  a.bins[i] = bin;
}

// Sort key of a list entry: the float32 of its FP64 depth (z > 0.2, so the
// float's bits order like the depths) above its primitive index.
__device__ inline uint64_t depth_key(double z, int64_t i) {
  return (static_cast<uint64_t>(__float_as_uint(__double2float_rn(z))) << 32) |
         static_cast<uint32_t>(i);
}

// Tile binning. A primitive's depth key goes to the list of every tile its
// box touches; the order of appends does not matter (the per-tile sort orders
// each list by its keys). The tiles are split into `parts` classes by tile
// index mod parts (a power of two): block b serves class b mod parts for the
// primitives of chunk b / parts.

// Calls f(tile) for each tile of box r in class `part` of `parts`: in each
// row, the box's columns whose tile index is part mod parts.
template <class F>
__device__ inline void for_class_tiles(const BinRec& r, int64_t tiles_x, int part, int parts,
                                       F&& f) {
  for (int y = r.ty0; y <= r.ty1; ++y) {
    const int64_t row = static_cast<int64_t>(y) * tiles_x;
    for (int tx = r.tx0 + static_cast<int>((part - (row + r.tx0)) & (parts - 1)); tx <= r.tx1;
         tx += parts)
      f(row + tx);
  }
}

// Images whose tiles fit kBinLdsTiles per class in at most kBinParts classes
// (parts = the smallest power of two that does it). A block first counts its
// chunk's entries per class tile in LDS, then reserves each touched tile's
// range in its list with one device atomic on the tile's cursor, then places
// the keys in those ranges with LDS atomics: one device atomic per (block,
// tile) instead of one per entry.
__global__ __launch_bounds__(kBinThreads) void raster_bin_lds(RasterArgs a, int pshift, int chunk) {
  extern __shared__ int cnt[];
  const int parts = 1 << pshift;
  const int part = static_cast<int>(blockIdx.x & (parts - 1));
  const int64_t first = static_cast<int64_t>(blockIdx.x >> pshift) * chunk;
  const int64_t last = min(first + chunk, a.n);
  const int64_t n_tiles = static_cast<int64_t>(a.tiles_x) * a.tiles_y;
  const int n_local = static_cast<int>((n_tiles - part + parts - 1) >> pshift);
  for (int m = threadIdx.x; m < n_local; m += kBinThreads) cnt[m] = 0;
  __syncthreads();
  for (int64_t i = first + threadIdx.x; i < last; i += kBinThreads) {
    const BinRec r = a.bins[i];
    for_class_tiles(r, a.tiles_x, part, parts, [&](int64_t t) { atomicAdd(&cnt[t >> pshift], 1); });
  }
  __syncthreads();
  for (int m = threadIdx.x; m < n_local; m += kBinThreads) {
    const int c = cnt[m];
    if (c > 0) cnt[m] = atomicAdd(a.cursor + (static_cast<int64_t>(m) << pshift) + part, c);
  }
  __syncthreads();
  for (int64_t i = first + threadIdx.x; i < last; i += kBinThreads) {
    const BinRec r = a.bins[i];
    const uint64_t key = depth_key(r.z, i);
    for_class_tiles(r, a.tiles_x, part, parts, [&](int64_t t) {
      const int pos = atomicAdd(&cnt[t >> pshift], 1);
      if (pos < a.cap) {
        a.lists[t * a.cap + pos] = key;
      } else {
        atomicMax(a.overflow, 1);
      }
    });
  }
}

// Larger images: one device atomic per entry on the tile's cursor, those of
// up to eight tiles issued before their results are used, so their latencies
// overlap. The tiles are split into kBinParts classes as above (each XCD of
// the chip, which takes every eighth workgroup, then appends to its own
// lists); slot (row y, j) of a box is column first(y) + kBinParts * j, where
// first(y) is the box's first column in this class.
__global__ void raster_bin(RasterArgs a) {
  const int part = static_cast<int>(blockIdx.x & (kBinParts - 1));
  const int64_t i = static_cast<int64_t>(blockIdx.x / kBinParts) * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const BinRec r = a.bins[i];
  const int w = r.tx1 - r.tx0 + 1, h = r.ty1 - r.ty0 + 1;
  if (w <= 0 || h <= 0) return;
  const int cw = (w + kBinParts - 1) / kBinParts;
  const int slots = cw * h;
  const uint64_t key = depth_key(r.z, i);
  for (int k0 = 0; k0 < slots; k0 += 8) {
    int64_t tl[8];
    int32_t pos[8];
    bool use[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + u;
      tl[u] = 0;
      pos[u] = 0;
      use[u] = false;
      if (k < slots) {
        const int y = r.ty0 + k / cw;
        const int64_t row = static_cast<int64_t>(y) * a.tiles_x;
        const int lead = static_cast<int>((part - (row + r.tx0)) & (kBinParts - 1));
        const int tx = r.tx0 + lead + kBinParts * (k % cw);
        if (tx <= r.tx1) {
          use[u] = true;
          tl[u] = row + tx;
          pos[u] = atomicAdd(a.cursor + tl[u], 1);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (use[u]) {
        if (pos[u] < a.cap) {
          a.lists[tl[u] * a.cap + pos[u]] = key;
        } else {
          atomicMax(a.overflow, 1);
        }
      }
    }
  }
}

// Per-tile depth sort. Key = (float32 of the FP64 depth, primitive index):
// rounding to float is monotone, so sorting the 64-bit keys orders the list
// by depth except inside runs of equal float depth, which a final pass puts
// in (FP64 depth, index) order; padding keys (all ones) sort last. Bitonic
// network over 256 EPT keys, EPT consecutive keys per thread in registers:
// strides below EPT are exchanged in registers, strides whose partner is in
// the same wavefront by lane shuffles, the rest through LDS.
template <int EPT>
__device__ void bitonic_keys(uint64_t (&v)[EPT], uint64_t* lds) {
  constexpr int M = 256 * EPT;
  const int t = static_cast<int>(threadIdx.x);
  for (int k = 2; k <= M; k <<= 1) {
    for (int j = k >> 1; j >= EPT; j >>= 1) {
      const int tj = j / EPT;  // partner thread t ^ tj holds the partner keys
      if (tj >= 64) {          // another wavefront: through LDS
        __syncthreads();
#pragma unroll
        for (int r = 0; r < EPT; ++r) lds[t * EPT + r] = v[r];
        __syncthreads();
      }
#pragma unroll
      for (int r = 0; r < EPT; ++r) {
        const int e = t * EPT + r, pe = e ^ j;
        const uint64_t o = tj >= 64 ? lds[pe] : __shfl_xor(v[r], tj, 64);
        const bool keep_min = ((e & k) == 0) == (e < pe);
        v[r] = keep_min ? (o < v[r] ? o : v[r]) : (o > v[r] ? o : v[r]);
      }
    }
#pragma unroll
    for (int jj = EPT / 2; jj >= 1; jj >>= 1) {
      if (jj < k) {
#pragma unroll
        for (int r = 0; r < EPT; ++r) {
          const int p = r ^ jj;
          if (p > r) {
            const bool up = ((t * EPT + r) & k) == 0;
            const uint64_t a = v[r], b = v[p];
            const uint64_t lo = a < b ? a : b, hi = a < b ? b : a;
            v[r] = up ? lo : hi;
            v[p] = up ? hi : lo;
          }
        }
      }
    }
  }
}

// Runs of equal float depth (in index order on entry): a stable insertion
// sort by FP64 depth, done by the thread that owns the run's first entry;
// then the sorted keys go back to the tile's list.
template <int T>
__device__ void order_runs_and_store(const RasterArgs& a, uint64_t* list, int cnt,
                                     uint64_t* lds) {
  const int t = static_cast<int>(threadIdx.x);
  for (int e = t; e < cnt; e += T) {
    const uint32_t hi = static_cast<uint32_t>(lds[e] >> 32);
    const bool start = e == 0 || static_cast<uint32_t>(lds[e - 1] >> 32) != hi;
    if (!start || e + 1 >= cnt || static_cast<uint32_t>(lds[e + 1] >> 32) != hi) continue;
    int end = e + 1;
    while (end < cnt && static_cast<uint32_t>(lds[end] >> 32) == hi) ++end;
    for (int i = e + 1; i < end; ++i) {
      const uint64_t key = lds[i];
      const double z = a.bins[static_cast<uint32_t>(key)].z;
      int p = i - 1;
      while (p >= e && a.bins[static_cast<uint32_t>(lds[p])].z > z) {
        lds[p + 1] = lds[p];
        --p;
      }
      lds[p + 1] = key;
    }
  }
  __syncthreads();
  for (int e = t; e < cnt; e += T) list[e] = lds[e];
}

template <int EPT>
__device__ void sort_tile(const RasterArgs& a, uint64_t* list, int cnt, uint64_t* lds) {
  const int t = static_cast<int>(threadIdx.x);
  // coalesced load through LDS into the blocked register layout
  for (int e = t; e < 256 * EPT; e += 256) lds[e] = e < cnt ? list[e] : ~0ull;
  __syncthreads();
  uint64_t v[EPT];
#pragma unroll
  for (int r = 0; r < EPT; ++r) v[r] = lds[t * EPT + r];
  bitonic_keys<EPT>(v, lds);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < EPT; ++r) lds[t * EPT + r] = v[r];
  __syncthreads();
  order_runs_and_store<256>(a, list, cnt, lds);
}

// Bucket sort of one tile's keys (257 .. 4096 of them) on the float depth
// bits, which order like the depths: bucket (bits - min) >> shift, with the
// shift that fits the tile's span of bits into kSortBuckets buckets, is
// monotone in the key, so sorting each bucket by the full key (depth bits,
// then index) sorts the list. An LDS histogram, a block scan of it and a
// scatter place the keys; the owner of eight consecutive buckets then sorts
// each of them by insertion. 512 threads a block: 49 KB of LDS allow three
// blocks per CU, whose 24 wavefronts hide the LDS latency that 12 (256 threads)
// leave bare (3 M primitives at 1920 x 1080: 275 -> 190 us; 1024 threads 193,
// and 98 against 77 us for 500 k primitives). Returns false, having changed nothing, when a
// bucket holds more than kSortBucketRun keys: the bitonic network takes
// that tile instead.
constexpr int kSortBuckets = 4096;
constexpr int kSortBucketRun = 32;
constexpr int kSortThreads = 512;

__device__ bool bucket_sort_tile(const RasterArgs& a, uint64_t* list, int cnt, uint64_t* out,
                                 int* bucket, uint32_t* red) {
  constexpr int BPT = kSortBuckets / kSortThreads, kWaves = kSortThreads / 64;  // buckets owned by each thread
  const int t = static_cast<int>(threadIdx.x), lane = t & 63, wave = t >> 6;
  // the keys' high words (float depth bits) are read from the list where
  // only they are needed, which keeps the keys out of registers
  const uint32_t* hw = reinterpret_cast<const uint32_t*>(list) + 1;
  uint32_t lo = 0xffffffffu, hi = 0u;
  for (int e = t; e < cnt; e += kSortThreads) {
    const uint32_t h = hw[2 * e];
    lo = min(lo, h);
    hi = max(hi, h);
  }
  for (int k = t; k < kSortBuckets; k += kSortThreads) bucket[k] = 0;
  for (int o = 32; o >= 1; o >>= 1) {
    lo = min(lo, static_cast<uint32_t>(__shfl_xor(static_cast<int>(lo), o, 64)));
    hi = max(hi, static_cast<uint32_t>(__shfl_xor(static_cast<int>(hi), o, 64)));
  }
  if (lane == 0) {
    red[wave] = lo;
    red[kWaves + wave] = hi;
  }
  __syncthreads();
  for (int w = 0; w < kWaves; ++w) {
    lo = min(lo, red[w]);
    hi = max(hi, red[kWaves + w]);
  }
  const uint32_t span = hi - lo;
  const int shift = span == 0 ? 0 : max(0, 32 - __clz(static_cast<int>(span)) - 12);
  for (int e = t; e < cnt; e += kSortThreads) atomicAdd(&bucket[(hw[2 * e] - lo) >> shift], 1);
  __syncthreads();
  int c[BPT];
  int sum = 0, cmax = 0;
#pragma unroll
  for (int k = 0; k < BPT; ++k) {
    c[k] = bucket[BPT * t + k];
    sum += c[k];
    cmax = max(cmax, c[k]);
  }
  if (__syncthreads_or(cmax > kSortBucketRun)) return false;
  // exclusive scan of the per-thread bucket totals over the block
  int incl = sum;
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  if (lane == 63) red[wave] = static_cast<uint32_t>(incl);
  __syncthreads();
  int run = incl - sum;
  for (int w = 0; w < wave; ++w) run += static_cast<int>(red[w]);
#pragma unroll
  for (int k = 0; k < BPT; ++k) {
    bucket[BPT * t + k] = run;
    run += c[k];
  }
  __syncthreads();
  for (int e = t; e < cnt; e += kSortThreads) {
    const uint64_t key = list[e];
    out[atomicAdd(&bucket[(static_cast<uint32_t>(key >> 32) - lo) >> shift], 1)] = key;
  }
  __syncthreads();
  // bucket b now ends at bucket[b] and starts where bucket b - 1 ends
  for (int k = 0; k < BPT; ++k) {
    const int b = BPT * t + k;
    const int s0 = b == 0 ? 0 : bucket[b - 1], s1 = bucket[b];
    for (int i = s0 + 1; i < s1; ++i) {
      const uint64_t v = out[i];
      int p = i - 1;
      while (p >= s0 && out[p] > v) {
        out[p + 1] = out[p];
        --p;
      }
      out[p + 1] = v;
    }
  }
  __syncthreads();
  order_runs_and_store<kSortThreads>(a, list, cnt, out);
  return true;
}

// Lists of at most kRankSort keys: each thread counts the keys below its own
// (they are distinct), which is its place: no barrier per step, and a list of
// a few keys costs a few steps (1540 tiles of about 4 keys: 18 -> 4 us against
// the bitonic network over 256).
constexpr int kRankSort = 256;

__device__ void rank_sort_tile(const RasterArgs& a, uint64_t* list, int cnt, uint64_t* out,
                               uint64_t* in) {
  const int t = static_cast<int>(threadIdx.x);
  if (t < cnt) in[t] = list[t];
  __syncthreads();
  if (t < cnt) {
    const uint64_t key = in[t];
    int rank = 0;
#pragma unroll 4
    for (int k = 0; k < cnt; ++k) rank += in[k] < key ? 1 : 0;
    out[rank] = key;
  }
  __syncthreads();
  order_runs_and_store<kSortThreads>(a, list, cnt, out);
}

__global__ __launch_bounds__(kSortThreads) void raster_sort(RasterArgs a) {
  __shared__ uint64_t lds[256 * 16];
  __shared__ alignas(8) int bucket[kSortBuckets];
  __shared__ uint32_t red[2 * kSortThreads / 64];
  const int64_t tile = blockIdx.x;
  const int cnt = min(a.cursor[tile], a.cap);
  if (cnt <= 1) return;
  uint64_t* list = a.lists + tile * a.cap;
  if (cnt <= kRankSort) {
    rank_sort_tile(a, list, cnt, lds, reinterpret_cast<uint64_t*>(bucket));
  } else if (!bucket_sort_tile(a, list, cnt, lds, bucket, red)) {
    // left to raster_sort_network, which this mark (the tile's count, bit
    // inverted) tells to take the tile and restore the count; every thread
    // read the cursor before the barrier inside the bucket sort
    if (threadIdx.x == 0) a.cursor[tile] = ~a.cursor[tile];
  }
}

// The tiles the bucket sort left: the bitonic network, whose registers would
// otherwise cap the occupancy of every tile's sort.
__global__ __launch_bounds__(256) void raster_sort_network(RasterArgs a) {
  __shared__ uint64_t lds[256 * 16];
  const int64_t tile = blockIdx.x;
  const int c = a.cursor[tile];
  if (c >= 0) return;
  const int cnt = min(~c, a.cap);
  uint64_t* list = a.lists + tile * a.cap;
  if (cnt <= 512) {
    sort_tile<2>(a, list, cnt, lds);
  } else if (cnt <= 1024) {
    sort_tile<4>(a, list, cnt, lds);
  } else if (cnt <= 2048) {
    sort_tile<8>(a, list, cnt, lds);
  } else {
    sort_tile<16>(a, list, cnt, lds);
  }
  __syncthreads();  // every thread has read the mark
  if (threadIdx.x == 0) a.cursor[tile] = ~c;
}

// A staged tile entry: pixel-space mean, conic (q = a dx^2 + 2 b dx dy + c dy^2),
// colour, opacity and the largest rho below the alpha clamp. Every field is
// FP64 so that the pixel loops convert nothing.
struct StageEntry {
  double u, v, a, b, c;
  double sigma, rmax;     // alpha = sigma min(rho, rmax)
  double c0, c1, c2;
};

// Totals of several per-lane values over the 64 lanes of a wavefront (every
// lane active) by halving exchanges: at each step a lane keeps half of the
// values it holds, adds its partner's partial sums of that half and passes
// the other half on, so the totals end up spread over the lanes instead of
// being reduced one value at a time. Partners: lane ^ 32 and lane ^ 16 (the
// permlane swaps), lane ^ 1 and lane ^ 2 (quad DPP); lane bits 2 and 3 are
// then summed with row rotations by 8 and 4.
__device__ inline float swap32_sum(float x, float y) {
  // lanes 0-31: x[l] + x[l + 32]; lanes 32-63: y[l - 32] + y[l]
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ inline float swap16_sum(float x, float y) {
  // rows 0 and 2 (lane bit 4 clear): x[l] + x[l ^ 16]; rows 1 and 3: y[l ^ 16] + y[l]
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

constexpr int kQuadXor1 = 0xB1;  // quad_perm [1, 0, 3, 2]
constexpr int kQuadXor2 = 0x4E;  // quad_perm [2, 3, 0, 1]
constexpr int kRowRor8 = 0x128;
constexpr int kRowRor4 = 0x124;

// Nine values: lane l ends with the total of value lane_slot9(l); lanes 0, 1,
// 2, 16, 17, 32, 33, 48, 49 hold the nine totals once each.
__device__ inline float lane_sums9(const float (&x)[9], int lane) {
  const float a0 = swap32_sum(x[0], x[1]), a1 = swap32_sum(x[2], x[3]);
  const float a2 = swap32_sum(x[4], x[5]), a3 = swap32_sum(x[6], x[7]);
  const float a4 = swap32_sum(x[8], x[8]);
  const float b0 = swap16_sum(a0, a1), b1 = swap16_sum(a2, a3), b2 = swap16_sum(a4, a4);
  const bool o1 = (lane & 1) != 0, o2 = (lane & 2) != 0;
  const float c0 = (o1 ? b1 : b0) + dpp_f<kQuadXor1>(o1 ? b0 : b1);
  const float c1 = b2 + dpp_f<kQuadXor1>(b2);
  float d = (o2 ? c1 : c0) + dpp_f<kQuadXor2>(o2 ? c0 : c1);
  d += dpp_f<kRowRor8>(d);
  d += dpp_f<kRowRor4>(d);
  return d;
}
__device__ inline bool lane_writes9(int lane) { return (lane & 0xE) == 0 || lane == 2; }
__device__ inline int lane_slot9(int lane) {
  return lane == 2 ? 8 : 4 * (lane & 1) + 2 * ((lane >> 4) & 1) + ((lane >> 5) & 1);
}

// Four values: lanes 0, 16, 32, 48 hold the totals of values 0, 2, 1, 3.
__device__ inline float lane_sums4(const float (&x)[4]) {
  float b = swap16_sum(swap32_sum(x[0], x[1]), swap32_sum(x[2], x[3]));
  b += dpp_f<kQuadXor1>(b);
  b += dpp_f<kQuadXor2>(b);
  b += dpp_f<kRowRor8>(b);
  b += dpp_f<kRowRor4>(b);
  return b;
}
__device__ inline bool lane_writes4(int lane) { return (lane & 0xF) == 0; }
__device__ inline int lane_slot4(int lane) { return 2 * ((lane >> 4) & 1) + ((lane >> 5) & 1); }

// Transmittance as t * 2^E (E a multiple of kRenorm). t is renormalised after
// every 64 staged entries, so at most 64 layers (each multiplying t by at
// least 0.01 going forward, or dividing it by at least 0.01 going back) pass
// between checks: t stays within [2^-500 1e-128, 1] in the forward and below
// 2^300 1e128 in the backward, normal doubles, and a pixel behind thousands of
// layers keeps an exact transmittance for the backward's recovery by division.
constexpr int kRenorm = 500;
// rho = exp(-q/2) = 2^(q * (-log2(e) / 2)); the constant is exact in float
// (half of the float log2 e), so this is the float exponential of -q/2
constexpr float kNegHalfLog2e = -0.72134752044448170368f;
__device__ inline RenderRec stage_entry(const RasterArgs& a, const uint64_t* list, int e,
                                        StageEntry* slot, int32_t* idx) {
  *idx = static_cast<int32_t>(static_cast<uint32_t>(list[e]));
  const RenderRec r = a.rec[*idx];
  StageEntry s;
  s.u = r.u;
  s.v = r.v;
  s.a = r.a;
  s.b = 0.5 * r.b2;
  s.c = r.c;
  s.sigma = opacity(r.sigma);
  s.rmax = s.sigma >= kClamp ? kClamp / s.sigma : 2.0;   // rho <= 1: no clamp below
  s.c0 = r.c0;
  s.c1 = r.c1;
  s.c2 = r.c2;
  *slot = s;
  return r;
}

// Where the ellipse q <= 9 of a record reaches, for culling an entry against
// the rectangles of pixel centres that a wavefront works on. On a horizontal
// line dy the ellipse spans dx = -(b/a) dy -+ (3/sqrt a) sqrt(1 - (dy/ey)^2),
// ey its vertical half-extent; over a band of lines the right end is largest
// at the line nearest to the right extreme point (dy = -(b/c) ex), the left
// end at the line nearest to its mirror image. FP32, kept conservative: the
// record's half-extents are rounded outward by 1e-5 and 0.01 pixel (which
// bounds the loss from the extreme point's rounding by 0.01 pixel), bands are
// widened by the rounding of their coordinates and spans by 0.02 pixel and
// 2e-6 of the sizes that enter. A NaN culls nothing. About 30 instructions a
// band, against some 70 for the minimum of q over the band's rectangle.
struct Reach {
  float u, v, ex, ey;   // centre relative to the tile's corner, half-extents
  float iey, slope, w;  // 1/ey, -b/a, 3/sqrt a
  float dyr, mx, my;    // dy of the right extreme point, margins
};

__device__ inline Reach reach_of(const RenderRec& r, double x0, double y0) {
  Reach e;
  e.u = static_cast<float>(r.u - x0);
  e.v = static_cast<float>(r.v - y0);
  e.ex = r.ex;
  e.ey = r.ey;
  e.iey = __builtin_amdgcn_rcpf(r.ey);
  const double hb = -0.5 * r.b2;
  e.slope = static_cast<float>(hb * __builtin_amdgcn_rcp(r.a));
  e.w = 3.f * static_cast<float>(__builtin_amdgcn_rsq(r.a));
  const float d = static_cast<float>(hb * __builtin_amdgcn_rcp(r.c)) * r.ex;
  e.dyr = fminf(fmaxf(d, -r.ey), r.ey);
  e.mx = fmaf(2e-6f, r.ex + fabsf(e.u), 0.02f);
  e.my = fmaf(4e-7f, fabsf(e.v), 1e-5f);
  return e;
}

// Bit k is set when the ellipse may reach a pixel centre of column k of the
// band of rows [row, row + ROWS) (tile-relative), columns COLS pixels wide.
template <int ROWS, int COLS>
__device__ inline uint32_t reach_band(const Reach& e, int row) {
  const float yl = (static_cast<float>(row) + 0.5f) - e.v - e.my;
  const float yh = (static_cast<float>(row + ROWS) - 0.5f) - e.v + e.my;
  const float dr = fminf(fmaxf(e.dyr, yl), yh), dl = fminf(fmaxf(-e.dyr, yl), yh);
  const float sr = dr * e.iey, sl = dl * e.iey;
  const float xr = e.u + e.mx + fmaf(e.slope, dr, e.w * __builtin_amdgcn_sqrtf(fmaxf(fmaf(-sr, sr, 1.f), 0.f)));
  const float xl = e.u - e.mx + fmaf(e.slope, dl, -e.w * __builtin_amdgcn_sqrtf(fmaxf(fmaf(-sl, sl, 1.f), 0.f)));
  uint32_t bits = 0;
#pragma unroll
  for (int k = 0; k < kTile / COLS; ++k) {
    const float lo = COLS * k + 0.5f, hi = COLS * k + (COLS - 0.5f);
    if (!(xr < lo) && !(xl > hi)) bits |= 1u << k;
  }
  return yl > e.ey || yh < -e.ey ? 0u : bits;
}

// Thread layout of the render kernels: a block of 256 / RPL threads per
// 16 x 16 tile, each lane RPL pixels. RPL = 1: wavefront w owns the 8 x 8
// quadrant (w & 1, w >> 1). RPL = 4: one wavefront owns the tile, lane l the
// pixels of column l & 15 in rows (l >> 4) + 4 j (row band j), so that an
// entry's dx terms, its wavefront totals and its atomics are shared by four
// pixels. An entry that cannot reach a quadrant or band skips it for the whole
// wavefront: of the pixels so evaluated, at 3 M primitives and 1920 x 1080 the
// ellipse covers 0.61 in 8 x 8 quadrants and 0.55 in 16 x 4 bands (0.44 with
// the bounding box alone).
template <int RPL>
struct TileMap {
  static_assert(RPL == 1 || RPL == 4, "rows per lane");
  int px, py0;     // the lane's column and first row
  int wave;
  double x0, y0;   // the tile's corner
  bool in_x;
  int height;
  __device__ bool in(int j) const { return in_x && py0 + 4 * j < height; }
  __device__ int64_t pixel(int j, int width) const {
    return static_cast<int64_t>(py0 + 4 * j) * width + px;
  }
};

template <int RPL>
__device__ inline TileMap<RPL> tile_map(const RasterArgs& a, int64_t tile) {
  TileMap<RPL> m;
  const int tx = static_cast<int>(tile % a.tiles_x), ty = static_cast<int>(tile / a.tiles_x);
  const int lane = static_cast<int>(threadIdx.x) & 63;
  m.wave = RPL == 4 ? 0 : __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  m.px = tx * kTile + (RPL == 4 ? lane & 15 : 8 * (m.wave & 1) + (lane & 7));
  m.py0 = ty * kTile + (RPL == 4 ? lane >> 4 : 8 * (m.wave >> 1) + (lane >> 3));
  m.x0 = tx * kTile;
  m.y0 = ty * kTile;
  m.in_x = m.px < a.width;
  m.height = a.height;
  return m;
}

// The units of the tile that an entry may reach: bit j is row band j (BANDS)
// or quadrant j (column half j & 1, row half j >> 1). kSlowBit: the entry's
// alpha can reach the clamp.
constexpr uint32_t kSlowBit = 16;

template <bool BANDS>
__device__ inline uint32_t unit_mask(const RenderRec& r, double x0, double y0) {
  const Reach e = reach_of(r, x0, y0);
  uint32_t mask = 0;
  if constexpr (BANDS) {
#pragma unroll
    for (int j = 0; j < 4; ++j) mask |= reach_band<4, 16>(e, 4 * j) << j;
  } else {
    mask = reach_band<8, 8>(e, 0) | (reach_band<8, 8>(e, 8) << 2);
  }
  return mask != 0 && opacity(r.sigma) >= kClamp ? mask | kSlowBit : mask;
}

// The part of a unit mask that concerns wavefront w.
template <int RPL>
__device__ inline uint32_t wave_units(uint32_t mask, int w) {
  return RPL == 4 ? mask & ~kSlowBit : (mask >> w) & 1u;
}

// Keeps a value in vector registers from here on: an entry's fields are read
// from LDS once, not again in every pixel's branch.
__device__ __forceinline__ void keep(double& x) { asm("" : "+v"(x)); }

// One pixel per thread. Each wavefront walks, in order, the staged entries
// that reach its quadrant, picked 64 at a time from a ballot by scalar bit
// scans (no list in LDS). Per entry: eight FP64 instructions for q and the
// support test, then rho in FP32, alpha, three colour sums and the
// transmittance in FP64. While no entry can reach the clamp and every pixel
// has E = 0 the clamp and the scale factor 2^E are left out (fast). Bound by
// the entries' reads from LDS (72 B per wavefront and entry) and by VALU
// issue, in about equal parts: 2.10 -> 1.55 ms at 3 M primitives and
// 1920 x 1080, 233 -> 174 us at 500 k and 1280 x 720 against 16 x 4 bands
// culled by bounding box with a compacted list in LDS. Two pixels per lane
// (half the LDS reads, half the waves) took 1.51 ms and 184 us, and twice the
// time on a few tiles.
__global__ __launch_bounds__(256) void raster_render_fwd(RasterArgs a) {
  constexpr int kBlock = 256;
  __shared__ StageEntry stage[kBlock];
  __shared__ uint32_t smask[kBlock];
  const int64_t tile = blockIdx.x;
  const TileMap<1> m = tile_map<1>(a, tile);
  const double cxp = m.px + 0.5, cyp = m.py0 + 0.5;
  const int cnt = __builtin_amdgcn_readfirstlane(min(a.cursor[tile], a.cap));
  const uint64_t* list = a.lists + tile * a.cap;
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const bool in = m.in(0);

  double C0 = 0.0, C1 = 0.0, C2 = 0.0;
  double t = 1.0, pw = 1.0;   // T = t * pw, pw = 2^E
  int E = 0;
  auto walk = [&](auto fast, uint64_t bal, const StageEntry* st) {
    constexpr bool kFast = decltype(fast)::value;
    while (bal != 0) {
      const StageEntry& s = st[__builtin_ctzll(bal)];
      bal &= bal - 1;
      const double dx = cxp - s.u, dy = cyp - s.v;
      const double q = fma(dy, fma(s.c, dy, s.b * (dx + dx)), s.a * dx * dx);
      if (in && q <= kSupport) {
        double rho = static_cast<double>(
            __builtin_amdgcn_exp2f(static_cast<float>(q) * kNegHalfLog2e));
        if constexpr (!kFast) rho = fmin(rho, s.rmax);
        const double al = s.sigma * rho;
        double w = al * t;
        if constexpr (!kFast) w *= pw;
        C0 = fma(w, s.c0, C0);
        C1 = fma(w, s.c1, C1);
        C2 = fma(w, s.c2, C2);
        t = fma(-al, t, t);
      }
    }
  };
  for (int base = 0; base < cnt; base += kBlock) {
    __syncthreads();
    const int e = base + static_cast<int>(threadIdx.x);
    uint32_t mask = 0;
    if (e < cnt) {
      int32_t idx;
      const RenderRec r = stage_entry(a, list, e, &stage[threadIdx.x], &idx);
      mask = unit_mask<false>(r, m.x0, m.y0);
    }
    smask[threadIdx.x] = mask;
    __syncthreads();
    for (int g = 0; g < kBlock && base + g < cnt; g += 64) {
      const uint32_t um = smask[g + lane];
      const uint64_t bal = __ballot(wave_units<1>(um, m.wave) != 0);
      if (__any((um & kSlowBit) != 0 || E != 0)) walk(std::false_type{}, bal, stage + g);
      else walk(std::true_type{}, bal, stage + g);
      if (t < 0x1p-500) {
        t *= 0x1p500;
        E -= kRenorm;
        pw = ldexp(1.0, E);
      }
    }
  }
  if (in) {
    const int64_t pix = m.pixel(0, a.width);
    a.image_out[3 * pix] = static_cast<float>(C0);
    a.image_out[3 * pix + 1] = static_cast<float>(C1);
    a.image_out[3 * pix + 2] = static_cast<float>(C2);
    a.pix_state[2 * pix] = t;
    a.pix_state[2 * pix + 1] = static_cast<double>(E);
  }
}

// Back to front over the same sorted list. With R_k the colour seen from
// layer k onwards in units of T_k (R_k = alpha_k c_k + (1 - alpha_k) R_{k+1},
// R = 0 behind the last layer), the colour behind i is S_i = T_i (1 -
// alpha_i) R_{i+1}, so dC/dalpha_i = T_i (c_i - R_{i+1}): no difference of
// large sums, whatever the depth. T_i is recovered from the forward's final
// transmittance, T_i = T_{i+1} / (1 - alpha_i).
//
// Only the upstream gradient's product with R enters: P = g . R obeys the same
// recursion as a scalar per pixel, P_i = P_{i+1} + alpha_i (g.c_i - P_{i+1}) (an
// instruction more than g.c_i - (1 - alpha_i) (g.c_i - P_{i+1}), which makes a NaN
// of an infinite colour), and dL/dalpha_i = T_i (g.c_i - P_{i+1}). All sums are taken in
// units of the opacity (alpha = sigma rho): with s = T rho dL/dalpha / T,
// the entry's sums are T rho g (colour / sigma), s (dL/dsigma) and the moments
// s (a dx + b dy), s (b dx + c dy), s dx^2, s dx dy, s dy^2, which the finish
// kernel scales by sigma and the constant factors once per primitive. At the
// clamp rho is rmax and s is 0.
// Rows per lane of the backward by the number of tiles (1024 SIMDs): with three
// tiles per SIMD or more, four rows per lane share the per-entry work (3.84 ms
// against 5.23 at 8160 tiles and 3 M primitives, 496 against 552 us at 3600
// tiles); below, one row per lane and four wavefronts per tile fill the chip
// (148 against 158 us at 2553 tiles, 101 against 178 at 920, 19 against 50 at
// 117).
constexpr int64_t kBwdRowsTiles = 3072;

template <int RPL, bool GEOM>
__global__ __launch_bounds__(256 / RPL) __attribute__((amdgpu_waves_per_eu(RPL == 4 ? 4 : 6)))
void raster_render_bwd(RasterArgs a) {
  constexpr int kBlock = 256 / RPL;
  __shared__ StageEntry stage[kBlock];
  __shared__ int32_t sidx[kBlock];
  __shared__ uint32_t smask[kBlock];
  {
    const RasterStamp st = *a.stamp;  // same for every thread: a uniform exit
    if (st.magic != kStampMagic || st.cap != a.cap || st.tiles_x != a.tiles_x ||
        st.tiles_y != a.tiles_y || st.n != a.n) {
      if (blockIdx.x == 0 && threadIdx.x == 0) *a.stale = 1;
      return;
    }
  }
  const int64_t tile = blockIdx.x;
  const TileMap<RPL> m = tile_map<RPL>(a, tile);
  const double cxp = m.px + 0.5, cyp = m.py0 + 0.5;
  const int cnt = __builtin_amdgcn_readfirstlane(min(a.cursor[tile], a.cap));
  const uint64_t* list = a.lists + tile * a.cap;

  double t[RPL], pw[RPL], P[RPL], g[RPL][3];
  int E[RPL];
  bool in[RPL];
#pragma unroll
  for (int j = 0; j < RPL; ++j) {
    in[j] = m.in(j);
    P[j] = 0.0;
    t[j] = 1.0;
    pw[j] = 1.0;
    E[j] = 0;
    g[j][0] = g[j][1] = g[j][2] = 0.0;
    if (in[j]) {
      const int64_t pix = m.pixel(j, a.width);
      t[j] = a.pix_state[2 * pix];
      E[j] = static_cast<int>(a.pix_state[2 * pix + 1]);
      pw[j] = ldexp(1.0, E[j]);
      g[j][0] = a.grad_image[3 * pix];
      g[j][1] = a.grad_image[3 * pix + 1];
      g[j][2] = a.grad_image[3 * pix + 2];
    }
  }
  const int lane = static_cast<int>(threadIdx.x & 63);
  const bool writer = GEOM ? lane_writes9(lane) : lane_writes4(lane);
  const int slot = GEOM ? lane_slot9(lane) : lane_slot4(lane);
  auto entry = [&](auto fast, int k, uint32_t bits) {
    constexpr bool kFast = decltype(fast)::value;
    StageEntry s = stage[k];
    keep(s.v);
    keep(s.c);
    keep(s.sigma);
    keep(s.c0);
    keep(s.c1);
    keep(s.c2);
    const double dx = cxp - s.u;
    const double A = s.a * dx * dx, B = s.b * (dx + dx);
    double gc0 = 0.0, gc1 = 0.0, gc2 = 0.0;
    // a lane's pixels share dx: it sums s, s dy and s dy^2 over them
    double q0 = 0.0, q1 = 0.0, q2 = 0.0;
#pragma unroll
    for (int j = 0; j < RPL; ++j) {
      if (RPL > 1 && ((bits >> j) & 1u) == 0) continue;  // uniform
      const double dy = (cyp + 4.0 * j) - s.v;
      const double q = fma(dy, fma(s.c, dy, B), A);
      if (in[j] && q <= kSupport) {
        const double rho = static_cast<double>(
            __builtin_amdgcn_exp2f(static_cast<float>(q) * kNegHalfLog2e));
        const double rc = kFast ? rho : fmin(rho, s.rmax);
        const double al = s.sigma * rc;
        const double om = 1.0 - al;
        t[j] *= rcp64(om);  // now T_i = t * pw
        const double w = rc * (kFast ? t[j] : t[j] * pw[j]);
        gc0 = fma(w, g[j][0], gc0);
        gc1 = fma(w, g[j][1], gc1);
        gc2 = fma(w, g[j][2], gc2);
        const double gc = fma(g[j][0], s.c0, fma(g[j][1], s.c1, g[j][2] * s.c2));
        const double d = gc - P[j];
        P[j] = fma(al, d, P[j]);
        const double sm = kFast || rho < s.rmax ? d * w : 0.0;
        q0 += sm;
        if constexpr (GEOM) {
          const double sy = sm * dy;
          q1 += sy;
          q2 = fma(sy, dy, q2);
        }
      }
    }
    // the entry's totals over the wavefront, one per writing lane
    float tot;
    if constexpr (GEOM) {
      const double qx = dx * q0;
      const float v[9] = {static_cast<float>(gc0), static_cast<float>(gc1),
                          static_cast<float>(gc2), static_cast<float>(q0),
                          static_cast<float>(fma(s.a, qx, s.b * q1)),
                          static_cast<float>(fma(s.b, qx, s.c * q1)),
                          static_cast<float>(dx * qx), static_cast<float>(dx * q1),
                          static_cast<float>(q2)};
      tot = lane_sums9(v, lane);
    } else {
      const float v[4] = {static_cast<float>(gc0), static_cast<float>(gc1),
                          static_cast<float>(gc2), static_cast<float>(q0)};
      tot = lane_sums4(v);
    }
    if (writer && tot != 0.f)
      unsafeAtomicAdd(a.grad_acc + kAccStride * static_cast<int64_t>(sidx[k]) + slot,
                      static_cast<double>(tot));
  };
  for (int end = cnt; end > 0; end -= kBlock) {
    const int base = max(0, end - kBlock);
    __syncthreads();
    const int e = base + static_cast<int>(threadIdx.x);
    uint32_t mask = 0;
    if (e < end) {
      const RenderRec r = stage_entry(a, list, e, &stage[threadIdx.x], &sidx[threadIdx.x]);
      mask = unit_mask<RPL == 4>(r, m.x0, m.y0);
    }
    smask[threadIdx.x] = mask;
    __syncthreads();
    for (int g0 = (end - base - 1) & ~63; g0 >= 0; g0 -= 64) {
      const uint32_t um = smask[g0 + lane];
      const uint32_t mine = wave_units<RPL>(um, m.wave);
      bool scaled = (um & kSlowBit) != 0;
#pragma unroll
      for (int j = 0; j < RPL; ++j) scaled = scaled || E[j] != 0;
      const bool slow = __any(scaled);
      auto walk = [&](auto fast) {
        uint64_t bal = __ballot(mine != 0);
        while (bal != 0) {
          const int k = 63 - __builtin_clzll(bal);
          bal &= ~(1ull << k);
          entry(fast, g0 + k, RPL == 1 ? 1u : __builtin_amdgcn_readlane(mine, k));
        }
      };
      if (slow) walk(std::false_type{});
      else walk(std::true_type{});
#pragma unroll
      for (int j = 0; j < RPL; ++j) {
        if (t[j] > 0x1p300 && E[j] < 0) {
          t[j] *= 0x1p-500;
          E[j] += kRenorm;
          pw[j] = ldexp(1.0, E[j]);
        }
      }
    }
  }
}

__global__ void raster_centre(float x, float y, float z, float* dst) {
  dst[0] = x;
  dst[1] = y;
  dst[2] = z;
}

hipError_t launch_centre(float x, float y, float z, float* dst, hipStream_t s) {
  hipLaunchKernelGGL(raster_centre, dim3(1), dim3(1), 0, s, x, y, z, dst);
  return hipGetLastError();
}

__global__ void raster_copy_flag(const int32_t* src, int32_t* dst) { *dst = *src; }

hipError_t launch_copy_flag(const int32_t* src, int32_t* dst, hipStream_t s) {
  hipLaunchKernelGGL(raster_copy_flag, dim3(1), dim3(1), 0, s, src, dst);
  return hipGetLastError();
}

template <int RPL, bool GEOM>
static void launch_bwd(const RasterArgs& a, int64_t n_tiles, hipStream_t s) {
  hipLaunchKernelGGL((raster_render_bwd<RPL, GEOM>), dim3(static_cast<unsigned>(n_tiles)),
                     dim3(256 / RPL), 0, s, a);
}

// Primitives per LDS-counting block: 1024 threads hide the latency of the
// record loads and LDS atomics that a block of 256 left bare (3 M primitives
// at 1920 x 1080: 366 -> 259 us, with four per thread; eight 278, two blocks
// per CU are then all that fit); fewer primitives take smaller chunks, of at least
// 1024: 128 blocks or more for each tile class from 131 072 primitives on, n/1024
// of them below (500 k at 1280 x 720: 171 -> 36 us, with one per thread 45, whose
// blocks send more device atomics; 12 k, 13 blocks: 48 -> 5 us).
static int64_t bin_chunk(int64_t n) {
  return kBinThreads * std::min<int64_t>(4, std::max<int64_t>(1, n / (kBinThreads * 128)));
}

hipError_t launch_raster(const RasterArgs& a, bool bwd, hipStream_t s) {
  const int64_t n_tiles = static_cast<int64_t>(a.tiles_x) * a.tiles_y;
  const unsigned gt = static_cast<unsigned>((n_tiles + 255) / 256);
  const unsigned gn = static_cast<unsigned>((a.n + 255) / 256);
  if (!bwd) {
    hipLaunchKernelGGL(raster_project, dim3(std::max(gt, gn)), dim3(256), 0, s, a);
    if (a.n > 0) {
      int pshift = 0;  // 2^pshift tile classes, the fewest that fit the LDS counters
      while ((1 << pshift) < kBinParts && ((n_tiles - 1) >> pshift) + 1 > kBinLdsTiles) ++pshift;
      if (((n_tiles - 1) >> pshift) + 1 <= kBinLdsTiles) {
        const int64_t chunk = bin_chunk(a.n);
        const unsigned gc = static_cast<unsigned>((a.n + chunk - 1) / chunk);
        const size_t lds = sizeof(int) * static_cast<size_t>(((n_tiles - 1) >> pshift) + 1);
        hipLaunchKernelGGL(raster_bin_lds, dim3(gc << pshift), dim3(kBinThreads), lds, s, a, pshift,
                           static_cast<int>(chunk));
      } else {
        hipLaunchKernelGGL(raster_bin, dim3(gn * kBinParts), dim3(256), 0, s, a);
      }
    }
    hipLaunchKernelGGL(raster_sort, dim3(static_cast<unsigned>(n_tiles)), dim3(kSortThreads), 0, s, a);
    hipLaunchKernelGGL(raster_sort_network, dim3(static_cast<unsigned>(n_tiles)), dim3(256), 0, s,
                       a);
    hipLaunchKernelGGL(raster_render_fwd, dim3(static_cast<unsigned>(n_tiles)), dim3(256), 0, s,
                       a);
  } else {
    if (a.n == 0) return hipGetLastError();
    const bool geom = a.grad_means != nullptr || a.grad_scales != nullptr || a.grad_rots != nullptr;
    hipLaunchKernelGGL(raster_zero_acc, dim3(gn), dim3(256), 0, s, a.grad_acc, a.n, a.stale);
    if (n_tiles >= kBwdRowsTiles) {
      geom ? launch_bwd<4, true>(a, n_tiles, s) : launch_bwd<4, false>(a, n_tiles, s);
    } else {
      geom ? launch_bwd<1, true>(a, n_tiles, s) : launch_bwd<1, false>(a, n_tiles, s);
    }
    if (geom) {
      hipLaunchKernelGGL(raster_finish_grads<true>, dim3(gn), dim3(256), 0, s, a);
    } else {
      hipLaunchKernelGGL(raster_finish_grads<false>, dim3(gn), dim3(256), 0, s, a);
    }
  }
  return hipGetLastError();
}

}  // namespace nasg
