// Scene dynamics (Sec. 3.4) and model expansion (Sec. 3.3) on the device.
//
//  * Rigid objects: Gaussians carry an object index; before an optimization
//    step the engine's object motion x -> R (x - p) + p + t (R the rotation of
//    the unit quaternion q / |q|) is applied to the means of the object's
//    Gaussians, and q / |q| is composed onto their orientation quaternions.
//    FP64 arithmetic, one rounding to FP32 per stored value.
//  * Relighting of the diffuse DC term: the DC colour C0 dc + 1/2 of each
//    channel is scaled by a per-Gaussian gain (one for all channels or one
//    per channel); a gain of exactly 1 leaves the coefficient untouched.
//  * Appending: new Gaussians join the end of the active pool (the frozen
//    pool moves up by their count); optimizer moments are extended with
//    zeros.  Written out of place into caller-sized tensors, row by row.
#include "internal.h"

namespace gs {
namespace {

__global__ __launch_bounds__(256) void k_object_transform(float* mean, float* quat, int64_t n,
                                                           const int32_t* object_of, const gs_transform* tf,
                                                           int32_t n_objects) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t o = object_of[i];
  if (o < 0 || o >= n_objects) return;
  const gs_transform T = tf[o];
  const double qn = sqrt((double)T.q[0] * T.q[0] + (double)T.q[1] * T.q[1] + (double)T.q[2] * T.q[2] +
                         (double)T.q[3] * T.q[3]);
  const double w = T.q[0] / qn, x = T.q[1] / qn, y = T.q[2] / qn, z = T.q[3] / qn;
  const double R[9] = {1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)};
  double d[3];
  for (int k = 0; k < 3; ++k) d[k] = (double)mean[k * n + i] - (double)T.pivot[k];
  for (int r = 0; r < 3; ++r)
    mean[r * n + i] = (float)(R[r * 3] * d[0] + R[r * 3 + 1] * d[1] + R[r * 3 + 2] * d[2] + (double)T.pivot[r] +
                              (double)T.t[r]);
  const double bw = quat[i], bx = quat[n + i], by = quat[2 * n + i], bz = quat[3 * n + i];
  quat[i] = (float)(w * bw - x * bx - y * by - z * bz);
  quat[n + i] = (float)(w * bx + x * bw + y * bz - z * by);
  quat[2 * n + i] = (float)(w * by - x * bz + y * bw + z * bx);
  quat[3 * n + i] = (float)(w * bz + x * by - y * bx + z * bw);
}

__global__ __launch_bounds__(256) void k_relight_dc(float* sh, int64_t n, const float* gain, int channels) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double c0 = 0.28209479177387814;   // 1 / (2 sqrt(pi)), the degree-0 basis function
  for (int c = 0; c < 3; ++c) {
    const float g = gain[(channels == 3 ? c : 0) * n + i];
    if (g == 1.0f) continue;
    const double dc = sh[c * n + i];
    sh[c * n + i] = (float)(((c0 * dc + 0.5) * (double)g - 0.5) / c0);
  }
}

// One tensor of an append: rows of old[0, na) | add[0, k) (zeros when add is
// null) | old[na, n_old), written to dst (row stride n_old + k).
struct AppendSeg {
  const uint32_t* old;
  const uint32_t* add;
  uint32_t* dst;
  int64_t n_old, na;
  int32_t row0;   // first row of the tensor among the launch's rows
};
constexpr int kAppendSegs = 16;
struct AppendArgs {
  AppendSeg seg[kAppendSegs];
  int32_t count;
  int64_t k;
};

// Bound by memory: every word of the model and moments is read and written
// once.  All tensors share one launch (one block row per tensor row); a
// thread writes one 16-byte aligned quad of the destination, its source four
// words at any word alignment, both streaming as nothing is read again: the
// append of 100k Gaussians to a 3M model with moments takes 0.60 ms (6.0 TB/s);
// word by word in 16 launches it took 1.10 ms.
typedef uint32_t U4 __attribute__((ext_vector_type(4)));
typedef U4 U4Unaligned __attribute__((aligned(4)));

__global__ __launch_bounds__(256) void k_append_rows(AppendArgs a) {
  int si = 0;
#pragma unroll
  for (int q = 1; q < kAppendSegs; ++q) si += q < a.count && (int)blockIdx.y >= a.seg[q].row0 ? 1 : 0;
  const AppendSeg s = a.seg[si];
  const int64_t r = (int)blockIdx.y - s.row0;
  const int64_t k = a.k, na = s.na, n = s.n_old + k;
  uint32_t* dst = s.dst + r * n;
  // quads lie on 16-byte boundaries of the destination: the first one may
  // start before the row, the last one end past it
  const int64_t lead = (int64_t)((reinterpret_cast<uintptr_t>(dst) >> 2) & 3u);
  const int64_t j = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4 - lead;
  if (j >= n) return;
  const uint32_t* old = s.old + r * s.n_old;
  const uint32_t* add = s.add ? s.add + r * k : nullptr;
  const uint32_t* src = nullptr;
  bool whole = j >= 0 && j + 4 <= n;
  if (j + 4 <= na) src = old + j;
  else if (j >= na + k) src = old + (j - k);
  else if (j >= na && j + 4 <= na + k) src = add ? add + (j - na) : nullptr;
  else whole = false;
  if (whole) {
    U4 v = {0u, 0u, 0u, 0u};
    if (src) v = __builtin_nontemporal_load(reinterpret_cast<const U4Unaligned*>(src));
    __builtin_nontemporal_store(v, reinterpret_cast<U4*>(dst + j));
    return;
  }
  for (int c = 0; c < 4; ++c) {
    const int64_t e = j + c;
    if (e < 0 || e >= n) continue;
    dst[e] = e < na ? old[e] : e >= na + k ? old[e - k] : add ? add[e - na] : 0u;
  }
}

}  // namespace

hipError_t launch_object_transform(const gs_params& p, const int32_t* object_of, const gs_transform* tf,
                                   int32_t n_objects, hipStream_t st) {
  if (p.n > 0 && n_objects > 0)
    hipLaunchKernelGGL(k_object_transform, dim3((unsigned)((p.n + 255) / 256)), dim3(256), 0, st, p.mean, p.quat,
                       (int64_t)p.n, object_of, tf, n_objects);
  return hipGetLastError();
}

hipError_t launch_relight_dc(const gs_params& p, const float* gain, int channels, hipStream_t st) {
  if (p.n > 0)
    hipLaunchKernelGGL(k_relight_dc, dim3((unsigned)((p.n + 255) / 256)), dim3(256), 0, st, p.sh, (int64_t)p.n,
                       gain, channels);
  return hipGetLastError();
}

hipError_t launch_append(const gs_params& old_p, const gs_params* old_m, const gs_params* old_v, int64_t na,
                         const gs_params& add, const gs_params& new_p, const gs_params* new_m,
                         const gs_params* new_v, const uint32_t* const* old_cols, const uint32_t* const* add_cols,
                         uint32_t* const* new_cols, int n_cols, hipStream_t st) {
  const int nk = (old_p.sh_degree + 1) * (old_p.sh_degree + 1);
  const int rows[5] = {3, 3, 4, 1, 3 * nk};
  const int64_t k = add.n;
  auto rows_of = [](const gs_params& t, int g) -> float* {
    float* r[5] = {t.mean, t.log_scale, t.quat, t.opacity_logit, t.sh};
    return r[g];
  };
  AppendArgs args;
  args.count = 0;
  args.k = k;
  int32_t total_rows = 0;
  int64_t longest = 0;
  auto flush = [&]() {
    if (total_rows > 0)   // + 3: a row's quads start at the 16-byte boundary before it
      hipLaunchKernelGGL(k_append_rows, dim3((unsigned)((longest + 3 + 1023) / 1024), (unsigned)total_rows), dim3(256),
                         0, st, args);
    args.count = 0;
    total_rows = 0;
    longest = 0;
  };
  auto copy = [&](const void* old, int64_t n_old, int64_t keep, const void* add_rows, void* dst, int nrows) {
    const int64_t dn = n_old + k;
    if (dn == 0 || nrows == 0) return;
    args.seg[args.count++] = AppendSeg{static_cast<const uint32_t*>(old), static_cast<const uint32_t*>(add_rows),
                                       static_cast<uint32_t*>(dst), n_old, keep, total_rows};
    total_rows += nrows;
    longest = dn > longest ? dn : longest;
    if (args.count == kAppendSegs) flush();
  };
  for (int g = 0; g < 5; ++g) {
    copy(rows_of(old_p, g), old_p.n, na, rows_of(add, g), rows_of(new_p, g), rows[g]);
    if (old_m) copy(rows_of(*old_m, g), na, na, nullptr, rows_of(*new_m, g), rows[g]);
    if (old_v) copy(rows_of(*old_v, g), na, na, nullptr, rows_of(*new_v, g), rows[g]);
  }
  for (int c = 0; c < n_cols; ++c) copy(old_cols[c], old_p.n, na, add_cols[c], new_cols[c], 1);
  flush();
  return hipGetLastError();
}

}  // namespace gs
