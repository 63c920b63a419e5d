// Disparity transformation, Sec. 3.3: roll-angle fit (Eqs. 14-28) and the
// transformation of Eq. (29), entirely on the device so that the call can be
// captured into a graph (no device-to-host copy).
//
// The energy of Eq. (23) and its gradient (Eq. 26) depend on the data only
// through ten sums over the selected pixels:
//   n, Su, Sv, Suu, Suv, Svv, Sd, Sdd, Sdu, Sdv.
// With y = v cos psi - u sin psi and y' = dy/dpsi:
//   alpha = A^-1 b,  A = [[n, Sy], [Sy, Syy]],  b = [Sd, Sdy]      (Eq. 21)
//   E(psi) = Sdd - alpha . b                                       (Eq. 23)
//   dE/dpsi = -2 alpha1 (Sdy' - alpha0 Sy' - alpha1 Syy')          (Eq. 26)
// The sums are accumulated in FP64 in a fixed order (per-thread grid-stride
// sums, a fixed tree per block, then a fixed tree over the block partials),
// so the fit is deterministic.
#include <algorithm>
#include <mutex>

#include "internal.h"

namespace stereo {
namespace {

constexpr int kRoadThreads = 256;
constexpr int kMom = 10;

struct Mom {
  double n, su, sv, suu, suv, svv, sd, sdd, sdu, sdv;
};

// out[j] = sum of a[j] over the workgroup's threads, by the tree that adds
// thread t + s to thread t for s = 128, 64, .. 1.  Wave w takes the sums
// j = w, w + 4, w + 8: the two widest steps read LDS, the others stay in the
// wave.  (Every step through LDS, ten sums by one wave and a barrier a step,
// took 2 us.)
template <int N>
__device__ __forceinline__ double row_down(double x) {   // lane + N of the row of 16
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const int lo = (int)(unsigned)b, hi = (int)(unsigned)(b >> 32);
  const unsigned l = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, 0x100 + N, 0xf, 0xf, false);
  const unsigned h = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, 0x100 + N, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)h << 32) | l);
}

__device__ __forceinline__ void sum_moments(const double (&a)[kMom], double (&red)[kMom][kRoadThreads],
                                            double (&out)[kMom]) {
#pragma unroll
  for (int j = 0; j < kMom; ++j) red[j][threadIdx.x] = a[j];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  for (int j = threadIdx.x >> 6; j < kMom; j += kRoadThreads / 64) {
    double v = (red[j][lane] + red[j][lane + 128]) + (red[j][lane + 64] + red[j][lane + 192]);
    v += __shfl_down(v, 32);
    v += __shfl_down(v, 16);
    v += row_down<8>(v);
    v += row_down<4>(v);
    v += row_down<2>(v);
    v += row_down<1>(v);
    if (lane == 0) out[j] = v;
  }
  __syncthreads();
}

// Rows by block, columns by thread: no division per pixel.  A thread's pixels
// are added in that order, kAhead of them loaded before the first is added
// (1280x720 13.7 -> 5.8 us, 1917x1075 27 -> 8.3 us; before, a load's latency
// each).
__global__ void __launch_bounds__(kRoadThreads)
road_moments_kernel(const float* __restrict__ disp, const uint8_t* __restrict__ mask,
                    int W, int H, double* __restrict__ partials) {
  __shared__ double red[kMom][kRoadThreads], sum[kMom];
  constexpr int kAhead = 8;
  double a[kMom];
#pragma unroll
  for (int j = 0; j < kMom; ++j) a[j] = 0.0;
  const uint8_t* const mk = mask ? mask : reinterpret_cast<const uint8_t*>(disp);
  int y = blockIdx.x, x0 = 0;
  while (y < H) {
    float d[kAhead];
    uint8_t in[kAhead];
    int yl = y, xl = x0;
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int64_t p = (int64_t)min(yl, H - 1) * W + min(xl + (int)threadIdx.x, W - 1);
      d[k] = disp[p];
      in[k] = mk[p];
      xl += kRoadThreads;
      if (xl >= W) { xl = 0; yl += gridDim.x; }
    }
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int xi = x0 + (int)threadIdx.x;
      const double v = (double)y, u = (double)xi, df = d[k];
      // NaN / inf: not a disparity
      if (y < H && xi < W && fabsf(d[k]) <= 3.402823466e38f && (!mask || in[k])) {
        a[0] += 1.0; a[1] += u; a[2] += v; a[3] += u * u; a[4] += u * v;
        a[5] += v * v; a[6] += df; a[7] += df * df; a[8] += df * u; a[9] += df * v;
      }
      x0 += kRoadThreads;
      if (x0 >= W) { x0 = 0; y += gridDim.x; }
    }
  }
  sum_moments(a, red, sum);
  if (threadIdx.x < kMom) partials[(int64_t)blockIdx.x * kMom + threadIdx.x] = sum[threadIdx.x];
}

struct Fit {
  double a0, a1, sdy, sy;
};

__device__ Fit alpha_cs(const Mom& m, double c, double s) {
  Fit f;
  f.sy = c * m.sv - s * m.su;
  const double syy = c * c * m.svv - 2.0 * s * c * m.suv + s * s * m.suu;
  f.sdy = c * m.sdv - s * m.sdu;
  const double det = m.n * syy - f.sy * f.sy;
  f.a0 = (syy * m.sd - f.sy * f.sdy) / det;
  f.a1 = (m.n * f.sdy - f.sy * m.sd) / det;
  return f;
}

__device__ double energy_cs(const Mom& m, double c, double s) {
  const Fit f = alpha_cs(m, c, s);
  return m.sdd - (f.a0 * m.sd + f.a1 * f.sdy);
}

__device__ double gradient_cs(const Mom& m, double c, double s) {
  const Fit f = alpha_cs(m, c, s);
  const double syp = -s * m.sv - c * m.su;
  const double syyp = s * c * (m.suu - m.svv) + (s * s - c * c) * m.suv;
  const double sdyp = -s * m.sdv - c * m.sdu;
  return -2.0 * f.a1 * (sdyp - f.a0 * syp - f.a1 * syyp);
}

__device__ double wrap_half_pi(double psi) {
  const double pi = 3.14159265358979323846;
  const double x = psi + pi / 2.0;
  // |x| < 2 pi but for angles out of range: there the remainder is x or, exactly, x -+ pi
  double w = fabs(x) < pi ? x : fabs(x) < 2.0 * pi ? x - copysign(pi, x) : fmod(x, pi);
  if (w <= 0.0) w += pi;
  return w - pi / 2.0;
}

// One block: thread b loads the partial sums of block b, then a fixed tree
// combines them (deterministic); one lane then runs the descent.  Rate:
// Eq. (28), lambda_k+1 = lambda_k g_k / (g_k - g_k+1); a step is halved while
// it raises the normalised energy or exceeds pi/4; a non-positive rate
// restarts at lambda0.  The lane's chain of sines, divisions and remainders
// bounds the launch: each angle's sine and cosine are formed once, for its
// energy, its gradient and as the next step's start (10.1 -> 5.9 us at 320x240;
// before, three times, and the tree through LDS).  Energy and gradient stay
// separate expressions: e_min cancels, and a plane shared by both, which the
// compiler fuses otherwise, moved it by up to 3e-10.
__global__ void __launch_bounds__(kRoadThreads)
road_fit_kernel(const double* __restrict__ partials, int nblocks, int W, int H,
                double psi0, double lambda0, double delta_psi, int max_iter,
                stereo_road_fit* __restrict__ out, stereo_plane_state* __restrict__ state) {
  __shared__ double red[kMom][kRoadThreads], mom[kMom];
  double a[kMom];
#pragma unroll
  for (int j = 0; j < kMom; ++j) a[j] = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += kRoadThreads) {
#pragma unroll
    for (int j = 0; j < kMom; ++j) a[j] += partials[(int64_t)b * kMom + j];
  }
  sum_moments(a, red, mom);
  if (threadIdx.x != 0) return;
  if (state) psi0 = state->psi;            // warm start from the previous frame
  const Mom m{mom[0], mom[1], mom[2], mom[3], mom[4], mom[5], mom[6], mom[7], mom[8], mom[9]};
  stereo_road_fit r;
  r.n_points = m.n;
  r.pad_ = 0;
  double psi = psi0;
  int iters = 0, converged = 0, flat = 0;
  double sp, cp;                           // of psi
  sincos(psi, &sp, &cp);
  Fit f0;
  if (m.n < 3.0) {
    flat = 1; converged = 1;
    f0.a0 = m.n > 0.0 ? m.sd / m.n : 0.0;
    f0.a1 = 0.0;
  } else {
    f0 = alpha_cs(m, cp, sp);
    if (!(fabs(f0.a1) >= 1e-6)) { flat = 1; converged = 1; }
  }
  if (!flat) {
    const double s = (double)max(W, H);
    const double scale = 1.0 / (m.n * s * s * f0.a1 * f0.a1);
    double lam = lambda0;
    double E = energy_cs(m, cp, sp) * scale;
    double g = gradient_cs(m, cp, sp) * scale;
    const double pi = 3.14159265358979323846;
    for (iters = 1; iters <= max_iter; ++iters) {
      double step = -lam * g, psi_new = psi;
      bool known = false;                  // psi_new, sp, cp belong to psi + step
      for (int h = 0; h < 64; ++h) {
        if (fabs(step) <= pi / 4.0) {
          psi_new = wrap_half_pi(psi + step);
          sincos(psi_new, &sp, &cp);
          known = true;
          if (energy_cs(m, cp, sp) * scale <= E * (1.0 + 1e-9)) break;
        }
        lam *= 0.5;
        step = -lam * g;
        known = false;
      }
      if (!known) {
        psi_new = wrap_half_pi(psi + step);
        sincos(psi_new, &sp, &cp);
      }
      const double g_new = gradient_cs(m, cp, sp) * scale;
      const bool done = fabs(step) < delta_psi;
      if (g_new == g) {
        psi = psi_new; converged = 1;
        break;
      }
      lam = lam * g / (g - g_new);
      if (!(lam > 0.0) || isinf(lam)) lam = lambda0;
      psi = psi_new;
      E = energy_cs(m, cp, sp) * scale;
      g = g_new;
      if (done) { converged = 1; break; }
    }
    if (iters > max_iter) iters = max_iter;
    f0 = alpha_cs(m, cp, sp);
  }
  r.psi = psi;
  r.alpha0 = f0.a0;
  r.alpha1 = f0.a1;
  r.e_min = (m.n >= 3.0) ? energy_cs(m, cp, sp) : 0.0;
  r.plane[0] = f0.a0;
  r.plane[1] = -f0.a1 * sp;
  r.plane[2] = f0.a1 * cp;
  r.iters = iters;
  r.converged = converged;
  r.flat = flat;
  *out = r;
  if (state && !flat) {                    // the next frame's plane
    state->plane[0] = r.plane[0];
    state->plane[1] = r.plane[1];
    state->plane[2] = r.plane[2];
    state->psi = psi;
    state->frames += 1;
  }
}

// Eq. (29): l' = l - a0 + a1 (u sin psi - v cos psi) + delta_t.  A thread walks
// down its column, so that it forms the sine and cosine once for several
// pixels (1280x720 6.7 -> 5.3 us, 1917x1075 12.1 -> 6.6 us).
__global__ void __launch_bounds__(256)
road_apply_kernel(const float* __restrict__ disp, int W, int H,
                  const stereo_road_fit* __restrict__ fit, float delta_t,
                  float* __restrict__ out) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= W) return;
  constexpr int kRows = 4;                 // rows loaded ahead
  const double psi = fit->psi, a0 = fit->alpha0, a1 = fit->alpha1;
  const double sp = sin(psi), cp = cos(psi);
  const int step = gridDim.y;
  for (int v0 = blockIdx.y; v0 < H; v0 += kRows * step) {
    float d[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) d[k] = disp[(int64_t)min(v0 + k * step, H - 1) * W + u];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
      const int v = v0 + k * step;
      if (v < H)
        out[(int64_t)v * W + u] = (float)((double)d[k] - a0 + a1 * ((double)u * sp - (double)v * cp) +
                                          (double)delta_t);
    }
  }
}

// Damage below the flattened road: mask = finite(l') && l' < delta_t - tau.
__global__ void __launch_bounds__(256)
damage_mask_kernel(const float* __restrict__ disp_t, int64_t n, float level,
                   uint8_t* __restrict__ mask) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float d = disp_t[i];
  mask[i] = (isfinite(d) && d < level) ? 1 : 0;
}

}  // namespace

hipError_t launch_damage_mask(const Plan& P, const float* disp_t, float delta_t, float tau,
                              uint8_t* mask, hipStream_t s) {
  const int64_t n = (int64_t)P.W * P.H;
  const float level = delta_t - tau;
  hipLaunchKernelGGL(damage_mask_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     disp_t, n, level, mask);
  return hipGetLastError();
}

// Fixed device buffer of the allocation-free road transform: room for the
// ten FP64 moment partials of up to kRoadScratchDoubles / 10 reduction
// blocks.  Every device the library runs on holds one copy for the life of
// the process; calls on one device share it.
static __device__ __align__(256) double scratch[kRoadScratchDoubles];

hipError_t road_scratch(double** out, size_t* bytes) {
  static std::mutex mu;
  static double* ptr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    // the array's name is a host-side stand-in: the device address of this
    // device's copy comes from the runtime, once per device
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    ptr[dev] = static_cast<double*>(p);
  }
  *out = ptr[dev];
  *bytes = sizeof(double) * (size_t)kRoadScratchDoubles;
  return hipSuccess;
}

hipError_t launch_road(const Plan& P, const float* disp, const uint8_t* mask,
                       double psi0, double lambda0, double delta_psi, int max_iter,
                       float delta_t, stereo_road_fit* fit, float* disp_t,
                       double* partials, hipStream_t s, stereo_plane_state* state) {
  hipLaunchKernelGGL(road_moments_kernel, dim3(P.road_blocks), dim3(kRoadThreads), 0, s,
                     disp, mask, P.W, P.H, partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(road_fit_kernel, dim3(1), dim3(kRoadThreads), 0, s, partials, P.road_blocks,
                     P.W, P.H, psi0, lambda0, delta_psi, max_iter, fit, state);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (disp_t) {
    const int nx = (P.W + 255) / 256, ny = std::max(1, std::min(P.H, 2048 / nx));
    hipLaunchKernelGGL(road_apply_kernel, dim3(nx, ny), dim3(256), 0, s,
                       disp, P.W, P.H, fit, delta_t, disp_t);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace stereo
