// Dispatch of the aggregation launches over the compiled window radii.
#include "bilateral_mfma16.h"

namespace stereo {
hipError_t launch_bilateral_r1(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r1(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);
hipError_t launch_bilateral_r2(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r2(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);
hipError_t launch_bilateral_r3(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r3(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);
hipError_t launch_bilateral_r4(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r4(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);
hipError_t launch_bilateral_r5(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r5(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);
hipError_t launch_bilateral_r6(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r6(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);
hipError_t launch_bilateral_r7(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r7(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);
hipError_t launch_bilateral_r8(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bilateral_persistent_r8(int, stereo_dtype, int, const void*, const int*, int, unsigned int*, int, hipStream_t);

hipError_t launch_bilateral_h2_r1(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r1(const void*, const Seg*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_r2(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r2(const void*, const Seg*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_r3(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r3(const void*, const Seg*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_r4(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r4(const void*, const Seg*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_r5(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r5(const void*, const Seg*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_r6(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r6(const void*, const Seg*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_r7(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r7(const void*, const Seg*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_r8(const Plan&, const BilArgs*, int, int, hipStream_t);
hipError_t launch_bilateral_h2_queue_r8(const void*, const Seg*, int, int, hipStream_t);

hipError_t launch_bwd16_r1(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bwd16_r2(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bwd16_r3(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bwd16_r4(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bwd16_r5(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bwd16_r6(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bwd16_r7(const Plan&, const BilArgs&, int, hipStream_t);
hipError_t launch_bwd16_r8(const Plan&, const BilArgs&, int, hipStream_t);

hipError_t launch_bilateral_bwd16(const Plan& P, const BilArgs& a, int pass, hipStream_t s) {
  if ((pass != 1 && pass != 2) || (a.d_first & 15)) return hipErrorInvalidValue;
  switch (P.R) {
    case 1: return launch_bwd16_r1(P, a, pass, s);
    case 2: return launch_bwd16_r2(P, a, pass, s);
    case 3: return launch_bwd16_r3(P, a, pass, s);
    case 4: return launch_bwd16_r4(P, a, pass, s);
    case 5: return launch_bwd16_r5(P, a, pass, s);
    case 6: return launch_bwd16_r6(P, a, pass, s);
    case 7: return launch_bwd16_r7(P, a, pass, s);
    case 8: return launch_bwd16_r8(P, a, pass, s);
    default: return hipErrorInvalidValue;
  }
}

namespace bilh {
// Zeros in the pad columns of every row, and in the rows outside the image,
// of the first blocks (all parts).  Row blockIdx.y of the stored rows; thread
// t: column t / 16 (of an image row: pad columns [0, R), then [W + R, pitch);
// of a row outside: all), level t % 16.
__global__ void __launch_bounds__(256) h2_pad_zero_kernel(uint16_t* __restrict__ h2,
                                                          uint16_t* __restrict__ h3, int nblk,
                                                          int64_t plane, int pitch, int W, int H,
                                                          int R) {
  const int st = blockIdx.y, y = st - (R & 1), bp = blockIdx.z;   // 2 block + part, then block
  uint16_t* const to = bp < 2 * nblk ? h2 + (int64_t)bp * plane : h3 + (int64_t)(bp - 2 * nblk) * plane;
  const bool out = y < 0 || y >= H;
  const int n = 16 * (out ? pitch : pitch - W);
  for (int t = blockIdx.x * 256 + threadIdx.x; t < n; t += gridDim.x * 256) {
    const int ci = t >> 4, l = t & 15;
    const int c = out || ci < R ? ci : W + ci;
    to[(int64_t)(st >> 1) * 32 * pitch + 128 * (c >> 2) + 8 * l + 4 * (st & 1) + (c & 3)] = 0;
  }
}
}  // namespace bilh

hipError_t launch_h2_pad_zero(uint16_t* h2, uint16_t* h3, int64_t plane, int pitch, int W, int H,
                              int R, int nblk, hipStream_t s) {
  if (!h2 || pitch < W + R || nblk <= 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((16 * (pitch - W) + 255) / 256), (unsigned)h2_rows(R, H),
                  (unsigned)((h3 ? 3 : 2) * nblk));
  hipLaunchKernelGGL(bilh::h2_pad_zero_kernel, grid, dim3(256), 0, s, h2, h3, nblk, plane, pitch, W,
                     H, R);
  return hipGetLastError();
}

hipError_t launch_bilateral(const Plan& P, const BilArgs& a, int mode, hipStream_t s) {
  switch (P.R) {
    case 1: return launch_bilateral_r1(P, a, mode, s);
    case 2: return launch_bilateral_r2(P, a, mode, s);
    case 3: return launch_bilateral_r3(P, a, mode, s);
    case 4: return launch_bilateral_r4(P, a, mode, s);
    case 5: return launch_bilateral_r5(P, a, mode, s);
    case 6: return launch_bilateral_r6(P, a, mode, s);
    case 7: return launch_bilateral_r7(P, a, mode, s);
    case 8: return launch_bilateral_r8(P, a, mode, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_bilateral_h2(const Plan& P, const BilArgs* a, int n, int mode, hipStream_t s) {
  switch (P.R) {
    case 1: return launch_bilateral_h2_r1(P, a, n, mode, s);
    case 2: return launch_bilateral_h2_r2(P, a, n, mode, s);
    case 3: return launch_bilateral_h2_r3(P, a, n, mode, s);
    case 4: return launch_bilateral_h2_r4(P, a, n, mode, s);
    case 5: return launch_bilateral_h2_r5(P, a, n, mode, s);
    case 6: return launch_bilateral_h2_r6(P, a, n, mode, s);
    case 7: return launch_bilateral_h2_r7(P, a, n, mode, s);
    case 8: return launch_bilateral_h2_r8(P, a, n, mode, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_bilateral_h2_queue(int R, const void* descs, const Seg* segs, int n,
                                     int duo, hipStream_t s) {
  switch (R) {
    case 1: return launch_bilateral_h2_queue_r1(descs, segs, n, duo, s);
    case 2: return launch_bilateral_h2_queue_r2(descs, segs, n, duo, s);
    case 3: return launch_bilateral_h2_queue_r3(descs, segs, n, duo, s);
    case 4: return launch_bilateral_h2_queue_r4(descs, segs, n, duo, s);
    case 5: return launch_bilateral_h2_queue_r5(descs, segs, n, duo, s);
    case 6: return launch_bilateral_h2_queue_r6(descs, segs, n, duo, s);
    case 7: return launch_bilateral_h2_queue_r7(descs, segs, n, duo, s);
    case 8: return launch_bilateral_h2_queue_r8(descs, segs, n, duo, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_bilateral_persistent(int engine, int R, stereo_dtype gdt, int levels, const void* pairs,
                                       const int* tiles, int n_tiles, unsigned int* counter,
                                       int n_groups, hipStream_t s) {
  switch (R) {
    case 1: return launch_bilateral_persistent_r1(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    case 2: return launch_bilateral_persistent_r2(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    case 3: return launch_bilateral_persistent_r3(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    case 4: return launch_bilateral_persistent_r4(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    case 5: return launch_bilateral_persistent_r5(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    case 6: return launch_bilateral_persistent_r6(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    case 7: return launch_bilateral_persistent_r7(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    case 8: return launch_bilateral_persistent_r8(engine, gdt, levels, pairs, tiles, n_tiles, counter, n_groups, s);
    default: return hipErrorInvalidValue;
  }
}

size_t bilateral_pair_bytes() { return sizeof(bil::BilPair); }

int h2_pitch(int R, int W) {
  switch (R) {
    case 1: return bilh::h2_pitch_for<1>(W);
    case 2: return bilh::h2_pitch_for<2>(W);
    case 3: return bilh::h2_pitch_for<3>(W);
    case 4: return bilh::h2_pitch_for<4>(W);
    case 5: return bilh::h2_pitch_for<5>(W);
    case 6: return bilh::h2_pitch_for<6>(W);
    case 7: return bilh::h2_pitch_for<7>(W);
    case 8: return bilh::h2_pitch_for<8>(W);
    default: return 0;
  }
}

void* bilateral_pair(const Plan& P, const BilArgs& a, void* out) {
  *static_cast<bil::BilPair*>(out) = bil::make_pair(P, a);
  return out;
}

}  // namespace stereo
