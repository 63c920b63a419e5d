// Operands and geometry of the bilateral aggregation, Eqs. (10)-(11), on the
// matrix cores with FP16 operands split in two: what the streamed kernels of
// bilateral_stream.h (forward and both backward passes) multiply and how the
// volumes they read are stored.
//
// As in the FP32 matrix-core kernel, the aggregated costs of a 4x4 block of
// pixels p and 16 levels d are the product E[p][d] = sum_q w(p, q) C(q, d)
// over the block's window union, with zero weights outside a pixel's own
// window.  Here every operand is carried as two FP16 numbers, x = x_hi + x_lo
// (x_hi the FP16 rounding of x, x_lo that of the remainder), and the product
// takes the three terms w_hi C_hi + w_hi C_lo + w_lo C_hi on
// v_mfma_f32_16x16x32_f16 with FP32 accumulation.  Each operand keeps about
// 22 significant bits and the dropped w_lo C_lo term is below 2^-22 of the
// product, so the sums are as accurate as FP32 products; the three FP16
// products take about a third of the matrix-core time of the FP32 ones.
// (The backward's second pass at large radii carries both operands in three
// BF16 numbers: kMaxWide in bilateral_stream.h.)
// Weights are scaled by 2^12 before the split (the selection and the
// normalised soft-argmin are scale-free), which keeps the low parts of small
// weights out of the FP16 subnormal range.
//
// Operand layout.  The K index of one product runs over 32 union positions:
// lane (m, g) (m = lane & 15, g = lane >> 4) holds 8 of them, a 2-row x
// 4-column patch of the union, for pixel m (A, weights) or level m (B,
// costs).  Patch 4 i + g of product i; the union ((4 + 2R) rows, 4 + 2R
// columns rounded up to whole column quads) has (R + 2) x ceil((4+2R)/4)
// patches, padded to a multiple of 4 with zero-weight patches.
//
// Costs.  The NCC writes two split-FP16 volumes, reference-anchored and
// target-anchored, so both volumes stage the same way.  Each is stored in
// blocks of 16 levels, [block][part][row pair][column quad][16 levels][2 rows]
// [4 columns] (columns shifted by R and rows by R & 1, so that a block's
// union starts at a column quad and a row pair): the 8 values of a lane's
// patch are 16 contiguous bytes, one operand read (16 levels x a patch) is
// 256 contiguous bytes read by ds_read_b128, and one halo row pair of a block
// part is HXP / 4 x 256 contiguous bytes.  The LDS returns 209 bytes per
// cycle to 16-byte reads but 119 to 8-byte ones (12 waves, this access
// pattern): with rows stored singly (two 8-byte reads per patch and part) the
// products of a pass took 2630 cycles, now 2000, near the 1800 of the matrix
// cores alone.  Rows and columns outside the image and the levels of
// the last block past D are zeros; their weights are zero or their outputs
// unused.
//
// Per pixel the result depends on the pixel's block and the levels only, so
// per-pair and queued launches are bitwise equal.  The summation order
// differs from the other engines': the three agree to rounding.
#pragma once
#include "bilateral_mfma.h"

namespace stereo {
namespace bilh {

using bil::BilPair;
typedef float f4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));

constexpr int kTW = kSegW;              // strip columns: four 4x4 blocks
constexpr float kFar = 1e30f;           // guide outside the image: zero weight
constexpr float kLog2WScale = 12.0f;    // weights scaled by 2^12 before the split

// Row pitch (halves) of the split-FP16 volumes for image width W at radius R.
template <int R>
struct HGeom {
  static constexpr int UH = 4 + 2 * R;                  // union rows of a 4x4 block
  static constexpr int UW = (4 + 2 * R + 3) & ~3;       // union columns, whole quads
  static constexpr int NRP = UH / 2;                    // row pairs
  static constexpr int NCQ = UW / 4;                    // column quads
  static constexpr int NP = NRP * NCQ;                  // 2x4 patches
  static constexpr int NI = (NP + 3) / 4;               // products (x3) per pass
  static constexpr int HXP = (4 * (kTW / 4 - 1) + UW + 7) & ~7;   // halo columns of a strip
  static constexpr int NQH = HXP / 4;                   // column quads per halo row
  static constexpr int STAB = NI * 64 * 8;              // spatial terms [i][lane][slot]
  static_assert(kTW + 2 * R <= HXP && 4 * (kTW / 4 - 1) + UW <= HXP, "halo columns");
};

template <int R>
inline int h2_pitch_for(int W) {
  return ((W + kTW - 1) / kTW) * kTW - kTW + HGeom<R>::HXP;
}

// The fields one tile needs; uniform across the workgroup.
struct View {
  const uint16_t* V;              // split-FP16 volume
  int64_t plane;                  // halves per block part: 16 h2_rows(R, H) pitch
  int pitch;                      // columns per row (a multiple of 8)
  const void* guide;
  int64_t g_pitch;
  int g_u8;                       // guide of uint8 (else FP32)
  int W, H, D;
  float ks2, kr2;
  float4* state;                  // selection state between sweeps of the levels
  int16_t* dint;                  // selection (mode 1)
  float* dsub;
  float* sm_m;                    // soft-argmin (mode 2)
  float* sm_logZ;
  float* sm_dh;
  float* disp;
  float invT;
  double delta_p, c0, c1, c2;
};

__host__ __device__ inline View view_of(const BilPair& a) {
  View v;
  v.V = a.h2;
  v.plane = a.h2_plane;
  v.pitch = a.h2_pitch;
  v.guide = a.guide;
  v.g_pitch = a.g_pitch;
  v.g_u8 = a.g_u8;
  v.state = reinterpret_cast<float4*>(a.state);
  v.W = a.W; v.H = a.H; v.D = a.D;
  v.ks2 = a.ks2;
  v.kr2 = a.kr2;
  v.dint = a.o.dint;
  v.dsub = a.o.dsub;
  v.sm_m = a.o.sm_m;
  v.sm_logZ = a.o.sm_logZ;
  v.sm_dh = a.o.sm_dh;
  v.disp = a.o.disp;
  v.invT = a.o.invT;
  v.delta_p = a.o.delta_p;
  v.c0 = a.o.c0; v.c1 = a.o.c1; v.c2 = a.o.c2;
  return v;
}

// v of another lane of the wave (index taken modulo 64).
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(
                                       4 * lane, __builtin_bit_cast(int, v)));
}

}  // namespace bilh
}  // namespace stereo
