// Operands and geometry of the bilateral aggregation, Eqs. (10)-(11), on the
// matrix cores with FP16 operands split in two: shared by the forward kernel
// (bilateral_stream.h) and the backward passes (bilateral_mfma16_bwd.h), whose
// tile staging is also here.
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

constexpr int kBR = 3;                  // block rows per tile
constexpr int kWaves = 4 * kBR;         // one 4x4 block per wave
constexpr int kThreads = 64 * kWaves;
constexpr int kTW = 16, kTH = 4 * kBR;  // tile in pixels
static_assert(kTW == kMfmaTileW && kTH == kMfmaTileH, "tile size shared with the batch tables");
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
  static constexpr int HY = kTH + 2 * R;                // halo rows
  static constexpr int HXP = (4 * (kTW / 4 - 1) + UW + 7) & ~7;   // halo columns
  static constexpr int NQH = HXP / 4;                   // column quads per halo row
  static constexpr int HP = HY / 2;                     // halo row pairs
  static constexpr int PAIRB = NQH * 256;               // bytes per halo row pair of a part
  static constexpr int PARTB = HP * PAIRB;              // bytes per part of a slab
  static constexpr int NWC = 2 * HY;                    // wave copies per slab
  static constexpr int KPW = (NWC + kWaves - 1) / kWaves;
  static constexpr int BUF = 2 * PARTB / 4;             // dwords per slab
  // the guide tile is laid out like a level of the slab, [row pair][column
  // quad][2 rows][4 columns] floats: a patch's guide offset (floats) is 8 x
  // its offset in 256-byte units
  static constexpr int GUIDE = HY * HXP;
  static constexpr int GPT = (GUIDE + kThreads - 1) / kThreads;
  static constexpr int STAB = NI * 64 * 8;              // spatial terms [i][lane][slot]
  static constexpr size_t base_bytes = sizeof(float) * (2 * (size_t)BUF + 2 * GUIDE);
  // the spatial terms are tabulated in LDS where it has room
  static constexpr bool kTable = base_bytes + sizeof(float) * STAB <= 160 * 1024;
  static constexpr size_t lds_bytes = base_bytes + (kTable ? sizeof(float) * STAB : 0);
  static_assert(kTW + 2 * R <= HXP && 4 * (kTW / 4 - 1) + UW <= HXP, "halo columns");
  static_assert(kTH % 2 == 0 && HY % 2 == 0, "halo rows come in pairs");
  static_assert(HP * NQH < 256, "patch offsets are packed in 8 bits");
  static_assert(lds_bytes <= 160 * 1024, "LDS budget");
  static_assert(PARTB < 65536, "lo-part offset must fit a DS immediate");
};

// Position (floats) of halo row yy, column xx in a guide tile.
template <int R>
__device__ __forceinline__ int guide_pos(int yy, int xx) {
  return ((yy >> 1) * HGeom<R>::NQH + (xx >> 2)) * 8 + 4 * (yy & 1) + (xx & 3);
}

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

// Slab of levels [d0, d0 + 16) (one stored block) of the tile at (x0, y0)
// into buf: [part][row pair][column quad][16 levels][2 rows][4 columns]
// halves, the same bytes as in the stored block.  One wave copy is half a
// halo row pair of one part (NQH x 128 bytes; with 24 halo columns 48 of the
// 64 lanes take part): copy k = wave + kWaves m is half k % HY of part k / HY.
// Row pairs clamp to the stored ones (image row y is row (y + (R & 1)) & 1 of
// pair (y + (R & 1)) >> 1; a row of the first or last pair outside the image
// holds zeros).  A copy's address is scalar but for the lane, so the border
// needs no path of its own.
template <int R>
struct Slab {
  using G = HGeom<R>;
  const uint16_t* base;           // block of d0, part 0, column quad of x0
  int64_t plane, rows;            // halves per part, per stored row pair
  int pair0, last;                // first halo row pair, last stored one

  __device__ __forceinline__ Slab(const View& v, int x0, int y0, int d0)
      : base(v.V + (int64_t)(2 * (d0 >> 4)) * v.plane + 32 * x0), plane(v.plane),
        rows(32 * (int64_t)v.pitch), pair0((y0 >> 1) - (R >> 1)),
        last((v.H - 1 + (R & 1)) >> 1) {}

  __device__ __forceinline__ void copy(int m, float* buf, int wave, int lane) const {
    const int k = wave + kWaves * m;
    if (k < G::NWC) {
      const int pr = k >= G::HY ? 1 : 0, h = k - pr * G::HY;
      int gp = pair0 + (h >> 1);
      gp = gp < 0 ? 0 : (gp > last ? last : gp);
      const uint16_t* src = base + pr * plane + gp * rows + (h & 1) * (G::NQH * 64);
      if (G::NQH == 8 || lane < G::NQH * 8)
        __builtin_amdgcn_global_load_lds((BILM_GLOBAL void*)(src + 8 * lane),
                                         (BILM_LOCAL void*)(buf + k * (G::NQH * 32)), 16, 0, 0);
    }
  }
  // every copy of this wave
  __device__ __forceinline__ void all(float* buf, int wave, int lane) const {
#pragma unroll
    for (int m = 0; m < G::KPW; ++m) copy(m, buf, wave, lane);
  }
};

// Guide of a tile's halo: the raw values are loaded into registers
// (unconditionally, clamped addresses) and turned into the scaled guide
// (sqrt(kr2) g, kFar outside the image) only when stored to LDS.  A value
// used right after its load waits at once, and that wait also covers the
// slab copies in flight; this way the loads of the next tile's guide overlap
// the last pass's products.
template <int R, typename GT>
struct GuideRaw {
  GT raw[HGeom<R>::GPT];
};

template <int R, typename GT>
__device__ __forceinline__ void guide_load(const View& v, int x0, int y0, GuideRaw<R, GT>& g) {
  using G = HGeom<R>;
  const GT* __restrict__ src = static_cast<const GT*>(v.guide);
#pragma unroll
  for (int k = 0; k < G::GPT; ++k) {
    const int i = threadIdx.x + k * kThreads;
    const int yy = i / G::HXP, xx = i % G::HXP;
    const int cy = min(max(y0 - R + yy, 0), v.H - 1), cx = min(max(x0 - R + xx, 0), v.W - 1);
    g.raw[k] = src[(int64_t)cy * v.g_pitch + cx];
  }
}

__device__ __forceinline__ float guide_value(uint8_t raw, unsigned z) {
  return (float)((unsigned)raw ^ z);
}
__device__ __forceinline__ float guide_value(float raw, unsigned z) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, raw) ^ z);
}

// (v, x0, y0): the tile the guide was loaded for
template <int R, typename GT>
__device__ __forceinline__ void guide_store(float* gs, const GuideRaw<R, GT>& g, const View& v,
                                            int x0, int y0) {
  using G = HGeom<R>;
  // an opaque zero: the conversion cannot move up into the load's branch
  unsigned z = 0u;
  asm volatile("" : "+s"(z));
  const float kr = sqrtf(v.kr2);
#pragma unroll
  for (int k = 0; k < G::GPT; ++k) {
    const int i = threadIdx.x + k * kThreads;
    const int yy = i / G::HXP, xx = i % G::HXP;
    const int gy = y0 - R + yy, gx = x0 - R + xx;
    const bool in = xx < kTW + 2 * R && gy >= 0 && gy < v.H && gx >= 0 && gx < v.W;
    if (i < G::GUIDE) gs[guide_pos<R>(yy, xx)] = in ? guide_value(g.raw[k], z) * kr : kFar;
  }
}

// x = hi + lo in FP16 (round to nearest); lo is the rounding of the
// remainder x - hi, which is exact in FP32 and formed by one mixed-precision
// FMA per value (the FP16 hi read from its half of the packed register).
// Written out so that each pair is packed where it is formed: left to the
// compiler, the FP32 remainders of a whole tile's weights stay live until
// the end of the weight loop and spill.
__device__ __forceinline__ void split8(const float (&w)[8], u4& hi, u4& lo) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    unsigned hb, lb;
    float r0, r1;
    asm volatile("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(hb) : "v"(w[2 * j]), "v"(w[2 * j + 1]));
    asm volatile("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]"
                 : "=v"(r0) : "v"(hb), "v"(w[2 * j]));
    asm volatile("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
                 : "=v"(r1) : "v"(hb), "v"(w[2 * j + 1]));
    asm volatile("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(lb) : "v"(r0), "v"(r1));
    hi[j] = hb;
    lo[j] = lb;
  }
}

// v of another lane of the wave (index taken modulo 64).
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(
                                       4 * lane, __builtin_bit_cast(int, v)));
}

}  // namespace bilh
}  // namespace stereo
