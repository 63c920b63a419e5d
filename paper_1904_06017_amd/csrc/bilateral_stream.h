// Bilateral cost aggregation, Eqs. (10)-(11), fused with winner-take-all
// selection and sub-pixel refinement (Sec. 3.2.2, Eq. 13) or the soft-argmin
// head, on the matrix cores with FP16 operands split in two: the products of
// bilateral_mfma16.h (same operands, same order, so the same bits), streamed
// down strips of the image.
//
// A workgroup owns a strip of kTW = 16 columns and walks down it one 4-row
// block row per phase.  The cost volume's row pairs pass through a ring in
// LDS, all NB level blocks (16 levels each) of a pair together, so each row
// pair of the halo is copied once per strip instead of once per tile, and a
// block's sums over all its levels form at the same time in NB accumulators.
// The K loop of a block (its window union, NI products of 32 positions) runs
// from top to bottom over S phases; the S groups of four waves (one wave per
// 4x4 block across the strip) hold S consecutive block rows, one phase apart,
// so that all of them read the same few row pairs at any time.  In every
// phase a wave forms the weights of its next NI / S products and multiplies
// them right away with the NB level blocks: weights (vector ALU), operand
// reads (LDS) and products (matrix cores) overlap in every wave and across
// the waves of a SIMD, and no weight is kept for longer than its product.
//
// What bounds it: per block row and SIMD (D = 64, R = 7) about 2400 cycles of
// products, 2400 of weights on the vector ALU and 2600 of LDS reads.  Products
// and vector ALU work overlap only in part on a SIMD (48 products of four waves
// take 870 cycles alone, with 192 FMAs 1320, with 48 exponentials 890), so 4000
// to 4300 cycles are the floor of a phase; it takes 5400.  The form before (a
// tile's weights kept in registers over passes of one level block each, every
// wave in the same phase between barriers) spent 10200 cycles on the first
// pass of a tile, vector ALU only, and 3600 on each other, matrix cores and
// LDS only.  Both volumes, kernel trace of 60 calls each, medians: 1280x720, R =
// 7, D = 64 0.498 -> 0.388 ms, D = 128 0.792 -> 0.727 ms; 640x480, R = 5, D = 48
// 0.116 -> 0.088 ms.
#pragma once
#include "bilateral_mfma16.h"

namespace stereo {
namespace bils {

using bil::BilPair;
using bilh::f4;
using bilh::h8;
using bilh::HGeom;
using bilh::kFar;
using bilh::kLog2WScale;
using bilh::kTW;
using bilh::lane_value;
using bilh::u4;
using bilh::View;

constexpr int kMaxNB = 4;               // level blocks per sweep

// Pass 2 of the backward reads C' = dE / W_p, whose range is that of the
// caller's gradient map: one pixel's may be 1e10 of another's.  FP16 parts
// share one scale over the image, so a value x keeps 2^-39 of the largest, and
// what lies 2^-39 below it is lost (a smooth map at R = 7: 6e-8 relative beside
// its like, 8e-5 at 1e-4 of the largest, nothing at 1e-10).  From R = kWideR on
// C' and the weights are split into three BF16 numbers instead, x = a + b + c
// (24 bits at FP32's range, as the FP32 form keeps), and the product takes the
// six terms down to 2^-24: aa, ab, ba, ac, bb, ca.  Three times the operand
// bytes of one part leave room for kMaxWide level blocks.  317x243, D = 40, R =
// 7: pass 2 takes 53 us (39 us on FP16 parts, 196 us on the vector ALU).
// A product over a block's union also meets values outside a pixel's own
// window, with weight 0, and 0 x infinity is NaN: so at these radii non-finite
// values stay out of the operands (C' 0, guide far off), and the pixels whose
// own window holds one are made NaN at the end.  Such a pixel has a non-finite
// aP; pass 1 raises a flag where it meets one, without which nothing is looked up.
constexpr int kMaxWide = 3;
constexpr float kMaxFloat = 3.402823466e38f;
constexpr int parts_of(int mode) { return mode == 5 ? 3 : 2; }
constexpr int max_blocks(int R, int mode, int duo) {
  return mode == 5 ? kMaxWide : duo && R > 2 ? kDuoBlocks : kMaxNB;
}
// Workgroups that share a CU.  A phase waits for the copies that it issues,
// about 1 us; at small radii its products do not fill that time, so there two
// workgroups of two groups each share a CU and one computes while the other
// waits (DUO: radii 1 and 2, and launches that duo_launch takes).  Match at
// 1280x720: R = 1, 16 levels 182 -> 134 us; R = 2, 64 levels 348 -> 279 us.
constexpr int held(int duo) { return duo ? 2 : 1; }

// Products of the S states of a block and the row pairs they read, relative
// to the block's first: state k takes products [ps(k), ps(k + 1)).  In phase
// t state k works on block row t - k, so it reads pairs lo(k) - 2 k .. hi(k) -
// 2 k relative to pair 2 t.
template <int R, int DUO>
struct Sched {
  using G = HGeom<R>;
  static constexpr int S = G::NI >= 4 && !DUO ? 4 : 2;
  // The group in state 0 also selects the levels of its last block: it gets
  // one product less than an even share where that leaves it one.
  static constexpr int ps(int k) {
    return k == 0 ? 0 : k == S ? G::NI : (G::NI / S > 1 || G::NI % S ? -1 : 0) +
           k * (G::NI / S) + (k < G::NI % S ? k : G::NI % S);
  }
  static constexpr int lo(int k) { return 4 * ps(k) / G::NCQ; }
  static constexpr int hi(int k) {
    return (4 * ps(k + 1) < G::NP ? 4 * ps(k + 1) - 1 : G::NP - 1) / G::NCQ;
  }
  static constexpr int wlo() {
    int m = 0;
    for (int k = 0; k < S; ++k) m = lo(k) - 2 * k < m ? lo(k) - 2 * k : m;
    return m;
  }
  static constexpr int whi() {
    int m = 0;
    for (int k = 0; k < S; ++k) m = hi(k) - 2 * k > m ? hi(k) - 2 * k : m;
    return m;
  }
};

// MODE 1: winner-take-all, 2: soft-argmin, 3 / 4: pass 1 / 2 of its backward,
// 5: pass 2 on BF16 parts (R >= kWideR).
template <int R, int NB, int MODE, int DUO>
struct SGeom {
  using G = HGeom<R>;
  using C = Sched<R, DUO>;
  static constexpr int S = C::S;
  static constexpr int kWaves = 4 * S, kThreads = 64 * kWaves;
  static constexpr int WLO = C::wlo(), WHI = C::whi();
  static constexpr int NSLOT = WHI - WLO + 1 + 2;        // pairs of a phase + the next two
  static constexpr int CHB = G::NQH * 256;               // bytes: a pair of one block and part
  static constexpr int PARTS = parts_of(MODE);
  static constexpr int SLOTB = NB * PARTS * CHB;
  // guide ring: a block's own pixels lie below the pairs of its first state
  static constexpr int GHI = WHI > (R + 3) / 2 ? WHI : (R + 3) / 2;
  static constexpr int NGS = GHI - WLO + 1 + 2;
  static constexpr int GSB = G::NQH * 32;                // bytes: a pair of the guide
  static constexpr int NGV = 2 * 2 * G::HXP;             // guide values of two pairs
  static constexpr int NCP = 4 * PARTS * NB;             // wave copies of two pairs
  static constexpr int KPW = (NCP + kWaves - 1) / kWaves;
  // Scratch of the group that finishes a block row.  MODE 1: a row of levels
  // per pixel; 3: C' of the block row, [level][4 rows][16 columns] dwords with
  // the level stride that spreads a write over the banks, two by phase; 4, 5:
  // the costs at its pixels, [wave][level][16 pixels], two by block row.
  static constexpr int EROW = 64 * NB + 16;
  static constexpr int CLEV = 65;                        // dwords per level (MODE 3)
  static constexpr int CBLK = 16 * NB * CLEV * 4;        // bytes of one of the two
  static constexpr int PBLK = 4 * NB * 1024;
  static constexpr int SCRATCH =
      MODE == 1 ? 64 * EROW : MODE == 3 ? 2 * CBLK : MODE >= 4 ? 2 * PBLK : 0;
  static constexpr size_t lds_bytes = (size_t)NSLOT * SLOTB + (size_t)NGS * GSB +
                                      sizeof(float) * G::STAB + SCRATCH;
  static_assert(held(DUO) * lds_bytes <= 160 * 1024, "LDS budget");
  static_assert((PARTS * NB - 1) * CHB < 65536, "operand offsets must fit a DS immediate");
  static_assert(NGV <= kThreads, "one guide value per thread");
};

// LDS of a launch, laid out for the most blocks whatever a sweep takes: ring,
// guide ring, spatial terms, scratch.
template <int R, int MODE, int DUO>
struct Lds {
  using Z = SGeom<R, max_blocks(R, MODE, DUO), MODE, DUO>;
  static constexpr int gring = Z::NSLOT * Z::SLOTB;
  static constexpr int tab = gring + Z::NGS * Z::GSB;
  static constexpr int scratch = tab + (int)sizeof(float) * HGeom<R>::STAB;
  static constexpr size_t bytes = Z::lds_bytes;
};

// A per-pair launch: the volumes of a pair (reference, then target), each cut
// into strips and each strip into nseg segments of len block rows.  A queued
// launch: n segments of many volumes, dealt one per workgroup and round.
struct Args {
  View v[2];
  int nvol, nseg, len, tx, br;
  int banded;                           // 1: XCD x owns a band of strips
  const BilPair* descs;
  const Seg* segs;
  int n;
};

// A backward pass (v[0] of Args: the split input volume, v.D = levels of the
// level tile, and the FP32 guide).  Six products per operand pair instead of
// three (twelve on BF16 parts): the weights, and the weights times the guide
// difference.  1280x720, D = 48, R = 5: pass 1 398 -> 270 us, pass 2 292 us
// either way (tiles of 32x16 pixels, their weights kept in registers, before).
struct Back {
  float* out;                           // pass 2: dC planar [D][H][W]
  uint16_t* h2out;                      // pass 1: C' S, split volume (as v): FP16 parts,
                                        // R >= kWideR the first two BF16 parts
  uint16_t* h3out;                      //   and the third, [block] planes of v.plane
  const uint16_t* h3;                   // pass 2 at R >= kWideR: that third part
  const float* cpix;                    // pass 2: C planar [D][H][W]
  const unsigned* gmax;                 // max |g'| over the image (float bits): the scale S
  unsigned* bad;                        // R >= kWideR: nonzero where some aP is not finite
  const float *sm_m, *sm_logZ, *sm_dh, *gD;
  float *aP, *A1, *A2, *Wp;             // Wp nullable
  float invT, one_minus_c1;
  int d_first;                          // level of the tile's first slice
  int d_all;                            // levels of the whole range (the bound on |d - dh|)
};

// Power-of-two scale that puts a bound m on |C'| in [2^13, 2^14) (bits: m
// as a float): FP16 keeps its range for every value up to the bound.  BF16 parts
// have FP32's range: the bound goes to 2^96, where window sums stay below
// overflow and the parts of values 2^-200 below it above underflow.
template <int R>
__device__ inline float cprime_scale(unsigned bits) {
  const int ex = (int)((bits >> 23) & 0xFF);
  if constexpr (R >= kWideR) {                        // ex = 255: a bound past FP32, < 2^160
    const int k = 96 - (ex == 0xFF ? 160 : ex - 126);
    return ldexpf(1.0f, k > 100 ? 100 : k);
  }
  if (ex == 0xFF || bits == 0) return 1.0f;          // non-finite or zero: no scaling
  int e = ex - 126;                                   // max = f 2^e, f in [0.5, 1)
  if (e < -80) e = -80;
  const int k = 14 - e;                               // scale 2^k, |k| <= 114
  return ldexpf(1.0f, k);
}

// x = hi + lo in FP16 (round to nearest) for a pair of values: lo rounds the
// remainder x - hi, which is exact in FP32.  Not inline assembly: the matrix
// cores read the results, and the compiler has to see that hazard.  m1 = -1,
// opaque, keeps the remainder one mixed-precision FMA.
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split_pair(float a, float b, float m1, unsigned& hi, unsigned& lo) {
  const h2 h = __builtin_convertvector((f2{a, b}), h2);
  const f2 r = {fmaf((float)h[0], m1, a), fmaf((float)h[1], m1, b)};
  hi = __builtin_bit_cast(unsigned, h);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector(r, h2));
}

// x = p[0] + p[1] + p[2] in BF16 (round to nearest, exact remainders) for a pair
// of values.
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ void split_wide(float x, float y, unsigned (&p)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    p[k] = __builtin_bit_cast(unsigned, __builtin_convertvector((f2{x, y}), b2));
    x -= __builtin_bit_cast(float, p[k] << 16);
    y -= __builtin_bit_cast(float, p[k] & 0xFFFF0000u);
  }
}

// value of lane q of this lane's row of 16
template <int Q>
__device__ __forceinline__ float row_value(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
      0, __builtin_bit_cast(int, v), 0x150 + Q /* row_newbcast */, 0xF, 0xF, true));
}

__device__ __forceinline__ int lane_int(int v, int lane) {
  return __builtin_amdgcn_ds_bpermute(4 * lane, v);
}

// the smallest of three, a NaN giving way to a number (one instruction; fminf
// would quiet every operand first)
__device__ __forceinline__ float min3(float a, float b, float c) {
  float r;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Priority of a wave with r products of the phase still to do: the waves of a
// SIMD then end a phase together instead of the oldest first and the youngest
// alone.
__device__ __forceinline__ void priority(int r) {
  if (r >= 3) __builtin_amdgcn_s_setprio(3);
  else if (r == 2) __builtin_amdgcn_s_setprio(2);
  else if (r == 1) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

template <int K>
struct Int {
  static constexpr int value = K;
};

template <int R, int MODE, int DUO, int NB>
struct Worker {
  using G = HGeom<R>;
  using C = Sched<R, DUO>;
  using Z = SGeom<R, NB, MODE, DUO>;
  using L = Lds<R, MODE, DUO>;
  static constexpr int S = C::S;
  static constexpr bool TWO = MODE >= 3;             // the second weight w (G(p) - G(q))

  char* ring;
  char* gring;
  char* scratch;
  const float* tab;
  int lane, wave, group, bx, li, lk;

  __device__ __forceinline__ explicit Worker(float* lds)
      : ring(reinterpret_cast<char*>(lds)), gring(ring + L::gring), scratch(ring + L::scratch),
        tab(reinterpret_cast<const float*>(ring + L::tab)) {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    group = wave >> 2;
    bx = wave & 3;
    li = lane & 15;
    lk = lane >> 4;
  }

  __device__ __forceinline__ int wrap(int s, int n) const { return s < 0 ? s + n : s >= n ? s - n : s; }

  // Block rows [b0, b0 + len) of the strip at column x0, levels [16 q0, 16
  // (q0 + NB)) of the volume's nblk level blocks.  first / last: the first /
  // last sweep of the strip's levels; between sweeps the selection state of a
  // pixel is kept in v.state.
  __device__ __forceinline__ void sweep(const View& v, const Back& bk, int x0, int b0, int len,
                                        int q0, int nblk) {
    const bool first = q0 == 0, last = q0 + NB >= nblk;
    const int pair0 = 2 * b0 - (R >> 1);             // stored pair of ring pair 0
    const int plast = (v.H - 1 + (R & 1)) >> 1;
    const uint32_t rows = 32u * (uint32_t)v.pitch;    // halves per row pair
    // this wave's copies of two row pairs: copy c = half c & 1 of part (c >> 1)
    // % PARTS of block (c / (2 PARTS)) % NB of pair c / (2 PARTS NB)
    constexpr int PARTS = Z::PARTS;
    const uint16_t* csrc[Z::KPW];
    int cdst[Z::KPW], cpair[Z::KPW];
#pragma unroll
    for (int m = 0; m < Z::KPW; ++m) {
      const int c = wave + Z::kWaves * m;
      cpair[m] = c >= 2 * PARTS * NB ? 1 : 0;
      const int w = c - cpair[m] * 2 * PARTS * NB, q = w / (2 * PARTS), half = w & 1;
      const int part = (w >> 1) - PARTS * q;
      const int blk = q0 + q;
      csrc[m] = (PARTS == 2 || part < 2 ? v.V + (int64_t)(2 * blk + part) * v.plane
                                        : bk.h3 + blk * v.plane) +
                32 * x0 + half * (G::NQH * 64);
      cdst[m] = (PARTS * q + part) * Z::CHB + half * (Z::CHB / 2);
    }
    // ring pairs j, j + 1 (j + 1 <= jmax) into their slots; slot: of pair j
    const int jmax = 2 * (len - 1) + G::NRP - 1;
    auto copy_pairs = [&](int j, int slot, char* __restrict__ wr) {
#pragma unroll
      for (int m = 0; m < Z::KPW; ++m) {
        const int pj = j + cpair[m];
        if (wave + Z::kWaves * m < Z::NCP && pj <= jmax) {
          int gp = pair0 + pj;
          gp = gp < 0 ? 0 : (gp > plast ? plast : gp);
          const int sl = wrap(slot + cpair[m], Z::NSLOT);
          const uint16_t* src = csrc[m] + (uint64_t)(uint32_t)gp * rows;
          if (G::NQH == 8 || lane < G::NQH * 8)
            __builtin_amdgcn_global_load_lds((BILM_GLOBAL void*)(src + 8 * lane),
                                             (BILM_LOCAL void*)(wr + sl * Z::SLOTB + cdst[m]),
                                             16, 0, 0);
        }
      }
    };
    // one value of guide pairs j, j + 1 per thread: raw, then scaled into LDS.
    // The thread's place is worked out at each use: kept, it would cost
    // registers of the products, and a spilled register's reload waits for
    // every copy in flight.
    const bool gw = wave < (Z::NGV + 63) / 64;       // waves that load guide values
    const float kr = sqrtf(v.kr2);
    auto guide_place = [&](int& gpr, int& grow, int& gcol) {
      int gi = threadIdx.x;
      asm volatile("" : "+v"(gi));
      gpr = gi / (2 * G::HXP);
      const int rem = gi - gpr * (2 * G::HXP);
      grow = rem / G::HXP;
      gcol = rem - grow * G::HXP;
      return gi < Z::NGV;
    };
    auto guide_raw = [&](int j) -> unsigned {
      int gpr, grow, gcol;
      guide_place(gpr, grow, gcol);
      const int y = 4 * b0 - R + 2 * (j + gpr) + grow, x = x0 - R + gcol;
      const int64_t o = (int64_t)min(max(y, 0), v.H - 1) * v.g_pitch + min(max(x, 0), v.W - 1);
      return v.g_u8 ? (unsigned)static_cast<const uint8_t*>(v.guide)[o]
                    : static_cast<const unsigned*>(v.guide)[o];
    };
    auto guide_put = [&](int j, int slot, unsigned raw) {
      int gpr, grow, gcol;
      const bool mine = guide_place(gpr, grow, gcol);
      const int y = 4 * b0 - R + 2 * (j + gpr) + grow, x = x0 - R + gcol;
      const float f = v.g_u8 ? (float)raw : __builtin_bit_cast(float, raw);
      const bool in = gcol < kTW + 2 * R && y >= 0 && y < v.H && x >= 0 && x < v.W;
      const int sl = wrap(slot + gpr, Z::NGS);
      const float fs = f * kr;
      const bool use = MODE == 5 ? in && fabsf(fs) <= kMaxFloat : in;
      if (mine)
        *reinterpret_cast<float*>(gring + sl * Z::GSB + (gcol >> 2) * 32 + grow * 16 +
                                  (gcol & 3) * 4) = use ? fs : kFar;
    };

    // the pairs of phase 0
#pragma unroll
    for (int j = 0; j <= Z::WHI; j += 2) copy_pairs(j, j, ring);
#pragma unroll
    for (int j = 0; j <= Z::GHI; j += 2)
      if (gw) guide_put(j, j, guide_raw(j));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    f4 acc[NB][2];
#pragma unroll
    for (int q = 0; q < NB; ++q) acc[q][0] = acc[q][1] = f4{0.f, 0.f, 0.f, 0.f};
    float Gp = 0.f, wsum = 0.f;
    // lane parts of the operand and guide addresses (patch column lk)
    const int olane = (bx + lk) * 256 + 16 * li, olane0 = bx * 256 + 16 * li;
    const int glane = (bx + lk) * 32 + 4 * (li & 7), glane0 = bx * 32 + 4 * (li & 7);

    // Selection state of the sweep before (E, E-, E+, E of the last level; its
    // level), read one phase ahead: at its use it would wait behind the copies.
    float4 st = make_float4(3.402823466e38f, 0.f, 0.f, 0.f);
    int stD = 0;
    // Backward: the scales and, of pass 1, -(m + log Z), g' and dh at the pixel
    // (st.x, st.y, st.z), of pass 2 the copies of its costs into the scratch.
    const float kr_inv = 1.0f / kr;
    float cscale = 1.0f;
    bool any_bad = false;
    if constexpr (MODE == 5) any_bad = __builtin_amdgcn_readfirstlane((int)*bk.bad) != 0;
    if constexpr (TWO)
      cscale = cprime_scale<R>(__builtin_bit_cast(
          unsigned, __builtin_bit_cast(float, *bk.gmax) * fabsf(bk.one_minus_c1) * bk.invT *
                        (float)(bk.d_all > 1 ? bk.d_all - 1 : 1)));
    auto fetch_state = [&](int b, char* __restrict__ swr) {
      int ln = lane;
      asm volatile("" : "+v"(ln));
      const int py = 4 * (b0 + b) + ((ln >> 2) & 3), px = x0 + 4 * bx + (ln & 3);
      const int64_t pix = py < v.H && px < v.W ? (int64_t)py * v.W + px : 0;
      if constexpr (MODE == 3) {
        st.x = -(bk.sm_m[pix] + bk.sm_logZ[pix]);
        st.y = bk.gD[pix] * (bk.one_minus_c1 * -bk.invT);
        st.z = bk.sm_dh[pix];
      } else if constexpr (MODE >= 4) {
        // copy c: 4 levels (lane >> 4) of the wave's 16 pixels (lane & 15)
        char* const dst = swr + (b & 1) * Z::PBLK + bx * NB * 1024;
#pragma unroll
        for (int c = 0; c < 4 * NB; ++c) {
          int d = 16 * q0 + 4 * c + (ln >> 4);
          d = d < v.D ? d : v.D - 1;
          __builtin_amdgcn_global_load_lds(
              (BILM_GLOBAL void*)(bk.cpix + (int64_t)d * v.H * v.W + pix),
              (BILM_LOCAL void*)(dst + 256 * c), 4, 0, 0);
        }
      } else if (MODE == 1) {
        st = v.state[pix];
        stD = v.dint[pix];
      } else {
        st = v.state[4 * pix + (ln >> 4)];
      }
    };
    // Selection over the block's levels: the lane holds E of pixel li at
    // levels 16 (q0 + q) + 4 lk .. + 3 in acc[q].
    auto finish = [&](int b, const char* __restrict__ srd) {
      int ln = lane;
      asm volatile("" : "+v"(ln));                  // worked out here, not kept live
      const int lk = ln >> 4, pr = (ln >> 2) & 3, pc = ln & 3, lane = ln;
      const int py = 4 * (b0 + b) + pr, px = x0 + 4 * bx + pc;
      const bool in = py < v.H && px < v.W;
      const int64_t pix = in ? (int64_t)py * v.W + px : 0;
      if constexpr (TWO) {
        // lane: levels 16 (q0 + q) + 4 lk + j of pixel li, acc[q][0] = sum w B,
        // acc[q][1] = sum w (G'(p) - G'(q)) B, both with the weights' 2^12
        float ca = 0.0f, cb = 0.0f;
        if constexpr (MODE == 3) {
          float ws = wsum;                             // W_p 2^12
          ws += __shfl_xor(ws, 16);
          ws += __shfl_xor(ws, 32);
          const float rinv = 1.0f / ws, oscale = (rinv * 4096.0f) * cscale;
          unsigned* const blk = reinterpret_cast<unsigned*>(scratch + (b & 1) * Z::CBLK) +
                                16 * pr + 4 * bx + pc;
#pragma unroll
          for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int d = 16 * q + 4 * lk + j;
              const float ev = acc[q][0][j] * rinv;
              const float Pd = __builtin_amdgcn_exp2f(fmaf(-ev, bk.invT, st.x) * 1.4426950408889634f);
              const float dE = in && d < v.D ? st.y * Pd * ((float)(bk.d_first + d) - st.z) : 0.0f;
              ca = fmaf(dE, ev, ca);
              cb = fmaf(dE, acc[q][1][j], cb);
              const float o = dE * oscale;             // S dE / W_p
              if constexpr (R >= kWideR) {             // split when it leaves
                blk[d * Z::CLEV] = __builtin_bit_cast(unsigned, fabsf(o) <= kMaxFloat ? o : 0.0f);
                continue;
              }
              const _Float16 hi = (_Float16)o, lo = (_Float16)(o - (float)hi);
              blk[d * Z::CLEV] = (unsigned)__builtin_bit_cast(uint16_t, hi) |
                                 ((unsigned)__builtin_bit_cast(uint16_t, lo) << 16);
            }
          ca += lane_value(ca, lane ^ 16);
          ca += lane_value(ca, lane ^ 32);
          cb += lane_value(cb, lane ^ 16);
          cb += lane_value(cb, lane ^ 32);
          // one lane per pixel adds this launch's sum (atomic adds without a
          // return value: no wait; one add per pixel and launch, so the order
          // is fixed)
          if (lk == 0 && in) {
            atomicAdd(bk.aP + pix, ca);
            atomicAdd(bk.A1 + pix, cb * (kr_inv / 4096.0f));
            if (bk.Wp) bk.Wp[pix] = ws * (1.0f / 4096.0f);
            if (R >= kWideR && !(fabsf(ca) <= kMaxFloat)) *bk.bad = 1u;
          }
        } else {
          float unscale = 1.0f / (4096.0f * cscale);
          if (any_bad) {                               // uniform; lane lk: every fourth row
            int hit = 0;
            for (int y = max(py - R, 0) + lk; y <= min(py + R, v.H - 1); y += 4)
              for (int x = max(px - R, 0); x <= min(px + R, v.W - 1); ++x)
                hit |= !(fabsf(bk.aP[(int64_t)y * v.W + x]) <= kMaxFloat);
            hit |= __shfl_xor(hit, 16);
            hit |= __shfl_xor(hit, 32);
            if (hit) unscale = __builtin_nanf("");
          }
          const float* const cp = reinterpret_cast<const float*>(srd + (b & 1) * Z::PBLK + bx * NB * 1024) +
                                  (ln & 15);
#pragma unroll
          for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const int dq = 16 * q + 4 * lk + j, d = 16 * q0 + dq;
              cb = fmaf(in && d < v.D ? cp[16 * dq] : 0.0f, acc[q][1][j], cb);
              if (in && d < v.D) bk.out[((int64_t)d * v.H + py) * v.W + px] = acc[q][0][j] * unscale;
            }
          cb += lane_value(cb, lane ^ 16);
          cb += lane_value(cb, lane ^ 32);
          if (lk == 0 && in) atomicAdd(bk.A2 + pix, -cb * unscale * kr_inv);
        }
        return;
      }
      f4 e[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) e[q] = acc[q][0] + acc[q][1];
      if constexpr (MODE == 1) {
        // the pixel's levels into the wave's scratch row, for the two around
        // the minimum
        char* const row = scratch + (bx * 16 + li) * Z::EROW;
#pragma unroll
        for (int q = 0; q < NB; ++q)
          *reinterpret_cast<f4*>(row + 64 * q + 16 * lk) = e[q];
        if (v.D < 16 * (q0 + NB)) {                    // uniform: levels past the range
#pragma unroll
          for (int q = 0; q < NB; ++q) {
            const int nvl = v.D - 16 * (q0 + q) - 4 * lk;
#pragma unroll
            for (int j = 0; j < 4; ++j) e[q][j] = nvl > j ? e[q][j] : __builtin_inff();
          }
        }
        float m = 3.402823466e38f;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          m = min3(m, e[q][0], e[q][1]);
          m = min3(m, e[q][2], e[q][3]);
        }
        m = min3(m, m, lane_value(m, lane ^ 16));
        m = min3(m, m, lane_value(m, lane ^ 32));
        // its first level: of the lane's, then of the pixel's four lanes
        int first_at = 16 * NB;
#pragma unroll
        for (int q = NB - 1; q >= 0; --q)
#pragma unroll
          for (int j = 3; j >= 0; --j) first_at = e[q][j] == m ? 16 * q + j : first_at;
        first_at += first_at < 16 * NB ? 4 * lk : 0;
        first_at = min(first_at, lane_int(first_at, lane ^ 16));
        first_at = min(first_at, lane_int(first_at, lane ^ 32));
        first_at = first_at < 16 * NB ? first_at : 0;  // no level below the largest float
        float bestE = m;
        int bestD = 16 * q0 + first_at;
        float Em = first_at > 0 ? *reinterpret_cast<const float*>(row + 4 * max(first_at - 1, 0)) : st.w;
        float Ep = *reinterpret_cast<const float*>(row + 4 * min(first_at + 1, 16 * NB - 1));
        if (!first) {
          // a minimum at the last level of the sweep before takes its upper
          // neighbour from this one
          if (stD == 16 * q0 - 1) st.z = *reinterpret_cast<const float*>(row);
          if (!(bestE < st.x)) {
            bestE = st.x; bestD = stD; Em = st.y; Ep = st.z;
          }
        }
        if (!last) {
          const float top = *reinterpret_cast<const float*>(row + 64 * NB - 4);
          if (lk == 0 && in) {
            v.state[pix] = make_float4(bestE, Em, Ep, top);
            v.dint[pix] = (int16_t)bestD;
          }
        } else if (lk == 0 && in) {
          v.dint[pix] = (int16_t)bestD;
          if (v.dsub) {
            float off = 0.0f;
            if (bestD > 0 && bestD < v.D - 1) {
              const float den = 2.0f * Em + 2.0f * Ep - 4.0f * bestE;
              if (den > 0.0f) off = (Em - Ep) / den;
            }
            v.dsub[pix] = (float)bestD + off;
          }
        }
      } else {
        // soft-argmin: each lane keeps (max, Z, S) of its quarter of every
        // block's levels; the four lanes of a pixel merge at the end
        constexpr float kNeg = -3.402823466e38f;
        float mr = kNeg, Zr = 0.0f, Sr = 0.0f, rinvP;
        if (first) {
          float ws = wsum;                             // W_p: the pixel's weights
          ws += __shfl_xor(ws, 16);
          ws += __shfl_xor(ws, 32);
          rinvP = 1.0f / ws;
        } else {
          mr = st.x; Zr = st.y; Sr = st.z; rinvP = st.w;
        }
        const float zscale = -v.invT * 1.4426950408889634f;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          const int dq = 16 * (q0 + q) + 4 * lk;
          const int nvl = v.D - dq;
          if (16 * (q0 + q) >= v.D) break;             // uniform
          float zv[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) zv[j] = nvl > j ? e[q][j] * rinvP * zscale : kNeg;
          const float M = fmaxf(mr, fmaxf(fmaxf(zv[0], zv[1]), fmaxf(zv[2], zv[3])));
          const float a = __builtin_amdgcn_exp2f(mr - M);
          Zr *= a;
          Sr *= a;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float ez = nvl > j ? __builtin_amdgcn_exp2f(zv[j] - M) : 0.0f;
            Zr += ez;
            Sr = fmaf((float)(dq + j), ez, Sr);
          }
          mr = M;
        }
        if (!last) {
          if (in) v.state[4 * pix + lk] = make_float4(mr, Zr, Sr, rinvP);
          return;
        }
        auto merge = [&](float om, float oZ, float oS) {
          const float M = fmaxf(mr, om);
          const float a = __builtin_amdgcn_exp2f(mr - M), c = __builtin_amdgcn_exp2f(om - M);
          Zr = fmaf(Zr, a, oZ * c);
          Sr = fmaf(Sr, a, oS * c);
          mr = M;
        };
        merge(lane_value(mr, lane ^ 16), lane_value(Zr, lane ^ 16), lane_value(Sr, lane ^ 16));
        merge(lane_value(mr, lane ^ 32), lane_value(Zr, lane ^ 32), lane_value(Sr, lane ^ 32));
        if (lk == 0 && in) {
          const float ln2 = 0.6931471805599453f;
          const float dh = Sr / Zr;
          v.sm_m[pix] = mr * ln2;
          v.sm_logZ[pix] = __builtin_amdgcn_logf(Zr) * ln2;
          v.sm_dh[pix] = dh;
          const double dd = dh;
          v.disp[pix] = (float)(dd - v.delta_p + (v.c0 + v.c1 * ((double)px - dd + v.delta_p) +
                                                  v.c2 * (double)py));
        }
      }
    };

    // Pass 1: C' of block row b, left in the scratch by the phase before, out to
    // the split volume by the group that formed it.  A chunk is the 4 columns
    // of a level of a stored row, 8 bytes of each half; 32 lanes write a quad's
    // 256 bytes.  The strip's 16 columns start R & 3 into a stored quad and a
    // block row R & 1 into a pair: chunks shared with a neighbour go out value
    // by value.
    auto flush = [&](int b) {
      constexpr int e = R & 1, QO = R & 3;
      constexpr int NPR = 2 + e, NQ = (kTW + QO + 3) / 4;
      const unsigned* const blk = reinterpret_cast<const unsigned*>(scratch + (b & 1) * Z::CBLK);
      int c = bx * 64 + lane;
      asm volatile("" : "+v"(c));
      const int l = (c >> 1) & 15, par = c & 1;
#pragma unroll 1
      for (int u = c >> 5; u < NPR * NQ * NB; u += 8) {
        const int q = u / (NPR * NQ), rem = u - q * (NPR * NQ);
        const int prn = rem / NQ, qd = rem - prn * NQ;
        const int row = 2 * prn + par - e, c0 = 4 * qd - QO;
        if (row < 0 || row > 3 || 4 * (b0 + b) + row >= v.H) continue;
        const unsigned* src = blk + (16 * q + l) * Z::CLEV + 16 * row;
        const int64_t o = (int64_t)(2 * q) * v.plane + (int64_t)(2 * (b0 + b) + prn) * rows +
                          128 * (((x0 + R) >> 2) + qd) + 8 * l + 4 * par;
        const bool whole = c0 >= 0 && c0 + 3 < kTW && x0 + c0 + 3 < v.W;
        if constexpr (R >= kWideR) {
          float f[4];
#pragma unroll
          for (int k = 0; k < 4; ++k)
            f[k] = __builtin_bit_cast(float, src[min(max(c0 + k, 0), kTW - 1)]);
          unsigned p01[3], p23[3];
          split_wide(f[0], f[1], p01);
          split_wide(f[2], f[3], p23);
#pragma unroll
          for (int part = 0; part < 3; ++part) {
            uint16_t* const to = part < 2 ? bk.h2out + o + part * v.plane
                                          : bk.h3out + o - (int64_t)q * v.plane;
            if (whole) *reinterpret_cast<uint2*>(to) = make_uint2(p01[part], p23[part]);
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (!whole && c0 + k >= 0 && c0 + k < kTW && x0 + c0 + k < v.W)
                to[k] = (uint16_t)((k < 2 ? p01 : p23)[part] >> (16 * (k & 1)));
          }
        } else if (whole) {
          const unsigned w0 = src[c0], w1 = src[c0 + 1], w2 = src[c0 + 2], w3 = src[c0 + 3];
          *reinterpret_cast<uint2*>(bk.h2out + o) =
              make_uint2((w0 & 0xFFFFu) | (w1 << 16), (w2 & 0xFFFFu) | (w3 << 16));
          *reinterpret_cast<uint2*>(bk.h2out + o + v.plane) =
              make_uint2((w0 >> 16) | (w1 & 0xFFFF0000u), (w2 >> 16) | (w3 & 0xFFFF0000u));
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (c0 + k < 0 || c0 + k >= kTW || x0 + c0 + k >= v.W) continue;
            const unsigned w = src[c0 + k];
            bk.h2out[o + k] = (uint16_t)w;
            bk.h2out[o + v.plane + k] = (uint16_t)(w >> 16);
          }
        }
      }
    };

    float m1 = -1.0f;
    asm volatile("" : "+s"(m1));
    int base = 0, gbase = 0;                          // ring slots of pair 2 t
    // State k of a block in the current phase: its products.
    auto products = [&](auto kc, const char* __restrict__ rd, const char* __restrict__ grd,
                        const float* __restrict__ tb) {
      constexpr int k = decltype(kc)::value;
      if constexpr (k == 0) {
        wsum = 0.f;
        // the guide at the lane's own pixel
        const int hr = (li >> 2) + R, hc = 4 * bx + (li & 3) + R;
        const int s0 = wrap(gbase + (R >> 1), Z::NGS);
        int sl = s0 + (hr >> 1) - (R >> 1);
        sl = sl >= Z::NGS ? sl - Z::NGS : sl;
        Gp = *reinterpret_cast<const float*>(grd + sl * Z::GSB + (hc >> 2) * 32 + (hr & 1) * 16 +
                                             (hc & 3) * 4);
      }
#pragma unroll
      for (int i = C::ps(k); i < C::ps(k + 1); ++i) {
        priority(C::ps(k + 1) - 1 - i);
        // patch 4 i + lk lies in pair r0 (lanes lk < thr) or r0 + 1, at column
        // lk + (4 i - NCQ pair)
        const int r0 = 4 * i / G::NCQ, thr = G::NCQ * (r0 + 1) - 4 * i;
        const int a0 = 4 * i - G::NCQ * r0, a1 = a0 - G::NCQ;
        const int rel = r0 - 2 * k;
        const int so = wrap(base + rel, Z::NSLOT) * Z::SLOTB;
        const int go = wrap(gbase + rel, Z::NGS) * Z::GSB;
        int oa = so + 256 * a0 + olane, ga = go + 32 * a0 + glane;
        if (thr < 4) {
          if (4 * i + 3 < G::NP) {
            const int so1 = wrap(base + rel + 1, Z::NSLOT) * Z::SLOTB;
            const int go1 = wrap(gbase + rel + 1, Z::NGS) * Z::GSB;
            oa = lk < thr ? oa : so1 + 256 * a1 + olane;
            ga = lk < thr ? ga : go1 + 32 * a1 + glane;
          } else if (4 * i + thr < G::NP) {
            const int so1 = wrap(base + rel + 1, Z::NSLOT) * Z::SLOTB;
            const int go1 = wrap(gbase + rel + 1, Z::NGS) * Z::GSB;
            oa = lk < thr ? oa : lk < G::NP - 4 * i ? so1 + 256 * a1 + olane : so + olane0;
            ga = lk < thr ? ga : lk < G::NP - 4 * i ? go1 + 32 * a1 + glane : go + glane0;
          }
        }
        if (4 * i + 3 >= G::NP && !(thr < 4 && 4 * i + thr < G::NP)) {
          // padding patches (zero weights) read the pair's first column
          oa = lk < G::NP - 4 * i ? oa : so + olane0;
          ga = lk < G::NP - 4 * i ? ga : go + glane0;
        }
        // weights of the product: 8 slots of the lane's patch
        const float gl = *reinterpret_cast<const float*>(grd + ga);
        const float4 s0 = *reinterpret_cast<const float4*>(tb + (i * 64 + lane) * 8);
        const float4 s1 = *reinterpret_cast<const float4*>(tb + (i * 64 + lane) * 8 + 4);
        const float g[8] = {row_value<0>(gl) - Gp, row_value<1>(gl) - Gp, row_value<2>(gl) - Gp,
                            row_value<3>(gl) - Gp, row_value<4>(gl) - Gp, row_value<5>(gl) - Gp,
                            row_value<6>(gl) - Gp, row_value<7>(gl) - Gp};
        const float sv[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
        float w[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = __builtin_amdgcn_exp2f(fmaf(-g[q], g[q], sv[q]));
        if constexpr (MODE == 5) {
          u4 wp[3], gp[3];                             // parts of w, w (G'(p) - G'(q))
#pragma unroll
          for (int j = 0; j < 4; ++j) {                // g = G'(q) - G'(p)
            unsigned pw[3], pg[3];
            split_wide(w[2 * j], w[2 * j + 1], pw);
            split_wide(-g[2 * j] * w[2 * j], -g[2 * j + 1] * w[2 * j + 1], pg);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              wp[k][j] = pw[k];
              gp[k][j] = pg[k];
            }
          }
#pragma unroll
          for (int q = 0; q < NB; ++q) {
            b8 b[3];
#pragma unroll
            for (int k = 0; k < 3; ++k)
              b[k] = __builtin_bit_cast(b8, *reinterpret_cast<const u4*>(rd + oa + (3 * q + k) * Z::CHB));
            f4 cw = i < 1 ? f4{0.f, 0.f, 0.f, 0.f} : acc[q][0];
            f4 cg = i < 1 ? f4{0.f, 0.f, 0.f, 0.f} : acc[q][1];
#pragma unroll
            for (int n = 2; n >= 0; --n)               // parts whose order is n, small ones first
#pragma unroll
              for (int k = 0; k <= n; ++k) {
                cw = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[k], __builtin_bit_cast(b8, wp[n - k]), cw, 0, 0, 0);
                cg = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[k], __builtin_bit_cast(b8, gp[n - k]), cg, 0, 0, 0);
              }
            acc[q][0] = cw;
            acc[q][1] = cg;
            __builtin_amdgcn_sched_barrier(0);
          }
          continue;
        }
        u4 hi, lo;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          unsigned hb, lb;
          split_pair(w[2 * j], w[2 * j + 1], m1, hb, lb);
          hi[j] = hb;
          lo[j] = lb;
        }
        const h8 aH = __builtin_bit_cast(h8, hi), aL = __builtin_bit_cast(h8, lo);
        if constexpr (MODE == 2 || MODE == 3) {
          // hi + lo as one mixed-precision FMA: two conversions and an addition
          // take 152 against 140 us (soft-argmin, 1280x720, D = 48, R = 5)
#pragma unroll
          for (int q = 0; q < 8; ++q) wsum += fmaf((float)aH[q], -m1, (float)aL[q]);
        }
        u4 ghi, glo;
        if constexpr (TWO) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {                // g = G'(q) - G'(p)
            unsigned hb, lb;
            split_pair(-g[2 * j] * w[2 * j], -g[2 * j + 1] * w[2 * j + 1], m1, hb, lb);
            ghi[j] = hb;
            glo[j] = lb;
          }
        }
        const h8 cH = __builtin_bit_cast(h8, ghi), cL = __builtin_bit_cast(h8, glo);
#pragma unroll
        for (int q = 0; q < NB; ++q) {
          const u4 bh = *reinterpret_cast<const u4*>(rd + oa + 2 * q * Z::CHB);
          const u4 bl = *reinterpret_cast<const u4*>(rd + oa + (2 * q + 1) * Z::CHB);
          const h8 bH = __builtin_bit_cast(h8, bh), bL = __builtin_bit_cast(h8, bl);
          if constexpr (TWO) {
            f4 cw = i < 1 ? f4{0.f, 0.f, 0.f, 0.f} : acc[q][0];
            f4 cg = i < 1 ? f4{0.f, 0.f, 0.f, 0.f} : acc[q][1];
            cw = __builtin_amdgcn_mfma_f32_16x16x32_f16(bH, aH, cw, 0, 0, 0);
            cg = __builtin_amdgcn_mfma_f32_16x16x32_f16(bH, cH, cg, 0, 0, 0);
            cw = __builtin_amdgcn_mfma_f32_16x16x32_f16(bL, aH, cw, 0, 0, 0);
            cg = __builtin_amdgcn_mfma_f32_16x16x32_f16(bL, cH, cg, 0, 0, 0);
            acc[q][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bH, aL, cw, 0, 0, 0);
            acc[q][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bH, cL, cg, 0, 0, 0);
            // keeps the operand reads of later blocks out of the registers
            if (q & 1) __builtin_amdgcn_sched_barrier(0);
            continue;
          }
          f4 c = i < 2 ? f4{0.f, 0.f, 0.f, 0.f} : acc[q][i & 1];
          // costs as the first operand: the result has a pixel per lane column
          // and four consecutive levels per lane
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(bH, aH, c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(bL, aH, c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(bH, aL, c, 0, 0, 0);
          acc[q][i & 1] = c;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    // Phase t: block row t enters, the groups hold block rows t - k in state
    // k; the copies of the next two pairs are in flight meanwhile.  A block's
    // selection runs at the start of the phase after its last products, so
    // that its stores have a phase to complete.
    int k = group == 0 ? 0 : S - group;               // state of this wave's group
    // The copies fill slots that no wave reads in the phase; as __restrict__
    // parameters the compiler knows that and does not wait for them before
    // the phase's first LDS read.
    auto phase = [&](int t, char* __restrict__ wr, const char* __restrict__ rd,
                     const char* __restrict__ grd, const float* __restrict__ tb,
                     char* __restrict__ swr, const char* __restrict__ srd) {
      const int b = t - k;                            // block row of this wave
      const int js = wrap(base + Z::WHI + 1, Z::NSLOT), gs = wrap(gbase + Z::GHI + 1, Z::NGS);
      copy_pairs(2 * t + Z::WHI + 1, js, wr);
      unsigned raw = 0;
      if (gw) raw = guide_raw(2 * t + Z::GHI + 1);
      if ((TWO || !first) && k == S - 1 && b >= 0 && b < len) fetch_state(b, swr);
      if (MODE == 3 && k == 1 && b >= S) flush(b - S);
      if (k == 0 && b >= S && b - S < len) {
        priority(3);
        finish(b - S, srd);
      }
      if (b >= 0 && b < len) {
        if (k == 0) products(Int<0>{}, rd, grd, tb);
        else if (k == 1) products(Int<1>{}, rd, grd, tb);
        else if constexpr (S > 2) {
          if (k == 2) products(Int<2>{}, rd, grd, tb);
          else products(Int<3>{}, rd, grd, tb);
        }
      }
      if (gw) guide_put(2 * t + Z::GHI + 1, gs, raw);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    };
    // the last block row's C' leaves one phase after its selection
    for (int t = 0; t < len + S + (MODE == 3 ? 1 : 0); ++t) {
      phase(t, ring, ring, gring, tab, scratch, scratch);
      base = wrap(base + 2, Z::NSLOT);
      gbase = wrap(gbase + 2, Z::NGS);
      k = k + 1 == S ? 0 : k + 1;
    }
  }
};

// Spatial terms of every lane's slots, 12 - |p - q|^2 log2(e) / sigma_s^2, -inf
// outside the pixel's window and for padding patches.
template <int R, int DUO>
__device__ __forceinline__ void spatial_table(float* t, float ks2) {
  using G = HGeom<R>;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int e = wave; e < G::NI * 8; e += 4 * Sched<R, DUO>::S) {
    const int i = e >> 3, s = e & 7;
    const int p = 4 * i + lk, rp = p / G::NCQ, cq = p - rp * G::NCQ;
    const int ty = 2 * rp + (s >> 2) - (li >> 2) - R, tx = 4 * cq + (s & 3) - (li & 3) - R;
    const bool in = p < G::NP && ty >= -R && ty <= R && tx >= -R && tx <= R;
    t[(i * 64 + lane) * 8 + s] =
        in ? fmaf(-(float)(ty * ty + tx * tx), ks2, kLog2WScale) : -__builtin_inff();
  }
}

// Every sweep of one segment.
template <int R, int MODE, int DUO>
__device__ __forceinline__ void segment(const View& v, const Back& bk, int x0, int b0, int len,
                                        float* lds) {
  const int nblk = (v.D + 15) / 16;
  for (int q0 = 0, nb = 0; q0 < nblk; q0 += nb) {
    constexpr int most = max_blocks(R, MODE, DUO);
    nb = sweep_blocks(nblk - q0, most);
    // the state a sweep leaves is read by the next one in the same wave (block
    // rows and lanes keep their waves): program order is enough.  A fence of
    // the whole device here cost 56 us a segment.
    if (most == 4 && nb == 4) Worker<R, MODE, DUO, most>(lds).sweep(v, bk, x0, b0, len, q0, nblk);
    else if (nb == 3) Worker<R, MODE, DUO, 3>(lds).sweep(v, bk, x0, b0, len, q0, nblk);
    else if (nb == 2) Worker<R, MODE, DUO, 2>(lds).sweep(v, bk, x0, b0, len, q0, nblk);
    else Worker<R, MODE, DUO, 1>(lds).sweep(v, bk, x0, b0, len, q0, nblk);
  }
}

template <int R, int MODE, int QUEUE, int DUO>
__global__ void __launch_bounds__((256 * Sched<R, DUO>::S), (held(DUO) * Sched<R, DUO>::S))
agg_stream_kernel(Args a, Back bk) {
  extern __shared__ float lds[];
  float* tab = lds + Lds<R, MODE, DUO>::tab / 4;
  if constexpr (QUEUE) {
    // round k of G workgroups covers entries [k G, (k + 1) G); workgroup b (XCD
    // b % 8) takes entry k G + (b % 8) G / 8 + b / 8, so that each XCD works on
    // a contiguous run of the list (neighbouring strips, longest first)
    const int G = (int)gridDim.x, b = (int)blockIdx.x;
    const int at = G % 8 == 0 ? (b % 8) * (G / 8) + b / 8 : b;
    float ks2 = __builtin_nanf("");
    for (int s = at; s < a.n; s += G) {
      const Seg e = a.segs[s];
      const View v = bilh::view_of(a.descs[e.desc]);
      // the pairs of a launch may differ in sigma_s; the last sweep's final
      // barrier is behind every read of the table, a sweep's first one ahead
      if (v.ks2 != ks2) {
        ks2 = v.ks2;
        spatial_table<R, DUO>(tab, ks2);
      }
      segment<R, MODE, DUO>(v, bk, e.x0, e.b0, e.len, lds);
    }
  } else {
    spatial_table<R, DUO>(tab, a.v[0].ks2);
    // banded: XCD x = b % 8 owns a band of strips; its workgroups run adjacent
    // strips of one vertical range at a time, whose shared halo columns meet
    // in its L2
    int c0 = 0, bc = a.tx, me = blockIdx.x, step = gridDim.x;
    if (a.banded) {
      const int bw = (a.tx + 7) / 8;
      c0 = (blockIdx.x % 8) * bw;
      bc = a.tx - c0 < bw ? (a.tx - c0 > 0 ? a.tx - c0 : 0) : bw;
      me = blockIdx.x / 8;
      step = gridDim.x / 8;
    }
    const int per = bc * a.nseg, n = a.nvol * per;
    for (int s = me; s < n; s += step) {
      const int vol = s >= per ? 1 : 0, rem = s - vol * per;
      const int seg = rem / bc, strip = c0 + rem - seg * bc;
      const int b0 = seg * a.len;
      const int len = min(a.len, a.br - b0);
      if (len > 0) segment<R, MODE, DUO>(a.v[vol], bk, strip * kTW, b0, len, lds);   // uniform
    }
  }
}

template <int R, int MODE, int QUEUE, int DUO>
hipError_t set_lds_attr() {
  static bool done = false;
  if (!done) {
    hipError_t e = hipFuncSetAttribute((const void*)agg_stream_kernel<R, MODE, QUEUE, DUO>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)Lds<R, MODE, DUO>::bytes);
    if (e != hipSuccess) return e;
    done = true;
  }
  return hipSuccess;
}

// Cut of nvol volumes of tx strips x br block rows over cus workgroups.  A
// segment costs its block rows plus the phases in which its groups fill and
// drain and its first row pairs arrive (S + 2); the cut with the smallest
// number of rounds x segment cost is taken, banded over the XCDs (strips that
// share halo columns on one L2) unless that costs more than 8 % (few strips).
// At 1280x720 both volumes of 80 strips take 3 segments a strip, 60 of an
// XCD's 32 workgroups' two rounds.
inline void cut_strips(int tx, int br, int nvol, int S, int cus, int& nseg, int& banded) {
  double best[2] = {1e30, 1e30};
  int at[2] = {1, 1};
  for (int k = 1; k <= br && k <= 64; ++k) {
    const int len = (br + k - 1) / k;
    if (k > 1 && len == (br + k - 2) / (k - 1)) continue;       // no shorter than with k - 1
    for (int b = 0; b < 2; ++b) {
      if (b && (cus % 8 || cus < 8)) continue;
      const long items = (long)nvol * (b ? (tx + 7) / 8 : tx) * k, w = b ? cus / 8 : cus;
      const double cost = (double)((items + w - 1) / w) * (len + S + 2);
      if (cost < best[b]) { best[b] = cost; at[b] = k; }
    }
  }
  banded = best[1] <= 1.08 * best[0] ? 1 : 0;
  nseg = at[banded];
}

// One or two volumes of a pair (the same size, radius and sigmas).
template <int R, int MODE, int DUO>
hipError_t launch_pair(const BilPair* p, int nvol, hipStream_t s, const Back& bk = Back{}) {
  Args a{};
  for (int k = 0; k < nvol; ++k) {
    const BilPair& b = p[k];
    if (!b.h2 || b.h2_pitch < bilh::h2_pitch_for<R>(b.W) || (b.h2_pitch & 7) ||
        b.h2_plane < 16 * (int64_t)h2_rows(R, b.H) * b.h2_pitch || b.W != p[0].W ||
        b.H != p[0].H || b.D != p[0].D || (MODE <= 2 && b.D > 16 * max_blocks(R, MODE, DUO) && !b.state))
      return hipErrorInvalidValue;
    a.v[k] = bilh::view_of(b);
  }
  hipError_t e = set_lds_attr<R, MODE, 0, DUO>();
  if (e != hipSuccess) return e;
  const int cus = held(DUO) * device_cus();            // workgroups at a time
  a.nvol = nvol;
  a.tx = (p[0].W + kTW - 1) / kTW;
  a.br = (p[0].H + 3) / 4;
  cut_strips(a.tx, a.br, nvol, Sched<R, DUO>::S, cus, a.nseg, a.banded);
  a.len = (a.br + a.nseg - 1) / a.nseg;
  const int grid = a.banded ? cus : std::min(cus, nvol * a.tx * a.nseg);
  hipLaunchKernelGGL((agg_stream_kernel<R, MODE, 0, DUO>), dim3(grid), dim3(256 * Sched<R, DUO>::S),
                     (Lds<R, MODE, DUO>::bytes), s, a, bk);
  return hipGetLastError();
}

template <int R>
hipError_t launch_args(const Plan& P, const BilArgs* a, int nvol, int mode, hipStream_t s) {
  if (nvol < 1 || nvol > 2 || (mode != 1 && mode != 2)) return hipErrorInvalidValue;
  BilPair p[2];
  for (int k = 0; k < nvol; ++k) p[k] = bil::make_pair(P, a[k]);
  if constexpr (R <= kDuoR) {
    const long rows = (long)nvol * ((P.W + kTW - 1) / kTW) * ((P.H + 3) / 4);
    if (R <= 2 || duo_launch((p[0].D + 15) / 16, rows, device_cus()))
      return mode == 2 ? launch_pair<R, 2, 1>(p, nvol, s) : launch_pair<R, 1, 1>(p, nvol, s);
  }
  if constexpr (R > 2)
    return mode == 2 ? launch_pair<R, 2, 0>(p, nvol, s) : launch_pair<R, 1, 0>(p, nvol, s);
  return hipErrorInvalidValue;
}

// Pass 1 or 2 of the backward for one level tile (at most 64 levels, float
// guide).
template <int R>
hipError_t launch_back(const Plan& P, const BilArgs& a, int pass, hipStream_t s) {
  const BilPair p = bil::make_pair(P, a);
  if (p.D > 16 * kMaxNB || p.g_u8 || !a.gmax || (pass == 1 && !a.h2_out) ||
      (pass == 2 && (!a.cpix || !a.E)) ||
      (R >= kWideR && (pass == 1 ? !a.h3_out : !a.h3)))
    return hipErrorInvalidValue;
  Back b{};
  b.out = a.E;
  b.h2out = a.h2_out;
  b.h3out = a.h3_out;
  b.h3 = a.h3;
  b.cpix = a.cpix;
  b.gmax = a.gmax;
  b.bad = a.gmax + 1;
  b.sm_m = a.sm_m;
  b.sm_logZ = a.sm_logZ;
  b.sm_dh = a.sm_dh;
  b.gD = a.gD;
  b.aP = a.aP;
  b.A1 = a.A1;
  b.A2 = a.A2;
  b.Wp = a.Wp;
  b.invT = p.o.invT;
  b.one_minus_c1 = p.o.one_minus_c1;
  b.d_first = a.d_first;
  b.d_all = P.D;
  return pass == 1 ? launch_pair<R, 3, 0>(&p, 1, s, b)
                   : launch_pair<R, (R >= kWideR ? 5 : 4), 0>(&p, 1, s, b);
}

// n segments over many volumes (descs, segs: device arrays).
template <int R, int DUO>
hipError_t launch_queue(const BilPair* descs, const Seg* segs, int n, hipStream_t s) {
  hipError_t e = set_lds_attr<R, 1, 1, DUO>();
  if (e != hipSuccess) return e;
  Args a{};
  a.descs = descs;
  a.segs = segs;
  a.n = n;
  const int grid = std::max(1, std::min(n, held(DUO) * device_cus()));
  hipLaunchKernelGGL((agg_stream_kernel<R, 1, 1, DUO>), dim3(grid), dim3(256 * Sched<R, DUO>::S),
                     (Lds<R, 1, DUO>::bytes), s, a, Back{});
  return hipGetLastError();
}

// duo: every volume of the list is one that duo_launch takes.
template <int R>
hipError_t launch_queue_r(const BilPair* descs, const Seg* segs, int n, int duo, hipStream_t s) {
  if constexpr (R <= 2) return launch_queue<R, 1>(descs, segs, n, s);
  else if constexpr (R <= kDuoR)
    return duo ? launch_queue<R, 1>(descs, segs, n, s) : launch_queue<R, 0>(descs, segs, n, s);
  else return launch_queue<R, 0>(descs, segs, n, s);
}

}  // namespace bils
}  // namespace stereo
