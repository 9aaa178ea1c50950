// hot_tiles.hip -- both passes as complex contractions on the FP16 matrix cores, at FP32 accuracy.
//
// Eq. 2 separates per trap: Delta_rev = (g U^2 + a U) + (g V^2 + b V), so
//   e^{i 2pi Delta_j^m} = X_m(c) Y_m(r),  X_m(c) = e^{i 2pi (g U_c^2 + a U_c)},  Y_m(r) = e^{i 2pi (g V_r^2 + b V_r)},
// and with the trap weights c_m = w_m e^{i theta_m}
//   pixel pass (Eq. 3)  S[r][c] = sum_m (c_m Y_m(r)) X_m(c),          phi = arg S
//   trap pass (Eq. 1)   T[r][m] = sum_c e^{i phi[r][c]} conj X_m(c),  V_m = (1/N) sum_r conj Y_m(r) T[r][m].
// The direct sums (k_iter, k_backward, k_forward) pay one sine and cosine per (pixel, trap) and pass; here
// a block computes 16 (rows + columns) of them per 16 traps for its tile of pixels, and the (pixel, trap)
// work is matrix products.
//
// Precision.  v_mfma_f32_16x16x32_f16 multiplies halves exactly and accumulates in FP32 at 16 times the
// rate of the FP32 products (16 cycles for 16 x 16 x 32 against 32 for 16 x 16 x 4).  Every real factor v
// (|v| <= 1) is carried as hi = f16(v), lo = f16(v - hi), which leaves |v - hi - lo| <= 2^-24, the
// rounding of an FP32 value just below 1, and a product is hi hi + hi lo + lo hi (the dropped lo lo is
// below 2^-24): three half products for one FP32 product.  (The adjoint scales by the larger component of
// G, so a factor there reaches sqrt 2, and both bounds above 1 are 2^-23.)  Measured against 64 bits over
// grids of 48 to 2048 pixels a side and 3 to 1000 traps, fields and gradients are as close as with FP32
// matrix products (2.3e-7 against 3.3e-7 relative for the adjoint of 8 x 512^2 x 64) and closer than the
// direct sums (7.2e-7), whose per-term arguments reach several revolutions.  The weights are scaled by a
// power of two so that the largest is below 1: a weight keeps an error of 2^-25 of the largest however
// small it is itself, while an FP32 sum rounds by as much at each of its terms.  Weights and G spread over
// 0 to 12 decades (512^2 x 100): masks 5.7e-7 .. 9.4e-7 rad rms from 64 bits at every spread (direct sums
// 1.7e-6 .. 4.8e-6, FP32 matrix products 6.9e-7 .. 1.3e-6), V within 2.1e-7 (2.6e-7, 2.0e-7), gradients
// 2.4e-7 .. 3.1e-7 relative (5.0e-7 .. 9.2e-7, 3.5e-7 .. 4.0e-7).  All the rest (arguments, sine and
// cosine, normalisation, trap sums) is FP32 or FP64 as in the other kernels.
//
// MFMA 16x16x32 operands: lane l = i + 16 g holds A[i][8 g ..+7] and B[8 g ..+7][i]; result D[i][j] is in
// lane j + 16 (i / 4), register i % 4.  Eight halves are four complex entries (re, im), so a product
// covers 16 traps (pixel pass) or 16 columns (trap pass):
//   pixel pass  Re S = (xr, xi) . (wr, -wi), Im S = (xr, xi) . (wi, wr): the second operand is the first
//               with its halves turned, in registers.  Columns are i, rows j, so a lane ends with four
//               consecutive pixels of one row.
//   epilogue    E = S / |S|, and the phase where it is wanted (a solve's last mask)
//   trap pass   Re T = (Er, Ei) . (xr, xi), Im T = (Ei, -Er) . (xr, xi), the lane's four E values being
//               its eight halves of the operand; T is folded over its 16 rows with conj Y in FP32 and the
//               lane groups are summed.
//
// What bounds it.  One iteration of 1024^2 x 256 is 8.6 GFLOP of products (5.1 us at the rate of the
// halves) and 17 to 19 us per launch (k_wide), against 108 us of the direct sums; 512^2 x 100 takes 6.9 us
// (15.4).  On the larger grid it is vector work beside the products (k_wide), on the smaller latency: 1.2 us
// from one launch to the next, 1.2 us until the first coefficients are there, 1 us more for V and the
// update, and after them phases of a few hundred instructions per wave at two waves per SIMD.
#include "hot_device.h"

#include <algorithm>

namespace hot {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma32(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, a), __builtin_bit_cast(half8v, b), c, 0, 0, 0);
}

// x + i y as two packed pairs of halves: hi = f16(x), f16(y), and lo = f16 of what hi leaves, each in
// one rounding from the very bits of hi (|x - hi - lo| <= 2^-24 for |x| <= 1).
struct Split {
  unsigned hi, lo;
};
__device__ __forceinline__ Split split(float x, float y) {
  const half2v h = {(_Float16)x, (_Float16)y};
  Split s;
  s.hi = __builtin_bit_cast(unsigned, h);
  asm("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixhi_f16 %0, %1, -1.0, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
      : "=&v"(s.lo)
      : "v"(s.hi), "v"(x), "v"(y));
  return s;
}
// ... of x - i y
__device__ __forceinline__ Split split_conj(float x, float y) {
  const half2v h = {(_Float16)x, (_Float16)(-y)};
  Split s;
  s.hi = __builtin_bit_cast(unsigned, h);
  asm("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]\n\t"
      "v_fma_mixhi_f16 %0, %1, -1.0, -%3 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
      : "=&v"(s.lo)
      : "v"(s.hi), "v"(x), "v"(y));
  return s;
}
// (a, b) -> (-b, a) and (a, b) -> (b, -a), halves of a word (exact)
__device__ __forceinline__ unsigned turn_p(unsigned v) {
  unsigned r;
  asm("v_pk_mul_f16 %0, %1, 1.0 op_sel:[1,0] op_sel_hi:[0,0] neg_lo:[1,0]" : "=v"(r) : "v"(v));
  return r;
}
__device__ __forceinline__ unsigned turn_m(unsigned v) {
  unsigned r;
  asm("v_pk_mul_f16 %0, %1, 1.0 op_sel:[1,0] op_sel_hi:[0,0] neg_hi:[1,0]" : "=v"(r) : "v"(v));
  return r;
}

// Two tiles' partial sums (re, im) of the four lane groups, summed over the groups: lane group 0
// gets tile a's re, group 1 tile b's re, group 2 tile a's im, group 3 tile b's im.  Each sum is
// (p0 + p2) + (p1 + p3) of the groups' partials.
__device__ __forceinline__ float2 swap32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  const unsigned x = r[0], y = r[1];  // (a bit_cast of the vector's element itself would read element 0)
  return make_float2(__builtin_bit_cast(float, x), __builtin_bit_cast(float, y));
}
__device__ __forceinline__ float2 swap16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
  const unsigned x = r[0], y = r[1];  // (a bit_cast of the vector's element itself would read element 0)
  return make_float2(__builtin_bit_cast(float, x), __builtin_bit_cast(float, y));
}
__device__ __forceinline__ float sum_groups(float2 a, float2 b) {
  const float2 p = swap32(a.x, a.y), q = swap32(b.x, b.y);
  const float2 r = swap16(p.x + p.y, q.x + q.y);
  return r.x + r.y;
}

// Between words of LDS that a wave's lanes write and other lanes of the same wave read: the wave's accesses
// are carried out in program order, and this keeps the compiler to it.  No instruction of its own.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A fragment of a table: 16 rows or columns x 16 traps of complex entries, each a word of two halves
// (re, im).  Entry (i, t) of the hi part is word 4 i + 132 (t / 4) + t % 4, of the lo part 64 words
// further: a lane's four consecutive traps are one 16-byte read (matrix operand with the traps as
// k), a lane's four consecutive i of one trap are four words 4 apart (matrix operand with i as k),
// and with 132 words per group of four traps both kinds of access reach every bank evenly.
constexpr int kFragWords = kTileFragWords;
constexpr int kTqWords = 132, kLoWords = 64;

// A caller's phase in revolutions, reduced in FP64 to the nearest turn: as in the tables' constants, arguments
// within half a turn of 0 round half as far as those of 0 .. 1.
__device__ __forceinline__ float phase_turn(float ph) {
  const double t = (double)ph * 0.15915494309189533577;  // 1 / (2 pi)
  return (float)(t - __builtin_rint(t));
}

// e^{i 2pi t} with the library's sine and cosine (the hardware's are about 5e-8 rms off).  Eq. 1 by itself
// takes E with it: three factors carry three such errors where the direct sum's term carries one, and V of
// 8 x 512^2 x 64 was 1.05e-7 off 64 bits (direct sums 9.9e-8); with E from here 7.7e-8.  The column table too
// gives 5.3e-8, but costs 1.5 us of 5.9 (trap pass of 512^2 x 100) and 3.6 of 14.7 (1024^2 x 256); E costs
// 0.5 of 10.6 us (8 x 512^2 x 64) and nothing that a call shows.
__device__ __forceinline__ float2 unit_turn(float t) {
  float s, c;
  sincospif(2.0f * t, &s, &c);
  return make_float2(c, s);
}

// E = e^{i phase_of(S)}: S / |S|, 1 where S = 0 or NaN (their phase is 0), 0 outside the grid.  After an
// infinite weight (`inf`) S is NaN and so is E.  A finite S is a sum of products of halves, multiples of
// 2^-48, over weights scaled to at most 1: |S|^2 neither underflows nor overflows.
__device__ __forceinline__ void unit_of(float x, float y, bool in, bool inf, float& er, float& ei) {
  const float n2 = __builtin_fmaf(x, x, y * y);
  const float inv = __builtin_amdgcn_rsqf(n2);
  const bool some = n2 > 0.0f || inf;
  er = in ? (some ? x * inv : 1.0f) : 0.0f;
  ei = in && some ? y * inv : 0.0f;
}

// sum over the lane's four rows of conj(y) t
__device__ __forceinline__ float2 fold_rows(const float2 (&y)[4], const f32x4& tre, const f32x4& tim) {
  float pr[2], pi[2];  // over rows (0, 1) and (2, 3)
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const float2 a = y[2 * h], c = y[2 * h + 1];
    const float tr0 = tre[2 * h], ti0 = tim[2 * h], tr1 = tre[2 * h + 1], ti1 = tim[2 * h + 1];
    pr[h] = __builtin_fmaf(c.x, tr1, __builtin_fmaf(c.y, ti1, __builtin_fmaf(a.x, tr0, a.y * ti0)));
    pi[h] = __builtin_fmaf(c.x, ti1, __builtin_fmaf(-c.y, tr1, __builtin_fmaf(a.x, ti0, -a.y * tr0)));
  }
  return make_float2(pr[0] + pr[1], pi[0] + pi[1]);
}

// The state and (MODE 0) V's words of trap threadIdx.x, loaded by the constructor and used by
// weights(): the accumulators were rewritten by the previous launch and come from beyond the L2, so the
// tables are built while these loads are in flight.
template <int NT, int MODE>
struct TrapInputs {
  static constexpr int NW = NT / 64;
  VAcc vacc;
  int off, M;
  TrapState s_first = {0.0f, 0.0f, 0.0f, 0.0f};
  unsigned long long w_first[kAccRegions] = {};
  __device__ __forceinline__ TrapInputs(const TrapState* st_in, const unsigned long long* acc_in, int T, int off_,
                                        int M_, float unscale)
      : vacc{acc_in, T, off_, unscale}, off(off_), M(M_) {
    const int tm = min((int)threadIdx.x, M - 1);
    if (MODE != 1 && MODE != 3 && __builtin_amdgcn_readfirstlane((int)threadIdx.x & ~63) < M) {
      s_first = st_in[off + tm];
      if (MODE == 0) vacc.load(tm, w_first);  // (acc_in is valid even when upd == 0)
    }
  }
  // c_m of all traps into cw [Mp] (after the GS/GSW update where upd asks for it; the lead block also
  // writes the new state and keeps V in hist); returns the exponent that scales the largest below 1.
  // `inf` tells of an infinite weight (and no NaN among them): a pair of halves cannot carry it (its low
  // half is NaN), so S is NaN where the direct sums leave it infinite and its phase NaN.  Ends with a
  // barrier; sh: 2 NW floats.
  __device__ __forceinline__ int weights(float2* cw, float* sh, int Mp, const TrapState* st_in, const float* vin,
                                         int upd, bool lead, TrapState* st_out, float2* hist, int* flag,
                                         bool& inf) const {
    const int wave = threadIdx.x >> 6;
    unsigned top = 0u;  // bits of the largest magnitude: in the order of the magnitudes, infinity and NaN above all
    auto take = [&](float w) { top = max(top, __builtin_bit_cast(unsigned, w) & 0x7fffffffu); };
    for (int m = M + (int)threadIdx.x; m < Mp; m += NT) cw[m] = make_float2(0.0f, 0.0f);
    if (MODE == 3) {
      for (int m = threadIdx.x; m < M; m += NT) {
        const float2 gm = make_float2(vin[2 * (off + m)], vin[2 * (off + m) + 1]);
        cw[m] = gm;
        take(gm.x);
        take(gm.y);
      }
    } else if (MODE == 2 || upd == 0) {
      for (int m = threadIdx.x; m < M; m += NT) {
        const TrapState s = m == (int)threadIdx.x ? s_first : st_in[off + m];
        cw[m] = trap_weight(s);
        take(s.w);
      }
    } else {
      unsigned long long w8[kAccRegions];
#pragma unroll
      for (int q = 0; q < kAccRegions; ++q) {
        w8[q] = w_first[q];
        asm volatile("" : "+v"(w8[q]));  // (the sum stays here)
      }
      const float2 v_first = vacc.sum(w8);
      if (lead && hist != nullptr) {
        if ((int)threadIdx.x < M) hist[off + threadIdx.x] = v_first;
        for (int m = NT + (int)threadIdx.x; m < M; m += NT) hist[off + m] = vacc(m);
      }
      auto emit = [&](int m, const TrapState& st) {
        if (lead) st_out[off + m] = st;
        cw[m] = trap_weight(st);
        take(st.w);
      };
      update_traps<NT, VAcc, decltype(emit), true>(vacc, st_in, off, M, upd, sh, nullptr, lead ? flag : nullptr, emit,
                                                   v_first, s_first);
    }
    top = wave_max_bits(top);
    unsigned* tops = reinterpret_cast<unsigned*>(sh + NW);
    if ((threadIdx.x & 63) == 0) tops[wave] = top;
    __syncthreads();
    top = tops[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) top = max(top, tops[w]);
    inf = __builtin_amdgcn_readfirstlane((int)top) == 0x7f800000;
    return __builtin_amdgcn_readfirstlane(__builtin_amdgcn_frexp_expf(__builtin_bit_cast(float, top)));
  }
};

// MODE 0: one iteration: GS/GSW update (upd 1 / 2, recomputed by every block from the previous mask's
//   fixed-point sums acc_in; 0: st_in as is), pixel pass, trap pass; the phase is written when not null.
//   Each trap's block sum is added to acc_out's region of the wave's XCD, block (0, 0, b) writes
//   hologram b's new state and clears its part of acc_zero, as in k_iter.  The figures of merit are not
//   taken here: that block leaves V in `hist` (when not null) and k_finish works on several masks at a
//   time (computed by one block before its pixel pass they held back the whole launch: 512^2 x 100 9.5
//   against 8.7 us).
// MODE 1: trap pass alone from the given phase (Eq. 1): per-block partials
// MODE 2: pixel pass alone from the given state (phase out)
// MODE 3: adjoint of Eq. 1: weights G_m (vin), grad[j] = (1/N) Im(e^{-i phi_j} S_j) for the given phase
//
// Grid (ceil(nx / 16 CW), ceil(ny / 16 RT), B), RT CW KH waves: wave (rt, cwv, part) has row tile rt,
// column tile cwv and share `part` of the trap tiles of each super-chunk (mc traps);
// the KH partial pixel sums of a tile meet in LDS and are added in a fixed order.  The waves build the
// tables together: a wave always has the same column tile tx and row tile ty, whose group constants
// (the phase about the tile's centre column or row, formed in FP64 and rounded once; K, slope, curvature)
// it forms for itself, so no barrier stands between them and the entries.  Columns past nx and rows past
// ny get the formula's values and pixels with E = 0; traps past M repeat trap M - 1 with weight 0.
// Dynamic LDS: tile_lds_bytes.
template <int RT, int CW, int KH, int MODE>
__global__ void __launch_bounds__(RT * CW * KH * 64, 2)
k_tile(const TrapCoef* __restrict__ coef, const TrapState* __restrict__ st_in,
       const unsigned long long* __restrict__ acc_in, int one_m, int one_off, int T, float unscale, int nx, int ny,
       int mc, int upd, const HoloDesc* __restrict__ hd, TrapState* __restrict__ st_out,
       const float* __restrict__ vin, float2* __restrict__ hist, int* __restrict__ flag, float inv_n,
       float* __restrict__ phase, float* __restrict__ grad, float2* __restrict__ partial,
       unsigned long long* __restrict__ acc_out, unsigned long long* __restrict__ acc_zero, float scale) {
  constexpr int NS = RT * CW, NW = NS * KH, NT = NW * 64;
  constexpr int XS = NW / CW, YS = NW / RT;  // waves sharing a column tile's (row tile's) table
  static_assert(NW % CW == 0 && NW % RT == 0, "whole waves per column and row tile");
  constexpr bool kPixel = MODE != 1, kTrap = MODE <= 1;
  extern __shared__ float4 lds4[];
  const int b = blockIdx.z;
  int M = one_m, off = one_off;
  if (one_m <= 0) {
    M = hd[b].m;
    off = hd[b].off;
  }
  const int Mp = (M + 15) & ~15;
  const int ntm = mc >> 4;
  unsigned* xf = reinterpret_cast<unsigned*>(lds4);              // [CW][ntm] X fragments
  unsigned* wf = xf + CW * ntm * kFragWords;                     // [RT][ntm] weighted Y fragments
  float4* yf = reinterpret_cast<float4*>(wf + RT * ntm * kFragWords);  // [RT][ntm][2][64] Y, FP32
  float4* refs = yf + RT * ntm * 128;                            // group constants {K, s, q}: [CW + RT][mc]
  float4* sx = refs + (CW + RT) * mc;                            // KH > 1: [NW][2][64] partial pixel sums
  float2* red = reinterpret_cast<float2*>(sx + (KH > 1 ? NW * 128 : 0));  // [NS][mc] trap sums
  float2* cw = red + NS * mc;                                    // [Mp] c_m
  float* sh = reinterpret_cast<float*>(cw + Mp);                 // [2 NW]

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int tw = wave % NS, part = wave / NS;    // the wave's pixels, and its share of the traps
  const int rt = tw / CW, cwv = tw - rt * CW;    // its row tile, and its group of column tiles
  const int row0 = blockIdx.y * (16 * RT), cb = blockIdx.x * (16 * CW);
  const int r = row0 + 16 * rt + li;
  const int c0 = cb + 16 * cwv + 4 * g;  // the lane's first column
  const size_t pix0 = (size_t)b * nx * ny + (size_t)r * nx + c0;

  const int ewofs = 16 * g + kTqWords * (li >> 2) + (li & 3);  // entry (4 g + v, trap li): + 4 v
  const int pofs = 4 * li + kTqWords * g;                      // entries (li, traps 4 g .. 4 g + 3)
  float fi[4], fq[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    fi[v] = (float)(4 * g + v - 8);
    fq[v] = fi[v] * fi[v];
  }

  // group constants of this wave's share of the tables, traps [k0, k0 + n): tile tx for the trap
  // tiles wave / CW, + XS, ..., and row tile ty for wave / RT, + YS, ...; written and read by this
  // wave alone
  const int tx = wave % CW, ty = wave % RT, jx = wave / CW, jy = wave / RT;
  float4* rx = refs + tx * mc;
  float4* ry = refs + (CW + ty) * mc;
  auto group = [&](const TrapCoef& k, double lin, double X) {
    const double kk = __builtin_fma(k.g, X * X, lin * X);
    double sl = __builtin_fma(4.0 * k.g, X, 2.0 * lin);
    sl -= __builtin_rint(sl);
    double q = 4.0 * k.g;
    q -= __builtin_rint(q);
    return make_float4((float)(kk - __builtin_rint(kk)), (float)sl, (float)q, 0.0f);
  };
  const double Xc = (double)(2 * (cb + 16 * tx + 8) - (nx - 1)), Yc = (double)(2 * (row0 + 16 * ty + 8) - (ny - 1));
  auto stage_refs = [&](int k0, int n) {
    for (int j = g; 16 * (jx + XS * j) < n; j += 4) {
      const int m = 16 * (jx + XS * j) + li;
      rx[m] = group(coef[off + min(k0 + m, M - 1)], coef[off + min(k0 + m, M - 1)].a, Xc);
    }
    for (int j = g; 16 * (jy + YS * j) < n; j += 4) {
      const int m = 16 * (jy + YS * j) + li;
      ry[m] = group(coef[off + min(k0 + m, M - 1)], coef[off + min(k0 + m, M - 1)].b, Yc);
    }
    wave_order();  // (the entries are formed from other lanes' constants)
  };
  auto entries = [&](const float4* ks, int tt, float2 (&e)[4]) {
    const float4 k = ks[16 * tt + li];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float t = __builtin_fmaf(k.z, fq[v], __builtin_fmaf(k.y, fi[v], k.x));
      e[v] = make_float2(__builtin_amdgcn_cosf(t), __builtin_amdgcn_sinf(t));
    }
  };
  auto put_x = [&](int tt) {
    float2 e[4];
    entries(rx, tt, e);
    unsigned* x = xf + (tx * ntm + tt) * kFragWords + ewofs;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const Split s = split(e[v].x, e[v].y);
      x[4 * v] = s.hi;
      x[4 * v + kLoWords] = s.lo;
    }
  };
  int wexp = 0;
  auto put_w = [&](int tt, int k0, const float2 (&e)[4]) {
    const float2 c = cw[k0 + 16 * tt + li];
    const float cx = __builtin_amdgcn_ldexpf(c.x, -wexp), cy = __builtin_amdgcn_ldexpf(c.y, -wexp);
    unsigned* w = wf + (ty * ntm + tt) * kFragWords + ewofs;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const Split s = split_conj(__builtin_fmaf(cx, e[v].x, -cy * e[v].y), __builtin_fmaf(cx, e[v].y, cy * e[v].x));
      w[4 * v] = s.hi;
      w[4 * v + kLoWords] = s.lo;
    }
  };
  auto put_y = [&](int tt, const float2 (&e)[4]) {
    float4* y = yf + (ty * ntm + tt) * 128 + lane;
    y[0] = make_float4(e[0].x, e[0].y, e[1].x, e[1].y);
    y[64] = make_float4(e[2].x, e[2].y, e[3].x, e[3].y);
  };
  auto get_y = [&](int f, float2 (&e)[4]) {
    const float4 y0 = yf[f * 128 + lane], y1 = yf[f * 128 + 64 + lane];
    e[0] = make_float2(y0.x, y0.y);
    e[1] = make_float2(y0.z, y0.w);
    e[2] = make_float2(y1.x, y1.y);
    e[3] = make_float2(y1.z, y1.w);
  };
  auto rebuild = [&](int k0, int n, bool weighted) {
    const int nt = n >> 4;
    __syncthreads();  // the previous super-chunk is no longer read
    stage_refs(k0, n);
    for (int tt = jx; tt < nt; tt += XS) put_x(tt);
    for (int tt = jy; tt < nt; tt += YS) {
      float2 e[4];
      entries(ry, tt, e);
      put_y(tt, e);
      if (weighted) put_w(tt, k0, e);
    }
    __syncthreads();
  };

  const int nsc = (Mp + mc - 1) / mc;
  const int n0 = min(mc, Mp), nt0 = n0 >> 4;
  const bool lead = blockIdx.x == 0 && blockIdx.y == 0;
  stage_refs(0, n0);
  __builtin_amdgcn_sched_barrier(0);
  const TrapInputs<NT, MODE> in(st_in, acc_in, T, off, M, unscale);
  __builtin_amdgcn_sched_barrier(0);
  for (int tt = jx; tt < nt0; tt += XS) put_x(tt);
  constexpr int YK = 4;  // this wave's first row fragments stay in registers until the weights are known
  float2 ey[YK][4];
#pragma unroll
  for (int j = 0; j < YK; ++j) {
    const int tt = jy + YS * j;
    if (tt < nt0) {
      entries(ry, tt, ey[j]);
      put_y(tt, ey[j]);
    }
  }
  for (int tt = jy + YS * YK; tt < nt0; tt += YS) {
    float2 e[4];
    entries(ry, tt, e);
    put_y(tt, e);
  }

  u32x4 eh, el, fh, fl;  // E = (Er, Ei) hi, lo and (Ei, -Er) hi, lo
  auto put_e = [&](const float* er, const float* ei) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const Split s = split(er[v], ei[v]);
      eh[v] = s.hi;
      el[v] = s.lo;
      fh[v] = turn_m(s.hi);
      fl[v] = turn_m(s.lo);
    }
  };
  auto inside = [&](int v) { return r < ny && c0 + v < nx; };

  if constexpr (kPixel) {
    bool inf;
    wexp = in.weights(cw, sh, Mp, st_in, vin, upd, lead, st_out, hist, flag, inf);
    // weighted Y of the first super-chunk
#pragma unroll
    for (int j = 0; j < YK; ++j) {
      const int tt = jy + YS * j;
      if (tt < nt0) put_w(tt, 0, ey[j]);
    }
    for (int tt = jy + YS * YK; tt < nt0; tt += YS) {
      float2 e[4];
      get_y(ty * ntm + tt, e);
      put_w(tt, 0, e);
    }
    __syncthreads();
    if (MODE == 0 && lead) {
      for (int m = threadIdx.x; m < M; m += NT) {
#pragma unroll
        for (int q = 0; q < kAccRegions; ++q) acc_zero[(size_t)q * T + off + m] = 0ull;
      }
    }

    f32x4 sre = {0.0f, 0.0f, 0.0f, 0.0f}, sim = sre;
    for (int s = 0; s < nsc; ++s) {
      const int k0 = s * mc, n = min(mc, Mp - k0), nt = n >> 4;
      if (s > 0) rebuild(k0, n, true);
      const int th = (nt + KH - 1) / KH;
      const int t0 = part * th, t1 = min(nt, t0 + th);
#pragma unroll 2
      for (int tt = t0; tt < t1; ++tt) {
        const unsigned* wb = wf + (rt * ntm + tt) * kFragWords + pofs;
        const u32x4 bh = *reinterpret_cast<const u32x4*>(wb), bl = *reinterpret_cast<const u32x4*>(wb + kLoWords);
        u32x4 ch, cl;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          ch[v] = turn_p(bh[v]);
          cl[v] = turn_p(bl[v]);
        }
        const unsigned* xb = xf + (cwv * ntm + tt) * kFragWords + pofs;
        const u32x4 ah = *reinterpret_cast<const u32x4*>(xb), al = *reinterpret_cast<const u32x4*>(xb + kLoWords);
        sre = mfma32(ah, bh, sre);
        sim = mfma32(ah, ch, sim);
        sre = mfma32(ah, bl, sre);
        sim = mfma32(ah, cl, sim);
        sre = mfma32(al, bh, sre);
        sim = mfma32(al, ch, sim);
      }
    }
    if constexpr (KH > 1) {
      float4* p = sx + wave * 128 + lane;
      p[0] = make_float4(sre[0], sre[1], sre[2], sre[3]);
      p[64] = make_float4(sim[0], sim[1], sim[2], sim[3]);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < KH; ++k) {
        const float4* p = sx + (tw + k * NS) * 128 + lane;
        const float4 a = p[0], c = p[64];
        const f32x4 ra = {a.x, a.y, a.z, a.w}, ia = {c.x, c.y, c.z, c.w};
        sre = k == 0 ? ra : sre + ra;
        sim = k == 0 ? ia : sim + ia;
      }
    }
    if constexpr (MODE == 3) {
      // (each pixel by one wave alone, which reads its phase before it writes: grad may be phase itself)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (inside(v) && v * KH / 4 == part) {
          const size_t px = pix0 + v;
          const float pr = phase_turn(phase[px]);
          grad[px] = __builtin_amdgcn_ldexpf(
              inv_n * (__builtin_amdgcn_cosf(pr) * sim[v] - __builtin_amdgcn_sinf(pr) * sre[v]), wexp);
        }
      }
    } else {
      if (phase != nullptr && part == 0) {  // (the last mask of a solve)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (inside(v)) phase[pix0 + v] = inf ? __builtin_nanf("") : phase_of(sim[v], sre[v]);
      }
      if constexpr (kTrap) {
        float er[4], ei[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) unit_of(sre[v], sim[v], inside(v), inf, er[v], ei[v]);
        put_e(er, ei);
      }
    }
  } else {
    float er[4], ei[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool in = inside(v);
      const float2 u = unit_turn(in ? phase_turn(phase[pix0 + v]) : 0.0f);
      er[v] = in ? u.x : 0.0f;
      ei[v] = in ? u.y : 0.0f;
    }
    put_e(er, ei);
    __syncthreads();
  }

  if constexpr (kTrap) {
    const int nblk = gridDim.x * gridDim.y, blk = blockIdx.y * gridDim.x + blockIdx.x;
    // super-chunks: the one whose tables are in LDS first
    for (int j = 0; j < nsc; ++j) {
      const int s = kPixel ? nsc - 1 - j : j;
      const int k0 = s * mc, n = min(mc, Mp - k0), nt = n >> 4;
      if (j > 0) rebuild(k0, n, false);
      const int th = (nt + KH - 1) / KH;
      const int t0 = part * th, t1 = min(nt, t0 + th);
      float* rw = reinterpret_cast<float*>(red) + 2 * (tw * mc + li) + (g >> 1);
      for (int tt = t0; tt < t1; tt += 2) {  // two trap tiles at a time
        f32x4 tre[2], tim[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int t = min(tt + p, t1 - 1);
          tre[p] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          tim[p] = tre[p];
          const unsigned* xb = xf + (cwv * ntm + t) * kFragWords + ewofs;
          u32x4 xh, xl;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            xh[v] = xb[4 * v];
            xl[v] = xb[4 * v + kLoWords];
          }
          tre[p] = mfma32(el, xh, tre[p]);
          tim[p] = mfma32(fl, xh, tim[p]);
          tre[p] = mfma32(eh, xl, tre[p]);
          tim[p] = mfma32(fh, xl, tim[p]);
          // (the large products last: every sum before them rounds finer)
          tre[p] = mfma32(eh, xh, tre[p]);
          tim[p] = mfma32(fh, xh, tim[p]);
        }
        float2 q[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          float2 yv[4];
          get_y(rt * ntm + min(tt + p, t1 - 1), yv);
          q[p] = fold_rows(yv, tre[p], tim[p]);
        }
        const float v = sum_groups(q[0], q[1]);
        if (tt + (g & 1) < t1) rw[32 * (tt + (g & 1))] = v;
      }
      __syncthreads();
      for (int m = threadIdx.x; m < n && k0 + m < M; m += NT) {
        float2 acc = red[m];
#pragma unroll
        for (int w = 1; w < NS; ++w) {
          acc.x += red[w * mc + m].x;
          acc.y += red[w * mc + m].y;
        }
        if constexpr (MODE == 0) {
          __hip_atomic_fetch_add(acc_out + (size_t)(xcc_id() & (kAccRegions - 1)) * T + off + k0 + m,
                                 pack_sum(acc, scale), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
          partial[(size_t)(off + k0 + m) * nblk + blk] = acc;
        }
      }
    }
  }
}

// The same for large grids: 64 x 64 pixels per block, eight waves.  What differs from k_tile is where
// the row factor lives.  A wave multiplies one row tile by all four column tiles, for half of the trap
// tiles (part 0 the even ones, part 1 the odd ones), so no other wave needs its weighted row entries:
// it computes them in registers, in the layout of the matrix operand (lane = row, four traps), between
// the products of the previous trap tile.  Only the column table stands in LDS, which then holds it for
// up to 256 traps at once: no super-chunks, no rebuilding and no barriers between them up to that count.
// The two partial sums of a tile meet through LDS, each wave finishing two of the four column tiles; in
// the trap pass it takes those two for all traps, with the row entries (lane = trap, four rows) in
// registers again.
//
// OCC: blocks that share a compute unit (1: up to 256 registers per wave; 2: up to 128, with half of the
// LDS each, so that one block's vector work overlaps the other's products).  Per iteration, against
// k_tile with 64 x 64 pixels per block: GSW 1024^2 x 256 24.2 -> 18.5 us (OCC 1; 19.7 with the
// registers of OCC 2), 2048^2 x 1000 305 -> 259 us (OCC 2; 285 with OCC 1), 64 holograms of 512^2 with
// 4..256 traps 195 -> 168 us (OCC 2; 191).  What bounds it: at 1024^2 x 256 about 38000 cycles, of which
// 9300 in the pixel pass and 11900 in the trap pass are at the issue rate of their vector instructions
// (4.5 cycles each, and 8 per product), 6500 build the column table while V is on its way, the rest is
// latency (update, exchange, barriers, last sums).
template <int MODE, int OCC>
__global__ void __launch_bounds__(512, 2 * OCC)
k_wide(const TrapCoef* __restrict__ coef, const TrapState* __restrict__ st_in,
       const unsigned long long* __restrict__ acc_in, int one_m, int one_off, int T, float unscale, int nx, int ny,
       int mc, int upd, const HoloDesc* __restrict__ hd, TrapState* __restrict__ st_out,
       const float* __restrict__ vin, float2* __restrict__ hist, int* __restrict__ flag, float inv_n,
       float* __restrict__ phase, float* __restrict__ grad, float2* __restrict__ partial,
       unsigned long long* __restrict__ acc_out, unsigned long long* __restrict__ acc_zero, float scale) {
  constexpr int NW = 8, NT = 512, CT = 4;
  constexpr bool kPixel = MODE != 1, kTrap = MODE <= 1;
  extern __shared__ float4 lds4[];
  const int b = blockIdx.z;
  int M = one_m, off = one_off;
  if (one_m <= 0) {
    M = hd[b].m;
    off = hd[b].off;
  }
  const int Mp = (M + 15) & ~15;
  const int ntm = mc >> 4;
  unsigned* xf = reinterpret_cast<unsigned*>(lds4);                      // [ntm][CT] X fragments
  float4* sx = reinterpret_cast<float4*>(xf + ntm * CT * kFragWords);     // 16 KB: column constants while the
  float2* red = reinterpret_cast<float2*>(sx);                            //   table is built, partial pixel sums,
  float4* rx = sx + (int)(threadIdx.x >> 6) * 128;                        //   trap sums [NW][mc]
  float2* rk = reinterpret_cast<float2*>(sx + 1024);                      // [4][mc] row constants {K, s}
  float* qv = reinterpret_cast<float*>(rk + 4 * mc);                      // [mc] curvature q
  float2* cw = reinterpret_cast<float2*>(qv + mc);                        // [Mp] c_m
  float* sh = reinterpret_cast<float*>(cw + Mp);                          // [2 NW]

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int rt = wave & 3, part = wave >> 2;
  const int row0 = blockIdx.y * 64, cb = blockIdx.x * 64;
  const int r = row0 + 16 * rt + li;
  const int c0 = cb + 32 * part + 4 * g;  // the lane's first column of the first tile it finishes
  const size_t pix0 = (size_t)b * nx * ny + (size_t)r * nx + c0;
  const int ewofs = 16 * g + kTqWords * (li >> 2) + (li & 3);  // entry (4 g + v, trap li): + 4 v
  const int pofs = 4 * li + kTqWords * g;                      // entries (li, traps 4 g .. 4 g + 3)
  const float fr = (float)(li - 8), frq = fr * fr;
  float fi[4], fq[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    fi[v] = (float)(4 * g + v - 8);
    fq[v] = fi[v] * fi[v];
  }

  // tables of the traps [k0, k0 + n): this wave fills column tile rt for the trap tiles part, part + 2,
  // ..., and forms the constants of column tile rt (for itself) and row tile rt (for all waves) of their
  // traps.  Lane group g takes the column (g even) or row constants (g odd) of trap tile
  // part + 2 (g / 2 + 2 round).
  const double Cg = g & 1 ? (double)(2 * (row0 + 16 * rt + 8) - (ny - 1)) : (double)(2 * (cb + 16 * rt + 8) - (nx - 1));
  struct RefCoef {
    double lin, q;
  };
  auto ref_load = [&](int k0, int round) {
    const TrapCoef* k = coef + off + min(k0 + 16 * (part + 2 * ((g >> 1) + 2 * round)) + li, M - 1);
    return RefCoef{g & 1 ? k->b : k->a, k->g};
  };
  auto ref_store = [&](const RefCoef& c, int n, int round) {
    const int i = (g >> 1) + 2 * round, m = 16 * (part + 2 * i) + li;
    if (m >= n) return;
    const double kk = __builtin_fma(c.q, Cg * Cg, c.lin * Cg);
    double sl = __builtin_fma(4.0 * c.q, Cg, 2.0 * c.lin);
    sl -= __builtin_rint(sl);
    double q = 4.0 * c.q;
    q -= __builtin_rint(q);
    const float2 ks = make_float2((float)(kk - __builtin_rint(kk)), (float)sl);
    if (g & 1) {
      rk[rt * mc + m] = ks;
    } else {
      rx[16 * i + li] = make_float4(ks.x, ks.y, (float)q, 0.0f);
      if (rt == 0) qv[m] = (float)q;
    }
  };
  auto build = [&](const RefCoef& first, int k0, int n) {
    const int nt = n >> 4;
    ref_store(first, n, 0);
    for (int round = 1; part + 4 * round < nt; ++round) ref_store(ref_load(k0, round), n, round);
    wave_order();  // (the entries are formed from other lanes' constants)
#pragma unroll 2
    for (int tt = part; tt < nt; tt += 2) {
      const int i = tt >> 1;
      const float4 k = rx[16 * i + li];
      unsigned* x = xf + (tt * CT + rt) * kFragWords + ewofs;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float t = __builtin_fmaf(k.z, fq[v], __builtin_fmaf(k.y, fi[v], k.x));
        const Split s = split(__builtin_amdgcn_cosf(t), __builtin_amdgcn_sinf(t));
        x[4 * v] = s.hi;
        x[4 * v + kLoWords] = s.lo;
      }
    }
  };

  const int nsc = (Mp + mc - 1) / mc;
  const int n0 = min(mc, Mp);
  const bool lead = blockIdx.x == 0 && blockIdx.y == 0;
  const RefCoef c_first = ref_load(0, 0);
  __builtin_amdgcn_sched_barrier(0);
  const TrapInputs<NT, MODE> in(st_in, acc_in, T, off, M, unscale);
  __builtin_amdgcn_sched_barrier(0);
  build(c_first, 0, n0);

  u32x4 eh[2], el[2], fh[2], fl[2];  // E = (Er, Ei) hi, lo and (Ei, -Er) hi, lo of the two tiles
  auto put_e = [&](int ct, const float* er, const float* ei) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const Split s = split(er[v], ei[v]);
      eh[ct][v] = s.hi;
      el[ct][v] = s.lo;
      fh[ct][v] = turn_m(s.hi);
      fl[ct][v] = turn_m(s.lo);
    }
  };
  auto inside = [&](int ct, int v) { return r < ny && c0 + 16 * ct + v < nx; };

  if constexpr (kPixel) {
    bool inf;
    const int wexp = in.weights(cw, sh, Mp, st_in, vin, upd, lead, st_out, hist, flag, inf);
    for (int m = threadIdx.x; m < M; m += NT) {  // (each thread rescales the weights it wrote)
      const float2 c = cw[m];
      cw[m] = make_float2(__builtin_amdgcn_ldexpf(c.x, -wexp), __builtin_amdgcn_ldexpf(c.y, -wexp));
    }
    __syncthreads();
    if (MODE == 0 && lead) {
      for (int m = threadIdx.x; m < M; m += NT) {
#pragma unroll
        for (int q = 0; q < kAccRegions; ++q) acc_zero[(size_t)q * T + off + m] = 0ull;
      }
    }

    f32x4 sre[CT], sim[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      sre[ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      sim[ct] = sre[ct];
    }
    struct RowOps {
      u32x4 bh, bl, ch, cl;
    };
    auto row_ops = [&](int k0, int tt) {  // c_m Y_m(row li) of traps 16 tt + 4 g .. + 3: (wr, -wi) and (wi, wr)
      const float4* k4 = reinterpret_cast<const float4*>(rk + rt * mc + 16 * tt + 4 * g);
      const float4* c4 = reinterpret_cast<const float4*>(cw + k0 + 16 * tt + 4 * g);
      const float4 q4 = *reinterpret_cast<const float4*>(qv + 16 * tt + 4 * g);
      const float4 ka = k4[0], kb = k4[1], ca = c4[0], cc = c4[1];
      const float K[4] = {ka.x, ka.z, kb.x, kb.z}, S[4] = {ka.y, ka.w, kb.y, kb.w}, Q[4] = {q4.x, q4.y, q4.z, q4.w};
      const float cx[4] = {ca.x, ca.z, cc.x, cc.z}, cy[4] = {ca.y, ca.w, cc.y, cc.w};
      RowOps o;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float t = __builtin_fmaf(Q[e], frq, __builtin_fmaf(S[e], fr, K[e]));
        const float yr = __builtin_amdgcn_cosf(t), yi = __builtin_amdgcn_sinf(t);
        const Split s = split_conj(__builtin_fmaf(cx[e], yr, -cy[e] * yi), __builtin_fmaf(cx[e], yi, cy[e] * yr));
        o.bh[e] = s.hi;
        o.bl[e] = s.lo;
        o.ch[e] = turn_p(s.hi);
        o.cl[e] = turn_p(s.lo);
      }
      return o;
    };
    for (int s = 0; s < nsc; ++s) {
      const int k0 = s * mc, n = min(mc, Mp - k0), nt = n >> 4;
      if (s > 0) {
        const RefCoef c = ref_load(k0, 0);
        __syncthreads();  // the previous super-chunk is no longer read
        build(c, k0, n);
        __syncthreads();
      }
      if (part < nt) {
        RowOps o = row_ops(k0, part);
        for (int tt = part; tt < nt; tt += 2) {
          const RowOps next = row_ops(k0, min(tt + 2, nt - 1));  // (the last one is not used)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const unsigned* xb = xf + (tt * CT + ct) * kFragWords + pofs;
            const u32x4 ah = *reinterpret_cast<const u32x4*>(xb), al = *reinterpret_cast<const u32x4*>(xb + kLoWords);
            sre[ct] = mfma32(ah, o.bh, sre[ct]);
            sim[ct] = mfma32(ah, o.ch, sim[ct]);
            sre[ct] = mfma32(ah, o.bl, sre[ct]);
            sim[ct] = mfma32(ah, o.cl, sim[ct]);
            sre[ct] = mfma32(al, o.bh, sre[ct]);
            sim[ct] = mfma32(al, o.ch, sim[ct]);
          }
          o = next;
        }
      }
    }
    // the two partial sums: a wave gives the tiles it does not finish to the other, one at a time
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const f32x4 gr = part == 0 ? sre[2 + i] : sre[i], gi = part == 0 ? sim[2 + i] : sim[i];
      if (i > 0) __syncthreads();
      float4* p = sx + wave * 128 + lane;
      p[0] = make_float4(gr[0], gr[1], gr[2], gr[3]);
      p[64] = make_float4(gi[0], gi[1], gi[2], gi[3]);
      __syncthreads();
      const float4* o = sx + (wave ^ 4) * 128 + lane;
      const float4 a = o[0], c = o[64];
      const f32x4 ra = {a.x, a.y, a.z, a.w}, ia = {c.x, c.y, c.z, c.w};
      if (part == 0) {
        sre[i] += ra;
        sim[i] += ia;
      } else {
        sre[i] = sre[2 + i] + ra;
        sim[i] = sim[2 + i] + ia;
      }
    }
    if constexpr (MODE == 3) {
#pragma unroll
      for (int ct = 0; ct < 2; ++ct) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (inside(ct, v)) {
            const size_t px = pix0 + 16 * ct + v;
            const float pr = phase_turn(phase[px]);
            grad[px] = __builtin_amdgcn_ldexpf(
                inv_n * (__builtin_amdgcn_cosf(pr) * sim[ct][v] - __builtin_amdgcn_sinf(pr) * sre[ct][v]), wexp);
          }
        }
      }
    } else {
      if (phase != nullptr) {  // (the last mask of a solve)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (inside(ct, v)) phase[pix0 + 16 * ct + v] = inf ? __builtin_nanf("") : phase_of(sim[ct][v], sre[ct][v]);
        }
      }
      if constexpr (kTrap) {
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          float er[4], ei[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) unit_of(sre[ct][v], sim[ct][v], inside(ct, v), inf, er[v], ei[v]);
          put_e(ct, er, ei);
        }
      }
    }
    if constexpr (kTrap) __syncthreads();  // (the trap sums take the place of the partial sums)
  } else {
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      float er[4], ei[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool in = inside(ct, v);
        const float2 u = unit_turn(in ? phase_turn(phase[pix0 + 16 * ct + v]) : 0.0f);
        er[v] = in ? u.x : 0.0f;
        ei[v] = in ? u.y : 0.0f;
      }
      put_e(ct, er, ei);
    }
    __syncthreads();
  }

  if constexpr (kTrap) {
    const int nblk = gridDim.x * gridDim.y, blk = blockIdx.y * gridDim.x + blockIdx.x;
    // super-chunks: the one whose table is in LDS first
    for (int j = 0; j < nsc; ++j) {
      const int s = kPixel ? nsc - 1 - j : j;
      const int k0 = s * mc, n = min(mc, Mp - k0), nt = n >> 4;
      if (j > 0) {
        const RefCoef c = ref_load(k0, 0);
        __syncthreads();  // the previous super-chunk's table and sums are no longer read
        build(c, k0, n);
        __syncthreads();
      }
      float* rw = reinterpret_cast<float*>(red) + 2 * (wave * mc + li) + (g >> 1);
      for (int tt = 0; tt < nt; tt += 2) {  // two trap tiles at a time
        f32x4 tre[2], tim[2];
        float2 q[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int t = min(tt + p, nt - 1);
          tre[p] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          tim[p] = tre[p];
          u32x4 xh[2];
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {
            const unsigned* xb = xf + (t * CT + 2 * part + ct) * kFragWords + ewofs;
            u32x4 xl;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              xh[ct][v] = xb[4 * v];
              xl[v] = xb[4 * v + kLoWords];
            }
            tre[p] = mfma32(el[ct], xh[ct], tre[p]);
            tim[p] = mfma32(fl[ct], xh[ct], tim[p]);
            tre[p] = mfma32(eh[ct], xl, tre[p]);
            tim[p] = mfma32(fh[ct], xl, tim[p]);
          }
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {  // (the large products last: every sum before them rounds finer)
            tre[p] = mfma32(eh[ct], xh[ct], tre[p]);
            tim[p] = mfma32(fh[ct], xh[ct], tim[p]);
          }
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int m = 16 * min(tt + p, nt - 1) + li;
          const float2 k = rk[rt * mc + m];
          const float qf = qv[m];
          float2 y[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float t = __builtin_fmaf(qf, fq[v], __builtin_fmaf(k.y, fi[v], k.x));
            y[v] = make_float2(__builtin_amdgcn_cosf(t), __builtin_amdgcn_sinf(t));
          }
          q[p] = fold_rows(y, tre[p], tim[p]);
        }
        const float v = sum_groups(q[0], q[1]);
        if (tt + (g & 1) < nt) rw[32 * (tt + (g & 1))] = v;
      }
      __syncthreads();
      for (int m = threadIdx.x; m < n && k0 + m < M; m += NT) {
        float2 acc = red[m];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
          acc.x += red[w * mc + m].x;
          acc.y += red[w * mc + m].y;
        }
        if constexpr (MODE == 0) {
          __hip_atomic_fetch_add(acc_out + (size_t)(xcc_id() & (kAccRegions - 1)) * T + off + k0 + m,
                                 pack_sum(acc, scale), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
          partial[(size_t)(off + k0 + m) * nblk + blk] = acc;
        }
      }
    }
  }
}

template <int RT, int CW, int KH, int MODE>
hipError_t tile_t(hipStream_t s, const SepArgs& a) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tile<RT, CW, KH, MODE>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
  if (attr != hipSuccess) return attr;
  const TileShape sh{RT, CW, 1, KH};
  const size_t lds = tile_lds_bytes(sh, a.sc, a.mmax);
  if (lds > (size_t)kLdsMax) return hipErrorInvalidValue;
  if (MODE == 0 && (!a.acc_in || !a.acc_out || !a.acc_zero || a.T < 1)) return hipErrorInvalidValue;
  dim3 grid(sh.gx(a.nx), sh.gy(a.ny), a.B);
  hipLaunchKernelGGL((k_tile<RT, CW, KH, MODE>), grid, dim3(sh.waves() * 64), lds, s, a.coef, a.st_in, a.acc_in,
                     a.B == 1 ? a.one_m : 0, a.B == 1 ? a.one_off : 0, a.T, a.acc_unscale, a.nx, a.ny, a.sc, a.upd,
                     a.hd, a.st_out, a.vin, a.hist, a.flag, a.inv_n, a.phase, a.grad, a.partial, a.acc_out, a.acc_zero,
                     a.acc_scale);
  return hipGetLastError();
}

template <int RT, int CW, int KH>
hipError_t tile_mode(hipStream_t s, const SepArgs& a) {
  switch (a.mode) {
    case 0: return tile_t<RT, CW, KH, 0>(s, a);
    case 1: return tile_t<RT, CW, KH, 1>(s, a);
    case 2: return tile_t<RT, CW, KH, 2>(s, a);
    case 3: return tile_t<RT, CW, KH, 3>(s, a);
    default: return hipErrorInvalidValue;
  }
}

template <int MODE, int OCC>
hipError_t wide_t(hipStream_t s, const SepArgs& a) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_wide<MODE, OCC>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
  if (attr != hipSuccess) return attr;
  const size_t lds = wide_lds_bytes(a.sc, a.mmax);
  if (lds > (size_t)kLdsMax || a.sc > kWideTraps) return hipErrorInvalidValue;
  if (MODE == 0 && (!a.acc_in || !a.acc_out || !a.acc_zero || a.T < 1)) return hipErrorInvalidValue;
  constexpr TileShape sh = kTileShapes[kTileWide];
  dim3 grid(sh.gx(a.nx), sh.gy(a.ny), a.B);
  hipLaunchKernelGGL((k_wide<MODE, OCC>), grid, dim3(512), lds, s, a.coef, a.st_in, a.acc_in, a.B == 1 ? a.one_m : 0,
                     a.B == 1 ? a.one_off : 0, a.T, a.acc_unscale, a.nx, a.ny, a.sc, a.upd, a.hd, a.st_out, a.vin,
                     a.hist, a.flag, a.inv_n, a.phase, a.grad, a.partial, a.acc_out, a.acc_zero, a.acc_scale);
  return hipGetLastError();
}

template <int MODE>
hipError_t wide_occ(hipStream_t s, const SepArgs& a) {
  return a.occ == 2 ? wide_t<MODE, 2>(s, a) : wide_t<MODE, 1>(s, a);
}

hipError_t wide_mode(hipStream_t s, const SepArgs& a) {
  switch (a.mode) {
    case 0: return wide_occ<0>(s, a);
    case 1: return wide_occ<1>(s, a);
    case 2: return wide_occ<2>(s, a);
    case 3: return wide_occ<3>(s, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_tile(hipStream_t s, const SepArgs& a) {
  if (a.nx < 1 || a.ny < 1 || a.mmax < 1 || a.mmax > kMaxTraps || a.sc < 16 || a.sc % 16 != 0)
    return hipErrorInvalidValue;
  switch (a.shape) {
    case kTile32: return tile_mode<2, 2, 1>(s, a);
    case kTile32Split: return tile_mode<2, 2, 2>(s, a);
    case kTileWide: return wide_mode(s, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace hot
