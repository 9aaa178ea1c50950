// hot_device.h -- device helpers shared by the kernel files: wave and block reductions, the phase
// of a complex number, the fixed-point trap sums, and the figures of merit with the GS/GSW update.
#pragma once

#include "hot_internal.h"

#include <type_traits>

namespace hot {

namespace {

constexpr float kInv2Pi = 0.159154943091895336f;  // FP32(1 / (2 pi))
constexpr float kTwoPi = 6.28318530717958648f;    // FP32(2 pi)

// Holograms of at least this many traps run the iteration kernels' update and pixel pass at a
// higher wave priority than their trap pass (measured: 768^2 x 49 traps 21.9 -> 20.2 us per
// iteration, 512^2 x 100 16.6 -> 15.2 us; 768^2 x 25 14.6 -> 15.5 us, 1024 x 768 x 8 7.4 -> 9.7 us).
constexpr int kPriorityTraps = 40;

// The XCD (accelerator complex die) the wave runs on: hardware register XCC_ID, bits 3:0.
__device__ __forceinline__ int xcc_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | ((4 - 1) << 11)) & 15; }

template <bool FRACT>
__device__ __forceinline__ float to_period(float t) {
  if constexpr (FRACT) return __builtin_amdgcn_fractf(t);
  return t;
}

// Wave-wide reductions.  DPP steps combine lanes inside each row of 16 (xor 1, xor 2, then the
// half-row and row mirrors), after which every lane of a row holds the row result; the four
// row results are then read from lanes 0, 16, 32, 48 and combined in that order, so the
// result is the same, deterministic value in every lane.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float rows_of(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  return (rows_of(v, 0) + rows_of(v, 16)) + (rows_of(v, 32) + rows_of(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  v = fmaxf(v, dpp<0x140>(v));
  return fmaxf(fmaxf(rows_of(v, 0), rows_of(v, 16)), fmaxf(rows_of(v, 32), rows_of(v, 48)));
}
__device__ __forceinline__ float wave_min(float v) {
  v = fminf(v, dpp<0xB1>(v));
  v = fminf(v, dpp<0x4E>(v));
  v = fminf(v, dpp<0x141>(v));
  v = fminf(v, dpp<0x140>(v));
  return fminf(fminf(rows_of(v, 0), rows_of(v, 16)), fminf(rows_of(v, 32), rows_of(v, 48)));
}

__device__ __forceinline__ unsigned wave_max_bits(unsigned v) {
  auto dpp_max = [&](auto ctrl) {
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, false));
  };
  dpp_max(std::integral_constant<int, 0xB1>{});
  dpp_max(std::integral_constant<int, 0x4E>{});
  dpp_max(std::integral_constant<int, 0x141>{});
  dpp_max(std::integral_constant<int, 0x140>{});
  auto row = [&](int lane) { return (unsigned)__builtin_amdgcn_readlane((int)v, lane); };
  return max(max(row(0), row(16)), max(row(32), row(48)));
}

// A caller's phase [rad] in revolutions, reduced to [0, 1] (1 is the same angle as 0): product and
// reduction in FP64, so a mask far outside [0, 2 pi) (an optimiser's drifting phase, say) loses
// nothing beyond its own FP32 rounding and stays inside the hardware sin/cos domain.  Once per pixel.
__device__ __forceinline__ float caller_phase_rev(float ph) {
  const double t = (double)ph * 0.15915494309189533577;  // 1 / (2 pi)
  return (float)(t - __builtin_floor(t));
}

__device__ __forceinline__ float wrap_phase(float ph) { return ph < 0.0f ? ph + kTwoPi : ph; }

// arg(x + i y) in [0, 2pi] (arg 0 = 0).  The octant is folded onto t = min(|x|,|y|) / max(|x|,|y|)
// in [0, 1], where atan t = t P(t^2) with P of degree 7: coefficients from a Lawson-weighted
// least-squares (near-minimax) fit to atan on [0, 1], max error 4e-8 in exact arithmetic and
// 1.4e-7 rad evaluated in FP32; the reciprocal adds at most 1.2e-7.  Then the octant and the
// quadrant are undone.
__device__ __forceinline__ float phase_of(float y, float x) {
  const float ax = __builtin_fabsf(x), ay = __builtin_fabsf(y);
  const float mx = __builtin_fmaxf(ax, ay), mn = __builtin_fminf(ax, ay);
  const float t = mx > 0.0f ? mn * __builtin_amdgcn_rcpf(mx) : 0.0f;
  const float s = t * t;
  float p = -4.054570390e-03f;
  p = __builtin_fmaf(p, s, 2.186296944e-02f);
  p = __builtin_fmaf(p, s, -5.591234356e-02f);
  p = __builtin_fmaf(p, s, 9.642198569e-02f);
  p = __builtin_fmaf(p, s, -1.390863004e-01f);
  p = __builtin_fmaf(p, s, 1.994656575e-01f);
  p = __builtin_fmaf(p, s, -3.332986079e-01f);
  p = __builtin_fmaf(p, s, 9.999993356e-01f);
  float r = p * t;
  if (ay > ax) r = 1.57079632679489662f - r;
  if (x < 0.0f) r = 3.14159265358979324f - r;
  if (y < 0.0f) r = kTwoPi - r;
  return r;
}

// Block-wide (NT threads) sums of a and b, max of c, min of d; every thread gets the
// results.  Waves reduce with wave_sum/max/min, lane 0 of each wave publishes to `sh`
// (4 * (NT / 64) floats, not reused by the caller), one barrier, then every thread combines
// the wave results in wave order.
template <int NT>
__device__ __forceinline__ void block_reduce(float* sh, float& a, float& b, float& c, float& d) {
  constexpr int W = NT / 64;
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_max(c);
  d = wave_min(d);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sh[wave] = a;
    sh[W + wave] = b;
    sh[2 * W + wave] = c;
    sh[3 * W + wave] = d;
  }
  __syncthreads();
  a = sh[0];
  b = sh[W];
  c = sh[2 * W];
  d = sh[3 * W];
  for (int w = 1; w < W; ++w) {
    a += sh[w];
    b += sh[W + w];
    c = fmaxf(c, sh[2 * W + w]);
    d = fminf(d, sh[3 * W + w]);
  }
}

// Block-wide sum of a (every thread gets it), combined in wave order as in block_reduce.
template <int NT>
__device__ __forceinline__ void block_sum(float* sh, float& a) {
  constexpr int W = NT / 64;
  a = wave_sum(a);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
  __syncthreads();
  a = sh[0];
  for (int w = 1; w < W; ++w) a += sh[w];
}

// V of trap k (local index) of a hologram: from an interleaved (re, im) array ...
struct VArray {
  const float* __restrict__ V;
  int off;
  __device__ float2 operator()(int k) const { return make_float2(V[2 * (off + k)], V[2 * (off + k) + 1]); }
};
// ... or from the fixed-point sums of the fused kernels: kAccRegions regions, each T = acc_stride(traps)
// 64-bit words from the next.
// A block adds its sum (re, im) of a trap as one word, pack_sum: re and im are rounded to
// integers in units of 1/scale, and the word is the 64-bit two's-complement value
// re + 2^32 im.  Words add like integers, so a sum of words is R + 2^32 I with R, I the sums of
// the parts; as long as |R| < 2^31 (the host picks scale so that any sum of N unit-modulus terms
// stays within 2^30), R is the low 32 bits read as signed, and I the high 32 bits plus one if R
// is negative.  V = (R, I) * unscale.
__device__ __forceinline__ unsigned long long pack_sum(float2 v, float scale) {
  const int re = (int)__builtin_rintf(v.x * scale), im = (int)__builtin_rintf(v.y * scale);
  return (unsigned long long)(long long)re + ((unsigned long long)(unsigned)im << 32);
}
static_assert(kAccRegions == 8, "VAcc sums eight regions");
struct VAcc {
  const unsigned long long* __restrict__ acc;
  int T, off;
  float unscale;
  // the eight words of trap k (loads only: nothing waits for them here) ...
  __device__ void load(int k, unsigned long long (&w8)[kAccRegions]) const {
#pragma unroll
    for (int r = 0; r < kAccRegions; ++r) w8[r] = acc[(size_t)r * T + off + k];
  }
  // ... and V from them: a tree of adds (exact, so the order is free), three dependent steps
  // instead of seven
  __device__ float2 sum(const unsigned long long (&w8)[kAccRegions]) const {
    const unsigned long long w = ((w8[0] + w8[1]) + (w8[2] + w8[3])) + ((w8[4] + w8[5]) + (w8[6] + w8[7]));
    const int re = (int)(unsigned)w;
    const int im = (int)((unsigned)(w >> 32) - (unsigned)(re >> 31));
    return make_float2((float)re * unscale, (float)im * unscale);
  }
  __device__ float2 operator()(int k) const {
    unsigned long long w8[kAccRegions];
    load(k, w8);
    return sum(w8);
  }
};

// Section 3 figures of merit and the GS/GSW update for one hologram, computed by one
// block from V (vmem(k) for its M traps) and the current state.
//   stats_row (3 floats) if non-null: e = sum I, u = 1 - (max-min)/(max+min), sigma = std(I)/mean(I)
//   mode 0: no update; 1 (GS): theta_m <- arg V_m; 2 (GSW): also w_m <- w_m <|V|>/|V_m|
// emit(m, state) is called once per trap m, by the thread that owns it.  <|V|> = 0 leaves
// the state unchanged and raises *flag (if non-null).  With PRE, trap threadIdx.x's V and state
// come from vpre / spre (loaded earlier by the caller) instead of memory.  |V_m|, <|V|> and the
// weight factor use the hardware square root and reciprocal (about 1 ulp each): this sits on the
// critical path at the start of every iteration launch.
template <int NT, class VGet, class Emit, bool PRE = false>
__device__ void update_traps(VGet vmem, const TrapState* __restrict__ st_in, int off, int M, int mode, float* sh,
                             float* stats_row, int* flag, Emit emit, float2 vpre = make_float2(0.0f, 0.0f),
                             TrapState spre = TrapState{}) {
  auto getv = [&](int k) {
    if (PRE && k == (int)threadIdx.x) return vpre;
    return vmem(k);
  };
  // PRE: the modulus of the thread's own V, its reciprocal and arg V do not need <|V|>; they are
  // formed here, so that their latency overlaps the block-wide sum instead of following it
  float own_amp = 0.0f, own_rcp = 0.0f, own_th = 0.0f;
  if (PRE && mode != 0 && (int)threadIdx.x < M) {
    own_amp = __builtin_amdgcn_sqrtf(vpre.x * vpre.x + vpre.y * vpre.y);
    own_rcp = __builtin_amdgcn_rcpf(own_amp);
    own_th = phase_of(vpre.y, vpre.x);
  }
  float sa = 0.0f, si = 0.0f, mx = -1.0f, mn = 3.0e38f;
  for (int k = threadIdx.x; k < M; k += NT) {
    const float2 v = getv(k);
    const float vr = v.x, vi = v.y;
    const float I = vr * vr + vi * vi;
    sa += __builtin_amdgcn_sqrtf(I);
    si += I;
    mx = fmaxf(mx, I);
    mn = fminf(mn, I);
  }
  if (stats_row) {
    block_reduce<NT>(sh, sa, si, mx, mn);
  } else {
    block_sum<NT>(sh, sa);  // the update needs only <|V|>
  }
  const float mean_abs = sa * __builtin_amdgcn_rcpf((float)M);
  if (stats_row) {
    const float mu = si / (float)M;
    float var = 0.0f, z0 = 0.0f, z1 = 0.0f, z2 = 0.0f;
    for (int k = threadIdx.x; k < M; k += NT) {
      const float2 v = getv(k);
      const float vr = v.x, vi = v.y;
      const float dI = vr * vr + vi * vi - mu;
      var += dI * dI;
    }
    block_reduce<NT>(sh + 4 * (NT / 64), var, z0, z1, z2);
    var /= (float)M;
    if (threadIdx.x == 0) {
      stats_row[0] = si;
      stats_row[1] = (mx + mn) > 0.0f ? 1.0f - (mx - mn) / (mx + mn) : 0.0f;
      stats_row[2] = mu > 0.0f ? sqrtf(var) / mu : 0.0f;
    }
  }
  const bool degenerate = mode != 0 && !(mean_abs > 0.0f);
  if (degenerate && flag && threadIdx.x == 0) *flag = 1;
  const float floor_abs = 1e-12f * mean_abs;
  for (int k = threadIdx.x; k < M; k += NT) {
    TrapState s = (PRE && k == (int)threadIdx.x) ? spre : st_in[off + k];
    if (mode != 0 && !degenerate) {
      float amp, rcp_amp, th;  // |V_m|, its reciprocal, arg V_m in [0, 2pi]
      if (PRE && k == (int)threadIdx.x) {
        amp = own_amp;
        rcp_amp = own_rcp;
        th = own_th;
      } else {
        const float2 v = getv(k);
        amp = __builtin_amdgcn_sqrtf(v.x * v.x + v.y * v.y);
        rcp_amp = __builtin_amdgcn_rcpf(amp);
        th = phase_of(v.y, v.x);
      }
      const bool tiny = amp < floor_abs;
      if (mode == 2) s.w *= mean_abs * (tiny ? __builtin_amdgcn_rcpf(floor_abs) : rcp_amp);
      if (!tiny) {
        s.theta_rad = th > 3.14159265358979324f ? th - kTwoPi : th;  // kept in (-pi, pi]
        s.theta_rev = s.theta_rad * kInv2Pi;
      }
    }
    emit(k, s);
  }
}

// The trap's complex weight c_m = w_m e^{i theta_m} (theta reduced to one period, exactly).
__device__ __forceinline__ float2 trap_weight(const TrapState& s) {
  const float t = s.theta_rev - __builtin_rintf(s.theta_rev);
  return make_float2(s.w * __builtin_amdgcn_cosf(t), s.w * __builtin_amdgcn_sinf(t));
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

}  // namespace

}  // namespace hot
