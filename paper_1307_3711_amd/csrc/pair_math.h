// pair_math.h -- one pair term, and a wave's chunk of pairs taken once, shared by the Coulomb
// kernels (force.hip describes the pair-once pass).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lc {

__device__ inline float rsq32(float x) { return __builtin_amdgcn_rsqf(x); }

// 1/sqrt(x) to FP64 rounding: with y0 from v_rsq_f64 and e = 1 - x y0^2 (computed with an
// FMA), 1/sqrt(x) = y0 (1 - e)^{-1/2} = y0 (1 + e/2 + 3e^2/8 + O(e^3)); the hardware estimate
// leaves |e| below about 2^-22, so the truncated series is exact to far below an FP64 ulp.
__device__ inline double rsq64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  const double p = __builtin_fma(0.375, e, 0.5);
  return __builtin_fma(y * e, p, y);
}

// x^{-3/2} to FP64 rounding in six instructions after the estimate, one less than the cube of
// rsq64: with Y = y0^2 rounded and e = 1 - x Y (exact up to one FMA rounding), x^{-3/2} =
// Y^{3/2} (1 - e)^{-3/2} = Y^{3/2} (1 + 3e/2 + 15e^2/8 + O(e^3)), and Y y0 is Y^{3/2} to 1.5 roundings.
// The series' FMA is written out: neither 3/2 nor 15/8 is an inline constant, and for the second one
// the compiler copies 3/2 into the result's registers before every FMA (two of 26 instructions).
// Measured on one card: a field of 50,021 charges taken in pairs 995 us, 1011 with the copies, 1053 with
// the cube of rsq64; the pair-once pass of the 20k argon cluster 154.4 us, 157.5 with the copies.
// A loop with the written-out FMA is not unrolled any more, so WRITTEN is for loops that unroll by hand.
template <bool WRITTEN>
__device__ inline double rsq64_cubed(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double y2 = y * y;
  const double e = __builtin_fma(-x, y2, 1.0);
  double p;
  if (WRITTEN) asm("v_fma_f64 %0, %1, %2, %3" : "=v"(p) : "v"(e), "s"(1.875), "v"(1.5));
  else p = __builtin_fma(1.875, e, 1.5);
  const double y3 = y2 * y;
  return __builtin_fma(y3 * e, p, y3);
}

__device__ inline float n3_rsq(float x) { return rsq32(x); }
__device__ inline double n3_rsq(double x) { return rsq64(x); }

// Pair arithmetic of the pair-once kernel: float (LC_FP32_ACC64) or double (LC_FP64).
// kFar places padding entries so far away that every field term they take part in is exactly zero:
// FP32 r^2 overflows to +inf and v_rsq_f32(+inf) = +0; FP64 r^2 = 1e300 stays finite (the
// refined 1/sqrt needs a finite argument) and (1/r)^3 = 1e-450 underflows to zero.  A potential
// term is zero in FP32; in FP64 it is 1e-150 times the charge, which the caller keeps at zero.
template <typename T> struct N3Type;
template <> struct N3Type<float> {
  using V4 = float4;
  static constexpr float kFar = 1e30f;
};
template <> struct N3Type<double> {
  using V4 = double4;
  static constexpr double kFar = 1e150;
};

__device__ inline float n3_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double n3_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Minimum-image separation in a periodic cube of side L (iL = 1/L): the nearest periodic copy
// of the partner (Sec. II periodic boundaries); a separation inside (-L/2, L/2) is unchanged.
// FP64 records hold coordinates, and the copy is the rounded multiple of L.
__device__ inline double min_image(double d, double L, double iL) { return __builtin_fma(-L, __builtin_rint(d * iL), d); }

// FP32 records of a periodic pass hold the cube on a 32-bit grid (coordinate x as the integer
// nearest x 2^32 / L, modulo 2^32; the charge as q (2^32 / L)^2): the wrapping integer
// difference of two records is the minimum-image separation in grid units, one subtraction and
// one conversion per component, and the pair terms in grid units are the field in physical
// units (the potential is 2^32 / L times its physical value).
__device__ inline float grid_sep(float a, float b) {
  return (float)(int32_t)(__float_as_uint(a) - __float_as_uint(b));
}

template <typename T, bool PBC>
__device__ inline T pair_sep(T a, T b, T L, T iL) {
  if constexpr (!PBC) return a - b;
  else if constexpr (sizeof(T) == 4) return grid_sep(a, b);
  else return min_image(a - b, L, iL);
}

// x from lane (l + 1) mod 64 for every lane l (DPP wave_rol:1).
__device__ inline float wave_rol1(float x) {
  // every lane of the wave has a source lane, so no "old" value is needed
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x134, 0xf, 0xf, false));
}
__device__ inline double wave_rol1(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, 0x134, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), 0x134, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Orders the LDS traffic of one wave around a point where lanes read what other lanes wrote.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Per-wave LDS slice: x, y, z, q arrays of the chunk twice (128 entries each) plus room for
// the prefetch of the rotation after the last one (up to 8 entries, read and discarded).
constexpr int kN3Slice = 136;
__host__ __device__ constexpr int n3_slices(int waves) { return waves * 4 * kN3Slice; }  // elements

// Between the stages of FP32 pair terms: keeps the reciprocal roots of a group of pairs together.
// FP32 instructions with vector operands go out for two waves of a SIMD at a time (2.4 to 2.9 cycles
// each with two waves or more; 4.2 with a scalar operand or DPP, 8.2 for v_rsq_f32), and a lone
// v_rsq_f32 among them costs about 30: a loop of the pair-once instructions takes 72 cycles a pair with
// its roots spread out, as the compiler schedules them, and 55 with eight of them in a row.  The
// pair-once pass of the 20k argon cluster: 91.9 -> 87.4 us, of 199,998 macroparticles 7.65 -> 7.28 ms.
template <typename T>
__device__ inline void rsq_fence() {
  if constexpr (sizeof(T) == 4) __builtin_amdgcn_sched_barrier(0x94);
}

// U rotations of the chunk from the register buffers (bx, by, bz, bq) holding their sources.
// PHI: also the potential, fp of the targets and (JSIDE) rp of the sources; self: the r whose
// target is the first rotation's source (-1: none), which its own potential leaves out.
template <typename T, int R, int U, bool US, bool UT, bool JSIDE, bool PBC, bool PHI = false>
__device__ inline void n3_steps(const T* bx, const T* by, const T* bz, const T* bq, const T* xi, const T* yi,
                                const T* zi, const T* qi, T eps2f, T* fx, T* fy, T* fz, T& rx, T& ry, T& rz, T L,
                                T iL, T* fp = nullptr, T* rp = nullptr, int self = -1) {
  constexpr int G = sizeof(T) == 8 || R > 4 ? 1 : R == 1 ? U : 2;  // rotations and targets of a group
  constexpr int GR = sizeof(T) == 4 ? R : 1;
#pragma unroll
  for (int u0 = 0; u0 < U; u0 += G) {
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += GR) {
      T dx[G][GR], dy[G][GR], dz[G][GR], inv[G][GR];
#pragma unroll
      for (int u = 0; u < G; ++u) {
#pragma unroll
        for (int r = 0; r < GR; ++r) {
          dx[u][r] = pair_sep<T, PBC>(xi[r0 + r], bx[u0 + u], L, iL);
          dy[u][r] = pair_sep<T, PBC>(yi[r0 + r], by[u0 + u], L, iL);
          dz[u][r] = pair_sep<T, PBC>(zi[r0 + r], bz[u0 + u], L, iL);
          T r2 = n3_fma(dx[u][r], dx[u][r], eps2f);
          r2 = n3_fma(dy[u][r], dy[u][r], r2);
          inv[u][r] = n3_fma(dz[u][r], dz[u][r], r2);
        }
      }
      if constexpr (sizeof(T) == 4 || PHI) {
        rsq_fence<T>();
#pragma unroll
        for (int u = 0; u < G; ++u)
#pragma unroll
          for (int r = 0; r < GR; ++r) inv[u][r] = n3_rsq(inv[u][r]);
        rsq_fence<T>();
      }
#pragma unroll
      for (int u = 0; u < G; ++u) {
#pragma unroll
        for (int r = 0; r < GR; ++r) {
          const int k = r0 + r;
          T r3;
          if constexpr (sizeof(T) == 4 || PHI) r3 = inv[u][r] * (inv[u][r] * inv[u][r]);
          else r3 = rsq64_cubed<true>(inv[u][r]);
          const T si = US ? r3 : bq[u0 + u] * r3;
          fx[k] = n3_fma(si, dx[u][r], fx[k]);
          fy[k] = n3_fma(si, dy[u][r], fy[k]);
          fz[k] = n3_fma(si, dz[u][r], fz[k]);
          if (JSIDE) {
            const T sr = UT ? r3 : qi[k] * r3;
            rx = n3_fma(sr, dx[u][r], rx);
            ry = n3_fma(sr, dy[u][r], ry);
            rz = n3_fma(sr, dz[u][r], rz);
          }
          if constexpr (PHI) {
            T pi = US ? inv[u][r] : bq[u0 + u] * inv[u][r];
            if (!JSIDE && u0 + u == 0 && k == self) pi = 0;
            fp[k] += pi;
            if (JSIDE) *rp = UT ? *rp + inv[u][r] : n3_fma(qi[k], inv[u][r], *rp);
          }
        }
        if (JSIDE && r0 + GR == R) {
          if constexpr (PHI) *rp = wave_rol1(*rp);
          rx = wave_rol1(rx);
          ry = wave_rol1(ry);
          rz = wave_rol1(rz);
        }
      }
    }
  }
}

// Sources of rotations [k, k + U) into registers.
template <typename T, int U, bool US>
__device__ inline void n3_load(const T* sx, int k, T* bx, T* by, T* bz, T* bq) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    bx[u] = sx[k + u];
    by[u] = sx[kN3Slice + k + u];
    bz[u] = sx[2 * kN3Slice + k + u];
    if (!US) bq[u] = sx[3 * kN3Slice + k + u];
  }
}

// One chunk of 64 sources (sb: x, y, z, q arrays of the chunk twice, kN3Slice apart) against
// the lane's R targets.  US: all sources of the chunk carry one charge (factored out by the
// caller); UT: likewise for the targets of the wave.  JSIDE: also the reaction sums
// sum_r q_r s_r (r_i - r_j) of the chunk's sources, returned in (ax, ay, az) of lane l for
// source l.  Software pipelined over two register buffers of U rotations: the sources of the next U
// rotations are read while the current U are used (the slice has kN3Slice >= 128 + U
// entries, so the read after the last rotation stays inside it).
template <typename T, int R, int U, bool US, bool UT, bool JSIDE, bool PBC, bool PHI = false>
__device__ inline void n3_chunk(const T* sb, int lane, const T* xi, const T* yi, const T* zi, const T* qi, T eps2f,
                                T* fx, T* fy, T* fz, T& ax, T& ay, T& az, T L, T iL, T* fp = nullptr,
                                T* ap = nullptr, int self = -1) {
  static_assert(128 + U <= kN3Slice && 64 % (2 * U) == 0, "prefetch stays inside the wave's slice");
  const T* sx = sb + lane;
  T rx = 0, ry = 0, rz = 0, rp = 0;  // running sums of source (lane + k) mod 64
  T ax_[U], ay_[U], az_[U], aq_[U], bx_[U], by_[U], bz_[U], bq_[U];
  n3_load<T, U, US>(sx, 0, ax_, ay_, az_, aq_);
  for (int k0 = 0; k0 < 64; k0 += 2 * U) {
    n3_load<T, U, US>(sx, k0 + U, bx_, by_, bz_, bq_);
    n3_steps<T, R, U, US, UT, JSIDE, PBC, PHI>(ax_, ay_, az_, aq_, xi, yi, zi, qi, eps2f, fx, fy, fz, rx, ry, rz, L, iL,
                                               fp, &rp, k0 == 0 ? self : -1);
    n3_load<T, U, US>(sx, k0 + 2 * U, ax_, ay_, az_, aq_);
    n3_steps<T, R, U, US, UT, JSIDE, PBC, PHI>(bx_, by_, bz_, bq_, xi, yi, zi, qi, eps2f, fx, fy, fz, rx, ry, rz, L, iL,
                                               fp, &rp);
  }
  ax = rx;
  ay = ry;
  az = rz;
  if constexpr (PHI) *ap = rp;
}

}  // namespace lc
