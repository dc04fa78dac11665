// field.hip -- the softened Coulomb field of charges on themselves with the default tiling
// (lc_field, lc_field_static), Sec. II:
//
//   E_i   = sum_{j != i} q_j (r_i - r_j) / (|r_i - r_j|^2 + eps^2)^{3/2}
//   phi_i = sum_{j != i} q_j / (|r_i - r_j|^2 + eps^2)^{1/2}        (when asked for)
// Part of force.hip's object: force.hip includes this file.
#include <algorithm>

#include "lc_internal.h"
#include "pair_math.h"

namespace lc {
namespace field_default {
namespace {

// One launch, straight from the caller's arrays to the caller's results.  A block of WAVES waves takes
// COLS targets and all sources, which it stages kChunk at a time in LDS in the pair type; the 64 lanes
// of a wave are COLS targets x 64 / COLS sources, so a block of 16 targets and 16 waves meets 64 sources
// at a time and a small n still fills the chip.  The partial sums of a target are added in a fixed
// order; sums run in the pair type over a lane's sources of one chunk (32, or 64 with 8 waves and 16
// targets), in FP64 beyond.  Only the step of sources that holds the block's own targets tests for
// them.
// Bound by launch and load latency below a few thousand charges, by VALU issue beyond.  Measured a
// call (field and potential): 1000 charges in FP64 12 us, 4099 with Kahan sums 21 us, against 120
// and 902 us with the one-sided tiling of force.hip that a default call took before (blocks of 512
// or 1024 targets: 2 and 5 of them on 256 compute units).  Two and four targets per lane were
// slower at every size from 4000 charges on (20,000 FP32: 222 and 243 us against 174 us): one
// block of 16 waves per compute unit instead of two waits at every chunk's barriers.
constexpr int kChunk = 2048;
constexpr int64_t kUnits = 256;     // compute units
constexpr int64_t kGrid = 1 << 20;  // blocks of a launch at most (they stride over the targets)

// The lane's target and its sums over a chunk (c: Kahan compensations).
template <typename T>
struct Lane {
  T x, y, z;
  T f[4], c[4];
};

template <typename T, bool KAHAN>
__device__ inline void add_term(T a, T b, T& f, T& c) {  // f += a b
  if (KAHAN) {
    const T y = n3_fma(a, b, -c), t = f + y;
    c = (t - f) - y;
    f = t;
  } else {
    f = n3_fma(a, b, f);
  }
}

// One source against the lane's target.  UNIFORM: the charge is left to the caller.  MASK: the
// source counts only if live, and in the potential only if not the target itself.
template <typename T, bool KAHAN, bool PHI, bool UNIFORM, bool MASK, typename V4>
__device__ inline void direct_pair(const V4 s, bool live, bool self, T eps2, Lane<T>& l) {
  const T dx = l.x - s.x, dy = l.y - s.y, dz = l.z - s.z;
  T r2 = n3_fma(dx, dx, eps2);
  r2 = n3_fma(dy, dy, r2);
  r2 = n3_fma(dz, dz, r2);
  T qinv = 0, sc;
  if constexpr (PHI || sizeof(T) == 4) {
    T inv = n3_rsq(r2);
    if (MASK && !live) inv = 0;
    qinv = UNIFORM ? inv : s.w * inv;
    sc = qinv * (inv * inv);
  } else {
    sc = rsq64_cubed<false>(r2);
    if (MASK && !live) sc = 0;
    if (!UNIFORM) sc *= s.w;
  }
  add_term<T, KAHAN>(sc, dx, l.f[0], l.c[0]);
  add_term<T, KAHAN>(sc, dy, l.f[1], l.c[1]);
  add_term<T, KAHAN>(sc, dz, l.f[2], l.c[2]);
  if (PHI) {
    if (MASK && self) qinv = 0;
    if (KAHAN) add_term<T, true>(qinv, T(1), l.f[3], l.c[3]);
    else l.f[3] += qinv;
  }
}

// The lane's share of a chunk: sources grp, grp + STEP, ... of the cnt in LDS.  self is the place of
// the lane's target among them; steps lo to hi hold the block's targets (the same in every lane).
template <typename T, int STEP, bool KAHAN, bool PHI, bool UNIFORM, typename V4>
__device__ inline void direct_chunk(const V4* src, int cnt, int grp, int lo, int hi, int self, T eps2, Lane<T>& l) {
  const int whole = cnt / STEP * STEP;
  lo = min(lo, whole);
#pragma unroll 4
  for (int k = 0; k < lo; k += STEP) direct_pair<T, KAHAN, PHI, UNIFORM, false>(src[k + grp], true, false, eps2, l);
  for (int k = lo; k < min(hi, cnt); k += STEP) {
    const bool live = k + grp < cnt;
    direct_pair<T, KAHAN, PHI, UNIFORM, true>(src[live ? k + grp : 0], live, k + grp == self, eps2, l);
  }
#pragma unroll 4
  for (int k = max(lo, hi); k < whole; k += STEP)
    direct_pair<T, KAHAN, PHI, UNIFORM, false>(src[k + grp], true, false, eps2, l);
  if (max(whole, hi) < cnt) {
    const bool live = whole + grp < cnt;
    direct_pair<T, KAHAN, PHI, UNIFORM, true>(src[live ? whole + grp : 0], live, false, eps2, l);
  }
}

template <typename T, int COLS, int WAVES, bool KAHAN, bool PHI>
__global__ __launch_bounds__(64 * WAVES) void k_field_direct(const double* __restrict__ xyzq, int64_t n,
                                                             double eps2d, double* E, double* phi) {
  using V4 = typename N3Type<T>::V4;
  constexpr int NC = PHI ? 4 : 3, GROUPS = 64 / COLS, STEP = GROUPS * WAVES, THREADS = 64 * WAVES;
  __shared__ V4 src[kChunk];
  double* red = reinterpret_cast<double*>(src);  // [wave][component][target], after the last chunk
  static_assert(sizeof(double) * WAVES * 4 * COLS <= sizeof(V4) * kChunk, "the block's partial sums fit");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t = lane % COLS, grp = GROUPS * wave + lane / COLS;
  const T eps2 = (T)eps2d;
  for (int64_t i0 = (int64_t)blockIdx.x * COLS; i0 < n; i0 += (int64_t)gridDim.x * COLS) {
    Lane<T> l;
    const int64_t i = i0 + t < n ? i0 + t : n - 1;  // lanes past the last target repeat it and store nothing
    l.x = (T)xyzq[i];
    l.y = (T)xyzq[n + i];
    l.z = (T)xyzq[2 * n + i];
    double e[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) e[k] = 0.0;
    for (int64_t j0 = 0; j0 < n; j0 += kChunk) {
      const int cnt = (int)(n - j0 < kChunk ? n - j0 : kChunk);
      const T q0 = (T)xyzq[3 * n + j0];
      int same = 1;
      __syncthreads();  // the sources and sums before these are read
      for (int k = tid; k < cnt; k += THREADS) {
        const int64_t j = j0 + k;
        V4 v;
        v.x = (T)xyzq[j];
        v.y = (T)xyzq[n + j];
        v.z = (T)xyzq[2 * n + j];
        v.w = (T)xyzq[3 * n + j];
        same &= v.w == q0;
        src[k] = v;
      }
      const bool uniform = __syncthreads_and(same);
      // the steps that hold the block's targets (COLS divides STEP: one, or in another chunk none)
      const bool own = PHI && i0 >= j0 && i0 < j0 + cnt;
      const int lo = own ? (int)(i0 - j0) / STEP * STEP : kChunk, hi = own ? lo + STEP : 0;
      const int self = own ? (int)(i - j0) : -1;
#pragma unroll
      for (int k = 0; k < 4; ++k) l.f[k] = l.c[k] = 0;
      if (uniform) direct_chunk<T, STEP, KAHAN, PHI, true>(src, cnt, grp, lo, hi, self, eps2, l);
      else direct_chunk<T, STEP, KAHAN, PHI, false>(src, cnt, grp, lo, hi, self, eps2, l);
      const double qs = uniform ? (double)q0 : 1.0;
#pragma unroll
      for (int k = 0; k < NC; ++k) e[k] += (double)l.f[k] * qs;
    }
    __syncthreads();  // the last chunk is read
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      for (int o = COLS; o < 64; o <<= 1) e[k] += __shfl_xor(e[k], o, 64);
      if (lane < COLS) red[(wave * NC + k) * COLS + t] = e[k];
    }
    __syncthreads();
    for (int v = tid; v < NC * COLS; v += THREADS) {
      const int k = v / COLS, c = v % COLS;
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) sum += red[(w * NC + k) * COLS + c];
      if (i0 + c < n) {
        if (k < 3) E[k * n + i0 + c] = sum;
        else phi[i0 + c] = sum;
      }
    }
  }
}

template <typename T, int COLS, int WAVES, bool KAHAN>
hipError_t launch_direct(int64_t n, const double* xyzq, double eps2, double* E, double* phi, hipStream_t st) {
  const int grid = (int)std::min<int64_t>((n + COLS - 1) / COLS, kGrid);
  if (phi) k_field_direct<T, COLS, WAVES, KAHAN, true><<<grid, 64 * WAVES, 0, st>>>(xyzq, n, eps2, E, phi);
  else k_field_direct<T, COLS, WAVES, KAHAN, false><<<grid, 64 * WAVES, 0, st>>>(xyzq, n, eps2, E, phi);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- each pair once
// The pair-once pass (force.hip) in its shape R = WJ = 4 (blocks of 256 charges, a thread block
// of 4 waves per tile), reading the caller's arrays and taking the potential along.  A tile (I, J),
// I <= J, leaves one row of sums for block I and, if I < J, one for block J.  The tiles go in
// strips of J so that a strip's rows fit the workspace: row (I, J) of the strip from J0 sits at
// J^2 - J0^2 + I, row (J, I) at J^2 - J0^2 + J + 1 + I, and a fold after each strip adds a charge's
// rows in a fixed order in FP64, and to the result of the strips before.
// Bound by VALU issue (pair_math.h has the rates); the potential adds two instructions a pair.  Measured
// a call: 20,000 charges with the potential in FP32 122 us, in FP64 196 us; 50,021 in FP64 without it
// 985 us, in four strips, against 2699, 1040 and 5245 us before; the one-sided kernels at their best
// tilings take 158, 311 and 1843 us.
constexpr int kPR = 4, kPB = 64 * kPR;  // targets per lane, charges per block

template <typename T, bool PHI>
struct PairLds {
  static constexpr int NC = PHI ? 4 : 3;
  T slice[4][4 * kN3Slice];  // a wave's sources, twice in a row
  T jres[NC][kPB];           // sums of the block's sources
  T ired[3][NC][kPB];        // sums of the targets by waves 1 to 3
};

template <typename T, bool PHI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 5)))
void k_field_pairs(const double* __restrict__ xyzq, int64_t n, double eps2d, T* __restrict__ rows, int64_t J0) {
  constexpr int NC = PHI ? 4 : 3, R = kPR;
  constexpr T kFar = N3Type<T>::kFar;
  __shared__ PairLds<T, PHI> s;
  const int64_t tile = J0 * (J0 + 1) / 2 + blockIdx.x;
  int64_t J = (int64_t)((sqrtf(8.0f * (float)tile + 1.0f) - 1.0f) * 0.5f);  // a guess, made exact below
  while (J * (J + 1) / 2 > tile) --J;
  while ((J + 1) * (J + 2) / 2 <= tile) ++J;
  const int64_t I = tile - J * (J + 1) / 2;
  const bool jside = I != J;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double *X = xyzq, *Y = xyzq + n, *Z = xyzq + 2 * n, *Q = xyzq + 3 * n;
  const int64_t i0 = I * kPB, jb = J * kPB + w * 64;

  // the lane's targets; places past the last charge lie so far away that they add nothing to a field
  const T qT = (T)Q[i0];
  T xi[R], yi[R], zi[R], qi[R];
  int same_t = 1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = i0 + r * 64 + lane;
    const bool live = i < n;
    xi[r] = live ? (T)X[i] : kFar;
    yi[r] = live ? (T)Y[i] : kFar;
    zi[r] = live ? (T)Z[i] : kFar;
    qi[r] = live ? (T)Q[i] : qT;
    same_t &= qi[r] == qT;
  }
  const bool ut = __all(same_t);
  const T eps2 = (T)eps2d;
  T f[4][R], a[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    a[k] = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) f[k][r] = 0;
  }
  if (jb < n) {  // the wave has sources
    const int64_t j = jb + lane;
    const bool live = j < n;
    const T q0 = (T)Q[jb];
    const T x = live ? (T)X[j] : kFar, y = live ? (T)Y[j] : kFar, z = live ? (T)Z[j] : kFar;
    const T q = live ? (T)Q[j] : T(0);
    // with the potential in FP64 a place past the last charge is one of charge 0: its 1/r of 1e-150 would
    // count among equal charges (FP32: 1/r is zero)
    const bool us = __all(PHI && sizeof(T) == 8 ? live && q == q0 : !live || q == q0);
    T* sb = s.slice[w];
    sb[lane] = sb[lane + 64] = x;
    sb[kN3Slice + lane] = sb[kN3Slice + lane + 64] = y;
    sb[2 * kN3Slice + lane] = sb[2 * kN3Slice + lane + 64] = z;
    sb[3 * kN3Slice + lane] = sb[3 * kN3Slice + lane + 64] = q;
    wave_lds_sync();
#define LC_CHUNK(US, UT, JS)                                                                                      \
  n3_chunk<T, R, 2, US, UT, JS, false, PHI>(sb, lane, xi, yi, zi, qi, eps2, f[0], f[1], f[2], a[0], a[1], a[2], T(0), T(0), \
                                         f[3], &a[3], w)
    if (jside) {
      if (us) {
        if (ut) LC_CHUNK(true, true, true);
        else LC_CHUNK(true, false, true);
      } else {
        if (ut) LC_CHUNK(false, true, true);
        else LC_CHUNK(false, false, true);
      }
    } else {
      if (us) LC_CHUNK(true, true, false);
      else LC_CHUNK(false, true, false);
    }
#undef LC_CHUNK
    if (us) {
#pragma unroll
      for (int k = 0; k < NC; ++k)
#pragma unroll
        for (int r = 0; r < R; ++r) f[k][r] *= q0;
    }
  }
  if (jside) {
    // E_j = sum_i q_i (r_j - r_i) s_ij = -(reaction sum); the potential keeps its sign
    const T qs = ut ? qT : T(1);
#pragma unroll
    for (int k = 0; k < NC; ++k) s.jres[k][w * 64 + lane] = (k < 3 ? -qs : qs) * a[k];
  }
  if (w > 0) {
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int r = 0; r < R; ++r) s.ired[w - 1][k][r * 64 + lane] = f[k][r];
  }
  __syncthreads();
  T* row = rows + (J * J - J0 * J0 + I) * NC * kPB;
  if (w == 0) {
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int l = r * 64 + lane;
        row[k * kPB + l] = ((f[k][r] + s.ired[0][k][l]) + s.ired[1][k][l]) + s.ired[2][k][l];
      }
  }
  if (jside) {
    row += (J + 1) * NC * kPB;
#pragma unroll
    for (int k = 0; k < NC; ++k) row[k * kPB + tid] = s.jres[k][tid];
  }
}

// A strip's rows of 64 charges of a block: kFoldWaves waves take them in turn, wave 0 adds the
// waves' sums in order.
template <typename T, bool PHI>
__global__ __launch_bounds__(64 * kFoldWaves) void k_field_fold(const T* __restrict__ rows, int64_t n, int64_t J0,
                                                                int64_t J1, double* E, double* phi) {
  constexpr int NC = PHI ? 4 : 3;
  __shared__ double red[kFoldWaves - 1][NC][64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const int64_t K = (int64_t)blockIdx.x * 64 / kPB;
  const int l = (int)(i - K * kPB);
  double e[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) e[k] = 0.0;
  // partners m < K (rows of the strip only if it holds J = K), then m = max(K, J0) .. J1 - 1
  const int64_t below = K >= J0 ? K : 0, from = K >= J0 ? K : J0;
  const int64_t total = below + (J1 - from);
  auto row_of = [&](int64_t v) {
    const int64_t J = from + (v - below);
    return rows + (v < below ? K * K - J0 * J0 + K + 1 + v : J * J - J0 * J0 + K) * NC * kPB + l;
  };
  int64_t v = w;
  for (; v + 3 * kFoldWaves < total; v += 4 * kFoldWaves) {
    T x[4][NC];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const T* r = row_of(v + u * kFoldWaves);
#pragma unroll
      for (int k = 0; k < NC; ++k) x[u][k] = r[k * kPB];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int k = 0; k < NC; ++k) e[k] += (double)x[u][k];
  }
  for (; v < total; v += kFoldWaves) {
    const T* r = row_of(v);
#pragma unroll
    for (int k = 0; k < NC; ++k) e[k] += (double)r[k * kPB];
  }
  if (w > 0) {
#pragma unroll
    for (int k = 0; k < NC; ++k) red[w - 1][k][lane] = e[k];
  }
  __syncthreads();
  if (w == 0 && i < n) {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      for (int q = 0; q < kFoldWaves - 1; ++q) e[k] += red[q][k][lane];
      double* out = k < 3 ? E + k * n + i : phi + i;
      *out = K < J0 ? *out + e[k] : e[k];  // an earlier strip has begun the sum
    }
  }
}

// Rows a strip may hold (the strip of blocks J0 .. J1 - 1 has J1^2 - J0^2).
template <typename T, bool PHI>
int64_t strip_rows() {
  return (int64_t)(LC_FIELD_STATIC_MAX_BYTES / (sizeof(T) * (PHI ? 4 : 3) * kPB));
}

template <typename T, bool PHI>
hipError_t launch_pairs(int64_t n, const double* xyzq, double eps2, double* E, double* phi, void* work,
                        hipStream_t st) {
  const int64_t nb = (n + kPB - 1) / kPB, cap = strip_rows<T, PHI>();
  for (int64_t J0 = 0; J0 < nb;) {
    int64_t J1 = J0;
    while (J1 < nb && (J1 + 1) * (J1 + 1) - J0 * J0 <= cap) ++J1;
    const int tiles = (int)(J1 * (J1 + 1) / 2 - J0 * (J0 + 1) / 2);
    k_field_pairs<T, PHI><<<tiles, 256, 0, st>>>(xyzq, n, eps2, (T*)work, J0);
    // blocks from J1 on have no rows in this strip
    const int64_t last = std::min<int64_t>(n, J1 * kPB);
    k_field_fold<T, PHI><<<(int)((last + 63) / 64), 64 * kFoldWaves, 0, st>>>((const T*)work, n, J0, J1, E, phi);
    J0 = J1;
  }
  return hipGetLastError();
}

}  // namespace
}  // namespace field_default

using namespace field_default;

// Each pair once past 4096 charges, as long as a strip can hold the rows of one J (up to 1,048,576
// charges in FP64 and 2,097,152 in FP32).  Up to there the direct kernel has one block of 16 targets per compute unit at
// most (4096 charges with the potential: 13.1 us in FP32 and 18.6 us in FP64, each pair once 18.6 and
// 22.2 us), beyond some have two (4099: 20.1 and 30.7 us against 18.8 and 22.2 us).  Kahan sums have
// no form that takes each pair once.
constexpr int64_t kPairsFrom = 16 * kUnits + 1;
bool strip_holds(int precision, int64_t n) {
  const int64_t nb = (n + kPB - 1) / kPB;
  return 2 * nb - 1 <= (precision == LC_FP64 ? strip_rows<double, true>() : strip_rows<float, true>());
}
bool field_pairs(int precision, int64_t n) {
  return precision != LC_FP32_KAHAN && n >= kPairsFrom && strip_holds(precision, n);
}

// Whether the one-sided kernel of force.hip takes a call that cannot take each pair once, for want of
// workspace or of rows in a strip.  Its blocks of 256 R targets (R = 4 in FP32, 2 in FP64) come in
// rounds of one per compute unit; with two rounds in FP32 and four in FP64 it is ahead of the direct kernel
// where the last round is nearly full: ms without the potential, one-sided and direct, FP32 520,000
// charges 92.8 and 95.8, 530,000 139 and 100, 780,000 203 and 217, 800,000 270 and 227; FP64 450,000
// 145 and 141, 520,000 170 and 187, 530,000 211 and 196, 600,000 240 and 251.  Beyond the strips it
// takes every call: FP32 2,100,000 1518 and 1561, FP64 1,060,000 743 and 776, 1,450,000 1340 and 1449.
bool field_one_sided(int precision, int64_t n) {
  if (precision == LC_FP32_KAHAN) return false;
  if (!strip_holds(precision, n)) return true;
  const bool wide = precision == LC_FP64;
  const int64_t round = kUnits * 256 * (wide ? 2 : 4), rounds = (n + round - 1) / round;
  return rounds >= (wide ? 4 : 2) && 100 * rounds * round <= (wide ? 110 : 105) * n;
}

size_t field_default_bytes(int precision, int64_t n) {
  if (!field_pairs(precision, n)) return 0;
  const int64_t nb = (n + kPB - 1) / kPB;
  const size_t row = (precision == LC_FP64 ? sizeof(double) : sizeof(float)) * 4 * kPB;
  return std::min<size_t>(LC_FIELD_STATIC_MAX_BYTES, (size_t)nb * (size_t)nb * row);
}

hipError_t launch_field_default(int precision, int64_t n, const double* xyzq, double eps2, double* E, double* phi,
                                void* work, size_t work_bytes, const ForceTiling& ft, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (field_pairs(precision, n) && work_bytes >= field_default_bytes(precision, n)) {
    if (precision == LC_FP64)
      return phi ? launch_pairs<double, true>(n, xyzq, eps2, E, phi, work, st)
                 : launch_pairs<double, false>(n, xyzq, eps2, E, phi, work, st);
    return phi ? launch_pairs<float, true>(n, xyzq, eps2, E, phi, work, st)
               : launch_pairs<float, false>(n, xyzq, eps2, E, phi, work, st);
  }
  if (field_one_sided(precision, n)) return launch_field_standalone(precision, n, xyzq, eps2, E, phi, work, ft, st);
  if (precision == LC_FP64) return launch_direct<double, 16, 16, false>(n, xyzq, eps2, E, phi, st);
  if (precision != LC_FP32_KAHAN) return launch_direct<float, 16, 16, false>(n, xyzq, eps2, E, phi, st);
  // Kahan sums of any size: up to a block of 16 targets per compute unit 16 waves each, beyond 8 waves
  // (20,000 charges: 223 against 243 us) with 16 targets, or with 8 where the last round of blocks
  // would leave more of the chip idle than their larger share of staging costs, about 8 % (4099: 21.3
  // against 24.8 us, 8200: 56 and 60, 8192: 49 and 46 us)
  const int64_t whole = (n + 16 * kUnits - 1) / (16 * kUnits), halves = (n + 8 * kUnits - 1) / (8 * kUnits);
  if (whole == 1) return launch_direct<float, 16, 16, true>(n, xyzq, eps2, E, phi, st);
  return 100 * 2 * whole <= 108 * halves ? launch_direct<float, 16, 8, true>(n, xyzq, eps2, E, phi, st)
                                         : launch_direct<float, 8, 8, true>(n, xyzq, eps2, E, phi, st);
}

}  // namespace lc
