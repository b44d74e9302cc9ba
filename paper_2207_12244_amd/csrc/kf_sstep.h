// Optimisation (Sec. II-C), the automatic fixed-count form of the float
// precisions: the same alternating Gauss-Newton scheme as kf_solve.hip, with
// each depth step solved by s-step conjugate gradients, S iterations per team
// synchronisation.
//
// Method. Jacobi-preconditioned CG on A x = b is CG on the symmetrically scaled
// system A' = D^-1/2 A D^-1/2, whose diagonal is 1, so A' = I - B with B the
// scaled couplings (spectrum inside (-1, 1)). One block forms the S products
// v_j = B^j r, reduces the 2 S moments <v_i, v_j>, i + j < 2 S, and then makes S
// iterations at once (Chronopoulos and Gear's s-step CG): the S directions
//   P := [v_0 .. v_S-1] + P B_c,   A'P := [v_j - v_j+1] + (A'P) B_c
// are made A'-conjugate to the previous block's, and the correction and the
// residual advance by P a and (A'P) a. B_c and a are S x S solves on the
// moments; the conjugation needs none of its own, because
// <A'P_i, v_j> = h_i+j with h_k = 0 for k < S - 1 and
// sum_i a_i h_i+j = -<r, v_j> (the residual is orthogonal to all earlier
// directions). In exact arithmetic these are CG's iterates; in FP32 they lie
// closer to FP64's than those of the pipelined recurrences (the correction is
// summed apart from x, the residual is formed from one update per S iterations).
//
// Bound and layout. A solve is a chain of dependent team-wide reductions, so it
// is bound by their latency: ~0.6 us for a word from one workgroup to another,
// ~1 us of reduction and polling around it. S iterations per reduction instead
// of one is what pays: 10 x 20 iterations make 60 (S = 4) or 110 (S = 2)
// synchronisations where pipelined CG makes 210 (640 x 480: 345 us on 228 tiles
// of 34 x 40, 637 us pipelined; 320 x 240: 256, 537; 160 x 120: 223, 502;
// 64 x 48: 210, 451; 4 tiles of 80 x 60 at 12 rows a thread: 756, 1050).
// Every workgroup holds its tile and a ghost frame S deep; thread (column,
// group) of the extended tile holds R vertically adjacent pixels, so the
// vertical neighbours of the stencil sit in its own registers and only the
// horizontal ones and the strip's two ends are read from LDS. The frame's rows
// are assembled like the owners' (from x shipped S + 1 deep with the scale step)
// and then advance by the same updates; the v_j that a frame pixel cannot form
// itself come from its owner beside the reduction, so a block costs one
// synchronisation and no second exchange. Of a block's 5.0 us at 640 x 480 the
// S stencil products take 0.8, the sums inside the workgroup 0.6, the wait for
// the other members' lines 0.75, the block's scalars 0.45.
#pragma once

#include "kf_device.h"

// Products and sums are contracted by expression, so that a keyframe's results do
// not depend on the kernel instance that solves it (alone, or in a batch).
#pragma clang fp contract(on)

namespace kf {

namespace {

constexpr int SS_NT = 512;            // threads per workgroup
constexpr int SS_NW = SS_NT / 64;

// a and b summed over the two halves of the wavefront: lanes 0-31 get a's, 32-63 b's.
__device__ inline double pair32(double a, double b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return __longlong_as_double(((long long)h[0] << 32) | (uint32_t)l[0]) +
         __longlong_as_double(((long long)h[1] << 32) | (uint32_t)l[1]);
}
// a and b summed over pairs of 16-lane rows: rows 0 and 2 get a's, rows 1 and 3 b's.
__device__ inline double pair16(double a, double b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return __longlong_as_double(((long long)h[0] << 32) | (uint32_t)l[0]) +
         __longlong_as_double(((long long)h[1] << 32) | (uint32_t)l[1]);
}
__device__ inline double row_sum16(double v) {   // every lane: the sum over its 16-lane row
  v += dpp_d<0x128, 0xf, true>(v);   // row_ror:8, 4, 2, 1
  v += dpp_d<0x124, 0xf, true>(v);
  v += dpp_d<0x122, 0xf, true>(v);
  v += dpp_d<0x121, 0xf, true>(v);
  return v;
}
__device__ inline double group_sum8(double v) {  // every lane: the sum over its aligned group of 8
  v += dpp_d<0xB1, 0xf, true>(v);    // quad_perm 1 0 3 2
  v += dpp_d<0x4E, 0xf, true>(v);    // quad_perm 2 3 0 1
  v += dpp_d<0x141, 0xf, true>(v);   // row_half_mirror
  return v;
}
// Wavefront totals of NV values in one pass: each exchange halves the values a
// lane still holds (10 additions for 8 values instead of 48), and lane group g
// of 64 / NV lanes ends with the total of value g.
template <int NV>
__device__ inline double wave_totals(const double* v) {
  static_assert(NV == 4 || NV == 8, "4 or 8 values");
  if constexpr (NV == 4) {
    return row_sum16(pair16(pair32(v[0], v[2]), pair32(v[1], v[3])));
  } else {
    const double a = pair16(pair32(v[0], v[4]), pair32(v[2], v[6]));   // rows: 0, 2, 4, 6
    const double c = pair16(pair32(v[1], v[5]), pair32(v[3], v[7]));   // rows: 1, 3, 5, 7
    const bool up = (threadIdx.x & 8) != 0;
    double keep = up ? c : a;
    keep += dpp_d<0x128, 0xf, true>(up ? a : c);
    return group_sum8(keep);
  }
}

// LDS of one workgroup: wavefront partials, totals, the block's scalars; then
// ss_arrays arrays of a.cells cells over the extended tile with a guard ring.
template <int S>
struct SsHead {
  static constexpr int NV = 2 * S;
  double wred[NV * SS_NW];   // per value and wavefront: the workgroup's sums
  double wsum[NV * SS_NW];   // the same of the team's partials that each wavefront has polled
  double tot[NV];        // team totals
  double w[S * S];       // W = P^T A' P, lower triangle
  double winv[S * S];    // the previous block's W^-1 (S = 4)
  double tz[10];         // its tau_k at [6 + k] (S = 4), zeros before
  double fac[14];        // its solve: 2 x 2 parts and a
  double tau;
  float coef[2][S * S + S];  // B_c (row-major), a, of this block and the one before
  int stop;              // 1: CG ends with this block, 2: before it
  int abort;
};

__device__ inline double rcp_d(double x) {   // 1 / x to about an ulp
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  return fma(y, fma(-x, y, 1.0), y);
}
template <int K>
__device__ inline double quad_bcast(double v) {   // lane K's value of each quad
  return dpp_d<K * 0x55, 0xf, true>(v);
}

// W = L D L^T and a = W^-1 (m_0 .. m_q-1) on the first q < S directions, or on
// those before a pivot that vanishes: the block's directions are dependent, CG
// has converged and ends with this block (returns false). The slow way, for a
// last block of fewer iterations, for convergence, and for a residual that is not
// finite.
template <int S>
__device__ __forceinline__ bool solve_leading(SsHead<S>* hd, const double* m, int q, double* a) {
  double L[S][S], D[S], iD[S];
  bool good = true;
#pragma unroll
  for (int i = 0; i < S; ++i) {
    D[i] = hd->w[i * S + i];
    a[i] = m[i];
#pragma unroll
    for (int j = 0; j < i; ++j) {
      double l = hd->w[i * S + j];
#pragma unroll
      for (int k = 0; k < j; ++k) l -= L[i][k] * L[j][k] * D[k];
      L[i][j] = l * iD[j];
      D[i] -= L[i][j] * l;
      a[i] -= L[i][j] * a[j];
    }
    if (i < q) good = good && D[i] > 1e-11 * fabs(m[2 * i] - m[2 * i + 1]);
    iD[i] = good ? 1.0 / D[i] : 0.0;
  }
#pragma unroll
  for (int i = S - 1; i >= 0; --i) {
    a[i] *= iD[i];
#pragma unroll
    for (int k = i + 1; k < S; ++k) a[i] -= L[k][i] * a[k];
    if (i >= q || iD[i] == 0.0) a[i] = 0.0;
    if (!(m[0] < (double)INFINITY)) a[i] = m[0] - m[0];   // shown, not passed over: x becomes NaN
  }
  return good;
}

// The S x S part of one block, by one wavefront. `prepare` forms what depends on
// the previous block alone, while the totals are on their way; `finish` takes
// the moments m[k] = <v_i, v_j>, i + j = k, and writes B_c and a for q <= S
// iterations. It lies on the critical path of every block, so it is kept short:
// with tau the power series inverse of a, h = -tau * m and so B_c = -W_prev^-1 C
// are linear in the moments, with coefficients that `prepare` has ready (S = 4:
// lane 4 j + i holds entry (i, j)), and W is inverted by 2 x 2 parts with two
// reciprocals.
template <int S>
struct BlockScalars;

template <>
struct BlockScalars<2> {
  double wi00, wi01, wi11, a0, ia;
  __device__ __forceinline__ void prepare(SsHead<2>* hd, int) {
    const double rd = hd->fac[3];
    wi00 = hd->fac[2] * rd;
    wi01 = -hd->fac[1] * rd;
    wi11 = hd->fac[0] * rd;
    a0 = hd->fac[4];
    ia = rcp_d(hd->fac[5]);
  }
  __device__ __forceinline__ bool finish(SsHead<2>* hd, float* coef, const double* m, bool first, int q,
                                         int lane) {
    double w00 = m[0] - m[1], w10 = m[1] - m[2], w11 = m[2] - m[3];
    const double g11 = w11;
    if (!first) {
      const double h1 = -m[0] * ia, h2 = -fma(a0, h1, m[1]) * ia;
      const double b00 = -wi01 * h1, b10 = -wi11 * h1;
      const double b01 = -fma(wi00, h1, wi01 * h2), b11 = -fma(wi01, h1, wi11 * h2);
      w00 = fma(h1, b10, w00);
      w10 = fma(h1, b00, fma(h2, b10, w10));
      w11 = fma(h1, b01, fma(h2, b11, w11));
      if (lane == 0) {
        coef[0] = (float)b00;
        coef[1] = (float)b01;
        coef[2] = (float)b10;
        coef[3] = (float)b11;
      }
    }
    const double det = fma(w00, w11, -w10 * w10);
    const double rd = rcp_d(det);
    double a[2] = {fma(w11, m[0], -w10 * m[1]) * rd, fma(w00, m[1], -w10 * m[0]) * rd};
    // a pivot is a difference of moments that carry FP32 rounding; this far
    // below its first term nothing of it is left
    bool good = w00 > 1e-11 * fabs(m[0] - m[1]) && det > 1e-11 * fabs(g11) * w00;
    if (!good || q < 2) {
      if (lane == 0) {
        hd->w[0] = w00;
        hd->w[2] = w10;
        hd->w[3] = w11;
      }
      __builtin_amdgcn_wave_barrier();
      good = solve_leading<2>(hd, m, q, a);
    }
    if (lane == 0) {
      coef[4] = (float)a[0];
      coef[5] = (float)a[1];
      hd->fac[0] = w00;
      hd->fac[1] = w10;
      hd->fac[2] = w11;
      hd->fac[3] = rd;
      hd->fac[4] = a[0];
      hd->fac[5] = a[1];
    }
    return good;
  }
};

template <>
struct BlockScalars<4> {
  double sg[4];   // h[k + i] = -sum_l sg[k - l] m[l]
  double mc[4];   // B_c(i, j) = sum_l mc[l] m[l]
  __device__ __forceinline__ void prepare(SsHead<4>* hd, int lane) {
    const int i = lane & 3, j = (lane >> 2) & 3;
    const double* f = hd->fac;   // A'^-1: 0-2, X: 3-6, Schur complement's inverse: 7-9, a: 10-13
    const double t0 = rcp_d(f[13]);
    const double t1 = -t0 * (f[12] * t0);
    const double t2 = -t0 * fma(f[12], t1, f[11] * t0);
    const double t3 = -t0 * fma(f[12], t2, fma(f[11], t1, f[10] * t0));
    // W^-1 = [A^-1 + X^T S^-1 X, -X^T S^-1; -S^-1 X, S^-1]
    const double y00 = fma(f[7], f[3], f[8] * f[5]), y01 = fma(f[7], f[4], f[8] * f[6]);
    const double y10 = fma(f[8], f[3], f[9] * f[5]), y11 = fma(f[8], f[4], f[9] * f[6]);
    const double v00 = fma(f[3], y00, fma(f[5], y10, f[0])), v01 = fma(f[3], y01, fma(f[5], y11, f[1]));
    const double v11 = fma(f[4], y01, fma(f[6], y11, f[2]));
    if (lane == 0) {
      double* w = hd->winv;
      w[0] = v00; w[1] = v01; w[2] = -y00; w[3] = -y10;
      w[4] = v01; w[5] = v11; w[6] = -y01; w[7] = -y11;
      w[8] = -y00; w[9] = -y01; w[10] = f[7]; w[11] = f[8];
      w[12] = -y10; w[13] = -y11; w[14] = f[8]; w[15] = f[9];
      double* t = hd->tz;
#pragma unroll
      for (int k = 0; k < 6; ++k) t[k] = 0.0;
      t[6] = t0; t[7] = t1; t[8] = t2; t[9] = t3;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < 4; ++k) sg[k] = hd->tz[3 + k + i];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      mc[l] = 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) mc[l] = fma(hd->winv[4 * i + k], hd->tz[3 + k + j - l], mc[l]);
    }
  }
  __device__ __forceinline__ bool finish(SsHead<4>* hd, float* coef, const double* m, bool first, int q,
                                         int lane) {
    const double g00 = m[0] - m[1], g11 = m[2] - m[3], g22 = m[4] - m[5], g33 = m[6] - m[7];
    double w00 = g00, w10 = m[1] - m[2], w11 = g11, w20 = g11, w21 = m[3] - m[4], w22 = g22;
    double w30 = w21, w31 = g22, w32 = m[5] - m[6], w33 = g33;
    if (!first) {
      const double bc = fma(mc[0], m[0], fma(mc[1], m[1], fma(mc[2], m[2], mc[3] * m[3])));
      double kk = 0.0;   // entry (i, j) of C^T B_c
      const double b0 = quad_bcast<0>(bc), b1 = quad_bcast<1>(bc), b2 = quad_bcast<2>(bc), b3 = quad_bcast<3>(bc);
      const double h0 = sg[0] * m[0];
      const double h1 = fma(sg[1], m[0], sg[0] * m[1]);
      const double h2 = fma(sg[2], m[0], fma(sg[1], m[1], sg[0] * m[2]));
      const double h3 = fma(sg[3], m[0], fma(sg[2], m[1], fma(sg[1], m[2], sg[0] * m[3])));
      kk = fma(h0, b0, fma(h1, b1, fma(h2, b2, h3 * b3)));
      if (lane < 16) {
        coef[4 * (lane & 3) + (lane >> 2)] = (float)bc;
        hd->w[4 * (lane & 3) + (lane >> 2)] = kk;
      }
      __builtin_amdgcn_wave_barrier();
      w00 -= hd->w[0];
      w10 -= hd->w[4]; w11 -= hd->w[5];
      w20 -= hd->w[8]; w21 -= hd->w[9]; w22 -= hd->w[10];
      w30 -= hd->w[12]; w31 -= hd->w[13]; w32 -= hd->w[14]; w33 -= hd->w[15];
    }
    const double da = fma(w00, w11, -w10 * w10), ra = rcp_d(da);
    const double x00 = fma(w20, w11, -w21 * w10) * ra, x01 = fma(w21, w00, -w20 * w10) * ra;
    const double x10 = fma(w30, w11, -w31 * w10) * ra, x11 = fma(w31, w00, -w30 * w10) * ra;
    const double s00 = w22 - fma(x00, w20, x01 * w21), s10 = w32 - fma(x10, w20, x11 * w21);
    const double s11 = w33 - fma(x10, w30, x11 * w31);
    const double ds = fma(s00, s11, -s10 * s10), rs = rcp_d(ds);
    const double i00 = w11 * ra, i01 = -w10 * ra, i11 = w00 * ra;
    const double t0 = m[2] - fma(x00, m[0], x01 * m[1]), t1 = m[3] - fma(x10, m[0], x11 * m[1]);
    double a[4];
    a[2] = fma(s11, t0, -s10 * t1) * rs;
    a[3] = fma(s00, t1, -s10 * t0) * rs;
    a[0] = fma(i00, m[0], i01 * m[1]) - fma(x00, a[2], x10 * a[3]);
    a[1] = fma(i01, m[0], i11 * m[1]) - fma(x01, a[2], x11 * a[3]);
    constexpr double tiny = 1e-11;   // as in the 2 x 2 case
    bool good = w00 > tiny * fabs(g00) && da > tiny * fabs(g11) * w00 && s00 > tiny * fabs(g22) &&
                ds > tiny * fabs(g33) * s00;
    if (!good || q < 4) {
      if (lane == 0) {
        double* w = hd->w;
        w[0] = w00;
        w[4] = w10; w[5] = w11;
        w[8] = w20; w[9] = w21; w[10] = w22;
        w[12] = w30; w[13] = w31; w[14] = w32; w[15] = w33;
      }
      __builtin_amdgcn_wave_barrier();
      good = solve_leading<4>(hd, m, q, a);
    }
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) coef[16 + k] = (float)a[k];
      double* f = hd->fac;
      f[0] = i00; f[1] = i01; f[2] = i11;
      f[3] = x00; f[4] = x01; f[5] = x10; f[6] = x11;
      f[7] = s11 * rs; f[8] = -s10 * rs; f[9] = s00 * rs;
#pragma unroll
      for (int k = 0; k < 4; ++k) f[10 + k] = a[k];
    }
    return good;
  }
};

// Whether the kernels of R rows per thread keep the static row inputs in LDS
// (larger tiles read them again in every Gauss-Newton iteration).
__host__ __device__ constexpr bool ss_resident(int rows) { return rows <= 6; }
// LDS arrays over the extended tile: x, the scaling, the static row inputs, and
// short strips' stencil operands.
__host__ __device__ constexpr bool ss_shift(int rows) { return rows >= 8; }
__host__ __device__ constexpr int ss_arrays(int rows) {
  return (ss_resident(rows) ? 10 : 4) + (ss_shift(rows) ? 0 : 2);
}

// What long strips exchange: their top and bottom pixels, and those of the
// wavefronts' first and last lanes (two buffers by turns).
template <int R>
struct SsEnds {
  float top[2][SS_NT], bottom[2][SS_NT];
  __align__(16) float edge[2][SS_NW + 2][2][(R + 3) & ~3];
};
__host__ __device__ constexpr size_t ss_align16(size_t n) { return (n + 15) & ~(size_t)15; }
__host__ __device__ constexpr size_t ss_head_bytes(int s, int rows) {
  return ss_align16(s == 2 ? sizeof(SsHead<2>) : sizeof(SsHead<4>)) +
         (ss_shift(rows) ? sizeof(float) * (4 * SS_NT + 4 * (SS_NW + 2) * (size_t)((rows + 3) & ~3)) : 0);
}

// A copy in a register of its own. (Left to the compiler, the copies of v share
// registers with what `take` loads into, and it waits for those loads at once.)
__device__ inline float copy_of(float v) {
  float c;
  asm("v_mov_b32 %0, %1" : "=v"(c) : "v"(v));
  return c;
}

// v of the lane before (0x138, wave_shr:1) or after (0x130, wave_shl:1); `old`
// at the wavefront's end.
template <int CTRL>
__device__ inline float lane_shift(float old, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Pixel data of the exchange region: agent-scope (written through to, and read
// from, the level that all XCDs share).
__device__ inline void st_float(KF_GLOBAL float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline float ld_float(const KF_GLOBAL float* p) {
  return __hip_atomic_load(const_cast<KF_GLOBAL float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Index of pixel (lx, ly) of a tw x th tile in its boundary frame.
template <int S>
__device__ inline int frame_index(int lx, int ly, int tw, int th, int tile_w) {
  constexpr int D = S + 1;
  if (ly < D) return ly * tile_w + lx;
  if (ly >= th - D) return (2 * D + ly - th) * tile_w + lx;
  return 2 * D * tile_w + (ly - D) * 2 * D + (lx < D ? lx : 2 * D + lx - tw);
}

// Tile of member b. Workgroups go to the 8 XCDs in turn; this gives those of one
// XCD a compact patch of tiles (runs of a path through vertical strips), whose
// pixel data then stays in its L2.
__device__ inline int tile_of(int b, int tx, int ty) {
  const int B = tx * ty, x = b & 7, n = B >> 3;
  const int rank = x * n + min(x, B & 7) + (b >> 3);
  const int strips = max(1, (int)(tx / sqrtf(0.125f * B) + 0.5f));
  const int w = (tx + strips - 1) / strips;
  const int s = rank / (w * ty), r = rank - s * w * ty, ws = min(w, tx - s * w);
  return (r / ws) * tx + s * w + r % ws;
}

// Member b of the team that solves keyframe `a`. R: pixels a thread
// holds (a.rows). VAR as in kf_solve.hip.
template <int R, int S, bool VAR>
__device__ __forceinline__ void sstep_member(const SolveArgs& a, const int b, unsigned char* smem) {
  constexpr int NV = 2 * S;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int W = a.W, H = a.H, N = W * H;
  const int B = a.tiles_x * a.tiles_y;
  SsHead<S>* hd = reinterpret_cast<SsHead<S>*>(smem);
  float* X = reinterpret_cast<float*>(smem + ss_head_bytes(S, R));
  float* SC = X + a.cells;
  float* ST = SC + a.cells;   // static row inputs (RowIn): z and 1 / sqrt(R), and all eight if RES
  constexpr bool RES = ss_resident(R);
  // The stencil operands that cross threads, in two buffers by turns. Short
  // strips write all their pixels (arrays like X, behind ST). Long ones (SHIFT)
  // write their top and bottom pixel, take the horizontal neighbours by lane
  // shifts, and write whole strips at a wavefront's first and last lane only:
  // LDS traffic bounds them (12 rows: 94 against 116 us of a 160 x 120 solve), while 4
  // rows are bound by latency, which the shifts lengthen (50 against 46 us, 640 x 480).
  constexpr bool SHIFT = ss_shift(R);
  float* V = ST + (RES ? 8 : 2) * a.cells;
  using Ends = SsEnds<R>;
  Ends* se = reinterpret_cast<Ends*>(smem + ss_align16(sizeof(SsHead<S>)));

  // ---- geometry: own tile, ghost frame up to S deep inside the image
  const int tile = tile_of(b, a.tiles_x, a.tiles_y);
  const int ox = (tile % a.tiles_x) * a.tile_w, oy = (tile / a.tiles_x) * a.tile_h;
  const int tw = min(a.tile_w, W - ox), th = min(a.tile_h, H - oy);
  const int gl = min(S, ox), gt = min(S, oy), gr = min(S, W - ox - tw), gb = min(S, H - oy - th);
  const int EW = gl + tw + gr, EH = gt + th + gb, st = EW + 2;
  const int c = threadIdx.x % EW, g = threadIdx.x / EW;
  const int ey0 = g * R;
  const bool live = ey0 < EH;
  int l0 = live ? (ey0 + 1) * st + c + 1 : st + 1;
  int u = ox - gl + c, vtop = oy - gt + ey0;

  for (int i = threadIdx.x; i < ss_arrays(R) * a.cells; i += SS_NT) X[i] = 0.0f;
  if constexpr (SHIFT) {
    static_assert(ss_align16(sizeof(SsHead<S>)) + sizeof(Ends) == ss_head_bytes(S, R), "layout");
    for (int i = threadIdx.x; i < (int)(sizeof(se->edge) / sizeof(float)); i += SS_NT) (&se->edge[0][0][0][0])[i] = 0.0f;
  }
  if (threadIdx.x == 0) hd->abort = 0;

  KF_GLOBAL DevScalars* scal = gp(a.scal);
  KF_GLOBAL int32_t* err = &scal->err;
  KF_GLOBAL uint64_t* parts = gp(a.parts);
  KF_GLOBAL float* halo = gp(reinterpret_cast<float*>(a.halo));   // [2][B][fw][S]
  const int fw = sstep_frame_words(a.tile_w, a.tile_h, S);

  // Per slot: its pixel's place in the exchange region, and what it is: an own
  // pixel (that ships its v_j, and x one pixel further in) or a ghost pixel.
  constexpr int OWN = 1 << 27, GHOST = 1 << 28, VPUB = 1 << 29, XPUB = 1 << 30;
  int meta[R];
  uint32_t own_bits = 0;
  auto word_of = [&](int pu, int pv) {
    const int tx = pu / a.tile_w, ty = pv / a.tile_h;
    const int bx = tx * a.tile_w, by = ty * a.tile_h;
    return (ty * a.tiles_x + tx) * fw +
           frame_index<S>(pu - bx, pv - by, min(a.tile_w, W - bx), min(a.tile_h, H - by), a.tile_w);
  };
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int ey = ey0 + j;
    meta[j] = 0;
    if (!live || ey >= EH) continue;
    const int v = vtop + j;
    // distances from the tile's edges (1: the edge row or column itself) and depths beyond them
    const int il = c - gl + 1, ir = gl + tw - c, it = ey - gt + 1, ib = gt + th - ey;
    if (il > 0 && ir > 0 && it > 0 && ib > 0) {
      own_bits |= 1u << j;
      meta[j] = OWN;
      int near = S + 2;   // distance from the nearest edge with a neighbour behind it
      if (gl > 0) near = min(near, il);
      if (gr > 0) near = min(near, ir);
      if (gt > 0) near = min(near, it);
      if (gb > 0) near = min(near, ib);
      if (near <= S + 1) meta[j] |= XPUB | (near <= S ? VPUB : 0) | word_of(u, v);
    } else {
      meta[j] = GHOST | word_of(u, v);
    }
  }
  // the ring of x beyond the ghost frame (depth S + 1), one cell per thread
  int ring_off = -1, ring_li = 0, ring_u = 0, ring_v = 0;
  {
    const int k = threadIdx.x;
    int cx, cy;
    if (k < EW) { cx = k; cy = -1; }
    else if (k < 2 * EW) { cx = k - EW; cy = EH; }
    else if (k < 2 * EW + EH) { cx = -1; cy = k - 2 * EW; }
    else { cx = EW; cy = k - 2 * EW - EH; }
    ring_u = ox - gl + cx;
    ring_v = oy - gt + cy;
    if (k < 2 * (EW + EH) && ring_u >= 0 && ring_u < W && ring_v >= 0 && ring_v < H) {
      ring_off = word_of(ring_u, ring_v);
      ring_li = (cy + 1) * st + cx + 1;
    }
  }

  const KF_GLOBAL float* pr = gp(static_cast<const float*>(a.prior));
  const KF_GLOBAL float* mu_g = pr;
  const KF_GLOBAL float* isn_g = pr + (size_t)N;
  const KF_GLOBAL float* gx_g = pr + 2 * (size_t)N;
  const KF_GLOBAL float* isx_g = pr + 3 * (size_t)N;
  const KF_GLOBAL float* gy_g = pr + 4 * (size_t)N;
  const KF_GLOBAL float* isy_g = pr + 5 * (size_t)N;
  KF_GLOBAL float* x_g = gp(static_cast<float*>(a.x));
  const KF_GLOBAL float* rho_g = gp(static_cast<const float*>(a.rho));
  const KF_GLOBAL float* var_g = gp(static_cast<const float*>(a.var));

  const float delta = (float)a.huber_delta, r_floor = (float)a.r_floor;
  const bool postfit = VAR && a.variant == KF_VARIANT_SCALE_POSTFIT;
  const bool tukey = VAR && a.robust == KF_ROBUST_TUKEY;
  double tau = scal->tau;
  const float x_shift = postfit ? (float)tau : 0.0f;
  int new_kf = 0;   // keyframe rule (Sec. II)
  if (VAR && a.lambda_trans > 0.0 && scal->frame_trans[a.buf] > a.lambda_trans) new_kf |= KF_NEW_KEYFRAME_TRANSLATION;
  if (VAR && a.lambda_inliers > 0 && scal->n_updated[a.buf] < a.lambda_inliers) new_kf |= KF_NEW_KEYFRAME_INLIERS;
  const uint32_t e0 = scal->epoch;
  uint32_t e = e0;

  __syncthreads();   // LDS cleared
  // x of the extended tile and its ring straight from the state (consistent at launch)
#pragma unroll
  for (int j = 0; j < R; ++j)
    if (meta[j] & (OWN | GHOST)) X[l0 + j * st] = x_g[(vtop + j) * W + u] - x_shift;
  if (ring_off >= 0) X[ring_li] = x_g[ring_v * W + ring_u] - x_shift;
  if (postfit && !new_kf) tau = 0.0;
  __syncthreads();

  // Team-wide totals of the NV per-thread values, handed to `use` in wavefront 2
  // (which leaves what the others need in hd). Every member writes its NV partial
  // sums as one line of epoch-tagged words; wavefront w of every member polls the
  // lines of members 8 Q w .. 8 Q (w + 1) - 1. A line has one writer and is
  // written once, so a poll that comes too early costs a second trip of the line;
  // the wavefronts first sleep for most of the ~0.6 us that a word takes (256
  // members, 8 values: 2.0 us per synchronisation, 2.7 without the sleep, 2.5
  // with a second hop through one member per value, 4.5 with the words of a value
  // side by side). The pixel data that `publish` ships has no tags: it is written
  // through, and complete, before the member's line, so whoever has seen all
  // lines may read it (`take`). `prep` (wavefront 2) and `aside` (everybody) need no
  // totals and run while they are on their way. The order of summation follows from the team's
  // size alone. Returns false if the team aborts.
  auto team_sync = [&](const double* vals, auto publish, auto take, auto prep, auto aside, auto use) -> bool {
    const uint32_t par = e & 1u;
    if (B > 1) publish(par);
    const double wt = wave_totals<NV>(vals);
    if (lane % (64 / NV) == 0) hd->wred[(lane / (64 / NV)) * SS_NW + wave] = wt;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    auto waves_sum = [&]() {   // lane (value, wavefront) of 8 x 8: every lane its value's sum
      return group_sum8(lane < NV * SS_NW ? hd->wred[lane] : 0.0);
    };
    if (B > 1) {
      if (wave == 0) {
        const double p = waves_sum();
        if ((lane & 7) == 0 && lane < NV * 8)
          st_word(parts + ((size_t)par * B + b) * 16 + (lane >> 3), Packed48::make_word(p, e));
      }
      aside();
      prep();
      const int Q = (B + 63) >> 6;
      const int m0 = wave * 8 * Q + (lane >> 3), k = lane & 7;
      double t = 0.0;
      if (wave * 8 * Q < B) {
        const KF_GLOBAL uint64_t* p = parts + (size_t)par * B * 16 + (k < NV ? k : 0);
        uint64_t w[4];
        unsigned spins = 0;
        uint64_t t0 = 0;
        bool dead = false;
        __builtin_amdgcn_s_sleep(12);
        while (true) {
          bool all = true;
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q < Q) w[q] = ld_word(p + min(m0 + 8 * q, B - 1) * 16);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (q < Q) all = all && Packed48::ready(w[q], e);
          if (__all(all)) break;
          if ((++spins & 63u) == 0u) {
            const uint64_t now = wall_clock64();
            if (t0 == 0) t0 = now;
            dead = now - t0 > a.timeout_ticks ||
                   (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ERR_TIMEOUT);
            if (__any(dead)) break;
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q < Q) t += m0 + 8 * q < B ? Packed48::value(w[q]) : 0.0;
        if (__any(dead) && lane == 0) {
          hd->abort = 1;
          __hip_atomic_fetch_or(err, ERR_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        t += dpp_d<0x128, 0xf, true>(t);
        t = pair16(t, t);
        t = pair32(t, t);
      }
      if (lane < NV) hd->wsum[lane * SS_NW + wave] = t;
      __syncthreads();
      if (hd->abort) return false;
      take(par);
    } else {
      prep();
      if (wave != 2) aside();
    }
    if (wave == 2) {
      const double t = B > 1 ? group_sum8(lane < NV * SS_NW ? hd->wsum[lane] : 0.0) : waves_sum();
      if ((lane & 7) == 0 && lane < NV * 8) hd->tot[lane >> 3] = t;
      __builtin_amdgcn_wave_barrier();
      double m[NV];
#pragma unroll
      for (int k = 0; k < NV; ++k) m[k] = hd->tot[k];
      use(m);
      if (B == 1) aside();
    }
    ++e;
    __syncthreads();
    return true;
  };

  // Static inputs of pixel i = (u, v): network log-depth and its inverse sigma,
  // the semi-dense measurement in log space (Sec. II-B last step: z = -ln rho,
  // 1 / sqrt(R) with R = max(v / rho^2, R_floor), 0 where there is none), and the
  // prior gradients to the right and below with their inverse sigmas (0 for an
  // edge that leaves the image: such an edge gets weight 0 without a branch).
  struct RowIn {
    float mu, isn, gx, isx, gy, isy;
  };
  auto semi = [&](float rho, float var, float& isr) -> float {
    const bool has = var > 0.0f;
    const float q = has ? rho : 1.0f;
    float Rv = (has ? var : 1.0f) / (q * q);
    Rv = Rv > r_floor ? Rv : r_floor;
    isr = has ? 1.0f / sqrt(Rv) : 0.0f;
    return has ? -log(q) : 0.0f;
  };
  auto row_in = [&](int pu, int pv) -> RowIn {
    const int i = pv * W + pu;
    RowIn q;
    q.mu = mu_g[i];
    q.isn = isn_g[i];
    q.gx = gx_g[i];
    q.isx = pu < W - 1 ? isx_g[i] : 0.0f;
    q.gy = gy_g[i];
    q.isy = pv < H - 1 ? isy_g[i] : 0.0f;
    if (!(pu < W - 1)) q.gx = 0.0f;
    if (!(pv < H - 1)) q.gy = 0.0f;
    return q;
  };
  const int cells = a.cells;
  // Read once per launch: the semi-dense measurement, and with RES all of a row's
  // inputs (the cells left of and above the extended tile hold the edges into it)
  constexpr int CH = R < 6 ? R : 2;   // rows whose loads are in flight together
#pragma unroll
  for (int j0 = 0; j0 < R; j0 += CH) {
#pragma unroll
    for (int j = j0; j < j0 + CH && j < R; ++j) {
      if (!(meta[j] & (OWN | GHOST))) continue;
      const int i = (vtop + j) * W + u;
      float* t = ST + l0 + j * st;
      t[0] = semi(rho_g[i], var_g[i], t[cells]);
      if constexpr (RES) {
        const RowIn q = row_in(u, vtop + j);
        t[2 * cells] = q.mu;
        t[3 * cells] = q.isn;
        t[4 * cells] = q.gx;
        t[5 * cells] = q.isx;
        t[6 * cells] = q.gy;
        t[7 * cells] = q.isy;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (RES) {
    if (ring_off >= 0 && ring_u < ox - gl) {
      ST[4 * cells + ring_li] = gx_g[ring_v * W + ring_u];
      ST[5 * cells + ring_li] = isx_g[ring_v * W + ring_u];
    }
    if (ring_off >= 0 && ring_v < oy - gt) {
      ST[6 * cells + ring_li] = gy_g[ring_v * W + ring_u];
      ST[7 * cells + ring_li] = isy_g[ring_v * W + ring_u];
    }
    __syncthreads();
  }

  int cg_total = 0;
  double n_valid = 0.0;
  const size_t plane = (size_t)B * fw * S;   // floats of one parity
  for (int gn = 0; gn < (new_kf ? 0 : a.n_gn); ++gn) {
#pragma unroll
    for (int j = 0; j < R; ++j) refresh(meta[j]);
    refresh(ring_off);
    refresh(u);
    refresh(vtop);
    refresh(l0);
    // ---- IRLS weights and 5-point normal equations at (x, tau) (Sec. II-C),
    //      scaled: couplings c / sqrt(d d'), residual (b - A x) / sqrt(d)
    float r[R], cl[R], cr[R], cv[R + 1];
    {
      float wu = 0.0f, gu = 0.0f;   // the edge above: its weight and prior gradient
      if (live) {
        float isd = 0.0f;
        if constexpr (RES) {
          gu = ST[6 * cells + l0 - st];
          isd = ST[7 * cells + l0 - st];
        } else if (vtop > 0) {
          gu = gy_g[(vtop - 1) * W + u];
          isd = isy_g[(vtop - 1) * W + u];
        }
        wu = edge_weight(X[l0 - st], X[l0], gu, isd, delta, tukey);
      }
      cv[0] = wu;
#pragma unroll
      for (int j0 = 0; j0 < R; j0 += CH) {
        RowIn qs[CH];
        float gls[CH], isls[CH];   // the edge to the left
        if constexpr (!RES) {
#pragma unroll
          for (int j = j0; j < j0 + CH && j < R; ++j) {
            if (!(meta[j] & (OWN | GHOST))) continue;
            qs[j - j0] = row_in(u, vtop + j);
            const int il = (vtop + j) * W + max(u - 1, 0);
            gls[j - j0] = gx_g[il];
            isls[j - j0] = u > 0 ? isx_g[il] : 0.0f;
          }
        }
#pragma unroll
        for (int j = j0; j < j0 + CH && j < R; ++j) {
          r[j] = cl[j] = cr[j] = cv[j + 1] = 0.0f;
          if (!(meta[j] & (OWN | GHOST))) {   // below the extended tile: no coupling to the row above
            cv[j] = 0.0f;
            continue;
          }
          const int l = l0 + j * st;
          const float* t = ST + l;
          const float zs = t[0], isr = t[cells];
          RowIn q = qs[j - j0];
          float gleft = gls[j - j0], isl = isls[j - j0];
          if constexpr (RES) {
            q.mu = t[2 * cells];
            q.isn = t[3 * cells];
            q.gx = t[4 * cells];
            q.isx = t[5 * cells];
            q.gy = t[6 * cells];
            q.isy = t[7 * cells];
            gleft = t[4 * cells - 1];
            isl = t[5 * cells - 1];
          }
          const float xi = X[l], xl = X[l - 1], xr = X[l + 1], xu = X[l - st], xd = X[l + st];
          const float wn = postfit ? 0.0f : huber_w((xi - q.mu) * q.isn, delta, tukey) * q.isn * q.isn;
          const float ws = huber_w((xi - (float)tau - zs) * isr, delta, tukey) * isr * isr;
          const float wr = edge_weight(xi, xr, q.gx, q.isx, delta, tukey);
          const float wl = edge_weight(xl, xi, gleft, isl, delta, tukey);
          const float wd = edge_weight(xi, xd, q.gy, q.isy, delta, tukey);
          const float bb = wn * q.mu + ws * ((float)tau + zs) - wr * q.gx + wl * gleft - wd * q.gy + wu * gu;
          const float d = wn + ws + wr + wl + wd + wu;
          const float sc = d > 0.0f ? 1.0f / sqrt(d) : 0.0f;   // d = 0: every term has weight 0, x stays
          SC[l] = sc;
          r[j] = (bb - (d * xi - wr * xr - wl * xl - wd * xd - wu * xu)) * sc;
          cl[j] = wl * sc;
          cr[j] = wr * sc;
          cv[j] *= sc;            // the edge above: this pixel's factor
          cv[j + 1] = wd * sc;    // the edge below: the other factor follows
          wu = wd;
          gu = q.gy;
        }
        // (the loads of all rows at once would take the registers of the rows)
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    // the other factor of each coupling (0 beyond the extended tile: those rows
    // only feed values that the owners' words replace)
    if (live) {
      cv[0] *= SC[l0 - st];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int l = l0 + j * st;
        cl[j] *= SC[l - 1];
        cr[j] *= SC[l + 1];
        if (j == R - 1) cv[j + 1] *= SC[l + st];
      }
    }

    // P and A'P; ev: the correction in the scaled system; pv: the block's v_0 .. v_S-1
    constexpr bool DEFER = R <= 4;
    float ev[R], P[S][R], AP[S][R], pv[DEFER ? S : 1][R];
    bool first = true;     // before the first block
    bool pending = false;  // the last block's directions are still to be formed
    bool fresh = true;     // no directions yet
    int cbuf = 0;          // hd->coef of the last block
    auto read_coef = [&](float* al, float (*bc)[S]) {
#pragma unroll
      for (int i = 0; i < S; ++i) {
        al[i] = hd->coef[cbuf][S * S + i];
#pragma unroll
        for (int k = 0; k < S; ++k) bc[i][k] = hd->coef[cbuf][i * S + k];
      }
    };
    auto directions = [&]() {   // DEFER: P := pv + P B_c, correction += P a
      float al[S], bc[S][S];
      read_coef(al, bc);
#pragma unroll
      for (int j = 0; j < R; ++j) {
        float pn[S], de = 0.0f;
#pragma unroll
        for (int k = 0; k < S; ++k) {
          pn[k] = pv[DEFER ? k : 0][j];
          if (!fresh) {
#pragma unroll
            for (int i = 0; i < S; ++i) pn[k] = fmaf(bc[i][k], P[i][j], pn[k]);
          }
        }
#pragma unroll
        for (int k = 0; k < S; ++k) {
          P[k][j] = pn[k];
          de = fmaf(al[k], pn[k], de);
        }
        ev[j] = fresh ? de : ev[j] + de;
      }
      fresh = false;
    };
    for (int left = a.n_cg; left > 0;) {
      const int q = left < S ? left : S;
      const bool last = left <= S;
#pragma unroll
      for (int j = 0; j < R; ++j) refresh(meta[j]);
      // ---- v_j = B^j r: own pixels and the ghost pixels within reach
      float v[S + 1][R];
#pragma unroll
      for (int j = 0; j < R; ++j) v[0][j] = r[j];
#pragma unroll
      for (int k = 0; k < S; ++k) {
        const int p = k & 1;
        if constexpr (SHIFT) {
          se->top[p][threadIdx.x] = v[k][0];
          se->bottom[p][threadIdx.x] = v[k][R - 1];
          if (lane == 0 || lane == 63) {
#pragma unroll
            for (int j = 0; j < R; ++j) se->edge[p][wave + 1][lane == 63][j] = v[k][j];
          }
        } else if (live) {
#pragma unroll
          for (int j = 0; j < R; ++j) V[p * cells + l0 + j * st] = v[k][j];
        }
        __syncthreads();
        // (outside the extended tile the couplings are 0 and any value will do)
        const float* vl = V + p * cells + l0;
        const float up = SHIFT ? se->bottom[p][max((int)threadIdx.x - EW, 0)] : vl[-st];
        const float dn = SHIFT ? se->top[p][min((int)threadIdx.x + EW, SS_NT - 1)] : vl[(live ? R : 0) * st];
        const float* edge = lane < 32 ? se->edge[p][wave][1] : se->edge[p][wave + 2][0];   // SHIFT
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const float left = SHIFT ? lane_shift<0x138>(edge[j], v[k][j]) : vl[j * st - 1];
          const float right = SHIFT ? lane_shift<0x130>(edge[j], v[k][j]) : vl[j * st + 1];
          const float above = j > 0 ? v[k][j > 0 ? j - 1 : 0] : up;
          const float below = j < R - 1 ? v[k][j < R - 1 ? j + 1 : j] : dn;
          v[k + 1][j] = cl[j] * left + cr[j] * right + cv[j] * above + cv[j + 1] * below;
        }
      }
      // ---- moments over the own pixels
      double m[NV];
#pragma unroll
      for (int k = 0; k < NV; ++k) m[k] = 0.0;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const bool own = (own_bits >> j) & 1u;
        double dv[S + 1];
#pragma unroll
        for (int k = 0; k <= S; ++k) dv[k] = k < S ? (double)(own ? v[k][j] : 0.0f) : (double)v[k][j];
#pragma unroll
        for (int k = 0; k < S; ++k) {
          m[2 * k] = fma(dv[k], dv[k], m[2 * k]);
          m[2 * k + 1] = fma(dv[k], dv[k + 1], m[2 * k + 1]);
        }
        if (j & 1) __builtin_amdgcn_sched_barrier(0);
      }
      auto publish = [&](uint32_t par) {
        KF_GLOBAL float* h = halo + (size_t)par * plane;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const int mt = meta[j];
          if (!(mt & VPUB)) continue;
          KF_GLOBAL uint64_t* t = (KF_GLOBAL uint64_t*)((KF_GLOBAL char*)h + (uint32_t)(mt & 0xffffff) * (S * 4u));
#pragma unroll
          for (int k = 1; k < S; k += 2)
            st_word(t + k / 2, ((uint64_t)__float_as_uint(v[k + 1][j]) << 32) | __float_as_uint(v[k][j]));
        }
      };
      auto take = [&](uint32_t par) {
        const KF_GLOBAL float* h = halo + (size_t)par * plane;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const int mt = meta[j];
          if (!(mt & GHOST)) continue;
          // (one word each: a wider load would be split into its registers, and
          // waited for, at once)
          const KF_GLOBAL float* t = (const KF_GLOBAL float*)((const KF_GLOBAL char*)h + (uint32_t)(mt & 0xffffff) * (S * 4u));
#pragma unroll
          for (int k = 1; k <= S; ++k) v[k][j] = ld_float(t + k - 1);
        }
      };
      BlockScalars<S> bs;
      auto prep = [&]() {
        if (wave == 2 && !first) bs.prepare(hd, lane);
      };
      auto aside = [&]() {
        if (DEFER && pending) directions();
      };
      auto use = [&](const double* t) {
        const bool some = t[0] != 0.0;
        bool good = false;
        if (some) good = bs.finish(hd, hd->coef[cbuf ^ 1], t, first, q, lane);
        if (lane == 0) hd->stop = some ? (good ? 0 : 1) : 2;
      };
      if (!team_sync(m, publish, take, prep, aside, use)) return;
      const int stop = hd->stop;
      if (stop == 2) {   // zero residual: nothing to add
        if (first) {
#pragma unroll
          for (int j = 0; j < R; ++j) ev[j] = 0.0f;
        }
        break;
      }
      // ---- the residual and A'P, which the next block starts from. P and the
      //      correction follow while its totals are on their way (DEFER: the
      //      copies of v take S registers a row), or here
      cbuf ^= 1;
      {
        float al[S], bc[S][S];
        read_coef(al, bc);
#pragma unroll
        for (int j = 0; j < R; ++j) {
          float pn[S], an[S];
#pragma unroll
          for (int k = 0; k < S; ++k) {
            pn[k] = v[k][j];
            an[k] = v[k][j] - v[k + 1][j];
            if (!first) {
              if constexpr (!DEFER) {
#pragma unroll
                for (int i = 0; i < S; ++i) pn[k] = fmaf(bc[i][k], P[i][j], pn[k]);
              }
              if (!last) {
#pragma unroll
                for (int i = 0; i < S; ++i) an[k] = fmaf(bc[i][k], AP[i][j], an[k]);
              }
            }
          }
          float de = 0.0f, dr = r[j];
#pragma unroll
          for (int k = 0; k < S; ++k) {
            if constexpr (DEFER) {
              pv[k][j] = copy_of(v[k][j]);
            } else {
              P[k][j] = pn[k];
              de = fmaf(al[k], pn[k], de);
            }
            AP[k][j] = an[k];
            dr = fmaf(-al[k], an[k], dr);
          }
          if constexpr (!DEFER) ev[j] = first ? de : ev[j] + de;
          r[j] = dr;
        }
      }
      cg_total += q;
      left -= q;
      const bool done = last || stop;
      if (DEFER && done) directions();
      pending = DEFER && !done;
      first = false;
      if (done) break;
    }

    // ---- x += D^-1/2 e; scale step: semi weights at (x_new, tau),
    //      tau = sum w (x - z) / sum w (R13)
    double vals[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) vals[k] = 0.0;
    refresh(u);
    refresh(vtop);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      refresh(meta[j]);
      if (!((own_bits >> j) & 1u)) continue;
      const int l = l0 + j * st;
      const float xn = fmaf(SC[l], ev[j], X[l]);
      X[l] = xn;
      const float zs = ST[l], isr = ST[cells + l];
      const float w = huber_w((xn - (float)tau - zs) * isr, delta, tukey) * isr * isr;
      vals[0] += (double)w * (double)(xn - zs);
      vals[1] += (double)w;
      vals[2] += isr > 0.0f ? 1.0 : 0.0;
    }
    auto publish_x = [&](uint32_t par) {
      KF_GLOBAL float* h = halo + (size_t)par * plane;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int mt = meta[j];
        if (mt & XPUB) st_float(h + (uint32_t)(mt & 0xffffff) * S, X[l0 + j * st]);
      }
    };
    auto take_x = [&](uint32_t par) {
      const KF_GLOBAL float* h = halo + (size_t)par * plane;
      float w[R], wr = 0.0f;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int mt = meta[j];
        if (mt & GHOST) w[j] = ld_float(h + (uint32_t)(mt & 0xffffff) * S);
      }
      if (ring_off >= 0) wr = ld_float(h + (size_t)ring_off * S);
#pragma unroll
      for (int j = 0; j < R; ++j)
        if (meta[j] & GHOST) X[l0 + j * st] = w[j];
      if (ring_off >= 0) X[ring_li] = wr;
    };
    auto use_tau = [&](const double* t) {
      if (lane == 0) {
        hd->tau = !postfit && t[1] > 0.0 ? t[0] / t[1] : tau;
        hd->tot[2] = t[2];
      }
    };
    if (!team_sync(vals, publish_x, take_x, [] {}, [] {}, use_tau)) return;
    tau = hd->tau;
    if (gn == 0) n_valid = hd->tot[2];
  }
  if (postfit && !new_kf) {
    // least-squares fit of the log-scale to the network: tau = mean(mu - y)
    double vals[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) vals[k] = 0.0;
#pragma unroll
    for (int j = 0; j < R; ++j)
      if ((own_bits >> j) & 1u) vals[0] += (double)mu_g[(vtop + j) * W + u] - (double)X[l0 + j * st];
    auto use_fit = [&](const double* t) {
      if (lane == 0) hd->tau = t[0] / (double)N;
    };
    if (!team_sync(vals, [](uint32_t) {}, [](uint32_t) {}, [] {}, [] {}, use_fit)) return;
    tau = hd->tau;
  }
  if (!new_kf) {
    const float add = postfit ? (float)tau : 0.0f;
#pragma unroll
    for (int j = 0; j < R; ++j)
      if ((own_bits >> j) & 1u) x_g[(vtop + j) * W + u] = X[l0 + j * st] + add;
  }
  if (b == 0 && threadIdx.x == 0) {
    // as in kf_solve.hip: a launch without synchronisations keeps the epoch base
    scal->epoch = e0 + (e != e0 ? a.epoch_span : 0u);
    scal->tau = tau;
    scal->cg_iterations = cg_total;
    scal->cg_rel_residual = 0.0;
    if (!new_kf) scal->n_valid = (int32_t)n_valid;
    scal->team_syncs = (int32_t)(e - e0);
    scal->new_keyframe = new_kf;
  }
}

template <int R, int S, bool VAR>
__global__ __launch_bounds__(SS_NT) void k_sstep(SolveArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  sstep_member<R, S, VAR>(a, blockIdx.x, smem);
}

}  // namespace

}  // namespace kf
