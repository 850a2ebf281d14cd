// HIP kernels for gfx950: the Ls-fused Wilson hop with fused fifth-dimension
// epilogues, fifth-dimension operators, FP64 BLAS for the outer solver and the
// batched block-CG kernels of the preconditioner.
//
// Thread layout of every site kernel: a workgroup owns `nsite_wg` 4D sites of
// a site list; its threads are (site, rhs, s) with s fastest, so one 4D site's
// Ls x nrhs spinors are handled by consecutive lanes (coalesced loads of the
// [rhs][site][chunk][s] layout, links staged once per site) and the
// fifth-dimension coupling is an exchange between neighbouring lanes (DPP row
// rotation, ds_bpermute or LDS, by the exchange mode below).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "internal.h"

namespace mspcg {

// ---------------------------------------------------------------- helpers
// Orders a wave's LDS stores before its following LDS loads of words other
// lanes of the same wave stored: wavefront-scope release/acquire fences (the
// compiler neither moves nor forwards memory accesses across them) around a
// wave barrier.
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename R>
__device__ inline void zero24(R v[24]) {
#pragma unroll
  for (int k = 0; k < 24; ++k) v[k] = 0;
}

// ---------------------------------------------------------------- fifth-dimension exchange
// The Ls values of one (4D site, rhs) sit on Ls consecutive lanes.  Coupling
// s to s-1 / s+1 is a cyclic rotation inside that group of lanes:
//  * Ls == 16: the group is one DPP row; row_ror moves the value in the same
//    VALU instruction stream, with no LDS traffic and no barrier;
//  * Ls divides 64: groups never straddle a wavefront; ds_bpermute;
//  * otherwise (Ls = 12, 24, ...): through LDS with workgroup barriers.
// (row_ror with all rows and banks enabled writes every lane: no "old" value)
__device__ inline int rot_prev_dpp(int x) { return __builtin_amdgcn_mov_dpp(x, 0x121, 0xF, 0xF, false); }
__device__ inline int rot_next_dpp(int x) { return __builtin_amdgcn_mov_dpp(x, 0x12F, 0xF, 0xF, false); }
__device__ inline float rot_prev_dpp(float x) { return __builtin_bit_cast(float, rot_prev_dpp(__builtin_bit_cast(int, x))); }
__device__ inline float rot_next_dpp(float x) { return __builtin_bit_cast(float, rot_next_dpp(__builtin_bit_cast(int, x))); }
__device__ inline double rot_prev_dpp(double x) {
  const int2 t = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(rot_prev_dpp(t.x), rot_prev_dpp(t.y)));
}
__device__ inline double rot_next_dpp(double x) {
  const int2 t = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(rot_next_dpp(t.x), rot_next_dpp(t.y)));
}
__device__ inline float perm(int addr, float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr, __builtin_bit_cast(int, x)));
}
__device__ inline double perm(int addr, double x) {
  const int2 t = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_ds_bpermute(addr, t.x), __builtin_amdgcn_ds_bpermute(addr, t.y)));
}

// Exchange modes, fixed per launch from Ls and nrhs (the kernels are
// instantiated per mode), and the lane layout that goes with them.  With DPP
// and ds_bpermute exchanges every 64-lane wave holds G = 64/Ls whole (site,
// rhs) groups of Ls lanes; the last 64 - G*Ls lanes of a wave are idle (4 of
// 64 for Ls = 12).  That layout is used where at most 8 lanes per wave idle
// and some workgroup of whole sites (all nrhs groups of a site together)
// fills whole waves; otherwise (Ls = 24; Ls = 12 with 8 right-hand sides) the
// groups are packed densely and exchange through LDS with barriers.
constexpr int kXDpp16 = 0, kXPerm = 1, kXLds = 2;
// Exchanges through LDS (and the M_5^{-1} transposition) give every thread a
// row of kRow values: the offsets inside a row are instruction immediates, and
// with an odd row length the rows of consecutive threads start on distinct
// banks.
constexpr int kRow = 25;
static inline int xmode(int Ls, int nrhs) {
  if (Ls == 16) return kXDpp16;
  if (Ls > 64) return kXLds;
  const int G = 64 / Ls;
  if (64 % Ls == 0) return kXPerm;
  if (64 - G * Ls > 8) return kXLds;
  for (int c = 1; nrhs * c <= 4 * G; ++c)
    if ((nrhs * c) % G == 0) return kXPerm;
  return kXLds;
}
// groups per wave of the layout (0: dense packing)
__host__ __device__ inline int groups_per_wave(int xm, int Ls) { return xm == kXLds ? 0 : 64 / Ls; }
// thread index of lane t of group g
__device__ inline int group_tid(int G, int Ls, int g, int t) { return G ? (g / G) * 64 + (g % G) * Ls + t : g * Ls + t; }
// threads of a workgroup of `groups` groups
static inline int layout_threads(int xm, int Ls, int groups) {
  const int G = groups_per_wave(xm, Ls);
  return G ? 64 * ((groups + G - 1) / G) : groups * Ls;
}

// v <- a v + b P_chi v (DAG = 0) or a v + b P_chi^+ v (DAG = 1) on the Ls column
// held one s per lane.  P_chi = P- S+ + P+ S-: chirality + (reals 0..11) takes
// s-1, chirality - (reals 12..23) takes s+1, with the -mf corner; the adjoint
// swaps the directions.  Must be reached by all threads of the workgroup.
template <int DAG, int XM, typename R>
__device__ inline void pchi_comb(R *lds, int nthr, int tid, int s, int Ls, R a, R b, R mf, R v[24]) {
  const R cm = (s > 0) ? R(1) : -mf;
  const R cp = (s < Ls - 1) ? R(1) : -mf;
  const R cu = b * (DAG ? cp : cm);
  const R cl = b * (DAG ? cm : cp);
  if (XM == kXDpp16) {
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = a * v[k] + cu * (DAG ? rot_next_dpp(v[k]) : rot_prev_dpp(v[k]));
#pragma unroll
    for (int k = 12; k < 24; ++k) v[k] = a * v[k] + cl * (DAG ? rot_prev_dpp(v[k]) : rot_next_dpp(v[k]));
  } else if (XM == kXPerm) {
    const int lane = tid & 63;
    const int am = 4 * ((s > 0) ? lane - 1 : lane + Ls - 1);
    const int ap = 4 * ((s < Ls - 1) ? lane + 1 : lane - (Ls - 1));
    const int au = DAG ? ap : am, al = DAG ? am : ap;
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = a * v[k] + cu * perm(au, v[k]);
#pragma unroll
    for (int k = 12; k < 24; ++k) v[k] = a * v[k] + cl * perm(al, v[k]);
  } else {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 24; ++k) lds[tid * kRow + k] = v[k];
    __syncthreads();
    const int tm = (s > 0) ? tid - 1 : tid + Ls - 1;
    const int tp = (s < Ls - 1) ? tid + 1 : tid - (Ls - 1);
    const int tu = DAG ? tp : tm;
    const int tl = DAG ? tm : tp;
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = a * v[k] + cu * lds[tu * kRow + k];
#pragma unroll
    for (int k = 12; k < 24; ++k) v[k] = a * v[k] + cl * lds[tl * kRow + k];
  }
}

// A <- A + P_chi B (DAG = 0) or A + P_chi^+ B (DAG = 1) on the Ls column held one
// s per lane (the directions and corners of pchi_comb): one exchange for a
// combination a u + b P u + c w + d P w of two columns.  Must be reached by
// all threads of the workgroup.
template <int DAG, int XM, typename R>
__device__ inline void pchi_add(R *lds, int nthr, int tid, int s, int Ls, R mf, R A[24], const R B[24]) {
  const R cm = (s > 0) ? R(1) : -mf;
  const R cp = (s < Ls - 1) ? R(1) : -mf;
  const R cu = DAG ? cp : cm;
  const R cl = DAG ? cm : cp;
  if (XM == kXDpp16) {
#pragma unroll
    for (int k = 0; k < 12; ++k) A[k] += cu * (DAG ? rot_next_dpp(B[k]) : rot_prev_dpp(B[k]));
#pragma unroll
    for (int k = 12; k < 24; ++k) A[k] += cl * (DAG ? rot_prev_dpp(B[k]) : rot_next_dpp(B[k]));
  } else if (XM == kXPerm) {
    const int lane = tid & 63;
    const int am = 4 * ((s > 0) ? lane - 1 : lane + Ls - 1);
    const int ap = 4 * ((s < Ls - 1) ? lane + 1 : lane - (Ls - 1));
    const int au = DAG ? ap : am, al = DAG ? am : ap;
#pragma unroll
    for (int k = 0; k < 12; ++k) A[k] += cu * perm(au, B[k]);
#pragma unroll
    for (int k = 12; k < 24; ++k) A[k] += cl * perm(al, B[k]);
  } else {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 24; ++k) lds[tid * kRow + k] = B[k];
    __syncthreads();
    const int tm = (s > 0) ? tid - 1 : tid + Ls - 1;
    const int tp = (s < Ls - 1) ? tid + 1 : tid - (Ls - 1);
    const int tu = DAG ? tp : tm;
    const int tl = DAG ? tm : tp;
#pragma unroll
    for (int k = 0; k < 12; ++k) A[k] += cu * lds[tu * kRow + k];
#pragma unroll
    for (int k = 12; k < 24; ++k) A[k] += cl * lds[tl * kRow + k];
  }
}

// Projected half spinor of (1 + pc P_chi) v for the hop in direction MU:
// h(s) = X(s) + Y(s) + cu X(s-1) + cl Y(s+1) with X, Y the two parts of the
// projection (P_chi takes the upper spins from s-1 and the lower ones from
// s+1, with the -mf corners folded into cu, cl), so no full M_phi v is formed.
// Must be reached by all threads of the workgroup.
template <int MU, int SGN, int XM, typename R>
__device__ inline void project_pre(R *lds, int nthr, int tid, int s, int Ls, R cu, R cl, const R v[24], R h[12]) {
  // w: the upper spins of v at s-1 and the lower spins at s+1 (rotated raw, so
  // that the signs of the projection fold into the multiply-adds)
  R w[24];
  if (XM == kXDpp16) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      w[k] = rot_prev_dpp(v[k]);
      w[12 + k] = rot_next_dpp(v[12 + k]);
    }
  } else if (XM == kXPerm) {
    const int lane = tid & 63;
    const int am = 4 * ((s > 0) ? lane - 1 : lane + Ls - 1);
    const int ap = 4 * ((s < Ls - 1) ? lane + 1 : lane - (Ls - 1));
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      w[k] = perm(am, v[k]);
      w[12 + k] = perm(ap, v[12 + k]);
    }
  } else {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 24; ++k) lds[tid * kRow + k] = v[k];
    __syncthreads();
    const int tm = (s > 0) ? tid - 1 : tid + Ls - 1;
    const int tp = (s < Ls - 1) ? tid + 1 : tid - (Ls - 1);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      w[k] = lds[tm * kRow + k];
      w[12 + k] = lds[tp * kRow + 12 + k];
    }
  }
  R X[12], Y[12], Xw[12], Yw[12];
  project_parts<MU, SGN>(v, X, Y);
  project_parts<MU, SGN>(w, Xw, Yw);
#pragma unroll
  for (int k = 0; k < 12; ++k) h[k] = fma(cl, Yw[k], fma(cu, Xw[k], X[k] + Y[k]));
}

// wt: the neighbour's weight (1, or 0 outside a block domain; only without M_phi on the input)
template <int MU, int SGN, int PRE, int XM, typename R>
__device__ inline void hop_dir(R *lds, int nthr, int tid, int s, int Ls, R cu, R cl, const R v[24], const R *U,
                               R acc[24], R wt) {
  R h[12];
  if (PRE)
    project_pre<MU, SGN, XM>(lds, nthr, tid, s, Ls, cu, cl, v, h);
  else
    project<MU, SGN>(v, h);
  hop_half<MU, SGN>(h, U, acc, wt);
}

__device__ inline uint32_t rot_prev_word(uint32_t x) { return (uint32_t)rot_prev_dpp((int)x); }
__device__ inline uint32_t rot_next_word(uint32_t x) { return (uint32_t)rot_next_dpp((int)x); }

// The stored words and norm of the upper spins at s-1 and the lower spins at
// s+1 (the part of the neighbouring lanes' inputs that M_phi mixes in).
// Must be reached by all threads of the workgroup.
template <int XM, typename S>
__device__ inline void exchange_pre_raw(float *lds, int nthr, int tid, int s, int Ls, const RawSite<S> &raw,
                                        RawSite<S> &w, float &nm, float &np) {
  if (XM == kXDpp16) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      w.set_word(i, rot_prev_word(raw.word(i)));
      w.set_word(6 + i, rot_next_word(raw.word(6 + i)));
    }
    nm = rot_prev_dpp(raw.n);
    np = rot_next_dpp(raw.n);
  } else if (XM == kXPerm) {
    const int lane = tid & 63;
    const int am = 4 * ((s > 0) ? lane - 1 : lane + Ls - 1);
    const int ap = 4 * ((s < Ls - 1) ? lane + 1 : lane - (Ls - 1));
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      w.set_word(i, (uint32_t)__builtin_amdgcn_ds_bpermute(am, (int)raw.word(i)));
      w.set_word(6 + i, (uint32_t)__builtin_amdgcn_ds_bpermute(ap, (int)raw.word(6 + i)));
    }
    nm = perm(am, raw.n);
    np = perm(ap, raw.n);
  } else {
    uint32_t *lw = reinterpret_cast<uint32_t *>(lds);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 12; ++i) lw[tid * kRow + i] = raw.word(i);
    lds[tid * kRow + 12] = raw.n;
    __syncthreads();
    const int tm = (s > 0) ? tid - 1 : tid + Ls - 1;
    const int tp = (s < Ls - 1) ? tid + 1 : tid - (Ls - 1);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      w.set_word(i, lw[tm * kRow + i]);
      w.set_word(6 + i, lw[tp * kRow + 6 + i]);
    }
    nm = lds[tm * kRow + 12];
    np = lds[tp * kRow + 12];
  }
}

// The same for BF16 inputs stored as v/n with a per-site norm n: the
// projection works on the stored values (widened to FP32) and n multiplies
// the link product as it is accumulated.  With M_phi on the input the
// neighbours' norms enter the mixing coefficients as n(s -+ 1)/n(s) (a zero
// site has no stored values and uses n = 1).  Taken with M_phi on the input and
// for Ls that are no multiple of four (otherwise hop_dir_b16_mm).  `one` is an opaque 1 that keeps
// each sum a multiply-add.
template <int MU, int SGN, int PRE, int XM, typename S>
__device__ inline void hop_dir_norm(float *lds, int nthr, int tid, int s, int Ls, float cu, float cl, float one,
                                    const RawSite<S> &raw, const float *U, float acc[24], bool out) {
  float v[24], X[12], Y[12], h[12];
  raw.decode_raw(v);
  project_parts<MU, SGN>(v, X, Y);
  float n = out ? 0.f : raw.n;
  if (PRE) {
    RawSite<S> w;
    float nm, np;
    exchange_pre_raw<XM>(lds, nthr, tid, s, Ls, raw, w, nm, np);
    float wv[24], Xw[12], Yw[12];
    w.decode_raw(wv);
    project_parts<MU, SGN>(wv, Xw, Yw);
    n = n > 0.f ? n : 1.f;
    const float rn = __builtin_amdgcn_rcpf(n);
    const float cu2 = cu * nm * rn, cl2 = cl * np * rn;
#pragma unroll
    for (int k = 0; k < 12; ++k) h[k] = fmaf(cl2, Yw[k], fmaf(cu2, Xw[k], fmaf(X[k], one, Y[k])));
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) h[k] = fmaf(X[k], one, Y[k]);
  }
  hop_half<MU, SGN>(h, U, acc, n);
}

// F16 inputs: the projected half spinor is formed in packed half precision
// on the stored words and multiplied by the link with FP32-accumulated dot
// products (hop_half_h16).  With M_phi on the input the three contributions
// n(s)(X + Y)(s), cu n(s-1) X(s-1) and cl n(s+1) Y(s+1) are scaled by the
// largest of their weights m, so that every coefficient is at most 1 and the
// half-precision sum cannot overflow; m multiplies the link product.
// U: the link as dot products read it; ra, rb: this lane's rows of it for the
// matrix cores (MM).
template <int MU, int SGN, int PRE, int XM, int MM>
__device__ inline void hop_dir_h16(float *lds, int nthr, int tid, int s, int Ls, float cu, float cl,
                                   const RawSite<_Float16> &raw, const uint32_t *U, const uint32_t *ra,
                                   const uint32_t *rb, float acc[24], bool out) {
  uint32_t wd[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) wd[i] = raw.word(i);
  half2_t X[6], Y[6], h[6];
  project_parts_h16<MU, SGN>(wd, X, Y);
  float m = out ? 0.f : raw.n;
  if (PRE) {
    RawSite<_Float16> w;
    float nm, np;
    exchange_pre_raw<XM>(lds, nthr, tid, s, Ls, raw, w, nm, np);
#pragma unroll
    for (int i = 0; i < 12; ++i) wd[i] = w.word(i);
    half2_t Xw[6], Yw[6];
    project_parts_h16<MU, SGN>(wd, Xw, Yw);
    const float n = raw.n, wu = cu * nm, wl = cl * np;
    m = fmaxf(n, fmaxf(fabsf(wu), fabsf(wl)));
    m = m > 0.f ? m : 1.f;
    const float rm = __builtin_amdgcn_rcpf(m);
    const _Float16 a = (_Float16)(n * rm), bu = (_Float16)(wu * rm), bl = (_Float16)(wl * rm);
#pragma unroll
    for (int k = 0; k < 6; ++k) h[k] = half2_t{a, a} * (X[k] + Y[k]) + (half2_t{bu, bu} * Xw[k] + half2_t{bl, bl} * Yw[k]);
  } else {
#pragma unroll
    for (int k = 0; k < 6; ++k) h[k] = X[k] + Y[k];
  }
  if constexpr (MM) hop_half_mm<MU, SGN>(h, ra, rb, acc, m);
  else hop_half_h16<MU, SGN>(h, U, acc, m);
}

// ---------------------------------------------------------------- M_5^{-1} along the fifth dimension
// v <- scale X v per chirality for X = sigma (1 + rho S)(1 - q S)^{-1}, S the
// chirality's shift of P_chi (chirality +, reals 0..11: s takes s-1; chirality
// -, reals 12..23: s takes s+1; S^Ls = -mf), or X^T (TR = 1: the shift runs the
// other way).  With sigma = b / alpha, rho = c / b and q = beta / alpha this is
// M_phi M_5^{-1} = (b + c P_chi)(alpha - beta P_chi)^{-1}; with rho = 0 and
// sigma = 1 / alpha it is M_5^{-1} alone (M_5 = alpha - beta P_chi, Eq. (5)).
// Both factors are functions of S, so X v is a first-order recurrence along s
// instead of a dense Ls x Ls product: with positions i counted along the shift
// (i = s, or Ls - 1 - s where the shift takes s+1),
//   u_0 = x_0 + wrap x_{Ls-1},  u_i = x_i + rho x_{i-1}          ((1 + rho S) x)
//   z_0 = u_0,                  z_i = u_i + q z_{i-1}            (no wrap-around)
//   (X x)_i = sigma (z_i + lambda_i z_{Ls-1})
// where wrap = -rho mf and lambda_i = gamma q^i, gamma = -q mf / (1 + mf q^Ls),
// restores the -mf corner of S (exact: (1 - q S)^{-1} = sum_k q^k S^k / (1 + mf q^Ls)).
// cf = [rho, wrap, q, sigma, lambda_0 .. lambda_{Ls-1}] in the compute type.
//
// The Ls values of one (site, rhs) sit on the Ls consecutive threads of its
// group; they are transposed through LDS (rows = positions i, one row of
// kRow words per thread: an odd stride, so a row store of all lanes
// and a column load of all lanes both spread over the banks), lane t of the
// group runs the recurrence of columns t, t + Ls, ... < 24, and the rows are
// read back.  A chirality whose shift takes s+1 is stored with its rows
// reversed, so every column runs toward increasing i.

template <typename R, int LSC>
__device__ inline void chain_columns(R *Tg, int t, int Ls_rt, const R *cf, R sig) {
  const int Ls = LSC > 0 ? LSC : Ls_rt;
  const R rho = cf[0], wrap = cf[1], q = cf[2];
  for (int k = t; k < 24; k += Ls) {
    R *c = Tg + k;
    if constexpr (LSC > 0) {  // the column in registers
      R x[LSC];
#pragma unroll
      for (int i = 0; i < LSC; ++i) x[i] = c[i * kRow];
      R prev = x[0];
      x[0] = fma(wrap, x[LSC - 1], x[0]);
#pragma unroll
      for (int i = 1; i < LSC; ++i) {
        const R cur = x[i];
        x[i] = fma(q, x[i - 1], fma(rho, prev, cur));
        prev = cur;
      }
      const R zl = x[LSC - 1];
#pragma unroll
      for (int i = 0; i < LSC; ++i) c[i * kRow] = sig * fma(cf[4 + i], zl, x[i]);
    } else {  // any Ls: in place in LDS
      R prev = c[0];
      R z = fma(wrap, c[(Ls - 1) * kRow], prev);
      c[0] = z;
      for (int i = 1; i < Ls; ++i) {
        const R cur = c[i * kRow];
        z = fma(q, z, fma(rho, prev, cur));
        c[i * kRow] = z;
        prev = cur;
      }
      for (int i = 0; i < Ls; ++i) c[i * kRow] = sig * fma(cf[4 + i], z, c[i * kRow]);
    }
  }
}

// lds: kRow * nthr values; G: groups per wave of the lane layout (0:
// dense packing, groups may straddle waves: workgroup barriers; otherwise the
// groups of a wave only touch that wave's rows).  Must be reached by all
// threads of the workgroup.
template <int TR, typename R, int LSC>
__device__ inline void m5_chain_t(R *lds, int tid, int s, int Ls_rt, int G, const R *cf, R scale, R v[24]) {
  const int Ls = LSC > 0 ? LSC : Ls_rt;
  R *Tg = lds + (size_t)(tid - s) * kRow;  // this group's rows
  const int rp = TR ? Ls - 1 - s : s;              // row of chirality + (reals 0..11)
  const int rm = TR ? s : Ls - 1 - s;              // row of chirality -
  // The idle lanes past a wave's last whole group (whole-wave layouts) form
  // no group: their rows would run into the next wave's, so they take no part.
  const bool own = G == 0 || ((tid & 63) - s) + Ls <= 64;
  if (G == 0) __syncthreads();                     // (earlier exchanges through the same words)
  if (own) {
#pragma unroll
    for (int k = 0; k < 12; ++k) Tg[rp * kRow + k] = v[k];
#pragma unroll
    for (int k = 12; k < 24; ++k) Tg[rm * kRow + k] = v[k];
  }
  if (G == 0) __syncthreads(); else wave_lds_sync();
  if (own) chain_columns<R, LSC>(Tg, s, Ls, cf, cf[3] * scale);
  if (G == 0) __syncthreads(); else wave_lds_sync();
  if (own) {
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = Tg[rp * kRow + k];
#pragma unroll
    for (int k = 12; k < 24; ++k) v[k] = Tg[rm * kRow + k];
  }
}

template <int TR, typename R>
__device__ inline void m5_chain(R *lds, int tid, int s, int Ls, int G, const R *cf, R scale, R v[24]) {
  switch (Ls) {
    case 8: m5_chain_t<TR, R, 8>(lds, tid, s, Ls, G, cf, scale, v); break;
    case 12: m5_chain_t<TR, R, 12>(lds, tid, s, Ls, G, cf, scale, v); break;
    case 16: m5_chain_t<TR, R, 16>(lds, tid, s, Ls, G, cf, scale, v); break;
    case 24: m5_chain_t<TR, R, 24>(lds, tid, s, Ls, G, cf, scale, v); break;
    case 32: m5_chain_t<TR, R, 32>(lds, tid, s, Ls, G, cf, scale, v); break;
    default: m5_chain_t<TR, R, 0>(lds, tid, s, Ls, G, cf, scale, v); break;
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs of the chip, each
// with its own L2.  Renumbering them so that every XCD works on one
// contiguous range of tiles keeps the neighbours a tile gathers (x, y and z
// hops land a few tiles away) in the same L2.  Bijective on [0, n).
__device__ inline int xcd_tile(int b, int n) {
  const int q = n >> 3, rem = n & 7, x = b & 7, k = b >> 3;
  return x * q + min(x, rem) + k;
}

// Workgroup sum of `val` per right-hand side into partial[tile * nrhs + r]
// (fixed order: deterministic).  Uses the LDS region as doubles.
__device__ inline void wg_partial(double *ldsd, int nthr, int tid, int Ls, int nrhs, int nsite_wg, int G, double val,
                                  double *partial, int tile) {
  __syncthreads();
  ldsd[tid] = val;
  __syncthreads();
  const int ngroups = nsite_wg * nrhs;
  if (tid < ngroups) {
    double acc = 0;
    for (int s = 0; s < Ls; ++s) acc += ldsd[group_tid(G, Ls, tid, s)];
    ldsd[nthr + tid] = acc;
  }
  __syncthreads();
  if (tid < nrhs) {
    double acc = 0;
    for (int g = 0; g < nsite_wg; ++g) acc += ldsd[nthr + g * nrhs + tid];
    partial[(size_t)tile * nrhs + tid] = acc;
  }
}

// ---------------------------------------------------------------- the hop kernel
// out(x) = epilogue( sum_mu [ P^{SGN_f}_mu U_mu(x) phi(x+mu) + P^{SGN_b}_mu U_mu(x-mu)^+ phi(x-mu) ] )
// with phi = M_phi in (PRE) or in; SGN_f = +1, SGN_b = -1 for H and the reverse
// for the daggered hop g5 H g5 = H^+.
// Workgroup = (s, rhs, site) threads: threadIdx.x = s, .y = rhs, .z = site.
// GLOBAL: the output list is the whole parity (site_cb a permutation of cb in
// column-sweep order); outputs and the `other`/dot operands are indexed by cb,
// neighbour tables and links by the position in the list.  Otherwise (block
// domains) tables and `other` indices are in the order of visit, outputs are
// indexed by a.self (nullptr: by the position in the list), and neighbours
// outside the domain enter with weight zero.
// 4-byte words of LDS for the links of one site
template <typename S, int MM>
__host__ __device__ constexpr int hop_link_words() {
  return MM ? kSiteWords : 144 * (int)sizeof(typename Traits<S>::R) / 4;
}
constexpr size_t kMaxLds = 160 * 1024;  // of a workgroup

// Occupancy the register allocation of the hop kernel is held to (waves per SIMD).
template <typename S> struct HopWaves { static constexpr int value = 4; };
template <> struct HopWaves<double> { static constexpr int value = 2; };
template <> struct HopWaves<float> { static constexpr int value = 3; };

template <typename S, int DAG, int PRE, int EPI, int DOT, int GLOBAL, int XM, int MM>
__global__ void __launch_bounds__(256, (HopWaves<S>::value)) hop_kernel(const HopArgs a) {
  using R = typename Traits<S>::R;
  extern __shared__ __align__(16) unsigned char smem[];
  const int Ls = a.Ls, nrhs = a.nrhs, nsw = a.nsite_wg;
  // lane -> (s, group = rhs + nrhs * site-in-workgroup); see groups_per_wave
  const int G = groups_per_wave(XM, Ls);
  const int nthr = blockDim.x * blockDim.y * blockDim.z;
  int s, r, sl, tid;
  bool lane_ok = true;
  if (XM == kXLds) {
    s = threadIdx.x, r = threadIdx.y, sl = threadIdx.z;
    tid = s + Ls * (r + nrhs * sl);
  } else {
    tid = threadIdx.x;
    const int lane = tid & 63, gi = lane / Ls;
    s = lane - gi * Ls;
    int g = (tid >> 6) * G + gi;
    lane_ok = gi < G && g < nrhs * nsw;  // idle lanes compute on the zero site and store nothing
    if (!lane_ok) g = 0;
    r = g % nrhs;
    sl = g / nrhs;
  }
  // links of this workgroup's sites ([nsite_wg][8][18], or the rows for the
  // matrix cores), then exchange rows [nthr][kRow] (LDS mode, M_5^{-1})
  constexpr int kSiteLinks = hop_link_words<S, MM>();
  R *Lk = reinterpret_cast<R *>(smem);
  uint32_t *Lw = reinterpret_cast<uint32_t *>(smem);
  R *lds = reinterpret_cast<R *>(Lw + nsw * kSiteLinks);
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int site = tile * nsw + sl;
  // The chain of dependent loads before the first spinor bounds a launch that
  // does not fill the chip several times over, and costs a wave of a full one
  // as much as two directions of the loop below: the neighbour row depends on
  // the list position alone, and with the full lattice so do the links (packed
  // in list order), so index, neighbour and link loads are all in flight at
  // once and only the spinors wait for one of them.
  const bool listed = site < a.nsites;
  const int row = listed ? site : 0;  // (inactive lanes compute on valid data and store nothing)
  const int cbr = listed ? a.site_cb[row] : -1;  // full lattice: cb; block domains: position of the site's links
  constexpr bool kUpd = EPI == EPI_M5DAG_MPHIDAG && DOT;  // variants that may update in place
  const bool has_upd = kUpd && a.upd_scal;
  const int ublk = (!GLOBAL && has_upd && listed) ? a.upd_blk[row] : -1;
  const bool active = lane_ok && (GLOBAL ? listed : cbr >= 0);

  // The eight neighbour indices are loaded once, with two 16-byte loads, and
  // kept in registers: no spinor load ever waits for an index load issued after
  // an earlier spinor load.
  // Block domains: a neighbour outside the domain is stored as -1 - n with n
  // an in-domain substitute whose data enters with weight zero (bit d of
  // outm).
  const int4 *nb4 = reinterpret_cast<const int4 *>(a.nbr + (size_t)row * 8);
  const int4 q0 = nb4[0], q1 = nb4[1];

  // the links of all sites of the workgroup, staged once into LDS (every link
  // is used by all Ls x nrhs lanes of its site); the lanes of a site stage that
  // site's links, in 16-byte words or, for the matrix cores, in colour rows.
  // The first kLinkBatch pieces of a lane are requested together (all of them
  // for Ls x nrhs >= 8): loaded one after the other they were 3 to 9 memory
  // latencies in a row (FP64, Ls = 24 to 8).  With the independent index loads:
  // FP64 dslash_eo on 8^4 x 8 11.7 -> 9.2 us, FP64 A on 24^3 x 64 x 24 7221 ->
  // 6773 us.
  constexpr bool kH16 = std::is_same<S, _Float16>::value;
  constexpr int per = 16 / sizeof(S);
  constexpr int nchunk = MM ? 24 : 144 / per;
  constexpr int kLinkBatch = (nchunk + 7) / 8;
  using Piece = typename std::conditional<MM != 0, LinkRow, uint4>::type;
  const int lstep = Ls * nrhs, lfirst = s + Ls * r;
  const S *lsrc = reinterpret_cast<const S *>(a.links) + (size_t)(GLOBAL ? row : (cbr >= 0 ? cbr : 0)) * 144;
  auto load_piece = [&](int c) {
    if constexpr (MM) return load_link_row(lsrc + c * 6);
    else return *reinterpret_cast<const uint4 *>(lsrc + c * per);
  };
  Piece lq[kLinkBatch];
  auto load_links = [&] {
#pragma unroll
    for (int j = 0; j < kLinkBatch; ++j)
      if (j * lstep < nchunk) lq[j] = load_piece(min(lfirst + j * lstep, nchunk - 1));
  };
  auto stage_piece = [&](int c, const Piece &q) {
    if constexpr (MM)  // piece c: colour row c % 3 of direction c / 3
      stage_link_row(q, Lw + sl * kSiteLinks + c * 2 * kRowWords);
    else if constexpr (kH16)  // F16: (A, B) pairs for the packed link product
      link_pairs_h16(q, Lw + sl * 144 + c * 8);
    else
      widen16<R>(reinterpret_cast<const S *>(&q), Lk + sl * 144 + c * per);
  };
  if (GLOBAL) load_links();

  const int cb = GLOBAL ? cbr : 0;
  // index of this site in the output (and what is read at the same site)
  const int self = GLOBAL ? cb : ((!DAG && a.self) ? a.self[row] : row);
  // A fused CG residual update (upd_scal set) stores out - alpha (result):
  // alpha is requested here, long before it is needed, and -alpha folds into
  // the epilogue's coefficients (all linear in the result).
  const bool upd = has_upd && active;
  double alpha_u = 0;
  if (upd) alpha_u = a.upd_scal[GLOBAL ? (size_t)r : ((size_t)ublk * nrhs + r) * kScal + 1];

  int nbw[8];
  int outm = 0;
  {
    const int qa[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      if (GLOBAL) {
        nbw[d] = qa[d];
      } else {
        nbw[d] = qa[d] ^ (qa[d] >> 31);  // (-1 - n = ~n)
        outm |= (int)((uint32_t)qa[d] >> 31) << d;
      }
    }
  }
  // Directions that some site of the wave has inside the domain.  The halo
  // sites of the first two block hops have one to three neighbours inside; they
  // are visited together, by the side of the block they lie on, and a wave of
  // them reads and computes its few directions only.  (Halo sites are 47% of
  // O1 and 38% of E2 for blocks of 8^3 x 16.  Hops 1 and 2 of 16^3 x 32, all
  // eight directions -> the live ones: FP32 Ls 16 261 -> 244 us, BF16 Ls 12
  // with 8 sources 1295 -> 1227, F16 Ls 24 263 -> 260; a block CG of six FP32
  // steps 3974 -> 3773.)  Four or more live directions keep the loads ahead.
  constexpr bool kSparse = !GLOBAL && !DAG;
  constexpr int kSparseMost = 3;
  uint32_t live = 0;
  if constexpr (kSparse) {
#pragma unroll
    for (int d = 0; d < 8; ++d)
      if (__ballot(active && !((outm >> d) & 1)) != 0) live |= 1u << d;
    live = __builtin_amdgcn_readfirstlane(live);
  }
  const bool sparse = kSparse && __builtin_popcount(live) <= kSparseMost;
  const S *in = reinterpret_cast<const S *>(a.in);
  const size_t rin = (size_t)r * a.in_stride;
  // neighbour n of this lane: chunk 0 at in_s + n * sstride, its chunks cstride
  // apart, its norm at nrm_s + n * Ls (one multiply-add per address)
  // (32 x 32 -> 64-bit products: one multiply-add each)
  const char *in_s = reinterpret_cast<const char *>(in + chunk_index<S>(rin, s, Ls, 0));
  const uint32_t cstride = (uint32_t)Ls * Chunk<S>::kReals;
  const uint32_t sstride = (uint32_t)Ls * 24 * sizeof(S);  // (bytes)
  const char *nrm_s = reinterpret_cast<const char *>(Traits<S>::kNorm ? a.in_norm + rin * Ls + s : nullptr);
  auto load_nbr = [&](RawSite<S> &dst, int n) {
    const uint64_t un = (uint32_t)n;
    dst.load_at(reinterpret_cast<const S *>(in_s + un * sstride), cstride,
                reinterpret_cast<const float *>(nrm_s + un * (uint32_t)(Ls * 4)));
  };
  // Neighbour spinors in flight ahead of the direction being computed.  FP64 at
  // two waves per SIMD has registers for one (none: A on 24^3 x 64 x 24 6745 us,
  // one: 6244; two waves with two: 7058, one wave with one: 6211).  The others
  // take two (block hops 1-4 on 24^3 x 64 x 24, F16: 2942 us with none, 2813 with
  // one, 2718 with two, 2712 with three).
  constexpr int kAhead = std::is_same<S, double>::value ? 1 : 2;
  RawSite<S> buf[kAhead + 1];
  if (!sparse) {
#pragma unroll
    for (int d = 0; d < kAhead; ++d) load_nbr(buf[d], nbw[d]);
  }

  if (!GLOBAL) load_links();
  if (lane_ok) {
#pragma unroll
    for (int j = 0; j < kLinkBatch; ++j) {
      const int c = lfirst + j * lstep;
      if (c < nchunk) stage_piece(c, lq[j]);
    }
    for (int c = lfirst + kLinkBatch * lstep; c < nchunk; c += lstep) stage_piece(c, load_piece(c));
  }
  __syncthreads();

  R acc[24];
  zero24(acc);
  const R *Lsite = Lk + sl * 144;
  const uint32_t *Lra = Lw + sl * kSiteLinks + (tid & 3) * kRowWords;
  const uint32_t *Lrb = Lw + sl * kSiteLinks + (4 + (tid & 1)) * kRowWords;
  // PRE: the input is M_phi in = b (1 + (c/b) P_chi) in; the factor b goes
  // into the final scale (handles are created only for b != 0)
  const R pc = PRE ? (R)(a.mphi_c / a.mphi_b) : R(0);
  const R pcu = pc * ((s > 0) ? R(1) : (R)(-a.mf));
  const R pcl = pc * ((s < Ls - 1) ? R(1) : (R)(-a.mf));
  // an opaque 1 (BF16, see hop_dir_norm)
  float one = 1.f;
  asm volatile("" : "+s"(one));
  // The eight directions are written out: as a loop over mu with a switch for
  // the code of a direction, each wave issued about 100 moves, copies and
  // address instructions more per mu, and the registers that they held left
  // FP64 no room to load ahead.  The scheduling barriers keep one direction's
  // registers from overlapping the next one's.  Loop -> written out with two
  // spinors ahead (FP64 one), 24^3 x 64 x 24: F16 block hops 1-4 2937 -> 2718 us,
  // F16 dslash_eo 469 -> 420, FP32 A 3129 -> 3030, FP64 A 6673 -> 6208.
  // (the sums exist from here on: without this the compiler moves the
  // multiply-adds of all directions into the later blocks that use them, and
  // keeps every product alive until then)
  auto pin_sums = [&]() {
#pragma unroll
    for (int k = 0; k < 24; ++k) asm volatile("" : "+v"(acc[k]));
  };
  auto product = [&](auto dc, const RawSite<S> &raw) {
    constexpr int d = decltype(dc)::value, mu = d >> 1;
    // (1 - g_mu) for the forward hop of H and the backward hop of H^+
    constexpr int sg = (DAG != 0) == ((d & 1) != 0) ? 1 : -1;
    const R *U = Lsite + d * 18;
    const uint32_t *ra = Lra + d * kLinkWords, *rb = Lrb + d * kLinkWords;
    const bool out = !GLOBAL && ((outm >> d) & 1);
    if constexpr (kH16) {
      hop_dir_h16<mu, sg, PRE, XM, MM>(lds, nthr, tid, s, Ls, pcu, pcl, raw, Lw + sl * 144 + d * 18, ra, rb, acc, out);
    } else if constexpr (MM != 0) {
      static_assert(!PRE, "M_phi mixes neighbouring s");
      hop_dir_b16_mm<mu, sg>(raw, ra, rb, acc, out ? 0.f : raw.n);
    } else if constexpr (Traits<S>::kNorm) {
      hop_dir_norm<mu, sg, PRE, XM>(lds, nthr, tid, s, Ls, pcu, pcl, one, raw, U, acc, out);
    } else {
      R v[24];
      raw.decode(v);
      hop_dir<mu, sg, PRE, XM>(lds, nthr, tid, s, Ls, pcu, pcl, v, U, acc, out ? R(0) : R(1));
    }
  };
  auto direction = [&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (d + kAhead < 8) load_nbr(buf[(d + kAhead) % (kAhead + 1)], nbw[d + kAhead < 8 ? d + kAhead : 0]);
    __builtin_amdgcn_sched_barrier(0);
    product(dc, buf[d % (kAhead + 1)]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto sparse_direction = [&](auto dc) {
    constexpr int d = decltype(dc)::value;
    if (!((live >> d) & 1)) return;
    RawSite<S> raw;
    load_nbr(raw, nbw[d]);
    product(dc, raw);
    pin_sums();
  };
  auto all = [](auto &&f) {
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
    f(std::integral_constant<int, 4>{});
    f(std::integral_constant<int, 5>{});
    f(std::integral_constant<int, 6>{});
    f(std::integral_constant<int, 7>{});
  };
  if constexpr (kSparse) {
    if (sparse) all(sparse_direction);
    else all(direction);
  } else {
    all(direction);
  }
  pin_sums();

  const R scale = (R)(PRE ? a.scale * a.mphi_b : a.scale);
  // (the opaque copy keeps the conversion, and so the wait for the load, here)
  asm volatile("" : "+v"(alpha_u));
  const R fu = upd ? -(R)alpha_u : R(1);
  if (EPI == EPI_M5INV) {
    m5_chain<DAG, R>(lds, tid, s, Ls, G, reinterpret_cast<const R *>(a.mat), scale, acc);
  } else if (EPI == EPI_MPHIDAG) {
    pchi_comb<1, XM, R>(lds, nthr, tid, s, Ls, (R)a.mphi_b, (R)a.mphi_c, (R)a.mf, acc);
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] *= scale;
  } else if (EPI == EPI_SCALE) {
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] *= scale;
  } else if (EPI == EPI_ADD_OTHER || EPI == EPI_M5INV_OTHER) {  // (full lattice)
    StoredOperand<S> o;
    o.load(reinterpret_cast<const S *>(a.other), a.other_norm, (size_t)r * a.other_stride + max(cb, 0), s, Ls);
    const R ow = o.norm();
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = fma(o.val(k), ow, scale * acc[k]);
    if (EPI == EPI_M5INV_OTHER) m5_chain<DAG, R>(lds, tid, s, Ls, G, reinterpret_cast<const R *>(a.mat), R(1), acc);
  }
  if (EPI == EPI_M5_OTHER || EPI == EPI_M5DAG_MPHIDAG) {
    // (outside the block domain the operand vanishes; those lanes load
    // nothing: a shared substitute site would draw the reads of every such
    // lane onto one cache line)
    const int oi = GLOBAL ? cb : (active ? (a.other_idx ? a.other_idx[site] : site) : -1);
    StoredOperand<S> o;
    o.zero();
    if (oi >= 0) o.load(reinterpret_cast<const S *>(a.other), a.other_norm, (size_t)r * a.other_stride + oi, s, Ls);
    const R ow = oi >= 0 ? o.norm() * fu : R(0);
    // M_5 = alpha - beta P_chi, M_5^+ = alpha - beta P_chi^+, M_phi^+ = b + c P_chi^+:
    //   M_5 o + scale h                 = (alpha o + scale h) + P_chi (-beta o)
    //   M_5^+ o + scale M_phi^+ h       = (alpha o + scale b h) + P_chi^+ (-beta o + scale c h)
    // (every coefficient times fu; the operand's norm with those of o)
    const R al = (R)a.m5_alpha * ow, mbe = (R)(-a.m5_beta) * ow;
    const R sb = (EPI == EPI_M5DAG_MPHIDAG ? scale * (R)a.mphi_b : scale) * fu;
    const R sc = (R)a.mphi_c * scale * fu;
    R B[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      const R ok = o.val(k);
      B[k] = EPI == EPI_M5DAG_MPHIDAG ? fma(ok, mbe, sc * acc[k]) : ok * mbe;
      acc[k] = fma(ok, al, sb * acc[k]);
    }
    pchi_add<EPI == EPI_M5DAG_MPHIDAG ? 1 : 0, XM, R>(lds, nthr, tid, s, Ls, (R)a.mf, acc, B);
  } else if (upd) {
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] *= fu;
  }

  R sumsq = 0;  // |out|^2 of the values as stored (DOT after a fused update)
  if (upd) {  // out <- out - alpha (result), read in place
    StoredOperand<S> ro;
    ro.load(reinterpret_cast<const S *>(a.out), a.out_norm, (size_t)r * a.out_stride + self, s, Ls);
    const R rn = ro.norm();
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = fma(ro.val(k), rn, acc[k]);
    if (DOT && !a.dotw)
      sumsq = store24_sumsq<S, R>(reinterpret_cast<S *>(a.out), a.out_norm, (size_t)r * a.out_stride + self, s, Ls,
                                  acc);
    else
      store24<R>(reinterpret_cast<S *>(a.out), a.out_norm, (size_t)r * a.out_stride + self, s, Ls, acc);
  } else if (active) {
    store24<R>(reinterpret_cast<S *>(a.out), a.out_norm, (size_t)r * a.out_stride + self, s, Ls, acc);
  }

  if (DOT) {  // Re<w, out>, or |out|^2 without w (of the values as stored, after a fused update)
    double val = 0;
    if (active) {
      R t = 0;
      if (a.dotw) {
        R w[24];
        load24<R>(reinterpret_cast<const S *>(a.dotw), a.dotw_norm, (size_t)r * a.dotw_stride + self, s, Ls, w);
#pragma unroll
        for (int k = 0; k < 24; ++k) t += w[k] * acc[k];
      } else if (upd) {
        t = sumsq;
      } else {
#pragma unroll
        for (int k = 0; k < 24; ++k) t += acc[k] * acc[k];
      }
      val = (double)t;
    }
    wg_partial(reinterpret_cast<double *>(smem), nthr, tid, Ls, nrhs, nsw, G, val, a.partial, tile);
  }
}

template <typename S>
static size_t hop_lds_bytes(const HopArgs &a, int nthr, int epi, int dot, int xm, int mm) {
  using R = typename Traits<S>::R;
  size_t b = (size_t)4 * (mm ? hop_link_words<S, 1>() : hop_link_words<S, 0>()) * a.nsite_wg;
  if (epi == EPI_M5INV || epi == EPI_M5INV_OTHER || xm == kXLds) b += (size_t)kRow * nthr * sizeof(R);
  if (dot) b = std::max(b, (size_t)2 * nthr * sizeof(double));
  return b;
}

// Types whose link products may run on the matrix cores: F16, and BF16 without
// M_phi on the input
template <typename S, int PRE> constexpr bool hop_can_mm() {
  return std::is_same<S, _Float16>::value || (std::is_same<S, bf16>::value && !PRE);
}

template <typename S, int DAG, int PRE, int EPI, int DOT, int GLOBAL, int MM>
static hipError_t launch_hop_t(const HopArgs &a, hipStream_t st) {
  const int xm = xmode(a.Ls, a.nrhs);
  const int nthr = layout_threads(xm, a.Ls, a.nsite_wg * a.nrhs);
  const int grid = (a.nsites + a.nsite_wg - 1) / a.nsite_wg;
  if (a.nsite_wg < 1 || nthr > 256 || grid < 1) return hipErrorInvalidValue;
  const dim3 blk = (xm == kXLds) ? dim3(a.Ls, a.nrhs, a.nsite_wg) : dim3(nthr);
  const size_t lds = hop_lds_bytes<S>(a, nthr, EPI, DOT, xm, MM);
  if (lds > kMaxLds) return hipErrorInvalidValue;
  switch (xm) {
    case kXDpp16:  // (Ls = 16: always on the matrix cores where they are used at all)
      if constexpr (MM || !hop_can_mm<S, PRE>())
        hipLaunchKernelGGL((hop_kernel<S, DAG, PRE, EPI, DOT, GLOBAL, kXDpp16, MM>), dim3(grid), blk, lds, st, a);
      break;
    case kXPerm: hipLaunchKernelGGL((hop_kernel<S, DAG, PRE, EPI, DOT, GLOBAL, kXPerm, MM>), dim3(grid), blk, lds, st, a); break;
    default: hipLaunchKernelGGL((hop_kernel<S, DAG, PRE, EPI, DOT, GLOBAL, kXLds, MM>), dim3(grid), blk, lds, st, a); break;
  }
  return hipGetLastError();
}

int hop_threads(int Ls, int nrhs, int nsite_wg) { return layout_threads(xmode(Ls, nrhs), Ls, nrhs * nsite_wg); }
int hop_groups_per_wave(int Ls, int nrhs) { return groups_per_wave(xmode(Ls, nrhs), Ls); }

bool hop_fits(int prec, int pre, int epi, int dot, const HopArgs &a) {
  const int nthr = hop_threads(a.Ls, a.nrhs, a.nsite_wg), xm = xmode(a.Ls, a.nrhs), mm = a.Ls % 4 == 0;
  size_t lds = 0;
  switch (prec) {
    case MSPCG_F64: lds = hop_lds_bytes<double>(a, nthr, epi, dot, xm, 0); break;
    case MSPCG_F32: lds = hop_lds_bytes<float>(a, nthr, epi, dot, xm, 0); break;
    case MSPCG_F16: lds = hop_lds_bytes<_Float16>(a, nthr, epi, dot, xm, mm); break;
    default: lds = hop_lds_bytes<bf16>(a, nthr, epi, dot, xm, mm && !pre); break;
  }
  return nthr <= 256 && lds <= kMaxLds;
}

template <typename S>
static hipError_t dispatch_hop(int dagger, int pre, int epi, int dot, int global, const HopArgs &a, hipStream_t st) {
  // F16 and BF16 link products run on the matrix cores wherever the lanes of a
  // site come in fours (every group of four lanes needs one link); other Ls take
  // dot products (F16, 24^3 x 64 x 24: 469 and 510 us a dslash_eo) or FP32
  // multiply-adds (BF16 daggered, 16^3 x 32 x 24: 59.7 and 63.9 us).
  const bool mm = a.Ls % 4 == 0;
  // the combinations used by the operators (anything else is rejected)
#define MSPCG_HOP(D, P, E, T, G)                                                \
  if (dagger == D && pre == P && epi == E && dot == T && (global != 0) == (G != 0)) \
    return mm ? launch_hop_t<S, D, P, E, T, G, hop_can_mm<S, P>()>(a, st) : launch_hop_t<S, D, P, E, T, G, 0>(a, st);
  MSPCG_HOP(0, 1, EPI_SCALE, 0, 1)          // M^4 in
  MSPCG_HOP(1, 0, EPI_MPHIDAG, 0, 1)        // (M^4)^+ in
  MSPCG_HOP(0, 1, EPI_M5INV, 0, 1)          // M_phi M_5^-1 M^4 in (first hop of D_PC)
  MSPCG_HOP(0, 0, EPI_M5_OTHER, 0, 1)       // M_5 psi + 1/2 H c
  if constexpr (std::is_same<S, double>::value) {
    MSPCG_HOP(0, 0, EPI_M5_OTHER, 1, 1)     //   ... with the fused |out|^2 (<p, A p> = |D_PC p|^2; the FP64 solvers)
    MSPCG_HOP(0, 0, EPI_ADD_OTHER, 0, 1)    // phi + 1/2 H c (source preparation)
    MSPCG_HOP(0, 1, EPI_M5INV_OTHER, 0, 1)  // M_5^-1 (phi + 1/2 H M_phi in) (reconstruction)
  }
  MSPCG_HOP(1, 0, EPI_M5INV, 0, 1)          // M_5^-+ M_phi^+ (M^4)^+ y
  MSPCG_HOP(1, 0, EPI_M5DAG_MPHIDAG, 0, 1)  // M_5^+ y + 1/2 M_phi^+ H^+ f
  MSPCG_HOP(1, 0, EPI_M5DAG_MPHIDAG, 1, 1)  //   ... with the fused <w, out>, or the residual update with its |r|^2
  MSPCG_HOP(0, 0, EPI_M5INV, 0, 0)          // the same four hops on block domains (M_phi p formed beforehand;
                                            // neighbours outside a domain enter with weight zero, which needs
                                            // the input unmixed: no M_phi on the input there)
  MSPCG_HOP(0, 0, EPI_M5_OTHER, 0, 0)
  MSPCG_HOP(0, 0, EPI_M5_OTHER, 1, 0)          //   ... with the fused |out|^2 (<p, A_s p> = |D_PC P_s p|^2)
  MSPCG_HOP(1, 0, EPI_M5INV, 0, 0)
  MSPCG_HOP(1, 0, EPI_M5DAG_MPHIDAG, 0, 0)
  MSPCG_HOP(1, 0, EPI_M5DAG_MPHIDAG, 1, 0)
#undef MSPCG_HOP
  return hipErrorInvalidValue;
}

hipError_t launch_hop(int prec, int dagger, int pre, int epi, int dot, int global, const HopArgs &a, hipStream_t st) {
  switch (prec) {
    case MSPCG_F64: return dispatch_hop<double>(dagger, pre, epi, dot, global, a, st);
    case MSPCG_F32: return dispatch_hop<float>(dagger, pre, epi, dot, global, a, st);
    case MSPCG_F16: return dispatch_hop<_Float16>(dagger, pre, epi, dot, global, a, st);
    case MSPCG_BF16: return dispatch_hop<bf16>(dagger, pre, epi, dot, global, a, st);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- fifth-dimension operator
// Non-temporal stores (NT) pay only where a wave fills the lines it writes: a
// store instruction writes one row of Ls x 16 bytes per site, and a line that
// holds the ends of two rows, or a site shared by two waves, reaches memory in
// parts.  They are used for rows of whole 64-byte segments (Ls a multiple of
// four), and for other Ls where a wave holds whole sites and a row has a segment
// of its own (FP64, with the most rows: Ls >= 8).  M_5^{-1}, ordinary -> non-temporal,
// us, used: FP64 Ls 24 on 24^3 x 48 570 -> 561, Ls 14 on 16^3 x 32 74 -> 63; FP32 Ls 6 and
// 16 on 24^3 x 48 90 -> 74 and 187 -> 180, F16 Ls 10 111 -> 83; not used: FP64 Ls 2 59 ->
// 81, Ls 5 167 -> 175, Ls 11 (packed lanes) 246 -> 317, FP32 Ls 13 (packed) 153 -> 194.
static bool op5_nontemporal(int prec, int Ls, int nrhs) {
  return Ls % 4 == 0 || (hop_groups_per_wave(Ls, nrhs) > 0 && Ls >= (prec == MSPCG_F64 ? 8 : 5));
}

template <typename S, int XM, bool NT>
__global__ void __launch_bounds__(256) op5_kernel(const Op5Args a) {
  using R = typename Traits<S>::R;
  extern __shared__ __align__(16) unsigned char smem[];
  const int Ls = a.Ls, nrhs = a.nrhs;
  const int G = groups_per_wave(XM, Ls);  // lane layout as in hop_kernel
  const int nthr = blockDim.x * blockDim.y * blockDim.z;
  int s, r, sl, tid;
  bool lane_ok = true;
  if (XM == kXLds) {
    s = threadIdx.x, r = threadIdx.y, sl = threadIdx.z;
    tid = s + Ls * (r + nrhs * sl);
  } else {
    tid = threadIdx.x;
    const int lane = tid & 63, gi = lane / Ls;
    s = lane - gi * Ls;
    int g = (tid >> 6) * G + gi;
    lane_ok = gi < G && g < nrhs * a.nsite_wg;
    if (!lane_ok) g = 0;
    r = g % nrhs;
    sl = g / nrhs;
  }
  R *lds = reinterpret_cast<R *>(smem);
  const int site = blockIdx.x * a.nsite_wg + sl;
  const bool active = lane_ok && site < a.nsites;
  R v[24];
  const size_t idx = (size_t)r * a.stride + (active ? site : 0);
  load24<R>(reinterpret_cast<const S *>(a.in), a.in_norm, idx, s, Ls, v);
  if (a.inv && a.dag)
    m5_chain<1, R>(lds, tid, s, Ls, G, reinterpret_cast<const R *>(a.chain), R(1), v);
  else if (a.inv)
    m5_chain<0, R>(lds, tid, s, Ls, G, reinterpret_cast<const R *>(a.chain), R(1), v);
  else if (a.dag)
    pchi_comb<1, XM, R>(lds, nthr, tid, s, Ls, (R)a.a, (R)a.b, (R)a.mf, v);
  else
    pchi_comb<0, XM, R>(lds, nthr, tid, s, Ls, (R)a.a, (R)a.b, (R)a.mf, v);
  if (active) store24<R, NT>(reinterpret_cast<S *>(a.out), a.out_norm, idx, s, Ls, v);
}

template <typename S, bool NT>
static void launch_op5_t(const Op5Args &a, dim3 grid, dim3 blk, size_t lds, hipStream_t st) {
  switch (xmode(a.Ls, a.nrhs)) {
    case kXDpp16: hipLaunchKernelGGL((op5_kernel<S, kXDpp16, NT>), grid, blk, lds, st, a); break;
    case kXPerm: hipLaunchKernelGGL((op5_kernel<S, kXPerm, NT>), grid, blk, lds, st, a); break;
    default: hipLaunchKernelGGL((op5_kernel<S, kXLds, NT>), grid, blk, lds, st, a); break;
  }
}

hipError_t launch_op5(int prec, const Op5Args &a, hipStream_t st) {
  const int xm = xmode(a.Ls, a.nrhs);
  const int nthr = layout_threads(xm, a.Ls, a.nsite_wg * a.nrhs);
  const int grid = (a.nsites + a.nsite_wg - 1) / a.nsite_wg;
  if (a.nsite_wg < 1 || nthr > 256 || grid < 1) return hipErrorInvalidValue;
  const size_t rsz = (prec == MSPCG_F64) ? 8 : 4;
  const size_t lds = (size_t)kRow * nthr * rsz;
  const dim3 blk = (xm == kXLds) ? dim3(a.Ls, a.nrhs, a.nsite_wg) : dim3(nthr);
  const bool nt = op5_nontemporal(prec, a.Ls, a.nrhs);
#define MSPCG_OP5(S) nt ? launch_op5_t<S, true>(a, dim3(grid), blk, lds, st) : launch_op5_t<S, false>(a, dim3(grid), blk, lds, st)
  switch (prec) {
    case MSPCG_F64: MSPCG_OP5(double); break;
    case MSPCG_F32: MSPCG_OP5(float); break;
    case MSPCG_F16: MSPCG_OP5(_Float16); break;
    case MSPCG_BF16: launch_op5_t<bf16, false>(a, dim3(grid), blk, lds, st); break;
    default: return hipErrorInvalidValue;
  }
#undef MSPCG_OP5
  return hipGetLastError();
}

// ---------------------------------------------------------------- conversion
// Non-temporal stores as in op5_kernel; the lanes are packed, so only rows of
// whole 128-byte lines, or of whole 64-byte segments and more than two lines,
// gain.  Ordinary -> non-temporal, us, 24^3 x 48, used: FP64 to FP64 Ls 24 567 -> 546,
// FP32 to FP64 Ls 8 146 -> 110, FP64 to FP64 Ls 20 on 16^3 x 32 94 -> 79; not used: FP64 to
// FP64 Ls 2 40 -> 117, 5 118 -> 220, 10 246 -> 306, 12 294 -> 307, F16 to FP64 Ls 5 97 -> 190.
template <typename SO, typename SI, bool NT>
__global__ void convert_kernel(SO *out, float *out_norm, const SI *in, const float *in_norm, long long n5, int Ls) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n5) return;
  const size_t site4 = (size_t)(i / Ls);
  const int s = (int)(i % Ls);
  using T = typename std::conditional<sizeof(SI) == 8 || sizeof(SO) == 8, double, float>::type;
  T v[24];
  load24<T>(in, in_norm, site4, s, Ls, v);
  store24<T, NT>(out, out_norm, site4, s, Ls, v);
}

template <typename SO, typename SI>
static void launch_convert_t(const Vec &out, const Vec &in, long long n5, int Ls, hipStream_t st) {
  const int blk = 256;
  const dim3 grid((n5 + blk - 1) / blk);
  SO *o = reinterpret_cast<SO *>(out.data);
  const SI *i = reinterpret_cast<const SI *>(in.data);
  if (Ls % 8 == 0 || (Ls % 4 == 0 && Ls > 16))
    hipLaunchKernelGGL((convert_kernel<SO, SI, true>), grid, dim3(blk), 0, st, o, out.norm, i, in.norm, n5, Ls);
  else
    hipLaunchKernelGGL((convert_kernel<SO, SI, false>), grid, dim3(blk), 0, st, o, out.norm, i, in.norm, n5, Ls);
}

template <typename SO>
static hipError_t convert_from(const Vec &out, const Vec &in, long long n5, int Ls, hipStream_t st) {
  switch (in.prec) {
    case MSPCG_F64: launch_convert_t<SO, double>(out, in, n5, Ls, st); break;
    case MSPCG_F32: launch_convert_t<SO, float>(out, in, n5, Ls, st); break;
    case MSPCG_F16: launch_convert_t<SO, _Float16>(out, in, n5, Ls, st); break;
    case MSPCG_BF16: launch_convert_t<SO, bf16>(out, in, n5, Ls, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_convert(const Vec &out, const Vec &in, int nrhs, long long nsites5, int Ls, hipStream_t st) {
  const long long n5 = nsites5 * nrhs;
  if (n5 <= 0) return hipSuccess;
  switch (out.prec) {
    case MSPCG_F64: return convert_from<double>(out, in, n5, Ls, st);
    case MSPCG_F32: return convert_from<float>(out, in, n5, Ls, st);
    case MSPCG_F16: return convert_from<_Float16>(out, in, n5, Ls, st);
    case MSPCG_BF16: return convert_from<bf16>(out, in, n5, Ls, st);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- FP64 BLAS
// Grid (kBlasGrid, nrhs) with a grid-stride loop over double2 pairs: the set
// of elements each thread sums, and the reduction tree, depend only on n.
__device__ inline void block_sum_store(double v, double *out) {
  __shared__ double sh[kBlasWG];
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int w = kBlasWG / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

__global__ void __launch_bounds__(kBlasWG) k_dot(const double *a, const double *b, long long n, double *partial) {
  const int r = blockIdx.y;
  const double2 *x = reinterpret_cast<const double2 *>(a + (size_t)r * n);
  const double2 *y = reinterpret_cast<const double2 *>(b + (size_t)r * n);
  const long long n2 = n / 2;
  double acc = 0;
  for (long long i = (long long)blockIdx.x * kBlasWG + threadIdx.x; i < n2; i += (long long)kBlasGrid * kBlasWG) {
    const double2 u = x[i], v = y[i];
    acc += u.x * v.x + u.y * v.y;
  }
  block_sum_store(acc, partial + (size_t)blockIdx.x * gridDim.y + r);
}

hipError_t blas_dot_partial(const double *a, const double *b, long long n, int nrhs, double *partial, hipStream_t st) {
  hipLaunchKernelGGL(k_dot, dim3(kBlasGrid, nrhs), dim3(kBlasWG), 0, st, a, b, n, partial);
  return hipGetLastError();
}

// partial[p][r] -> out[r], and what the solvers form from it; one workgroup per
// right-hand side.  Bound by latency: each thread sums eight strands (fixed
// order: deterministic), whose loads are guarded and follow one another.  4096
// partials: 15 us with 256 threads of one strand, 5 us so; 44000 take 28 us.
constexpr int kReduceWG = 1024, kReduceStrands = 8;
__global__ void __launch_bounds__(kReduceWG) k_reduce(const double *partial, int nparts, int nrhs, double *out,
                                                      const ReduceOp op) {
  __shared__ double sh[kReduceWG / 64];
  const int r = blockIdx.x;
  // The scalars of the solvers are requested with the partial sums, not after
  // them, and as vector loads (scalar ones would all be waited for before the
  // first partial sum is requested).
  double rho = 0, rho_new = 0, stop = -1, last_beta = 0;
  if (op.scal) {
    int vr = r;
    asm("" : "+v"(vr));
    rho = op.scal[kRho * nrhs + vr];
    rho_new = op.scal[kRR * nrhs + vr];
    stop = op.scal[kStop * nrhs + vr];
    last_beta = op.scal[kBeta * nrhs + min((int)(threadIdx.x & 63), nrhs - 1)];
  }
  double acc[kReduceStrands];
#pragma unroll
  for (int j = 0; j < kReduceStrands; ++j) acc[j] = 0;
  for (int p0 = threadIdx.x; p0 < nparts; p0 += kReduceWG * kReduceStrands) {
#pragma unroll
    for (int j = 0; j < kReduceStrands; ++j) {
      const int p = p0 + j * kReduceWG;
      if (p < nparts) acc[j] += partial[(size_t)p * nrhs + r];
    }
  }
#pragma unroll
  for (int w = kReduceStrands / 2; w > 0; w >>= 1)
#pragma unroll
    for (int j = 0; j < w; ++j) acc[j] += acc[j + w];
  double v = acc[0];
#pragma unroll
  for (int w = 32; w > 0; w >>= 1) v += __shfl_down(v, w, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  const bool on = stop >= 0.0, dropped = op.ahead && __ballot(last_beta < 0.0) != 0;
  if (threadIdx.x != 0) return;
  v = 0;
#pragma unroll
  for (int w = 0; w < kReduceWG / 64; ++w) v += sh[w];
  out[r] = v;
  if (op.mode == 1) {  // v = <p, A p>
    if (op.ahead && on && !dropped) op.scal[kRho * nrhs + r] = rho = rho_new;
    op.scal[kAlpha * nrhs + r] = (on && !dropped && v != 0.0) ? rho / v : 0.0;
  } else if (op.mode == 2) {  // v = rho_new
    op.scal[kBeta * nrhs + r] = v <= stop ? -1.0 : (on && rho != 0.0) ? v / rho : 0.0;
  }
  if (op.host) {  // the value, then its tag, in host memory
    __hip_atomic_store(op.host->rr + r, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(op.host->tag + r, op.tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

hipError_t blas_reduce(const double *partial, int nparts, int nrhs, double *out, hipStream_t st, const ReduceOp &op) {
  hipLaunchKernelGGL(k_reduce, dim3(nrhs), dim3(kReduceWG), 0, st, partial, nparts, nrhs, out, op);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kBlasWG) k_update_xr(double *xv, double *rv, const double *pv, const double *qv,
                                                       const double *alpha, long long n, double *partial) {
  const int r = blockIdx.y;
  const double al = alpha[r];
  double2 *x = reinterpret_cast<double2 *>(xv + (size_t)r * n);
  double2 *rr = reinterpret_cast<double2 *>(rv + (size_t)r * n);
  const double2 *p = reinterpret_cast<const double2 *>(pv + (size_t)r * n);
  const double2 *q = reinterpret_cast<const double2 *>(qv + (size_t)r * n);
  const long long n2 = n / 2;
  double acc = 0;
  for (long long i = (long long)blockIdx.x * kBlasWG + threadIdx.x; i < n2; i += (long long)kBlasGrid * kBlasWG) {
    double2 xi = x[i], ri = rr[i];
    const double2 pi = p[i], qi = q[i];
    xi.x += al * pi.x; xi.y += al * pi.y;
    ri.x -= al * qi.x; ri.y -= al * qi.y;
    store16(x + i, xi);
    store16(rr + i, ri);
    acc += ri.x * ri.x + ri.y * ri.y;
  }
  block_sum_store(acc, partial + (size_t)blockIdx.x * gridDim.y + r);
}

hipError_t blas_update_xr(double *x, double *r, const double *p, const double *q, const double *alpha, long long n,
                          int nrhs, double *partial, hipStream_t st) {
  hipLaunchKernelGGL(k_update_xr, dim3(kBlasGrid, nrhs), dim3(kBlasWG), 0, st, x, r, p, q, alpha, n, partial);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kBlasWG) k_xpay(double *pv, const double *zv, const double *beta, long long n) {
  const int r = blockIdx.y;
  const double be = beta[r];
  double2 *p = reinterpret_cast<double2 *>(pv + (size_t)r * n);
  const double2 *z = reinterpret_cast<const double2 *>(zv + (size_t)r * n);
  const long long n2 = n / 2;
  for (long long i = (long long)blockIdx.x * kBlasWG + threadIdx.x; i < n2; i += (long long)kBlasGrid * kBlasWG) {
    double2 pi = p[i];
    const double2 zi = z[i];
    pi.x = zi.x + be * pi.x;
    pi.y = zi.y + be * pi.y;
    store16(p + i, pi);
  }
}

hipError_t blas_xpay(double *p, const double *z, const double *beta, long long n, int nrhs, hipStream_t st) {
  hipLaunchKernelGGL(k_xpay, dim3(kBlasGrid, nrhs), dim3(kBlasWG), 0, st, p, z, beta, n);
  return hipGetLastError();
}

// x += alpha p and p = z + beta p in one pass (the x update of an iteration
// waits for beta: five passes over memory instead of the 3 + 3 of an update of
// x and one of p).  Bound by memory.
__global__ void __launch_bounds__(kBlasWG) k_update_xp(double *xv, double *pv, const double *zv, const double *scal,
                                                       long long n, int nrhs, int ahead) {
  const int r = blockIdx.y;
  const double *beta = scal + kBeta * nrhs;
  const double al = scal[kAlpha * nrhs + r], be = beta[r];
  double any_be = 0;
  if (nrhs > 1) any_be = beta[min((int)(threadIdx.x & 63), nrhs - 1)];
  double2 *x = reinterpret_cast<double2 *>(xv + (size_t)r * n);
  double2 *p = reinterpret_cast<double2 *>(pv + (size_t)r * n);
  const double2 *z = reinterpret_cast<const double2 *>(zv + (size_t)r * n);
  const long long n2 = n / 2;
  for (long long i = (long long)blockIdx.x * kBlasWG + threadIdx.x; i < n2; i += (long long)kBlasGrid * kBlasWG) {
    double2 xi = x[i], pi = p[i];
    const double2 zi = z[i];
    xi.x += al * pi.x;
    xi.y += al * pi.y;
    pi.x = zi.x + be * pi.x;
    pi.y = zi.y + be * pi.y;
    store16(x + i, xi);
    // (seen by the first lanes of a wave, 32 at least: n2 is a multiple of 32)
    if (!(ahead && (nrhs == 1 ? be < 0.0 : __ballot(any_be < 0.0) != 0))) store16(p + i, pi);
  }
}

hipError_t blas_update_xp(double *x, double *p, const double *z, const double *scal, long long n, int nrhs, int ahead,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_update_xp, dim3(kBlasGrid, nrhs), dim3(kBlasWG), 0, st, x, p, z, scal, n, nrhs, ahead);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kBlasWG) k_axpy(double *xv, const double *pv, const double *alpha, long long n) {
  const int r = blockIdx.y;
  const double al = alpha[r];
  double2 *x = reinterpret_cast<double2 *>(xv + (size_t)r * n);
  const double2 *p = reinterpret_cast<const double2 *>(pv + (size_t)r * n);
  const long long n2 = n / 2;
  for (long long i = (long long)blockIdx.x * kBlasWG + threadIdx.x; i < n2; i += (long long)kBlasGrid * kBlasWG) {
    double2 xi = x[i];
    const double2 pi = p[i];
    xi.x += al * pi.x;
    xi.y += al * pi.y;
    store16(x + i, xi);
  }
}

hipError_t blas_axpy(double *x, const double *p, const double *alpha, long long n, int nrhs, hipStream_t st) {
  hipLaunchKernelGGL(k_axpy, dim3(kBlasGrid, nrhs), dim3(kBlasWG), 0, st, x, p, alpha, n);
  return hipGetLastError();
}

__global__ void __launch_bounds__(kBlasWG) k_axpby(double *ov, double a, const double *xv, double b, const double *yv,
                                                   long long n) {
  const int r = blockIdx.y;
  double2 *o = reinterpret_cast<double2 *>(ov + (size_t)r * n);
  const double2 *x = reinterpret_cast<const double2 *>(xv + (size_t)r * n);
  const double2 *y = reinterpret_cast<const double2 *>(yv + (size_t)r * n);
  const long long n2 = n / 2;
  for (long long i = (long long)blockIdx.x * kBlasWG + threadIdx.x; i < n2; i += (long long)kBlasGrid * kBlasWG) {
    const double2 xi = x[i], yi = y[i];
    store16(o + i, make_double2(a * xi.x + b * yi.x, a * xi.y + b * yi.y));
  }
}

hipError_t blas_axpby(double *out, double a, const double *x, double b, const double *y, long long n, int nrhs,
                      hipStream_t st) {
  hipLaunchKernelGGL(k_axpby, dim3(kBlasGrid, nrhs), dim3(kBlasWG), 0, st, out, a, x, b, y, n);
  return hipGetLastError();
}

__global__ void k_solver_scalars(int mode, int nrhs, const int *active, double *rho, const double *x1, double *out,
                                 const double *x2, const double *x3) {
  const int r = threadIdx.x;
  if (r >= nrhs) return;
  const bool on = active[r] != 0;
  const double rn = x1[r];
  if (mode == 1)
    out[r] = (on && rho[r] != 0.0) ? rn / rho[r] : 0.0;
  else
    out[r] = (on && x3[r] != 0.0) ? -x2[r] / x3[r] : 0.0;
  if (on) rho[r] = rn;
}

hipError_t solver_scalars(int mode, int nrhs, const int *active, double *rho, const double *x1, double *out,
                          hipStream_t st, const double *x2, const double *x3) {
  if ((mode != 1 && mode != 2) || (mode == 2 && (!x2 || !x3))) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_solver_scalars, dim3(1), dim3(64), 0, st, mode, nrhs, active, rho, x1, out, x2, x3);
  return hipGetLastError();
}

// ---------------------------------------------------------------- block preconditioner
// The B_e list is ordered block by block, each block padded to a multiple of
// 64 sites, so with nsite_wg dividing 64 every workgroup lies in one block.
// M_phi v = b v + c P_chi v for the Ls values of one (site, rhs) held on
// consecutive threads of a block kernel (layout tid = s + Ls (rhs + nrhs site)),
// exchanged through LDS; all threads of the workgroup must reach it.
template <typename R>
__device__ inline void block_mphi(R *lds, int nthr, int tid, int s, int Ls, const BlockArgs &b, R v[24]) {
  pchi_comb<0, kXLds, R>(lds, nthr, tid, s, Ls, (R)b.mphi_b, (R)b.mphi_c, (R)b.mf, v);
}

template <typename S, bool NT>
__global__ void __launch_bounds__(256) k_block_gather(const BlockArgs b, Vec xs, Vec rs, Vec ps, Vec mps,
                                                       const double *rg, long long rg_stride, const double *rr,
                                                       double n_total, double *partial) {
  using R = typename Traits<S>::R;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nthr = blockDim.x, tid = threadIdx.x, Ls = b.Ls, G = b.nrhs * Ls;
  const int sl = tid / G, rem = tid - sl * G, r = rem / Ls, s = rem - r * Ls;
  const int site = blockIdx.x * b.nsite_wg + sl;
  const int cb = site < b.nsites ? b.be_cb[site] : -1;
  const size_t o = (size_t)r * rs.stride + site;
  double val = 0;
  R v[24];
  zero24(v);
  if (cb >= 0) {
    const double scale = rr ? (rr[r] > 0 ? sqrt(n_total / rr[r]) : 0.0) : 1.0;
    double t[24];
    load24<double>(rg, nullptr, (size_t)r * rg_stride + cb, s, Ls, t);
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = (R)(scale * t[k]);
    store24<R, NT>(reinterpret_cast<S *>(rs.data), rs.norm, o, s, Ls, v);
    // the values as stored, so that r and p start identical and the sum matches them
    stored_values<S>(v);
    store24<R, NT>(reinterpret_cast<S *>(ps.data), ps.norm, o, s, Ls, v);
    if (xs.data) {  // (the fixed-k solve sets x in its first update instead)
      R z[24];
      zero24(z);
      store24<R, NT>(reinterpret_cast<S *>(xs.data), xs.norm, o, s, Ls, z);
    }
    R acc = 0;
#pragma unroll
    for (int k = 0; k < 24; ++k) acc += v[k] * v[k];
    val = (double)acc;
  }
  block_mphi<R>(reinterpret_cast<R *>(smem), nthr, tid, s, Ls, b, v);
  if (cb >= 0) store24<R, NT>(reinterpret_cast<S *>(mps.data), mps.norm, o, s, Ls, v);
  wg_partial(reinterpret_cast<double *>(smem), nthr, tid, Ls, b.nrhs, b.nsite_wg, 0, val, partial, blockIdx.x);
}

template <typename S, bool NT>
__global__ void __launch_bounds__(256) k_block_scatter(const BlockArgs b, double *zg, long long zg_stride, Vec xs,
                                                        Vec ps, const double *scal, int mode, const double *rg,
                                                        long long rg_stride, const double *rr, double n_total,
                                                        double *partial) {
  using R = typename Traits<S>::R;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nthr = blockDim.x, tid = threadIdx.x, Ls = b.Ls, G = b.nrhs * Ls;
  const int sl = tid / G, rem = tid - sl * G, r = rem / Ls, s = rem - r * Ls;
  const int site = blockIdx.x * b.nsite_wg + sl;
  const int cb = site < b.nsites ? b.be_cb[site] : -1;
  double val = 0;
  if (cb >= 0) {
    const double inv = rr ? (rr[r] > 0 ? sqrt(rr[r] / n_total) : 0.0) : 1.0;
    const size_t o = (size_t)r * xs.stride + site;
    R v[24];
    if (mode == 2) zero24(v); else load24<R>(reinterpret_cast<const S *>(xs.data), xs.norm, o, s, Ls, v);
    if (mode != 0) {  // the last inner iteration's x update, not stored: x + alpha p
      const int blk = b.be_blk[site];
      const R al = (R)scal[((size_t)blk * b.nrhs + r) * kScal + 1];
      R pv[24];
      load24<R>(reinterpret_cast<const S *>(ps.data), ps.norm, o, s, Ls, pv);
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = fma(al, pv[k], v[k]);
    }
    double z[24], t[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) z[k] = inv * (double)v[k];
    if (zg) store24<double, NT>(zg, nullptr, (size_t)r * zg_stride + cb, s, Ls, z);  // (none: only the partials)
    if (rg) {
      load24<double>(rg, nullptr, (size_t)r * rg_stride + cb, s, Ls, t);
#pragma unroll
      for (int k = 0; k < 24; ++k) val += z[k] * t[k];
    }
  }
  wg_partial(reinterpret_cast<double *>(smem), nthr, tid, Ls, b.nrhs, b.nsite_wg, 0, val, partial, blockIdx.x);
}

// The outer direction update fused with the scatter: p(cb) = v / scale +
// beta p(cb) (first: p = v / scale) with v as in k_block_scatter, so the
// preconditioned residual z is never stored.  With xg the outer solution's
// pending update x += alpha p happens here too, where p is read anyway.
template <typename S, bool NT>
__global__ void __launch_bounds__(256) k_block_scatter_xpay(const BlockArgs b, double *pg, double *xg,
                                                             long long pg_stride, Vec xs, Vec ps, const double *scal,
                                                             int mode, const double *rr, double n_total,
                                                             const double *alpha, const double *beta, int first) {
  using R = typename Traits<S>::R;
  const int tid = threadIdx.x, Ls = b.Ls, G = b.nrhs * Ls;
  const int sl = tid / G, rem = tid - sl * G, r = rem / Ls, s = rem - r * Ls;
  const int site = blockIdx.x * b.nsite_wg + sl;
  const int cb = site < b.nsites ? b.be_cb[site] : -1;
  if (cb < 0) return;
  const double inv = rr ? (rr[r] > 0 ? sqrt(rr[r] / n_total) : 0.0) : 1.0;
  const size_t o = (size_t)r * xs.stride + site;
  R v[24];
  if (mode == 2) zero24(v); else load24<R>(reinterpret_cast<const S *>(xs.data), xs.norm, o, s, Ls, v);
  if (mode != 0) {
    const R al = (R)scal[((size_t)b.be_blk[site] * b.nrhs + r) * kScal + 1];
    R pv[24];
    load24<R>(reinterpret_cast<const S *>(ps.data), ps.norm, o, s, Ls, pv);
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = fma(al, pv[k], v[k]);
  }
  const size_t g = (size_t)r * pg_stride + cb;
  double pn[24];
  if (first) {
#pragma unroll
    for (int k = 0; k < 24; ++k) pn[k] = inv * (double)v[k];
  } else {
    load24<double>(pg, nullptr, g, s, Ls, pn);
    const double be = beta[r];
    if (xg) {
      const double oal = alpha[r];
      double x[24];
      load24<double>(xg, nullptr, g, s, Ls, x);
#pragma unroll
      for (int k = 0; k < 24; ++k) x[k] = fma(oal, pn[k], x[k]);
      store24<double, NT>(xg, nullptr, g, s, Ls, x);
    }
#pragma unroll
    for (int k = 0; k < 24; ++k) pn[k] = fma(be, pn[k], inv * (double)v[k]);
  }
  store24<double, NT>(pg, nullptr, g, s, Ls, pn);
}

template <typename S, bool NT>
__global__ void __launch_bounds__(256) k_block_update_xr(const BlockArgs b, Vec xv, Vec rv, Vec pv, Vec qv,
                                                          const double *scal, double *partial) {
  using R = typename Traits<S>::R;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nthr = blockDim.x, tid = threadIdx.x, Ls = b.Ls, G = b.nrhs * Ls;
  const int sl = tid / G, rem = tid - sl * G, r = rem / Ls, s = rem - r * Ls;
  const int site = blockIdx.x * b.nsite_wg + sl;
  const int blk = site < b.nsites ? b.be_blk[site] : -1;
  double val = 0;
  if (blk >= 0) {
    const R al = (R)scal[((size_t)blk * b.nrhs + r) * kScal + 1];
    const size_t o = (size_t)r * xv.stride + site;
    R x[24], rr[24], p[24], q[24];
    load24<R>(reinterpret_cast<const S *>(xv.data), xv.norm, o, s, Ls, x);
    load24<R>(reinterpret_cast<const S *>(rv.data), rv.norm, o, s, Ls, rr);
    load24<R>(reinterpret_cast<const S *>(pv.data), pv.norm, o, s, Ls, p);
    load24<R>(reinterpret_cast<const S *>(qv.data), qv.norm, o, s, Ls, q);
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      x[k] += al * p[k];
      rr[k] -= al * q[k];
    }
    store24<R, NT>(reinterpret_cast<S *>(xv.data), xv.norm, o, s, Ls, x);
    store24<R, NT>(reinterpret_cast<S *>(rv.data), rv.norm, o, s, Ls, rr);
    // the norm is taken of the stored (rounded) residual
    stored_values<S>(rr);
    R acc = 0;
#pragma unroll
    for (int k = 0; k < 24; ++k) acc += rr[k] * rr[k];
    val = (double)acc;
  }
  wg_partial(reinterpret_cast<double *>(smem), nthr, tid, Ls, b.nrhs, b.nsite_wg, 0, val, partial, blockIdx.x);
}

// r -= alpha Ap with the partial |r|^2 (every iteration but the last, where
// k_block_update_xr also updates x)
template <typename S, bool NT>
__global__ void __launch_bounds__(256) k_block_update_r(const BlockArgs b, Vec rv, Vec qv, const double *scal,
                                                        double *partial) {
  using R = typename Traits<S>::R;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nthr = blockDim.x, tid = threadIdx.x, Ls = b.Ls, G = b.nrhs * Ls;
  const int sl = tid / G, rem = tid - sl * G, r = rem / Ls, s = rem - r * Ls;
  const int site = blockIdx.x * b.nsite_wg + sl;
  const int blk = site < b.nsites ? b.be_blk[site] : -1;
  double val = 0;
  if (blk >= 0) {
    const R al = (R)scal[((size_t)blk * b.nrhs + r) * kScal + 1];
    const size_t o = (size_t)r * rv.stride + site;
    R rr[24], q[24];
    load24<R>(reinterpret_cast<const S *>(rv.data), rv.norm, o, s, Ls, rr);
    load24<R>(reinterpret_cast<const S *>(qv.data), qv.norm, o, s, Ls, q);
#pragma unroll
    for (int k = 0; k < 24; ++k) rr[k] -= al * q[k];
    store24<R, NT>(reinterpret_cast<S *>(rv.data), rv.norm, o, s, Ls, rr);
    stored_values<S>(rr);
    R acc = 0;
#pragma unroll
    for (int k = 0; k < 24; ++k) acc += rr[k] * rr[k];
    val = (double)acc;
  }
  wg_partial(reinterpret_cast<double *>(smem), nthr, tid, Ls, b.nrhs, b.nsite_wg, 0, val, partial, blockIdx.x);
}

// x += alpha p, then p = r + beta p (the x update of k_block_update_xr moved
// here, where p is read anyway), and M_phi p for the next first hop (from the
// values as stored)
template <typename S, bool NT>
__global__ void __launch_bounds__(256) k_block_update_xp(const BlockArgs b, Vec xv, Vec pv, Vec mpv, Vec rv,
                                                         const double *scal, int first) {
  using R = typename Traits<S>::R;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nthr = blockDim.x, tid = threadIdx.x, Ls = b.Ls, G = b.nrhs * Ls;
  const int sl = tid / G, rem = tid - sl * G, r = rem / Ls, s = rem - r * Ls;
  const int site = blockIdx.x * b.nsite_wg + sl;
  const int blk = site < b.nsites ? b.be_blk[site] : -1;
  const size_t o = (size_t)r * pv.stride + site;
  R p[24];
  zero24(p);
  if (blk >= 0) {
    const double *sc = scal + ((size_t)blk * b.nrhs + r) * kScal;
    const R al = (R)sc[1], be = (R)sc[2];
    R x[24], rr[24];
    if (first) zero24(x);  // (x_0 = 0: not read)
    else load24<R>(reinterpret_cast<const S *>(xv.data), xv.norm, o, s, Ls, x);
    load24<R>(reinterpret_cast<const S *>(pv.data), pv.norm, o, s, Ls, p);
    load24<R>(reinterpret_cast<const S *>(rv.data), rv.norm, o, s, Ls, rr);
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      x[k] += al * p[k];
      p[k] = rr[k] + be * p[k];
    }
    store24<R, NT>(reinterpret_cast<S *>(xv.data), xv.norm, o, s, Ls, x);
    store24<R, NT>(reinterpret_cast<S *>(pv.data), pv.norm, o, s, Ls, p);
    stored_values<S>(p);
  }
  block_mphi<R>(reinterpret_cast<R *>(smem), nthr, tid, s, Ls, b, p);
  if (blk >= 0) store24<R, NT>(reinterpret_cast<S *>(mpv.data), mpv.norm, o, s, Ls, p);
}

// one workgroup per (block, rhs): a fixed-shape tree sum of that block's
// workgroup partials (deterministic), then the CG scalar update
__global__ void __launch_bounds__(256) k_block_scalars(int mode, int nrhs, int nsite_wg, const int *be_off,
                                                       const double *partial, double *scal) {
  __shared__ double sh[256];
  const int blk = blockIdx.x, r = blockIdx.y;
  const int w0 = be_off[blk] / nsite_wg, w1 = be_off[blk + 1] / nsite_wg;
  double sum = 0;
  for (int w = w0 + (int)threadIdx.x; w < w1; w += 256) sum += partial[(size_t)w * nrhs + r];
  sh[threadIdx.x] = sum;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  sum = sh[0];
  double *sc = scal + ((size_t)blk * nrhs + r) * kScal;
  if (mode == 0) {
    sc[1] = (sum > 0.0 && sc[0] > 0.0) ? sc[0] / sum : 0.0;
  } else if (mode == 1) {
    sc[2] = (sc[0] > 0.0) ? sum / sc[0] : 0.0;
    sc[0] = sum;
  } else {
    sc[0] = sum;
    sc[1] = sc[2] = 0.0;
  }
}

static inline int block_threads(const BlockArgs &b) { return b.nsite_wg * b.nrhs * b.Ls; }
static inline int block_grid(const BlockArgs &b) { return (b.nsites + b.nsite_wg - 1) / b.nsite_wg; }
static inline size_t block_lds(const BlockArgs &b) { return (size_t)2 * block_threads(b) * sizeof(double); }
// the kernels that form M_phi p exchange 24 reals per thread through LDS
template <typename S>
static inline size_t block_lds_mphi(const BlockArgs &b) {
  return std::max(block_lds(b), (size_t)kRow * block_threads(b) * sizeof(typename Traits<S>::R));
}

#define MSPCG_PREC_SWITCH(prec, ...)                        \
  switch (prec) {                                           \
    case MSPCG_F64: { using S = double; __VA_ARGS__; } break;   \
    case MSPCG_F32: { using S = float; __VA_ARGS__; } break;    \
    case MSPCG_F16: { using S = _Float16; __VA_ARGS__; } break; \
    case MSPCG_BF16: { using S = bf16; __VA_ARGS__; } break;    \
    default: return hipErrorInvalidValue;                   \
  }

// The lanes of the block kernels are packed: non-temporal stores (NT) only for rows
// of whole 64-byte segments (see op5_kernel).  Ordinary -> non-temporal, us, 24^3 x 48, 16
// blocks, gather and scatter alone in FP32, used: Ls 4 352 -> 315, 20 1739 -> 1668; not
// used: Ls 2 217 -> 364, 5 489 -> 721, 13 1160 -> 1435.  (With one iteration on 16^3 x 32
// at Ls 10 to 14 the two differ by 3%.)
#define MSPCG_BLOCK_SWITCH(prec, Ls, ...)       \
  if ((Ls) % 4 == 0) {                          \
    constexpr bool NT = true;                   \
    MSPCG_PREC_SWITCH(prec, __VA_ARGS__)        \
  } else {                                      \
    constexpr bool NT = false;                  \
    MSPCG_PREC_SWITCH(prec, __VA_ARGS__)        \
  }

hipError_t block_gather(int prec, const BlockArgs &b, const Vec &xs, const Vec &rs, const Vec &ps, const Vec &mps,
                        const Vec &rglob, const double *rr, double n_total, double *partial, hipStream_t st) {
  if (rglob.prec != MSPCG_F64 || block_threads(b) > 256) return hipErrorInvalidValue;
  MSPCG_BLOCK_SWITCH(prec, b.Ls, hipLaunchKernelGGL((k_block_gather<S, NT>), dim3(block_grid(b)),
                     dim3(block_threads(b)), block_lds_mphi<S>(b), st, b, xs, rs, ps, mps,
                     (const double *)rglob.data, rglob.stride, rr, n_total, partial));
  return hipGetLastError();
}

hipError_t block_scatter(int prec, const BlockArgs &b, const Vec &zglob, const Vec &xs, const Vec &ps,
                         const double *scal, int mode, const Vec &rglob, const double *rr, double n_total,
                         double *partial, hipStream_t st) {
  if (zglob.prec != MSPCG_F64 || block_threads(b) > 256 || mode < 0 || mode > 2) return hipErrorInvalidValue;
  MSPCG_BLOCK_SWITCH(prec, b.Ls, hipLaunchKernelGGL((k_block_scatter<S, NT>), dim3(block_grid(b)),
                     dim3(block_threads(b)), block_lds(b), st, b, (double *)zglob.data, zglob.stride, xs, ps, scal,
                     mode, (const double *)rglob.data, rglob.stride, rr, n_total, partial));
  return hipGetLastError();
}

hipError_t block_scatter_xpay(int prec, const BlockArgs &b, const Vec &pglob, double *xglob, const Vec &xs,
                              const Vec &ps, const double *scal, int mode, const double *rr, double n_total,
                              const double *alpha, const double *beta, int first, hipStream_t st) {
  if (pglob.prec != MSPCG_F64 || block_threads(b) > 256 || mode < 0 || mode > 2) return hipErrorInvalidValue;
  MSPCG_BLOCK_SWITCH(prec, b.Ls, hipLaunchKernelGGL((k_block_scatter_xpay<S, NT>), dim3(block_grid(b)),
                     dim3(block_threads(b)), 0, st, b, (double *)pglob.data, xglob, pglob.stride, xs, ps, scal, mode,
                     rr, n_total, alpha, beta, first));
  return hipGetLastError();
}

hipError_t block_scalars(int mode, const BlockArgs &b, const double *partial, double *scal, hipStream_t st) {
  const int n = b.nblocks * b.nrhs;
  (void)n;
  hipLaunchKernelGGL(k_block_scalars, dim3(b.nblocks, b.nrhs), dim3(256), 0, st, mode, b.nrhs, b.nsite_wg, b.be_off,
                     partial, scal);
  return hipGetLastError();
}

hipError_t block_update_xr(int prec, const BlockArgs &b, const Vec &x, const Vec &r, const Vec &p, const Vec &Ap,
                           const double *scal, double *partial, hipStream_t st) {
  if (block_threads(b) > 256) return hipErrorInvalidValue;
  MSPCG_BLOCK_SWITCH(prec, b.Ls, hipLaunchKernelGGL((k_block_update_xr<S, NT>), dim3(block_grid(b)),
                     dim3(block_threads(b)), block_lds(b), st, b, x, r, p, Ap, scal, partial));
  return hipGetLastError();
}

hipError_t block_update_r(int prec, const BlockArgs &b, const Vec &r, const Vec &Ap, const double *scal,
                          double *partial, hipStream_t st) {
  if (block_threads(b) > 256) return hipErrorInvalidValue;
  MSPCG_BLOCK_SWITCH(prec, b.Ls, hipLaunchKernelGGL((k_block_update_r<S, NT>), dim3(block_grid(b)),
                     dim3(block_threads(b)), block_lds(b), st, b, r, Ap, scal, partial));
  return hipGetLastError();
}

hipError_t block_update_xp(int prec, const BlockArgs &b, const Vec &x, const Vec &p, const Vec &mp, const Vec &r,
                           const double *scal, int first, hipStream_t st) {
  if (block_threads(b) > 256) return hipErrorInvalidValue;
  MSPCG_BLOCK_SWITCH(prec, b.Ls, hipLaunchKernelGGL((k_block_update_xp<S, NT>), dim3(block_grid(b)),
                     dim3(block_threads(b)), block_lds_mphi<S>(b), st, b, x, p, mp, r, scal, first));
  return hipGetLastError();
}

// ---------------------------------------------------------------- link packing
template <typename S>
__global__ void k_pack_links(S *out, const double *gauge, const int *order, const int *lex_of_cb, const int *nbr_lex,
                             int Vh, int Lt, int Lxyz, double tbc) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // (list position, d)
  if (i >= Vh * 8) return;
  const int cb = order[i >> 3], d = i & 7, mu = d >> 1, bw = d & 1;
  const int x = lex_of_cb[cb];
  const int t = x / Lxyz;
  const int src = bw ? nbr_lex[(size_t)cb * 8 + d] : x;
  const double sign = (mu == 3 && ((!bw && t == Lt - 1) || (bw && t == 0))) ? tbc : 1.0;
  const double *U = gauge + ((size_t)src * 4 + mu) * 18;
  S *o = out + (size_t)i * 18;
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) {
      double re, im;
      if (!bw) { re = U[(a * 3 + b) * 2]; im = U[(a * 3 + b) * 2 + 1]; }
      else { re = U[(b * 3 + a) * 2]; im = -U[(b * 3 + a) * 2 + 1]; }
      re *= sign;
      im *= sign;
      if constexpr (std::is_same<S, bf16>::value) {
        o[(a * 3 + b) * 2].bits = float_to_bf16((float)re);
        o[(a * 3 + b) * 2 + 1].bits = float_to_bf16((float)im);
      } else {
        o[(a * 3 + b) * 2] = (S)re;
        o[(a * 3 + b) * 2 + 1] = (S)im;
      }
    }
}

hipError_t pack_links(int prec, void *out, const double *gauge, const int *order, const int *lex_of_cb,
                      const int *nbr_lex, int Vh, int Lt, int Lxyz, double tbc, hipStream_t st) {
  const int n = Vh * 8, blk = 256;
  MSPCG_PREC_SWITCH(prec, hipLaunchKernelGGL(k_pack_links<S>, dim3((n + blk - 1) / blk), dim3(blk), 0, st,
                                             reinterpret_cast<S *>(out), gauge, order, lex_of_cb, nbr_lex, Vh, Lt, Lxyz,
                                             tbc));
  return hipGetLastError();
}

}  // namespace mspcg
