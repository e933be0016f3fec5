// Wilson hopping stencil kernels (arXiv:1106.4964 Sec. II, eq. 1-2) with
// fused epilogues: the device templates and their launchers.  Each storage
// precision and link format is instantiated in a translation unit of its own
// (stencil_<prec>.hip), so the kernels compile in parallel.
//
// For each of the 8 directions the neighbour spinor is loaded, spin-projected
// to a 2x3 half spinor with (1 -+ gamma_mu), both colour vectors are
// multiplied by U_mu(x) or U_mu(x-mu)^dag and the result is added back, the
// lower two spin components being fixed multiples of the upper two (chiral
// basis).  stencil_split_kernel shares a site between four threads, one per
// direction; stencil_kernel does a site's 8 hops in one thread.  Both treat
// KR right-hand sides per thread and add the same terms in the same order
// (the two hops of a direction, then the directions by mu), so that a result
// does not depend on the shape that the tuner took.  The epilogue forms
// G(a*in + b*hop) + sum_j c_j G_j(v_j) at the output site, which covers
// D_w(m), H_w = gamma5 D_w(-rho), and the Clenshaw update of the polynomial
// sign function (Sec. V) in one pass.
#pragma once

#include "ops.h"

namespace ovl {

struct Shape {
  int kr;    // vectors per thread
  int bs;    // threads per block (sites per block when rin); 256 = split directions
  int pipe;  // >= 2: split directions, one vector per thread (one kernel for every depth: all its loads are in flight)
  int rin;   // 1: the nrhs/kr vector groups are the y-dimension of the block
  int tm;    // block order (StencilArgs::tmaj): 0 by h, 1 t-major, >= 2 z-slabs of tm planes
};

// Launches the stencil in shape sh for one storage precision (one function
// per translation unit).
void launch_stencil_f64(const StencilArgs& A, int recon, int nrhs, Shape sh, hipStream_t s);
void launch_stencil_f32(const StencilArgs& A, int recon, int nrhs, Shape sh, hipStream_t s);
void launch_stencil_f16(const StencilArgs& A, int recon, int nrhs, Shape sh, hipStream_t s);
void launch_stencil_bf16(const StencilArgs& A, int recon, int nrhs, Shape sh, hipStream_t s);

namespace {

// Half-spinor projection (1 + SGN*gamma_mu) psi -> h[2][3] and the
// reconstruction of the lower spin components from U*h.  Chiral basis:
//   mu=0: (1-g1): h0=s0+i s3, h1=s1+i s2, lower=(-i h1,-i h0); (1+g1): signs of i flip
//   mu=1: (1-g2): h0=s0+s3,   h1=s1-s2,   lower=(-h1, h0);     (1+g2): h0=s0-s3, h1=s1+s2, lower=(h1,-h0)
//   mu=2: (1-g3): h0=s0+i s2, h1=s1-i s3, lower=(-i h0, i h1); (1+g3): signs of i flip
//   mu=3: (1-g4): h0=s0-s2,   h1=s1-s3,   lower=(-h0,-h1);     (1+g4): h0=s0+s2, h1=s1+s3, lower=(h0,h1)
// h_k = s_k + phase * s_partner with phase +1, -1, +i, -i coded 0, 1, 2, 3
// (code ^ 1 negates).
template <int PH, typename T>
__device__ inline Cx<T> proj1(Cx<T> a, Cx<T> b) {
  if constexpr (PH == 0) return {a.re + b.re, a.im + b.im};
  else if constexpr (PH == 1) return {a.re - b.re, a.im - b.im};
  else if constexpr (PH == 2) return {a.re - b.im, a.im + b.re};  // + i b
  else return {a.re + b.im, a.im - b.re};                          // - i b
}

template <int MU, int SGN, typename T>
__device__ inline void project(const Cx<T>* s, Cx<T> (*h)[3]) {
  constexpr int p0 = MU < 2 ? 3 : 2, p1 = MU < 2 ? 2 : 3;
  constexpr int f = SGN < 0 ? 0 : 1;
  constexpr int ph0 = (MU == 0 ? 2 : MU == 1 ? 0 : MU == 2 ? 2 : 1) ^ f;
  constexpr int ph1 = (MU == 0 ? 2 : MU == 1 ? 1 : MU == 2 ? 3 : 1) ^ f;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    h[0][c] = proj1<ph0>(s[c], s[3 * p0 + c]);
    h[1][c] = proj1<ph1>(s[3 + c], s[3 * p1 + c]);
  }
}

// acc += s * ph * w for the phase ph coded as in proj1 (0: +1, 1: -1, 2: +i,
// 3: -i), two FMAs (the sign of s is a source modifier).
template <int PH, typename T>
__device__ inline void addph(Cx<T>& a, Cx<T> w, T s) {
  if constexpr (PH == 0) {
    a.re = ffma(s, w.re, a.re);
    a.im = ffma(s, w.im, a.im);
  } else if constexpr (PH == 1) {
    a.re = ffma(-s, w.re, a.re);
    a.im = ffma(-s, w.im, a.im);
  } else if constexpr (PH == 2) {  // + i w = (-w.im, w.re)
    a.re = ffma(-s, w.im, a.re);
    a.im = ffma(s, w.re, a.im);
  } else {  // - i w = (w.im, -w.re)
    a.re = ffma(s, w.im, a.re);
    a.im = ffma(-s, w.re, a.im);
  }
}

// re + i im += u h  (CONJ: conj(u) h), four FMAs.
template <bool CONJ, typename T>
__device__ inline void cmac(T& re, T& im, Cx<T> u, Cx<T> h) {
  re = ffma(u.re, h.re, re);
  im = ffma(u.re, h.im, im);
  if constexpr (CONJ) {
    re = ffma(u.im, h.im, re);
    im = ffma(-u.im, h.re, im);
  } else {
    re = ffma(-u.im, h.im, re);
    im = ffma(u.im, h.re, im);
  }
}

// sum_b u_b h_b (CONJ: conj(u_b) h_b), one FMA chain per real part (4
// instructions per complex multiply-add).
template <bool CONJ, typename T>
__device__ inline Cx<T> row3(Cx<T> u0, Cx<T> u1, Cx<T> u2, const Cx<T>* h) {
  T re = T(0), im = T(0);
  cmac<CONJ>(re, im, u0, h[0]);
  cmac<CONJ>(re, im, u1, h[1]);
  cmac<CONJ>(re, im, u2, h[2]);
  return {re, im};
}

// w[s] = U h[s]  (DAG = false)  or  U^dag h[s]  (DAG = true)
template <bool DAG, typename T>
__device__ inline void colour_mul(const Cx<T> (*u)[3], const Cx<T> (*h)[3], Cx<T> (*w)[3]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int a = 0; a < 3; ++a)
      w[s][a] = DAG ? row3<true>(u[0][a], u[1][a], u[2][a], h[s]) : row3<false>(u[a][0], u[a][1], u[a][2], h[s]);
}

// ------------------------------------------------------- F16 operands
// An F16 spinor is 12 dwords, dword c holding complex component
// c = 3*spin + colour as (re, im) halves.  v_fma_mix_f32 takes an f16 half of
// a dword as an operand and computes in f32, so the spin projection and the
// epilogue read the stored halves directly: one instruction per real
// instead of a conversion plus the arithmetic.
//   mix_pm<HB, HA, NEG>(b, a) = (NEG ? -1 : +1) * half(b, HB) + half(a, HA)
//   mix_fma<HA>(a, s, c)      = half(a, HA) * s + c
// (half 0 = low, 1 = high; s and c in f32; s uniform, in an SGPR).
#define OVL_MIX_PM(HB, HA, K)                                                                             \
  asm("v_fma_mix_f32 %0, %1, " K ", %2 op_sel:[" #HB ",0," #HA "] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(b), \
      "v"(a))
template <int HB, int HA, bool NEG>
__device__ inline float mix_pm(uint32_t b, uint32_t a) {
  float d;
  if constexpr (HB == 0 && HA == 0) {
    if constexpr (NEG) OVL_MIX_PM(0, 0, "-1.0"); else OVL_MIX_PM(0, 0, "1.0");
  } else if constexpr (HB == 0 && HA == 1) {
    if constexpr (NEG) OVL_MIX_PM(0, 1, "-1.0"); else OVL_MIX_PM(0, 1, "1.0");
  } else if constexpr (HB == 1 && HA == 0) {
    if constexpr (NEG) OVL_MIX_PM(1, 0, "-1.0"); else OVL_MIX_PM(1, 0, "1.0");
  } else {
    if constexpr (NEG) OVL_MIX_PM(1, 1, "-1.0"); else OVL_MIX_PM(1, 1, "1.0");
  }
  return d;
}
#undef OVL_MIX_PM

template <int HA>
__device__ inline float mix_fma(uint32_t a, float s, float c) {
  float d;
  if constexpr (HA == 0)
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(a), "s"(s), "v"(c));
  else
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(a), "s"(s), "v"(c));
  return d;
}

// a + ph * b for complex components given as (re, im) f16 dwords
template <int PH>
__device__ inline Cx<float> proj1_f16(uint32_t a, uint32_t b) {
  if constexpr (PH == 0) return {mix_pm<0, 0, false>(b, a), mix_pm<1, 1, false>(b, a)};
  else if constexpr (PH == 1) return {mix_pm<0, 0, true>(b, a), mix_pm<1, 1, true>(b, a)};
  else if constexpr (PH == 2) return {mix_pm<1, 0, true>(b, a), mix_pm<0, 1, false>(b, a)};  // + i b
  else return {mix_pm<1, 0, false>(b, a), mix_pm<0, 1, true>(b, a)};                          // - i b
}

// (1 + SGN gamma_mu) psi -> h[2][3] straight from the raw F16 dwords
template <int MU, int SGN>
__device__ inline void project_f16(const uint32_t* s, Cx<float> (*h)[3]) {
  constexpr int p0 = MU < 2 ? 3 : 2, p1 = MU < 2 ? 2 : 3;
  constexpr int f = SGN < 0 ? 0 : 1;
  constexpr int ph0 = (MU == 0 ? 2 : MU == 1 ? 0 : MU == 2 ? 2 : 1) ^ f;
  constexpr int ph1 = (MU == 0 ? 2 : MU == 1 ? 1 : MU == 2 ? 3 : 1) ^ f;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    h[0][c] = proj1_f16<ph0>(s[c], s[3 * p0 + c]);
    h[1][c] = proj1_f16<ph1>(s[3 + c], s[3 * p1 + c]);
  }
}

__device__ inline uint32_t raw_word(const SpinorRaw<OVL_F16>& r, int c) {
  const uint4 v = r.b[c / 4];
  const int k = c % 4;
  return k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w;
}

// F16 links are converted to f32 once per thread and then hidden from the
// optimiser: otherwise it folds the conversions into the colour products as
// v_fma_mix_f32, which issues at about 70% of the rate of v_fma_f32
// (measured on MI355X: 35 vs 51 T lane-instructions/s) and would run 72 of
// them per direction and vector instead of 12 conversions per link.
template <int P>
__device__ inline void opaque_link(Cx<typename Prec<P>::real> (*u)[3]) {
  if constexpr (P == OVL_F16) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) asm("" : "+v"(u[i][j].re), "+v"(u[i][j].im));
  }
}

// Hopping weights of the epilogue: b on the upper spins, and on the lower
// spins b, or -b when the output takes gamma5.
template <typename T>
__device__ inline void hop_weights(const StencilArgs& A, T& bu, T& bl) {
  bu = static_cast<T>(A.b);
  bl = A.g5 ? -bu : bu;
}

// Epilogue at the output site: G(a*in + b*hop) + sum_j c_j G_j(v_j), G = 1
// or gamma5, then the store; acc holds hop.
template <int P, int NV>
__device__ inline void epilogue(const StencilArgs& A, size_t off, int p, int h, Cx<typename Prec<P>::real>* acc) {
  using real = typename Prec<P>::real;
  const real au = static_cast<real>(A.a), al = A.g5 ? -au : au;
  real bu, bl;
  hop_weights(A, bu, bl);
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = (c >= 6 ? bl : bu) * acc[c];
  if constexpr (P == OVL_F16) {
    SpinorRaw<P> r;
    spinor_load_raw<P>(static_cast<const char*>(A.in) + off, p, h, A.g.Nh, r);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const uint32_t x = raw_word(r, c);
      const float s = c >= 6 ? al : au;
      acc[c] = {mix_fma<0>(x, s, acc[c].re), mix_fma<1>(x, s, acc[c].im)};
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const char* vb = static_cast<const char*>(A.v[j]) + off + (static_cast<size_t>(p) * 3 * A.g.Nh + h) * 16;
      SpinorRaw<P> v;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(vb + static_cast<size_t>(k) * A.g.Nh * 16));
        v.b[k] = make_uint4(t.x, t.y, t.z, t.w);
      }
      const float cu = static_cast<float>(A.cv[j]);
      const float cl = ((A.g5v >> j) & 1) ? -cu : cu;
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const uint32_t x = raw_word(v, c);
        const float s = c >= 6 ? cl : cu;
        acc[c] = {mix_fma<0>(x, s, acc[c].re), mix_fma<1>(x, s, acc[c].im)};
      }
    }
  } else {
    Cx<real> s[12];
    SpinorIO<P>::load(static_cast<const char*>(A.in) + off, p, h, A.g.Nh, s);
#pragma unroll
    for (int c = 0; c < 12; ++c) addph<0>(acc[c], s[c], c >= 6 ? al : au);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      SpinorIO<P>::load_nt(static_cast<const char*>(A.v[j]) + off, p, h, A.g.Nh, s);
      const real cu = static_cast<real>(A.cv[j]);
      const real cl = ((A.g5v >> j) & 1) ? -cu : cu;
#pragma unroll
      for (int c = 0; c < 12; ++c) addph<0>(acc[c], s[c], c >= 6 ? cl : cu);
    }
  }
  SpinorIO<P>::store_nt(static_cast<char*>(A.out) + off, p, h, A.g.Nh, acc);
}

// Site i of logical block lb, for blocks of bs sites: parity p and half
// index h; false past the end.
__device__ inline bool tile_site(const StencilArgs& A, int lb, int bs, int i, int& p, int& h) {
  int hb;
  if (A.npar == 2) {
    p = lb & 1;
    hb = lb >> 1;
  } else {
    p = A.par0;
    hb = lb;
  }
  if (A.tmaj >= 2) {
    // z-slabs of Z = tmaj planes: consecutive blocks cover one slab's
    // (x, y, z) half-slice at t, then the same slab at t + 1, ..., before the
    // next slab, so a site's t-neighbours are read 2 Z Lx Ly / 2 half-sites
    // apart in launch order instead of Lx Ly Lz (a slice of the whole lattice)
    const int Z = A.tmaj, bps = (Z * A.g.sz + bs - 1) / bs;
    const int per_slab = bps * A.g.Lt;
    const int slab = hb / per_slab, r = hb - slab * per_slab;
    const int t = r / bps, j = r - t * bps;
    const int z0 = slab * Z;
    const int len = min(Z, A.g.Lz - z0) * A.g.sz;  // the last slab may be thinner
    const int hl = j * bs + i;
    h = t * A.g.st + z0 * A.g.sz + hl;
    return hl < len;
  }
  if (A.tmaj) {
    const int tile = hb / A.g.Lt, t = hb - tile * A.g.Lt;
    const int hl = tile * bs + i;
    h = t * A.g.st + hl;
    return hl < A.g.st;
  }
  h = hb * bs + i;
  return h < A.g.Nh;
}

// Output site (parity p, half index h) of this thread; false past the end.
__device__ inline bool stencil_site(const StencilArgs& A, int& p, int& h) {
  return tile_site(A, xcd_remap(blockIdx.x, gridDim.x), static_cast<int>(blockDim.x), static_cast<int>(threadIdx.x),
                   p, h);
}

// ------------------------------------------------------- split directions
// One workgroup of four waves per tile of 64 sites: wave w computes the two
// hops of direction mu = w for KR vectors of every site, and the four partial
// sums meet in LDS (one vector at a time, 24 KB in FP32), where the vector's
// 16-byte output blocks are dealt out over the waves for the epilogue.
//
// Against one thread per site and all directions:
//  - all loads of a wave (two links, 2 KR spinors) are requested before the
//    first use, so it waits for memory once instead of once per direction;
//    small lattices have four times the waves.  4^4 FP64: 6.3 -> 4.2 us a
//    launch; 8^3x16 F16, 12 rhs: 10.1 -> 7.4 us; 16^3x32 F16, 1 rhs: 10.3 ->
//    9.2 us, FP64: 33.9 -> 32.3 us.
//  - a quarter of the sites in flight per XCD, so that neighbours and links
//    are found in its L2: 24^3x64 F16, 12 rhs, no extra vectors: 1.10 ->
//    0.53 million KiB FETCH_SIZE a launch.
//  - the two hops of a direction share the addition (hops).
// 24^3x64 (H_w / Clenshaw step with three extra vectors, us): F16 12 rhs
// 435 / 635 -> 395 / 600, FP32-12 1 rhs 85 / 115 -> 76 / 110, FP64 1 rhs
// 228 / 304 -> 214 / 299, FP64 12 rhs 2132 / 2794 -> 1989 / 3001.
// What bounds it there: with three extra vectors HBM (3.1 GB at 5.2 TB/s);
// without, the reads between L1 and L2 (34 million 128-byte requests in 0.4 ms
// for F16, 11 TB/s; 93 million in 0.88 ms for FP32, 13 TB/s) and the FP32
// instructions (1120 a site and vector, about 70% of the issue rate).
//
// Uniform base + 32-bit lane offset for every load, so that the address
// arithmetic stays in scalar registers.
template <int P>
__device__ inline void raw_spinor_at(const char* base, uint32_t off, int Nh, SpinorRaw<P>& r) {
#pragma unroll
  for (int j = 0; j < 12 / Prec<P>::cpb; ++j)
    r.b[j] = *reinterpret_cast<const uint4*>(base + static_cast<size_t>(j) * Nh * 16 + off);
}

template <int P, int R>
__device__ inline void raw_link_at(const char* base, uint32_t h, int Nh, LinkRaw<P, R>& r) {
  using F = LinkFmt<P, R>;
#pragma unroll
  for (int k = 0; k < F::K; ++k)
    __builtin_memcpy(&r.w[k * F::E / 4],
                     __builtin_assume_aligned(base + static_cast<size_t>(k) * Nh * F::E + h * F::E, F::E), F::E);
}

// The 3x3 link from raw data.  F16: converted once per link and hidden from
// the optimiser (see opaque_link) before row 2 is rebuilt, so that the
// rebuild runs in v_fma_f32 as well.
template <int P, int R>
__device__ inline void raw_link_unpack(const LinkRaw<P, R>& r, Cx<typename Prec<P>::real> (*u)[3]) {
  if constexpr (P == OVL_F16 && R == 12) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      u[k / 3][k % 3] = ScalarIO<P>::load1(reinterpret_cast<const char*>(&r.w[k]));
      asm("" : "+v"(u[k / 3][k % 3].re), "+v"(u[k / 3][k % 3].im));
    }
    reconstruct_row2(u);
  } else {
    link_unpack<P, R>(r, u);
    opaque_link<P>(u);
  }
}

// Half spinor of direction MU (SGN -1: forward, +1: backward) from raw data.
template <int P, int MU, int SGN>
__device__ inline void raw_project(const SpinorRaw<P>& sr, Cx<typename Prec<P>::real> (*hs)[3]) {
  if constexpr (P == OVL_F16) {
    uint32_t sw[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) sw[c] = raw_word(sr, c);
    project_f16<MU, SGN>(sw, hs);
  } else {
    Cx<typename Prec<P>::real> s[12];
    spinor_unpack<P>(sr, s);
    project<MU, SGN>(s, hs);
  }
}

// ph * (a - f) for the phase ph coded as in proj1.
template <int PH, typename T>
__device__ inline Cx<T> phase_diff(Cx<T> a, Cx<T> f) {
  if constexpr (PH == 0) return {a.re - f.re, a.im - f.im};
  else if constexpr (PH == 1) return {f.re - a.re, f.im - a.im};
  else if constexpr (PH == 2) return {f.im - a.im, a.re - f.re};
  else return {a.im - f.im, f.re - a.re};
}

// Ends the arithmetic of these numbers here: the compiler otherwise puts off
// a direction's products until the next ones' operands are loaded, and all
// eight hops' operands then want registers (256 VGPRs and scratch).
template <typename T>
__device__ inline void keep(T& x) {
  using E = std::remove_all_extents_t<T>;
  E* e = reinterpret_cast<E*>(&x);
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / sizeof(E); ++i) asm volatile("" : "+v"(e[i].re), "+v"(e[i].im));
}

// Both hops of direction MU for KR vectors,
// U_mu(x)(1 - gamma_mu) in(x+mu) + U_mu(x-mu)^dag (1 + gamma_mu) in(x-mu),
// into val[k] (SPLIT, or MU = 0) or added to it.  With f and g the two
// transported half spinors, the upper spins are f + g and the lower spins a
// phase times g - f, each rounded once: 24 instructions where adding the two
// hops one after the other takes 48.  (g's colour products accumulated onto f,
// and g - f = (f + g) - 2 f, would save 12 more, but round once more: H_w in
// FP32 6.21e-8 from the 64-bit result against 5.96e-8, and at F16 storage 4.66
// of 10^4 stored reals other than the exact ones' rounding, where this has 4.24
// and the hops added one after the other 4.34.)
template <int P, int R, int MU, int KR, bool SPLIT>
__device__ inline void hops(const StencilArgs& A, const char* in, int p, int h, int x, int y, int z, int t,
                            Cx<typename Prec<P>::real> (*val)[12]) {
  using real = typename Prec<P>::real;
  using LF = LinkFmt<P, R>;
  const int Nh = A.g.Nh, q = 1 - p;
  int nb[8];
  site_neighbors(A.g, h, x, y, z, t, nb);
  const uint32_t hf = static_cast<uint32_t>(nb[MU]), hb = static_cast<uint32_t>(nb[MU + 4]);
  const char* src = in + static_cast<size_t>(q) * (12 / Prec<P>::cpb) * Nh * 16;
  const char* lk = static_cast<const char*>(A.links) + static_cast<size_t>(MU) * 2 * LF::K * Nh * LF::E;
  const size_t lpar = static_cast<size_t>(LF::K) * Nh * LF::E;
  SpinorRaw<P> sf[KR], sb[KR];
  LinkRaw<P, R> lf, lb;
  raw_link_at<P, R>(lk + p * lpar, static_cast<uint32_t>(h), Nh, lf);
  auto forward = [&](int k) { raw_spinor_at<P>(src + k * A.vstride, hf * 16u, Nh, sf[k]); };
  auto backward = [&](int k) { raw_spinor_at<P>(src + k * A.vstride, hb * 16u, Nh, sb[k]); };
  if constexpr (SPLIT)
#pragma unroll
    for (int k = 0; k < KR; ++k) forward(k);
  auto load_back = [&] {
    raw_link_at<P, R>(lk + q * lpar, hb, Nh, lb);
    if constexpr (SPLIT)
#pragma unroll
      for (int k = 0; k < KR; ++k) backward(k);
  };
  // both hops' operands in flight at once while they fit the registers
  constexpr bool ahead = SPLIT && 2 * (sizeof(SpinorRaw<P>) * KR + sizeof(LinkRaw<P, R>)) <= 680;
  if constexpr (ahead) {
    load_back();
    __builtin_amdgcn_sched_barrier(0);
  }
  Cx<real> u[3][3], f[KR][2][3];
  raw_link_unpack<P, R>(lf, u);
#pragma unroll
  for (int k = 0; k < KR; ++k) {
    Cx<real> hs[2][3];
    if constexpr (!SPLIT) forward(k);
    raw_project<P, MU, -1>(sf[k], hs);
    colour_mul<false>(u, hs, f[k]);
  }
  if constexpr (ahead) __builtin_amdgcn_sched_barrier(0);
  if constexpr (!SPLIT) keep(f);
  if constexpr (!ahead) load_back();
  raw_link_unpack<P, R>(lb, u);
  constexpr int l0 = MU == 0 ? 2 : MU == 1 ? 0 : MU == 2 ? 2 : 0;
  constexpr int l1 = MU == 0 ? 2 : MU == 1 ? 1 : MU == 2 ? 3 : 0;
  constexpr int s0 = MU < 2 ? 1 : 0, s1 = MU < 2 ? 0 : 1;
#pragma unroll
  for (int k = 0; k < KR; ++k) {
    Cx<real> hs[2][3], g[2][3];
    if constexpr (!SPLIT) backward(k);
    raw_project<P, MU, +1>(sb[k], hs);
    colour_mul<true>(u, hs, g);
    auto put = [&](int c, Cx<real> v) { val[k][c] = SPLIT || MU == 0 ? v : val[k][c] + v; };
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      put(c, f[k][0][c] + g[0][c]);
      put(3 + c, f[k][1][c] + g[1][c]);
      put(6 + c, phase_diff<l0>(g[s0][c], f[k][s0][c]));
      put(9 + c, phase_diff<l1>(g[s1][c], f[k][s1][c]));
    }
  }
  if constexpr (!SPLIT) keep(*reinterpret_cast<Cx<real>(*)[KR][12]>(val));
}

// One thread: one output site and KR consecutive vectors of the batch, so
// each link is loaded and rebuilt once per KR right-hand sides.  With
// RIN = false the group of KR vectors is blockIdx.y (one pass over the
// lattice per group); with RIN = true it is threadIdx.y, so all groups of a
// site tile run in the same workgroup and share its links and neighbour
// spinors through L1/L2 (one pass over the lattice for the whole batch).
template <int P, int R, int NV, int KR, bool RIN>
__global__ __launch_bounds__(RIN ? 512 : 256) void stencil_kernel(StencilArgs A) {
  using real = typename Prec<P>::real;
  const Geo& g = A.g;
  int p, h;
  if (!stencil_site(A, p, h)) return;
  const int group = RIN ? threadIdx.y : blockIdx.y;
  const size_t voff = static_cast<size_t>(group) * KR * A.vstride;
  const char* in = static_cast<const char*>(A.in) + voff;

  int x, y, z, t;
  site_coords(g, p, h, x, y, z, t);

  Cx<real> acc[KR][12];
  hops<P, R, 0, KR, false>(A, in, p, h, x, y, z, t, acc);
  hops<P, R, 1, KR, false>(A, in, p, h, x, y, z, t, acc);
  hops<P, R, 2, KR, false>(A, in, p, h, x, y, z, t, acc);
  hops<P, R, 3, KR, false>(A, in, p, h, x, y, z, t, acc);

#pragma unroll
  for (int k = 0; k < KR; ++k) epilogue<P, NV>(A, voff + k * A.vstride, p, h, acc[k]);
}

// Epilogue of one 16-byte output block u (components u*cpb ...): a = the sum
// of the hops, rin and rv the same block of the input and the extra vectors.
template <int P, int NV>
__device__ inline void split_block(const StencilArgs& A, size_t off, int u, const u32x4_t& rin, const u32x4_t* rv,
                                   Cx<typename Prec<P>::real>* a) {
  using real = typename Prec<P>::real;
  constexpr int cpb = Prec<P>::cpb;
  real bu, bl;
  hop_weights(A, bu, bl);
#pragma unroll
  for (int j = 0; j < cpb; ++j) a[j] = (u * cpb + j >= 6 ? bl : bu) * a[j];
#pragma unroll
  for (int q = 0; q <= NV; ++q) {
    const u32x4_t raw = q == 0 ? rin : rv[q == 0 ? 0 : q - 1];
    const real cu = static_cast<real>(q == 0 ? A.a : A.cv[q == 0 ? 0 : q - 1]);
    const real cl = (q == 0 ? A.g5 != 0 : ((A.g5v >> (q == 0 ? 0 : q - 1)) & 1) != 0) ? -cu : cu;
    if constexpr (P == OVL_F16) {
      const uint32_t wd[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
      for (int j = 0; j < cpb; ++j) {
        const float s = u * cpb + j >= 6 ? cl : cu;
        a[j] = {mix_fma<0>(wd[j], s, a[j].re), mix_fma<1>(wd[j], s, a[j].im)};
      }
    } else {
      Cx<real> x[cpb];
      Block<P>::load(&raw, x);
#pragma unroll
      for (int j = 0; j < cpb; ++j) addph<0>(a[j], x[j], u * cpb + j >= 6 ? cl : cu);
    }
  }
  u32x4_t v;
  Block<P>::store(&v, a);
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(static_cast<char*>(A.out) + off));
}

template <int P, int R, int NV, int KR>
__global__ __launch_bounds__(256) void stencil_split_kernel(StencilArgs A) {
  using real = typename Prec<P>::real;
  constexpr int cpb = Prec<P>::cpb, NB = 12 / cpb;
  constexpr int CH = 24 * sizeof(real) / 16, CPU = CH / NB;  // 16-byte chunks per vector and per output block
  constexpr int UW = (NB + 3) / 4;                           // output blocks per wave and vector
  __shared__ u32x4_t part[4][CH][64];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const Geo& g = A.g;
  int p, h;
  const bool ok = tile_site(A, xcd_remap(blockIdx.x, gridDim.x), 64, lane, p, h);
  if (!ok) h = 0;  // lanes past the end compute site 0 and store nothing
  const size_t voff = static_cast<size_t>(blockIdx.y) * KR * A.vstride;
  const char* in = static_cast<const char*>(A.in) + voff;
  int x, y, z, t;
  site_coords(g, p, h, x, y, z, t);
  Cx<real> val[KR][12];
  switch (w) {
    case 0: hops<P, R, 0, KR, true>(A, in, p, h, x, y, z, t, val); break;
    case 1: hops<P, R, 1, KR, true>(A, in, p, h, x, y, z, t, val); break;
    case 2: hops<P, R, 2, KR, true>(A, in, p, h, x, y, z, t, val); break;
    default: hops<P, R, 3, KR, true>(A, in, p, h, x, y, z, t, val); break;
  }

  // Output blocks of this wave: block 4 i + (w + k) % 4 of vector k.  The
  // epilogue's operands are requested here, before the exchange: requested
  // with the hops' operands they cost registers the hops need (F16, 12 rhs,
  // 24^3x64, three extra vectors: 692 us against 596), and vector by vector
  // they cost one memory latency each.
  u32x4_t rin[KR][UW], rv[KR][UW][NV == 0 ? 1 : NV];
  const uint32_t hoff = static_cast<uint32_t>(h) * 16u;
  auto block_off = [&](int k, int u) {
    return voff + k * A.vstride + (static_cast<size_t>(p) * NB + u) * g.Nh * 16;
  };
#pragma unroll
  for (int k = 0; k < KR; ++k)
#pragma unroll
    for (int i = 0; i < UW; ++i) {
      const int u = 4 * i + ((w + k) & 3);
      if (u < NB) {
        const size_t off = block_off(k, u);
        rin[k][i] = *reinterpret_cast<const u32x4_t*>(static_cast<const char*>(A.in) + off + hoff);
#pragma unroll
        for (int j = 0; j < NV; ++j)
          rv[k][i][j] = __builtin_nontemporal_load(
              reinterpret_cast<const u32x4_t*>(static_cast<const char*>(A.v[j]) + off + hoff));
      }
    }

#pragma unroll
  for (int k = 0; k < KR; ++k) {
    if (k > 0) __syncthreads();
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      u32x4_t v;
      __builtin_memcpy(&v, reinterpret_cast<const char*>(val[k]) + 16 * c, 16);
      part[w][c][lane] = v;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < UW; ++i) {
      const int u = 4 * i + ((w + k) & 3);
      if (u < NB && ok) {
        Cx<real> b[4][cpb], a[cpb];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int c = 0; c < CPU; ++c) {
            const u32x4_t v = part[s][u * CPU + c][lane];
            __builtin_memcpy(reinterpret_cast<char*>(b[s]) + 16 * c, &v, 16);
          }
#pragma unroll
        for (int j = 0; j < cpb; ++j) a[j] = ((b[0][j] + b[1][j]) + b[2][j]) + b[3][j];
        split_block<P, NV>(A, block_off(k, u) + hoff, u, rin[k][i], rv[k][i], a);
      }
    }
  }
}

template <int P, int R, int NV>
void launch_k(const StencilArgs& A0, int nrhs, Shape sh, hipStream_t s) {
  StencilArgs A = A0;
  A.tmaj = sh.tm;
  const bool split = sh.pipe || (sh.bs == 256 && !sh.rin);
  const int sites = split ? 64 : sh.bs;  // per block
  int hblocks;
  if (sh.tm >= 2) {
    OVL_REQUIRE(sh.tm <= A.g.Lz, OVL_E_ARG, "stencil: slab thicker than the lattice");
    hblocks = ((A.g.Lz + sh.tm - 1) / sh.tm) * A.g.Lt * ((sh.tm * A.g.sz + sites - 1) / sites);
  } else if (sh.tm == 1) {
    hblocks = ((A.g.st + sites - 1) / sites) * A.g.Lt;
  } else {
    hblocks = (A.g.Nh + sites - 1) / sites;
  }
  if (split) {
    dim3 grid(hblocks * A.npar, nrhs / sh.kr), block(256);
    OVL_REQUIRE(sh.kr >= 1 && sh.kr <= (P == OVL_F64 ? 2 : 4), OVL_E_ARG, "stencil: unsupported vectors per thread");
    if (sh.kr == 1) hipLaunchKernelGGL((stencil_split_kernel<P, R, NV, 1>), grid, block, 0, s, A);
    else if (sh.kr == 2) hipLaunchKernelGGL((stencil_split_kernel<P, R, NV, 2>), grid, block, 0, s, A);
    if constexpr (P != OVL_F64) {
      if (sh.kr == 3) hipLaunchKernelGGL((stencil_split_kernel<P, R, NV, 3>), grid, block, 0, s, A);
      else if (sh.kr == 4) hipLaunchKernelGGL((stencil_split_kernel<P, R, NV, 4>), grid, block, 0, s, A);
    }
    return;
  }
  if (sh.rin) {
    const int groups = nrhs / sh.kr;
    OVL_REQUIRE(sh.bs * groups <= 512, OVL_E_ARG, "stencil: block too large");
    dim3 grid(hblocks * A.npar), block(sh.bs, groups);
    switch (sh.kr) {
      case 1: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 1, true>), grid, block, 0, s, A); break;
      case 2: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 2, true>), grid, block, 0, s, A); break;
      case 3: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 3, true>), grid, block, 0, s, A); break;
      case 4: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 4, true>), grid, block, 0, s, A); break;
      default: throw Error(OVL_E_ARG, "stencil: unsupported vectors per thread");
    }
    return;
  }
  dim3 grid(hblocks * A.npar, nrhs / sh.kr), block(sh.bs);
  switch (sh.kr) {
    case 1: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 1, false>), grid, block, 0, s, A); break;
    case 2: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 2, false>), grid, block, 0, s, A); break;
    case 3: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 3, false>), grid, block, 0, s, A); break;
    case 4: hipLaunchKernelGGL((stencil_kernel<P, R, NV, 4, false>), grid, block, 0, s, A); break;
    default: throw Error(OVL_E_ARG, "stencil: unsupported vectors per thread");
  }
}

template <int P, int R>
void launch_pr(const StencilArgs& A, int nrhs, Shape sh, hipStream_t s) {
  switch (A.nv) {
    case 0: launch_k<P, R, 0>(A, nrhs, sh, s); break;
    case 1: launch_k<P, R, 1>(A, nrhs, sh, s); break;
    case 2: launch_k<P, R, 2>(A, nrhs, sh, s); break;
    case 3: launch_k<P, R, 3>(A, nrhs, sh, s); break;
    default: throw Error(OVL_E_ARG, "stencil: at most 3 extra vectors");
  }
  OVL_HIP(hipGetLastError());
}

}  // namespace
}  // namespace ovl
