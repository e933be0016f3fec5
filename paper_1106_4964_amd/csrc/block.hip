// Tall-skinny block operations between a set of FP64 basis vectors V
// (eigenvectors, Krylov or subspace bases) and a batch of R <= 12 spinors:
//
//   block_dot   : C[i][r] = V_i^dag psi_r             (FP64 accumulation)
//   block_axpy  : Y_r     = [Y_r] + sum_i V_i K[i][r]
//   lowmode_project (eq. 6-7 of arXiv:1106.4964):
//       psi_h = psi - sum_i (V_i^dag psi) V_i,
//       w     = [gamma5] sum_i sign(lambda_i) (V_i^dag psi) V_i
//
// Both sweeps read V exactly once.  Elements are walked in "rows"
// (parity p, complex index c) of N/2 sites, so a complex number is addressed
// the same way whatever the storage precision of the batch.
//
// All three are contractions in FP64.  From three vectors on, block_dot and the
// projection run on the FP64 matrix cores (v_mfma_f64_16x16x4_f64): a complex
// product of the basis with the batch is two real ones against the columns
// (psi_re, psi_im) and (psi_im, -psi_re) of every right-hand side, two columns per
// vector, so 12 vectors take two 16-column tiles and up to 8 take one.  One and two
// vectors are bound by the basis alone and take FP64 FMAs.
#include <algorithm>
#include <string>

#include "ops.h"

namespace ovl {
namespace {

template <int P>
__device__ inline size_t cx_offset(int row, int h, int Nh) {
  constexpr int cpb = Prec<P>::cpb;
  const int p = row / 12, c = row % 12;
  const size_t blk = (static_cast<size_t>(p) * (12 / cpb) + c / cpb) * Nh + h;
  return blk * 16 + (c % cpb) * (16 / cpb);
}

template <int P>
__device__ inline Cx<double> load_cx(const char* base, int row, int h, int Nh) {
  Cx<typename Prec<P>::real> v = ScalarIO<P>::load1(base + cx_offset<P>(row, h, Nh));
  return {static_cast<double>(v.re), static_cast<double>(v.im)};
}

// Basis elements are read once per sweep: non-temporal, so the batch's
// blocks (reused across the 24 rows of a site tile) stay in L2.
__device__ inline Cx<double> load_basis_at(const char* p) {
  typedef double f64x2_t __attribute__((ext_vector_type(2)));
  const f64x2_t v = __builtin_nontemporal_load(reinterpret_cast<const f64x2_t*>(p));
  return {v.x, v.y};
}

template <int P>
__device__ inline void store_cx(char* base, int row, int h, int Nh, Cx<double> v) {
  using real = typename Prec<P>::real;
  ScalarIO<P>::store1(base + cx_offset<P>(row, h, Nh), Cx<real>{static_cast<real>(v.re), static_cast<real>(v.im)});
}

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Lane l of a 16x16x4 FP64 matrix instruction supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and holds D[l / 16 + 4 v][l % 16], v = 0..3.
__device__ inline f64x4_t mfma64(double a, double b, f64x4_t c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int PJ_TILE = 32;  // sites per unit of block_dot
constexpr int PJ_PAD = 33;   // padded row of a unit in LDS

// partial[(kb*ell + i)*R + r] = sum over K-block kb's units of conj(V_i) psi_r.
// A unit is 32 sites of one row; a block of NW waves runs through a
// contiguous range of units, wave w for the mw <= 16 modes from (blockIdx.x NW
// + w) mw (rows past them repeat the last mode; skipping their loads puts
// branches between the loads: 3 and 4 vectors, 20 modes, a third slower).  The
// matrix instruction wants 16 modes side by side, memory wants one: a load that
// touches 16 modes (64 or 128 bytes of each) reached 2.6 TB/s, whatever was in
// flight, so a wave loads 512 bytes of two modes at a time into registers (the
// next unit, while the current one is used) and turns the unit in its own part
// of LDS (units of 64 sites leave room for one block of four waves a CU: 50
// modes at 16^3x32 took 315 us against 238).  The batch's unit is shared by the
// block, in two buffers, so one barrier per unit is enough.  The rows of a site
// tile follow each other, so the batch's 16-byte blocks, which hold several
// rows, come from cache.
// 24^3x64, 100 modes, 12 F16 vectors: 5.42 ms with FP64 FMAs on an LDS copy of
// the batch (LDS-bound: one 16-byte read per 8 FMAs), 3.59 ms now; the basis is
// 17 GB, 2.7 ms at 6.35 TB/s, the matrix instructions 2.2 ms.
template <int P, int NW, int NT>
__global__ __launch_bounds__(NW * 64) void dot_kernel(int Nh, int ell, int mw, const char* V, size_t vstrideV,
                                                      const char* psi, size_t vstrideP, int R, double2* partial) {
  constexpr int RM = NT == 1 ? 8 : OVL_MAX_RHS, PI = (RM * PJ_TILE + 64 * NW - 1) / (64 * NW);
  using real = typename Prec<P>::real;
  __shared__ double2 vt[NW][16][PJ_PAD];
  __shared__ double2 pt[2][RM][PJ_PAD];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, q = lane >> 4;
  const int tiles = (Nh + PJ_TILE - 1) / PJ_TILE;
  const long units = 24L * tiles;
  const int u0 = static_cast<int>(units * blockIdx.y / gridDim.y);
  const int u1 = static_cast<int>(units * (blockIdx.y + 1) / gridDim.y);
  const int i0 = (blockIdx.x * NW + wave) * mw;
  f64x4_t acc[2][NT];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[k][n] = f64x4_t{0.0, 0.0, 0.0, 0.0};

  double2 vr[8];  // the unit in flight (a second one: 3.79 against 3.59 ms)
  Cx<real> pr[PI];
  const int site = lane & 31, half = lane >> 5;
  bool in = false;  // of the unit in flight: this lane's site exists
  auto request = [&](int u) {
    const int row = u % 24, h = u / 24 * PJ_TILE + site, hl = min(h, Nh - 1);
    in = h < Nh;
    const size_t voff = (static_cast<size_t>(row) * Nh + hl) * 16, poff = cx_offset<P>(row, hl, Nh);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const Cx<double> v = load_basis_at(V + static_cast<size_t>(min(i0 + min(2 * m + half, mw - 1), ell - 1)) * vstrideV + voff);
      vr[m] = make_double2(v.re, v.im);
    }
#pragma unroll
    for (int k = 0; k < PI; ++k) {
      const int r = min((k * NW + wave) * 2 + half, R - 1);
      pr[k] = ScalarIO<P>::load1(psi + static_cast<size_t>(r) * vstrideP + poff);
    }
  };
  const bool part = j & 1;
  int rr[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) rr[n] = min(8 * n + (j >> 1), R - 1);
  if (u0 < u1) request(u0);
  for (int u = u0; u < u1; ++u) {
    const int buf = u & 1;
#pragma unroll
    for (int m = 0; m < 8; ++m) vt[wave][2 * m + half][site] = vr[m];
#pragma unroll
    for (int k = 0; k < PI; ++k)
      if ((k * NW + wave) * 2 + half < R)
        pt[buf][(k * NW + wave) * 2 + half][site] =
            in ? make_double2(static_cast<double>(pr[k].re), static_cast<double>(pr[k].im)) : make_double2(0.0, 0.0);
    request(min(u + 1, u1 - 1));  // past the end the last unit again
    __syncthreads();
#pragma unroll 4
    for (int s = 0; s < PJ_TILE / 4; ++s) {
      const double2 a = vt[wave][j][4 * s + q];
      double b1[NT], b2[NT];
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const double2 f = pt[buf][rr[n]][4 * s + q];
        b1[n] = part ? f.y : f.x;
        b2[n] = part ? -f.x : f.y;
      }
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[0][n] = mfma64(a.x, b1[n], acc[0][n]);
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[1][n] = mfma64(a.y, b2[n], acc[1][n]);
    }
  }
  double* out = reinterpret_cast<double*>(partial) + static_cast<size_t>(blockIdx.y) * ell * R * 2;
#pragma unroll
  for (int n = 0; n < NT; ++n)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = i0 + q + 4 * v, col = 16 * n + j;
      if (q + 4 * v < mw && i < ell && col < 2 * R) out[static_cast<size_t>(i) * R * 2 + col] = acc[0][n][v] + acc[1][n][v];
    }
}

// The same for one or two vectors with FP64 FMAs: 2 or 4 of the matrix
// instruction's 16 columns would be used, and a wave with 9 modes of 16 loads as
// long as one with 16.  A wave runs through the units (64 sites of one row) of
// its block for IW modes, 1 KB of each at a time, the next unit in flight; the
// batch's elements, the same for all waves of the block, come through L1.  No LDS
// and no barrier.  Bound by the basis, 6.5-6.8 TB/s.  FP64, one vector (two), with
// dot_kernel and with this, us: 24^3x64, 33 modes 1203 -> 839 (1218 -> 913), 100
// modes 2611 -> 2556 (2612 -> 2677), 130 modes 4233 -> 3369 (4235 -> 3518);
// 16^3x32, 33 modes 190 -> 128, 100 modes 403 -> 382; 8^3x16, 33 modes 18.7 -> 14.2.
template <int P, int R, int IW>
__global__ __launch_bounds__(512) void dot_small_kernel(int Nh, int ell, const char* V, size_t vstrideV,
                                                        const char* psi, size_t vstrideP, double2* partial) {
  using real = typename Prec<P>::real;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = (blockIdx.x * (blockDim.x >> 6) + wave) * IW;
  if (i0 >= ell) return;
  const long units = 24L * ((Nh + 63) / 64);
  const int u0 = static_cast<int>(units * blockIdx.y / gridDim.y);
  const int u1 = static_cast<int>(units * (blockIdx.y + 1) / gridDim.y);
  Cx<double> acc[IW][R], va[2][IW];
  Cx<real> pa[2][R];
  bool in[2];
#pragma unroll
  for (int m = 0; m < IW; ++m)
#pragma unroll
    for (int r = 0; r < R; ++r) acc[m][r] = {0.0, 0.0};
  auto request = [&](int d, int u) {
    const int row = u % 24, h0 = u / 24 * 64, l = min(lane, Nh - 1 - h0);
    in[d] = lane == l;
    const char* v = V + (static_cast<size_t>(row) * Nh + h0) * 16;
#pragma unroll
    for (int m = 0; m < IW; ++m)  // past the last mode: the basis' first line
      va[d][m] = load_basis_at((i0 + m < ell ? v + static_cast<size_t>(i0 + m) * vstrideV : V) +
                               static_cast<uint32_t>(i0 + m < ell ? l * 16 : 0));
    const char* p = psi + cx_offset<P>(row, h0, Nh);
#pragma unroll
    for (int r = 0; r < R; ++r) pa[d][r] = ScalarIO<P>::load1(p + r * vstrideP + static_cast<uint32_t>(l * 16));
    __builtin_amdgcn_sched_barrier(0);
  };
  auto use = [&](int d) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double re = in[d] ? static_cast<double>(pa[d][r].re) : 0.0;
      const double im = in[d] ? static_cast<double>(pa[d][r].im) : 0.0;
#pragma unroll
      for (int m = 0; m < IW; ++m) {
        Cx<double>& a = acc[m][r];
        a.re = fma(va[d][m].re, re, a.re);
        a.im = fma(va[d][m].re, im, a.im);
        a.re = fma(va[d][m].im, im, a.re);
        a.im = fma(-va[d][m].im, re, a.im);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  int u = u0;
  if (u < u1) request(0, u);
  for (; u + 2 < u1; u += 2) {
    request(1, u + 1);
    use(0);
    request(0, u + 2);
    use(1);
  }
  if (u + 1 < u1) {
    request(1, u + 1);
    use(0);
    use(1);
  } else if (u < u1) {
    use(0);
  }
#pragma unroll
  for (int m = 0; m < IW; ++m)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double re = acc[m][r].re, im = acc[m][r].im;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        re += __shfl_xor(re, o, 64);
        im += __shfl_xor(im, o, 64);
      }
      if (lane == 0 && i0 + m < ell)
        partial[(static_cast<size_t>(blockIdx.y) * ell + i0 + m) * R + r] = make_double2(re, im);
    }
}

// C[k] = sum_b partial[b*n + k], n = ell R: 64 sums of every 64th block each,
// added pairwise.  (One thread per sum, 512 reads in turn, took 54-213 us.)
__global__ __launch_bounds__(256) void dot_reduce_kernel(int n, int G, const double2* partial, double2* C) {
  __shared__ double2 red[64][4];
  const int kl = threadIdx.x & 3, bl = threadIdx.x >> 2;
  const int k = blockIdx.x * 4 + kl;
  double re = 0.0, im = 0.0;
  if (k < n) {
#pragma unroll 4
    for (int b = bl; b < G; b += 64) {
      const double2 v = partial[static_cast<size_t>(b) * n + k];
      re += v.x;
      im += v.y;
    }
  }
  red[bl][kl] = make_double2(re, im);
  for (int o = 32; o > 0; o >>= 1) {
    __syncthreads();
    if (bl < o) {
      re += red[bl + o][kl].x;
      im += red[bl + o][kl].y;
      red[bl][kl] = make_double2(re, im);
    }
  }
  if (bl == 0 && k < n) C[k] = make_double2(re, im);
}

// x[m], lane group g (16 lanes): element (m, g) -> x[t], group q: element (q, t).
__device__ inline void turn(double2 (&x)[4]) {
  uint32_t d[4][4];
  __builtin_memcpy(d, x, sizeof(d));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    swap32(d[0][k], d[2][k]);
    swap32(d[1][k], d[3][k]);
    swap16(d[0][k], d[1][k]);
    swap16(d[2][k], d[3][k]);
  }
  __builtin_memcpy(x, d, sizeof(d));
}

// The second sweep of a projection of three and more vectors:
// psi_h = psi - sum_i C_i V_i and w = [gamma5] sum_i s_i C_i V_i.
// A block of four waves makes the 16-byte output blocks u of 256 / cpb sites of
// one parity; a wave the 64 sites of one complex row, four tiles of 16 sites,
// which are the rows of the matrix product, against the coefficients' columns
// (c_re, c_im) and (-c_im, c_re).  A step is four modes, each loaded as 1 KB by
// one instruction and turned into (16 sites x 4 modes) by lane swaps (loads of
// 256 bytes from each of four modes were a third slower).  The modes of positive
// and of negative sign are summed apart (order: first nsp steps of four modes with
// s = +1, then the others, -1 filling up a step), which halves the columns:
// psi_h = psi - (S+ + S-), w = S+ - S-.  The sums pass through LDS, where the rows
// of a 16-byte block meet.
// 24^3x64, 100 modes, 12 F16 vectors: 4.93 ms with one thread per element and
// FP64 FMAs (4-byte stores), 3.95 ms now.
template <int P, int NT>
__global__ __launch_bounds__(256) void project_kernel(int Nh, const char* V, size_t vstrideV, const char* psi,
                                                      char* psih, char* w, size_t vstrideP, int R,
                                                      const double2* __restrict__ coef,
                                                      const int* __restrict__ order, int nsp, int ns, int g5w) {
  constexpr int cpb = Prec<P>::cpb, NB = 12 / cpb, SG = 256 / cpb;  // sites per block
  constexpr int LD = 8 * NT + 9;  // padded row of the LDS exchange: 16 or 24 columns are used
  using real = typename Prec<P>::real;
  __shared__ double ex[4][64 * LD];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, q = lane >> 4;
  const int groups = (Nh + SG - 1) / SG;
  const int pu = blockIdx.x / groups, h0 = (blockIdx.x - pu * groups) * SG;  // pu = p NB + u
  // wave: complex wave % cpb of the block, sites h0 + 64 (wave / cpb) ...
  V += (static_cast<size_t>(pu * cpb + wave % cpb) * Nh) * 16;
  const uint32_t hoff = static_cast<uint32_t>(min(h0 + wave / cpb * 64 + lane, Nh - 1)) * 16u;
  int rr[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) rr[n] = min(8 * n + (j >> 1), R - 1);
  const bool part = j & 1;
  const int m0 = -static_cast<int>(q == 0), m1 = -static_cast<int>(q == 1), m2 = -static_cast<int>(q == 2),
            m3 = -static_cast<int>(q == 3);

  auto sum = [&](int s0, int s1, f64x4_t (*acc)[NT]) {
    constexpr int DP = 3;
    double2 va[DP][4], cf[DP][NT];
    bool some[DP];
    int i[4];  // the modes of the next request, looked up one request ahead
    auto look = [&](int s) {
#pragma unroll
      for (int m = 0; m < 4; ++m) i[m] = order[4 * s + m];
    };
    auto request = [&](int d, int s) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const Cx<double> v = load_basis_at(V + static_cast<size_t>(max(i[m], 0)) * vstrideV + hoff);
        va[d][m] = make_double2(v.re, v.im);
      }
      const int iq = (i[0] & m0) | (i[1] & m1) | (i[2] & m2) | (i[3] & m3);  // i[q], without branches
#pragma unroll
      for (int n = 0; n < NT; ++n) cf[d][n] = coef[max(iq, 0) * R + rr[n]];
      some[d] = iq >= 0;  // applied at the use: a select here would wait for the load
      look(min(s + 1, s1 - 1));
    };
    auto use = [&](int d) {
      turn(va[d]);
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const double b1 = some[d] ? part ? cf[d][n].y : cf[d][n].x : 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t][n] = mfma64(va[d][t].x, b1, acc[t][n]);
      }
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const double b2 = some[d] ? part ? cf[d][n].x : -cf[d][n].y : 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t][n] = mfma64(va[d][t].y, b2, acc[t][n]);
      }
    };
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int n = 0; n < NT; ++n) acc[t][n] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    if (s0 == s1) return;
    // no branch between a request and its use: where two paths meet, the
    // compiler waits for the later of their loads, and nothing stays in flight
    look(s0);
#pragma unroll
    for (int d = 0; d < DP - 1; ++d) request(d, min(s0 + d, s1 - 1));
    int s = s0;
    for (; s + DP <= s1; s += DP) {
#pragma unroll
      for (int d = 0; d < DP; ++d) {
        request((d + DP - 1) % DP, min(s + d + DP - 1, s1 - 1));
        __builtin_amdgcn_sched_barrier(0);  // requests first
        use(d);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < DP - 1; ++d)
      if (s + d < s1) use(d);
  };
  // element (tile t, row q + 4 v, column 16 n + j) of this wave's sums in LDS
  auto slot = [&](int t, int n, int v) -> double& {
    return ex[wave][(t * 16 + q + 4 * v) * LD + (n == 0 ? j : 16 + (j & 7))];
  };
  f64x4_t acc[4][NT];
  auto park = [&] {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (n == 0 || j < 8) slot(t, n, v) = acc[t][n][v];
  };
  // one output, 16-byte blocks put together from LDS: out = [base] + sgn sums
  auto store = [&](const char* base, char* out, double sgn, bool lower) {
    __syncthreads();
    for (int k = threadIdx.x; k < R * SG; k += 256) {
      const int r = k / SG, e = k - r * SG, h = h0 + e;
      if (h >= Nh) continue;
      const size_t off = r * vstrideP + (static_cast<size_t>(pu) * Nh + h) * 16;
      Cx<real> y[cpb];
      if (base) Block<P>::load(base + off, y);
#pragma unroll
      for (int c = 0; c < cpb; ++c) {
        const double* x = &ex[e / 64 * cpb + c][e % 64 * LD + 2 * r];
        const double f = (lower && (pu % NB) * cpb + c >= 6) ? -sgn : sgn;
        const double b0 = base ? static_cast<double>(y[c].re) : 0.0, b1 = base ? static_cast<double>(y[c].im) : 0.0;
        y[c] = {static_cast<real>(b0 + f * x[0]), static_cast<real>(b1 + f * x[1])};
      }
      Block<P>::store(out + off, y);
    }
  };

  // one copy of the loop for both signs; S+ waits in LDS
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    sum(side ? nsp : 0, side ? ns : nsp, acc);
    if (side == 0) park();
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (n == 0 || j < 8) {
          const double a = slot(t, n, v), b = acc[t][n][v];
          slot(t, n, v) = a + b;
          acc[t][n][v] = a - b;
        }
  store(psi, psih, -1.0, false);
  __syncthreads();
  park();
  store(nullptr, w, 1.0, g5w != 0);
}

// The FMA form of the second reading, for block_axpy (FP64 vectors) and for the
// projection of one or two vectors: a thread is a site and one of its 16-byte
// blocks of rows.  MODE 0: Y_r = f sum_i V_i K_ir, 1: Y_r += the same (f = +-1),
// 2: the projection, as above.  Bound by the basis; the 4 R FMAs per 16 bytes reach
// 13 TB/s at 12 vectors.  Where the lattice fills the CUs, one load in flight per
// thread reads best, with the rows of a site tile in consecutive blocks: more
// loads in flight wait on each other.  On small lattices U modes are read ahead
// (DEEP).  FP64 update, 100 modes, us, with matrix instructions (1 and 2 vectors:
// 8 modes ahead, some read twice), U modes ahead, one load:
//              24^3x64           16^3x32          8^3x16
//    1 vector  2944 2888 2765    427 423 386      25  24  49
//    4         3397 3359 3328    483 467 431      29  26  56
//   12         4022 4089 4110    606 581 528      44  36  67
template <int P, int R, int MODE, bool DEEP>
__global__ __launch_bounds__(256) void sweep_kernel(int Nh, int ell, const char* V, size_t vstrideV, const char* in,
                                                    char* Y, char* w, size_t vstrideP,
                                                    const double2* __restrict__ coef, const int* __restrict__ order,
                                                    int nsp, int ns, int g5w, double f) {
  constexpr int cpb = Prec<P>::cpb, NB = 12 / cpb, U = cpb == 1 ? (R <= 4 ? 8 : 4) : cpb == 2 ? 4 : 2;
  using real = typename Prec<P>::real;
  const int tiles = (Nh + 255) / 256, b = blockIdx.x;
  const int pu = DEEP ? b / tiles : b % (2 * NB);  // p NB + u
  const int h = (DEEP ? b % tiles : b / (2 * NB)) * 256 + threadIdx.x;
  if (h >= Nh) return;
  V += static_cast<size_t>(pu * cpb) * Nh * 16;
  const uint32_t hoff = static_cast<uint32_t>(h) * 16u;
  const size_t off = (static_cast<size_t>(pu) * Nh + h) * 16;
  Cx<double> acc[2][R][cpb];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    Cx<real> y[cpb];
    if (MODE == 1) Block<P>::load(Y + r * vstrideP + off, y);
#pragma unroll
    for (int c = 0; c < cpb; ++c) {
      acc[0][r][c] = acc[1][r][c] = {0.0, 0.0};
      if (MODE == 1) acc[0][r][c] = {f * static_cast<double>(y[c].re), f * static_cast<double>(y[c].im)};
    }
  }
  auto sum = [&](int k0, int k1, Cx<double> (*a)[cpb]) {
    if (MODE == 2)
      while (k1 > k0 && order[k1 - 1] < 0) --k1;  // the padding of the last quad
    auto mode = [&](int k) { return MODE == 2 ? order[k] : k; };
    Cx<double> va[2][U][cpb];
    auto load = [&](Cx<double>* x, int k) {
      const char* v = V + static_cast<size_t>(mode(k)) * vstrideV;
#pragma unroll
      for (int c = 0; c < cpb; ++c) x[c] = load_basis_at(v + static_cast<size_t>(c) * Nh * 16 + hoff);
    };
    auto add = [&](const Cx<double>* x, int k) {
      const double2* cm = coef + mode(k) * R;
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < cpb; ++c) {
          Cx<double>& y = a[r][c];
          y.re = fma(x[c].re, cm[r].x, y.re);
          y.im = fma(x[c].re, cm[r].y, y.im);
          y.re = fma(-x[c].im, cm[r].y, y.re);
          y.im = fma(x[c].im, cm[r].x, y.im);
        }
    };
    auto request = [&](int d, int k) {
#pragma unroll
      for (int m = 0; m < U; ++m) load(va[d][m], k + m);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto use = [&](int d, int k) {
#pragma unroll
      for (int m = 0; m < U; ++m) add(va[d][m], k + m);
      __builtin_amdgcn_sched_barrier(0);
    };
    if (!DEEP) {
#pragma unroll 1
      for (int k = k0; k < k1; ++k) {
        load(va[0][0], k);
        add(va[0][0], k);
      }
      return;
    }
    // the modes past the last whole group first, then group after group
    const int rest = (k1 - k0) % U;
    int k = k0 + rest, n = (k1 - k0) / U;
#pragma unroll
    for (int m = 0; m < U - 1; ++m)
      if (m < rest) load(va[0][m], k0 + m);
    if (n > 0) request(1, k);
#pragma unroll
    for (int m = 0; m < U - 1; ++m)
      if (m < rest) add(va[0][m], k0 + m);
    for (; n > 2; n -= 2, k += 2 * U) {
      request(0, k + U);
      use(1, k);
      request(1, k + 2 * U);
      use(0, k + U);
    }
    if (n == 2) request(0, k + U);
    if (n > 0) use(1, k);
    if (n == 2) use(0, k + U);
  };
  auto store = [&](const char* base, char* out, Cx<double> (*a)[cpb], double sgn, bool lower) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      Cx<real> y[cpb];
      if (base) Block<P>::load(base + r * vstrideP + off, y);
#pragma unroll
      for (int c = 0; c < cpb; ++c) {
        const double g = (lower && (pu % NB) * cpb + c >= 6) ? -sgn : sgn;
        const double b0 = base ? static_cast<double>(y[c].re) : 0.0, b1 = base ? static_cast<double>(y[c].im) : 0.0;
        y[c] = {static_cast<real>(b0 + g * a[r][c].re), static_cast<real>(b1 + g * a[r][c].im)};
      }
      Block<P>::store(out + r * vstrideP + off, y);
    }
  };
  if constexpr (MODE == 2) {
    sum(0, 4 * nsp, acc[0]);
    sum(4 * nsp, 4 * ns, acc[1]);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int c = 0; c < cpb; ++c) {
        const Cx<double> a = acc[0][r][c], b = acc[1][r][c];
        acc[0][r][c] = a + b;
        acc[1][r][c] = a - b;
      }
    store(in, Y, acc[0], -1.0, false);
    store(nullptr, w, acc[1], 1.0, g5w != 0);
  } else {
    sum(0, ell, acc[0]);
    store(nullptr, Y, acc[0], f, false);
  }
}

// In-place basis rotation V[:, j] = sum_{i<K} V[:, i] S[i + K j], j < k.
// Each block stages all K values of RT consecutive elements of one row in
// LDS, so every element is read once and rewritten by the same block.
constexpr int RT = 8;
__global__ __launch_bounds__(256) void rotate_kernel(int Nh, int K, int k, char* V, size_t vstride,
                                                     const double2* S) {
  extern __shared__ Cx<double> vt[];  // [K][RT]
  const int row = blockIdx.y;
  const int h0 = blockIdx.x * RT;
  for (int idx = threadIdx.x; idx < K * RT; idx += blockDim.x) {
    const int i = idx / RT, e = idx % RT;
    vt[idx] = (h0 + e < Nh) ? load_cx<OVL_F64>(V + i * vstride, row, h0 + e, Nh) : Cx<double>{0.0, 0.0};
  }
  __syncthreads();
  const int e = threadIdx.x % RT;
  for (int j = threadIdx.x / RT; j < k; j += blockDim.x / RT) {
    Cx<double> acc = {0.0, 0.0};
    const double2* sj = S + static_cast<size_t>(K) * j;
    for (int i = 0; i < K; ++i) {
      const double2 c = sj[i];
      acc = acc + vt[i * RT + e] * Cx<double>{c.x, c.y};
    }
    if (h0 + e < Nh) store_cx<OVL_F64>(V + j * vstride, row, h0 + e, Nh, acc);
  }
}

// Waves of a dot_kernel block: the tiles of 16 modes in equal groups of at most
// eight (each group reads the batch again).  A wave loads as long for a part of a
// tile as for a whole one, so up to 8 vectors take 5 or 6 waves where those do
// (24^3x64, FP64, 4 vectors, 130 modes: twice 7 waves 4310 us, twice 5 3692; the
// projection at 14x18x10x34, FP32, 5 vectors, 7% less).  With two column tiles the
// matrix instructions weigh more and 7 waves are ahead (F16, 12 vectors, 72 modes,
// 24^3x64: 3210 against 3360 us), and three waves, though 14% ahead of four alone,
// leave less of the basis in the Infinity Cache for the second reading (that
// projection, 37 modes: 290 us with four, 300 with three).
int dot_waves(int ell, int R) {
  const int tiles = (ell + 15) / 16, groups = (tiles + 7) / 8, nw = (tiles + groups - 1) / groups;
  return nw == 3 ? 4 : R > 8 && (nw == 5 || nw == 6) ? 7 : nw;
}

// Batches up to this take dot_small_kernel.  With two vectors dot_kernel is ahead by
// 2% at 100 modes already, where its tiles are full, and behind by 4-33% elsewhere.
constexpr int DOT_SMALL_R = 2;

// Modes a wave and waves a block of dot_small_kernel: groups of at most 64 modes
// (each reads the batch again), spread evenly over up to eight waves.
void dot_small_split(int ell, int& iw, int& nw, int& groups) {
  groups = (ell + 63) / 64;
  iw = (ell + 8 * groups - 1) / (8 * groups);
  nw = ((ell + groups - 1) / groups + iw - 1) / iw;
  groups = (ell + iw * nw - 1) / (iw * nw);
}

// K-blocks of block_dot: what the 256 CUs hold at once (dot_small_kernel: 16 waves a
// CU, as eight modes of one vector leave registers for; a third more blocks than
// that made a second, nearly empty round: 24^3x64, 20 modes 615 against 530 us;
// dot_kernel: by LDS), and at least four units each, which cost less than the
// partial sums of more blocks.
int dot_blocks(const ovl_geom* g, int ell, int R) {
  if (R <= DOT_SMALL_R) {
    int iw, nw, groups;
    dot_small_split(ell, iw, nw, groups);
    const long units = 24L * ((g->geo.Nh + 63) / 64);
    return static_cast<int>(std::max(1L, std::min((units + 3) / 4, 256L * (16 / nw) / groups)));
  }
  const long units = 24L * ((g->geo.Nh + PJ_TILE - 1) / PJ_TILE);
  const int nw = dot_waves(ell, R), groups = (ell + 16 * nw - 1) / (16 * nw);
  const long held = 256L * ((160 << 10) / ((nw * 16 + 2 * OVL_MAX_RHS) * PJ_PAD * 16));
  return static_cast<int>(std::max(1L, std::min((units + 3) / 4, held / groups)));
}

template <int P, int NW, int NT>
void dot_go(const ovl_geom* g, const void* V, int ell, const void* psi, int R, double2* part, int G, hipStream_t s) {
  const int groups = (ell + 16 * NW - 1) / (16 * NW), mw = (ell + NW * groups - 1) / (NW * groups);
  hipLaunchKernelGGL((dot_kernel<P, NW, NT>), dim3(groups, G), dim3(64 * NW), 0, s, g->geo.Nh, ell, mw, static_cast<const char*>(V), spinor_vec_bytes(g, OVL_F64),
                     static_cast<const char*>(psi), spinor_vec_bytes(g, P), R, part);
}

template <int P, int NT, int NW = 8>
void dot_mt(const ovl_geom* g, const void* V, int ell, const void* psi, int R, double2* part, int G, hipStream_t s) {
  constexpr int next = NW == 4 ? 2 : NT == 2 && NW == 7 ? 4 : NW - 1;  // the counts that dot_waves gives
  if constexpr (NW > 1)
    if (dot_waves(ell, R) < NW) return dot_mt<P, NT, next>(g, V, ell, psi, R, part, G, s);
  dot_go<P, NW, NT>(g, V, ell, psi, R, part, G, s);
}

template <int P, int R, int IW = 8>
void dot_small_go(const ovl_geom* g, const void* V, int ell, const void* psi, double2* part, int G, hipStream_t s) {
  int iw, nw, groups;
  dot_small_split(ell, iw, nw, groups);
  if constexpr (IW > 1)
    if (iw < IW) return dot_small_go<P, R, IW - 1>(g, V, ell, psi, part, G, s);
  hipLaunchKernelGGL((dot_small_kernel<P, R, IW>), dim3(groups, G), dim3(64 * nw), 0, s, g->geo.Nh, ell,
                     static_cast<const char*>(V), spinor_vec_bytes(g, OVL_F64), static_cast<const char*>(psi),
                     spinor_vec_bytes(g, P), part);
}

// C = V^dag psi with the per-block partials in `part` (ell * G * R entries).
void dot_prec(const ovl_geom* g, const void* V, int ell, const void* psi, int prec, int R, double2* C, double2* part,
              int G, hipStream_t s) {
  auto go = [&](auto P) {
    constexpr int p = decltype(P)::value;
    if (R == 1) dot_small_go<p, 1>(g, V, ell, psi, part, G, s);
    else if (R == 2) dot_small_go<p, 2>(g, V, ell, psi, part, G, s);
    else if (R <= 8) dot_mt<p, 1>(g, V, ell, psi, R, part, G, s);
    else dot_mt<p, 2>(g, V, ell, psi, R, part, G, s);
  };
  switch (prec) {
    case OVL_F64: go(std::integral_constant<int, OVL_F64>{}); break;
    case OVL_F32: go(std::integral_constant<int, OVL_F32>{}); break;
    case OVL_F16: go(std::integral_constant<int, OVL_F16>{}); break;
    case OVL_BF16: go(std::integral_constant<int, OVL_BF16>{}); break;
    default: throw Error(OVL_E_PRECISION, "unknown precision");
  }
  OVL_HIP(hipGetLastError());
  hipLaunchKernelGGL(dot_reduce_kernel, dim3((ell * R + 3) / 4), dim3(256), 0, s, ell * R, G,
                     static_cast<const double2*>(part), C);
  OVL_HIP(hipGetLastError());
}

// One load in flight per thread needs the CUs full of waves: 24 rows of 16 Ki sites
// are three quarters of what they hold (FP64 update, 1 vector, 100 modes, ahead / one
// load: 10^3x20, 960 blocks, 0.93 / 1.00; 12^3x24, 1944 blocks, 1.09 / 1.00).
bool sweep_deep(int Nh) { return Nh < 16384; }

template <int P, int R, int MODE>
void sweep_go(const ovl_geom* g, const void* V, int ell, const void* in, void* Y, void* w, const double2* K,
              const int* order, int nsp, int ns, int g5w, double f, hipStream_t s) {
  const int Nh = g->geo.Nh;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((Nh + 255) / 256 * (24 / Prec<P>::cpb)), dim3(256), 0, s, Nh, ell,
                       static_cast<const char*>(V), spinor_vec_bytes(g, OVL_F64), static_cast<const char*>(in),
                       static_cast<char*>(Y), static_cast<char*>(w), spinor_vec_bytes(g, P), K, order, nsp, ns, g5w, f);
  };
  if (sweep_deep(Nh)) go(sweep_kernel<P, R, MODE, true>);
  else go(sweep_kernel<P, R, MODE, false>);
  OVL_HIP(hipGetLastError());
}

// Y_r = [Y_r] + f sum_i V_i K_ir for FP64 vectors.
template <int MODE, int R = OVL_MAX_RHS>
void update(const ovl_geom* g, const void* V, int ell, void* Y, int nrhs, const double2* K, double f, hipStream_t s) {
  if constexpr (R > 1)
    if (nrhs < R) return update<MODE, R - 1>(g, V, ell, Y, nrhs, K, f, s);
  sweep_go<OVL_F64, R, MODE>(g, V, ell, nullptr, Y, nullptr, K, nullptr, 0, 0, 0, f, s);
}

template <int P>
void project_go(const ovl_lowmodes* lm, const void* psi, void* psih, void* w, int R, const double2* C, int g5w,
                hipStream_t s) {
  const ovl_geom* g = &lm->geom;
  if (R == 1)
    return sweep_go<P, 1, 2>(g, lm->V, lm->ell, psi, psih, w, C, lm->dev_order, lm->steps_pos, lm->steps, g5w, 1.0, s);
  if (R == 2)
    return sweep_go<P, 2, 2>(g, lm->V, lm->ell, psi, psih, w, C, lm->dev_order, lm->steps_pos, lm->steps, g5w, 1.0, s);
  constexpr int cpb = Prec<P>::cpb;
  const int Nh = g->geo.Nh, blocks = 2 * (12 / cpb) * ((Nh + 256 / cpb - 1) / (256 / cpb));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, Nh, static_cast<const char*>(lm->V),
                       spinor_vec_bytes(g, OVL_F64), static_cast<const char*>(psi), static_cast<char*>(psih),
                       static_cast<char*>(w), spinor_vec_bytes(g, P), R, C, lm->dev_order, lm->steps_pos, lm->steps, g5w);
  };
  if (R <= 8) go(project_kernel<P, 1>);
  else go(project_kernel<P, 2>);
  OVL_HIP(hipGetLastError());
}

}  // namespace

void block_dot(const ovl_geom* g, const void* V, int ell, const void* psi, int prec, int R, double2* C,
               hipStream_t s) {
  OVL_REQUIRE(R >= 1 && R <= OVL_MAX_RHS && ell >= 1, OVL_E_ARG, "block_dot: 1 <= R <= 12, ell >= 1");
  const int G = dot_blocks(g, ell, R);
  WsBuf part(static_cast<size_t>(ell) * G * R * sizeof(double2), s);
  dot_prec(g, V, ell, psi, prec, R, C, static_cast<double2*>(part.p), G, s);
}

void block_axpy(const ovl_geom* g, const void* V, int ell, const double2* K, void* Y, int R, bool keep,
                hipStream_t s) {
  OVL_REQUIRE(R >= 1 && R <= OVL_MAX_RHS && ell >= 1, OVL_E_ARG, "block_axpy: 1 <= R <= 12, ell >= 1");
  if (keep) update<1>(g, V, ell, Y, R, K, 1.0, s);
  else update<0>(g, V, ell, Y, R, K, 1.0, s);
}

namespace {
// coef = c1 + c2, beta = sqrt(n2), inv = 1 / beta (as a complex scalar).
__global__ void lanczos_scalars_kernel(int n, const double2* c1, const double2* c2, double2* coef, const double* n2,
                                       double* beta, double* inv) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) coef[i] = make_double2(c1[i].x + c2[i].x, c1[i].y + c2[i].y);
  if (threadIdx.x == 0) {
    const double b = sqrt(n2[0]);
    beta[0] = b;
    inv[0] = 1.0 / b;
    inv[1] = 0.0;
  }
}
}  // namespace

// Nothing of a step needs the host: coefficients, norm and scale stay on the
// device (the host took part six times a step before, about 15 us).
void lanczos_step(const ovl_geom* g, const void* Q, int n, void* w, void* next, double2* coef, double* beta,
                  double2* scratch, hipStream_t s) {
  double2 *c1 = scratch, *c2 = scratch + n;
  double* sc = reinterpret_cast<double*>(scratch + 2 * n);  // norm (2), 1 / beta (2)
  const size_t v64 = spinor_vec_bytes(g, OVL_F64);
  for (double2* c : {c1, c2}) {
    block_dot(g, Q, n, w, OVL_F64, 1, c, s);
    update<1>(g, Q, n, w, 1, c, -1.0, s);
  }
  blas_norm2(OVL_F64, v64 / 16, w, 1, v64, sc, s);
  hipLaunchKernelGGL(lanczos_scalars_kernel, dim3(1), dim3(256), 0, s, n, c1, c2, coef, sc, beta, sc + 2);
  OVL_HIP(hipGetLastError());
  blas_axpby(OVL_F64, w, sc + 2, OVL_F64, next, nullptr, static_cast<size_t>(g->N), 1, s);
}

namespace {
// The scalars of lanczos_fused from D[R i] = s_i = q_i^dag u, D[R i + 1] = t_i =
// q_i^dag y (i < j), D[R j] = u^dag u, D[R j + 1] = u^dag y; R = 1: there is no y.
template <int R>
__global__ __launch_bounds__(256) void lanczos_fused_scalars_kernel(int j, const double2* D, double* alpha,
                                                                    double* beta, double* sc) {
  double v[3] = {0.0, 0.0, 0.0};  // s^dag s, s^dag t
  for (int i = threadIdx.x; i < j; i += 256) {
    const double2 a = D[R * i], b = D[R * i + R - 1];
    v[0] += a.x * a.x + a.y * a.y;
    v[1] += a.x * b.x + a.y * b.y;
    v[2] += a.x * b.y - a.y * b.x;
  }
  __shared__ double red[3][256];
#pragma unroll
  for (int k = 0; k < 3; ++k) red[k][threadIdx.x] = v[k];
  for (int o = 128; o > 0; o >>= 1) {
    __syncthreads();
    if (threadIdx.x < o)
#pragma unroll
      for (int k = 0; k < 3; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + o];
  }
  if (threadIdx.x) return;
  double b2 = D[R * j].x - red[0][0];
  if (b2 < 0.0) b2 = 0.0;  // rounding; a NaN stays
  const double b = sqrt(b2), last = j > 0 ? D[R * (j - 1)].x : 0.0;  // s_{j-1}
  if (j > 0) {
    alpha[j - 1] += last;
    beta[j - 1] = b;
  }
  if constexpr (R == 2) {
    const double2 uy = D[2 * j + 1];
    const double pr = (uy.x - red[1][0]) / b2, pi = (uy.y - red[2][0]) / b2;  // q_j^dag y / beta
    alpha[j] = pr - last;
    sc[0] = 1.0 / b;
    sc[1] = pr;
    sc[2] = pi;
  }
}

// u *= c, y = c y - (p + i q) u (the new one) for sc = {c, p, q}.
__global__ __launch_bounds__(256) void lanczos_next_kernel(size_t n, const double* sc, double2* u, double2* y) {
  const double c = sc[0], p = sc[1], q = sc[2];
  for (size_t i = blockIdx.x * 256ul + threadIdx.x; i < n; i += gridDim.x * 256ul) {
    const double2 a = u[i], b = y[i], z = make_double2(c * a.x, c * a.y);
    u[i] = z;
    y[i] = make_double2(c * b.x - (p * z.x - q * z.y), c * b.y - (p * z.y + q * z.x));
  }
}
}  // namespace

// With q = (u - Q s) / beta, beta^2 = u^dag u - s^dag s, and y = H u: q_j^dag y =
// (u^dag y - s^dag t) / beta, and (y - Q t - q q_j^dag y) / beta is H q without its
// parts along Q and q, because H Q s lies in their span; along q it has beta
// s_{j-1} (the recurrence), so q_j^dag H q = q_j^dag y / beta - s_{j-1}.  One step's second
// pass and the next step's first pass are then one reading of Q for the dots and
// one for the updates; lanczos_step reads it four times.  Bound by those readings,
// 92 GB for 60 steps at 16^3x32: ovl_hw_bound 39.6 ms with four, 23.3 ms now.
void lanczos_fused(const ovl_geom* g, void* Q, int j, bool last, double* alpha, double* beta, double2* scratch,
                   hipStream_t s) {
  const size_t v64 = spinor_vec_bytes(g, OVL_F64);
  char* u = static_cast<char*>(Q) + static_cast<size_t>(j) * v64;
  double* sc = reinterpret_cast<double*>(scratch + 2 * (j + 1));
  auto scalars = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1), dim3(256), 0, s, j, scratch, alpha, beta, sc);
    OVL_HIP(hipGetLastError());
  };
  block_dot(g, Q, j + 1, u, OVL_F64, last ? 1 : 2, scratch, s);
  if (last) return scalars(lanczos_fused_scalars_kernel<1>);
  scalars(lanczos_fused_scalars_kernel<2>);
  if (j > 0) update<1>(g, Q, j, u, 2, scratch, -1.0, s);
  const size_t n = v64 / 16;
  hipLaunchKernelGGL(lanczos_next_kernel, dim3(static_cast<unsigned>(std::min<size_t>((n + 255) / 256, 8192))),
                     dim3(256), 0, s, n, sc, reinterpret_cast<double2*>(u), reinterpret_cast<double2*>(u + v64));
  OVL_HIP(hipGetLastError());
}

void block_rotate_inplace(const ovl_geom* g, void* V, int K, const double2* S, int k, hipStream_t s) {
  OVL_REQUIRE(k >= 1 && k <= K, OVL_E_ARG, "rotate: need 1 <= k <= K");
  const size_t lds = static_cast<size_t>(K) * RT * sizeof(Cx<double>);
  OVL_REQUIRE(lds <= 64 * 1024, OVL_E_ARG, "rotate: basis too large (K <= 512)");
  const int Nh = g->geo.Nh;
  dim3 grid((Nh + RT - 1) / RT, 24);
  hipLaunchKernelGGL(rotate_kernel, grid, dim3(256), lds, s, Nh, K, k, static_cast<char*>(V),
                     spinor_vec_bytes(g, OVL_F64), S);
  OVL_HIP(hipGetLastError());
}

namespace {
// The projection with caller-provided scratch: C (ell * nrhs coefficients)
// and the split-K partials of pass 1 (ell * G * nrhs).
void lowmode_project_ws(const ovl_lowmodes* lm, const void* psi, void* psih, void* w, int prec, int nrhs, int g5w,
                        double2* C, double2* part, int G, hipStream_t s) {
  OVL_REQUIRE(nrhs >= 1 && nrhs <= OVL_MAX_RHS && lm->ell >= 1, OVL_E_ARG,
              "projection: 1 <= nrhs <= 12 and at least one low mode");
  dot_prec(&lm->geom, lm->V, lm->ell, psi, prec, nrhs, C, part, G, s);
  switch (prec) {
    case OVL_F64: project_go<OVL_F64>(lm, psi, psih, w, nrhs, C, g5w, s); break;
    case OVL_F32: project_go<OVL_F32>(lm, psi, psih, w, nrhs, C, g5w, s); break;
    case OVL_F16: project_go<OVL_F16>(lm, psi, psih, w, nrhs, C, g5w, s); break;
    case OVL_BF16: project_go<OVL_BF16>(lm, psi, psih, w, nrhs, C, g5w, s); break;
    default: throw Error(OVL_E_PRECISION, "unknown precision");
  }
}

// Scratch of the allocation-free projection: one array per GPU, in device
// memory for the life of the process.  Host code never uses the array's
// name as an address; the kernels receive the per-device pointer that
// hipGetSymbolAddress returns.
constexpr size_t kStaticScratchBytes = size_t(16) << 20;
constexpr int kStaticMinBlocks = 64;  // fewest K-blocks of pass 1 accepted
// Largest ell * nrhs for which the coefficients (rounded up to 256 bytes)
// and kStaticMinBlocks sets of partials fit.
constexpr size_t kMaxStaticEllRhs = (kStaticScratchBytes - 256) / (sizeof(double2) * (kStaticMinBlocks + 1));
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per
// device with that device current.
void* static_scratch() {
  int dev = -1;
  OVL_HIP(hipGetDevice(&dev));
  OVL_REQUIRE(dev >= 0 && dev < kMaxDevices, OVL_E_ARG, "device index out of range for the static scratch table");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      throw Error(OVL_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

void lowmode_project(const ovl_lowmodes* lm, const void* psi, void* psih, void* w, int prec, int nrhs, int g5w,
                     hipStream_t s) {
  OVL_REQUIRE(nrhs >= 1 && nrhs <= OVL_MAX_RHS, OVL_E_ARG, "projection supports 1 to 12 right-hand sides");
  WsBuf cbuf(static_cast<size_t>(lm->ell) * nrhs * sizeof(double2), s);
  const int G = dot_blocks(&lm->geom, lm->ell, nrhs);
  WsBuf part(static_cast<size_t>(lm->ell) * G * nrhs * sizeof(double2), s);
  lowmode_project_ws(lm, psi, psih, w, prec, nrhs, g5w, static_cast<double2*>(cbuf.p),
                     static_cast<double2*>(part.p), G, s);
}

// Same projection with its scratch in the static per-device array.  Pass 1
// keeps dot_blocks() K-blocks while they fit (then the result is bit-identical
// to lowmode_project), else as many as fit, at least kStaticMinBlocks.
// Every partial and coefficient slot is written before it is read, so
// nothing needs clearing between calls.
void lowmode_project_static(const ovl_lowmodes* lm, const void* psi, void* psih, void* w, int prec, int nrhs,
                            hipStream_t s) {
  OVL_REQUIRE(nrhs >= 1 && nrhs <= OVL_MAX_RHS, OVL_E_ARG, "projection supports 1 to 12 right-hand sides");
  OVL_REQUIRE(static_cast<size_t>(lm->ell) * nrhs <= kMaxStaticEllRhs, OVL_E_ARG,
              "ovl_lowmodes_project_noalloc: ell * nrhs = " + std::to_string(lm->ell * nrhs) +
                  " exceeds what its 16 MiB static scratch holds (ell * nrhs <= " +
                  std::to_string(kMaxStaticEllRhs) + ")");
  const size_t unit = static_cast<size_t>(lm->ell) * nrhs * sizeof(double2);  // one coefficient set
  const size_t c_bytes = (unit + 255) / 256 * 256;
  const size_t fit = (kStaticScratchBytes - c_bytes) / unit;  // >= kStaticMinBlocks by the check above
  const int G = static_cast<int>(std::min<size_t>(dot_blocks(&lm->geom, lm->ell, nrhs), fit));
  char* base = static_cast<char*>(static_scratch());
  lowmode_project_ws(lm, psi, psih, w, prec, nrhs, 0, reinterpret_cast<double2*>(base),
                     reinterpret_cast<double2*>(base + c_bytes), G, s);
}

}  // namespace ovl
