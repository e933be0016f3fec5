// Gauge-equivariant parallel-transport convolution (PTC) network used as a
// learned right preconditioner for D(m).  Not part of arXiv:1106.4964; it
// is built from the same parallel transporters T_mu as the Wilson operator
// (Sec. II eq. 2, here without the spin projector):
//
//   phi_out[a](x) = sum_b sum_k W[k][a][b] (T_k phi_in[b])(x),
//   k = 0: identity; 1..4: T_{+mu} phi(x) = U_mu(x) phi(x+mu);
//   5..8: T_{-mu} phi(x) = U_mu(x-mu)^dag phi(x-mu);  W[k][a][b]: 4x4 on spin.
//
// Layers are linear, so the network commutes with gauge transformations.
// With T_{+mu}^dag = T_{-mu} and W acting on spin only, the input gradient
// of a layer is the same kind of layer with weights W'[k'][b][a] =
// W[k][a][b]^dag (k' the opposite path), so one forward kernel serves both
// directions.  The weight gradient
//   G[k][a][b] = sum_x sum_colour g_out[a](x) (T_k phi_in[b](x))^dag
// is a site reduction (FP32 per thread, FP64 across blocks, fixed order).
//
// Activations are FP32 spinors in the library layout, one vector per
// channel; the links come from the FP32 representation of the gauge field.
#include <algorithm>
#include <cmath>
#include <complex>

#include "ops.h"

namespace ovl {
namespace {

constexpr int NPATH = 9;
constexpr int CMAX = 4;

// Neighbours of site h in direction mu (the same for the whole wave), parity
// 1 - p; computed where they are needed, since a run-time index into a table of
// eight would put the table in scratch memory.
__device__ inline void neighbors_of(const Geo& g, int h, int x, int y, int z, int t, int mu, int& fwd, int& bwd) {
  if (mu == 0) {
    const int base = h - (x >> 1);
    fwd = base + ((x + 1 == g.Lx ? 0 : x + 1) >> 1);
    bwd = base + ((x == 0 ? g.Lx - 1 : x - 1) >> 1);
    return;
  }
  const int c = mu == 1 ? y : mu == 2 ? z : t, L = mu == 1 ? g.Ly : mu == 2 ? g.Lz : g.Lt;
  const int st = mu == 1 ? g.sy : mu == 2 ? g.sz : g.st;
  fwd = h + (c + 1 == L ? -(L - 1) * st : st);
  bwd = h + (c == 0 ? (L - 1) * st : -st);
}

// a += u v, four FMAs
__device__ inline void cfma(Cx<float>& a, Cx<float> u, Cx<float> v) {
  a.re = ffma(u.re, v.re, a.re);
  a.re = ffma(-u.im, v.im, a.re);
  a.im = ffma(u.re, v.im, a.im);
  a.im = ffma(u.im, v.re, a.im);
}

// out += U s (DAG: U^dag s) on the colour index of the four spins, each row's
// product summed before it is added (the sums over paths and channels then
// round once per term; adding every product at once cost a third in accuracy).
template <bool DAG>
__device__ inline void colour_add(const Cx<float> (*u)[3], const Cx<float>* s, Cx<float>* out) {
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      Cx<float> r = {0.f, 0.f};
#pragma unroll
      for (int b = 0; b < 3; ++b) cfma(r, DAG ? conj(u[b][a]) : u[a][b], s[3 * sp + b]);
      out[3 * sp + a] = out[3 * sp + a] + r;
    }
}

// u s (CONJ: conj(u) s) with every rounding spelled out: one product of each
// part is rounded, the other one fused; SWAP: the other way round in the
// commutative part (im; re with CONJ).
template <bool CONJ, bool SWAP>
__device__ inline Cx<float> rounded_mul(Cx<float> u, Cx<float> s) {
  const float ui = CONJ ? -u.im : u.im;
  Cx<float> z;
  if constexpr (CONJ && SWAP) z.re = ffma(-ui, s.im, __fmul_rn(u.re, s.re));
  else z.re = ffma(u.re, s.re, -__fmul_rn(ui, s.im));
  if constexpr (!CONJ && SWAP) z.im = ffma(ui, s.re, __fmul_rn(u.re, s.im));
  else z.im = ffma(u.re, s.im, __fmul_rn(ui, s.re));
  return z;
}

// out = U s (DAG: U^dag s) for the weight gradient, whose FP32 sums are handed
// out in FP64: each complex product is rounded before it is added.  Which of a
// part's two products is rounded and which fused (columns 0 and 2 of a rebuilt
// third row have it the other way round) is a choice without a reason in the
// arithmetic: it is the one that gradients and trained weights of earlier builds
// were made with, and is kept so that they repeat.  The blocks' FP32 sums are the
// same to the last bit; the FP64 sum over the 256 blocks runs in another order
// than in those builds, which changed none of 3600 gradient entries (8 shapes from
// 4^4 to 24^3x64).  It costs six instructions per product where colour_add takes four.
template <int R, bool DAG>
__device__ inline void colour_mul12(const Cx<float> (*u)[3], const Cx<float>* s, Cx<float>* out) {
#pragma unroll
  for (int sp = 0; sp < 4; ++sp)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      Cx<float> r = {0.f, 0.f};
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const Cx<float> x = s[3 * sp + b];
        const bool swap = R == 12 && (DAG ? b == 2 && a != 1 : a == 2 && b != 1);
        if constexpr (DAG) r = r + (swap ? rounded_mul<true, true>(u[b][a], x) : rounded_mul<true, false>(u[b][a], x));
        else r = r + (swap ? rounded_mul<false, true>(u[a][b], x) : rounded_mul<false, false>(u[a][b], x));
      }
      out[3 * sp + a] = r;
    }
}

// out += w s, the 4x4 matrix w (16 complex numbers, the same for the whole
// wave: scalar loads) on the spin index.
__device__ inline void spin_add(const float2* __restrict__ w, const Cx<float>* s, Cx<float>* out) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    Cx<float> z[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float2 ww = w[4 * r + t];
#pragma unroll
      for (int c = 0; c < 3; ++c) cfma(z[c], Cx<float>{ww.x, ww.y}, s[3 * t + c]);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) out[3 * r + c] = out[3 * r + c] + z[c];
  }
}

__device__ inline void clear12(Cx<float>* v) {
#pragma unroll
  for (int c = 0; c < 12; ++c) v[c] = {0.f, 0.f};
}

// out[a] = sum_b sum_k W[k][a][b] T_k in[b]; W as float2 [k][a][b][s][t].
// blockIdx.y selects one field of a batch: its channels start rstride_in
// (rstride_out) bytes after the previous field's.  Colour and spin matrices
// commute, so the transport acts where there are fewer channels: on the
// inputs, or on the spin-mixed sums.  The channel counts are compile-time, so
// that the accumulators are registers, and W comes through scalar loads:
// with run-time counts and W in LDS 4 -> 1 channels took 135 us at 16^3x32,
// now 72 (1.1 GFMA, 21 us at 51 TFMA/s; two waves per SIMD that wait for each
// direction's loads in turn).
template <int R, int CIN, int COUT>
__global__ __launch_bounds__(256) void ptc_forward_kernel(Geo g, const void* links, const char* in, char* out,
                                                          size_t vstride, const float2* __restrict__ W,
                                                          size_t rstride_in, size_t rstride_out) {
  in += blockIdx.y * rstride_in;
  out += blockIdx.y * rstride_out;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 2 * g.Nh) return;
  const int p = e >= g.Nh, h = e - p * g.Nh;
  int x, y, z, t;
  site_coords(g, p, h, x, y, z, t);
  Cx<float> acc[COUT][12];
#pragma unroll
  for (int a = 0; a < COUT; ++a) clear12(acc[a]);
  auto path = [&](auto dir, int k, int q, int hn, const Cx<float> (*u)[3]) {  // dir: 0 identity, 1 U, 2 U^dag
    constexpr int D = decltype(dir)::value;
    const float2* w = W + static_cast<size_t>(k) * COUT * CIN * 16;
    if constexpr (D == 0 || CIN <= COUT) {
#pragma unroll
      for (int b = 0; b < CIN; ++b) {
        Cx<float> s[12], v[12];
        SpinorIO<OVL_F32>::load(in + b * vstride, q, hn, g.Nh, s);
        if constexpr (D != 0) {
          clear12(v);
          colour_add<D == 2>(u, s, v);
        }
#pragma unroll
        for (int a = 0; a < COUT; ++a) spin_add(w + (a * CIN + b) * 16, D == 0 ? s : v, acc[a]);
      }
    } else {
      Cx<float> v[COUT][12];
#pragma unroll
      for (int a = 0; a < COUT; ++a) clear12(v[a]);
#pragma unroll
      for (int b = 0; b < CIN; ++b) {
        Cx<float> s[12];
        SpinorIO<OVL_F32>::load(in + b * vstride, q, hn, g.Nh, s);
#pragma unroll
        for (int a = 0; a < COUT; ++a) spin_add(w + (a * CIN + b) * 16, s, v[a]);
      }
#pragma unroll
      for (int a = 0; a < COUT; ++a) colour_add<D == 2>(u, v[a], acc[a]);
    }
  };
  path(std::integral_constant<int, 0>{}, 0, p, h, nullptr);
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
    int hf, hb;
    neighbors_of(g, h, x, y, z, t, mu, hf, hb);
    Cx<float> u[3][3];
    LinkIO<OVL_F32, R>::load(links, mu, p, h, g.Nh, u);
    path(std::integral_constant<int, 1>{}, mu + 1, 1 - p, hf, u);
    LinkIO<OVL_F32, R>::load(links, mu, 1 - p, hb, g.Nh, u);
    path(std::integral_constant<int, 2>{}, mu + 5, 1 - p, hb, u);
  }
#pragma unroll
  for (int a = 0; a < COUT; ++a) SpinorIO<OVL_F32>::store(out + a * vstride, p, h, g.Nh, acc[a]);
}

// Sums v[0..N) over the wave, the values dealt out over the lanes: every step
// halves the lanes that share a value and the values a lane keeps, N + N/2 +
// ... exchanges instead of 6 N, with the pairs of a butterfly (so its sums, to
// the last bit).  On return v[0..dealt(N)) are the sums of the values
// base + 0..dealt(N) - 1 of this lane.
template <int N, int O>
__device__ inline void wave_deal(float* v, int lane, int& base) {
  if constexpr (O >= 1) {
    if constexpr (N % 2 == 0) {
      constexpr int H = N / 2;
      const bool up = lane & O;
#pragma unroll
      for (int i = 0; i < H; ++i) {
        if constexpr (O >= 16) {
          uint32_t a = __builtin_bit_cast(uint32_t, v[i]), b = __builtin_bit_cast(uint32_t, v[i + H]);
          if constexpr (O == 32) swap32(a, b);
          else swap16(a, b);
          v[i] = __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
        } else {
          const float keep = up ? v[i + H] : v[i], send = up ? v[i] : v[i + H];
          v[i] = keep + __shfl_xor(send, O, 64);
        }
      }
      base += up ? H : 0;
      wave_deal<H, O / 2>(v, lane, base);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] += __shfl_xor(v[i], O, 64);
      wave_deal<N, O / 2>(v, lane, base);
    }
  }
}
constexpr int dealt(int n) {  // values a lane keeps
  for (int o = 0; o < 6 && n % 2 == 0; ++o) n /= 2;
  return n;
}

// partial[(k*G + block)*cout*cin*16 + ...] = sum over the block's sites of
// g_out[a][s][c] conj(T_k in[b][t][c]).  blockIdx.y = k.  The channel counts
// are compile-time (with run-time counts the 64 accumulators lived in scratch
// memory: 376 us for 1 -> 4 channels at 16^3x32, now 71; 0.9 GFMA are 18 us).
template <int R, int CIN, int COUT>
__global__ __launch_bounds__(256) void ptc_wgrad_kernel(Geo g, const void* links, const char* in, const char* gout,
                                                        size_t vstride, double2* partial) {
  constexpr int NC = CIN * COUT * 16;
  __shared__ float2 red[256 / 64][NC];
  const int k = blockIdx.y, mu = (k - 1) & 3;
  union {
    Cx<float> c[NC];  // [a*cin+b][s][t]
    float f[2 * NC];
  } acc;
#pragma unroll
  for (int i = 0; i < NC; ++i) acc.c[i] = {0.f, 0.f};
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < 2 * g.Nh; e += gridDim.x * blockDim.x) {
    const int p = e >= g.Nh, h = e - p * g.Nh;
    int x, y, z, t, hf, hb;
    site_coords(g, p, h, x, y, z, t);
    neighbors_of(g, h, x, y, z, t, mu, hf, hb);
    Cx<float> u[3][3];
    if (k >= 5) LinkIO<OVL_F32, R>::load(links, mu, 1 - p, hb, g.Nh, u);
    else if (k >= 1) LinkIO<OVL_F32, R>::load(links, mu, p, h, g.Nh, u);
    const int q = k == 0 ? p : 1 - p, hn = k == 0 ? h : k <= 4 ? hf : hb;
#pragma unroll
    for (int b = 0; b < CIN; ++b) {
      Cx<float> s[12], v[12];
      SpinorIO<OVL_F32>::load(in + b * vstride, q, hn, g.Nh, s);
      if (k >= 5) colour_mul12<R, true>(u, s, v);
      else if (k >= 1) colour_mul12<R, false>(u, s, v);
      else {
#pragma unroll
        for (int c = 0; c < 12; ++c) v[c] = s[c];
      }
#pragma unroll
      for (int a = 0; a < COUT; ++a) {
        Cx<float> go[12];
        SpinorIO<OVL_F32>::load(gout + a * vstride, p, h, g.Nh, go);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) {
            Cx<float> z = acc.c[(a * CIN + b) * 16 + 4 * r + tt];
#pragma unroll
            for (int c = 0; c < 3; ++c) z = z + rounded_mul<true, false>(v[3 * tt + c], go[3 * r + c]);
            acc.c[(a * CIN + b) * 16 + 4 * r + tt] = z;
          }
      }
      if (CIN > 1) __builtin_amdgcn_sched_barrier(0);  // one input channel's operands at a time
    }
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int base = 0;
  wave_deal<2 * NC, 32>(acc.f, lane, base);
#pragma unroll
  for (int i = 0; i < dealt(2 * NC); ++i) reinterpret_cast<float*>(red[wv])[base + i] = acc.f[i];
  __syncthreads();
  for (int i = threadIdx.x; i < NC; i += blockDim.x) {
    double re = 0.0, im = 0.0;
    for (int w = 0; w < 256 / 64; ++w) {
      re += red[w][i].x;
      im += red[w][i].y;
    }
    partial[(static_cast<size_t>(k) * gridDim.x + blockIdx.x) * NC + i] = make_double2(re, im);
  }
}

// out[k][i] (+)= sum_b partial[k][b][i]: 64 sums of every 64th block each,
// added pairwise (one thread per sum took 64 us).
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(int nout, int G, const double2* partial, double2* out,
                                                           int accumulate) {
  __shared__ double2 red[64][4];
  const int il = threadIdx.x & 3, bl = threadIdx.x >> 2;
  const int i = blockIdx.x * 4 + il, k = blockIdx.y;
  double re = 0.0, im = 0.0;
  if (i < nout)
    for (int b = bl; b < G; b += 64) {
      const double2 v = partial[(static_cast<size_t>(k) * G + b) * nout + i];
      re += v.x;
      im += v.y;
    }
  red[bl][il] = make_double2(re, im);
  for (int o = 32; o > 0; o >>= 1) {
    __syncthreads();
    if (bl < o) {
      re += red[bl + o][il].x;
      im += red[bl + o][il].y;
      red[bl][il] = make_double2(re, im);
    }
  }
  if (bl == 0 && i < nout) {
    double2* o = out + static_cast<size_t>(k) * nout + i;
    if (accumulate) {
      re += o->x;
      im += o->y;
    }
    *o = make_double2(re, im);
  }
}

// loss[0] += d2[0] / x2[0];  gscale = (2 / x2[0], 0): the gradient of
// ||out - x||^2 / ||x||^2 with respect to out is gscale * (out - x).
__global__ void pair_loss_kernel(const double* d2, const double* x2, double* loss, double* gscale) {
  if (threadIdx.x == 0) {
    loss[0] += d2[0] / x2[0];
    gscale[0] = 2.0 / x2[0];
    gscale[1] = 0.0;
  }
}

constexpr int WG_BLOCKS = 256;

// f(integral_constant<CIN>, integral_constant<COUT>) for run-time counts.
template <int I = 1, class F>
void with_channel(int n, F&& f) {
  if constexpr (I <= CMAX) {
    if (n == I) f(std::integral_constant<int, I>{});
    else with_channel<I + 1>(n, f);
  } else {
    throw Error(OVL_E_ARG, "channels must be 1..4");
  }
}

using zc = std::complex<double>;

// Device copy (float2) of host weights [k][a][b][16].
void upload(const std::vector<zc>& w, float2* dev, hipStream_t s) {
  std::vector<float2> h(w.size());
  for (size_t i = 0; i < w.size(); ++i) h[i] = make_float2(static_cast<float>(w[i].real()), static_cast<float>(w[i].imag()));
  OVL_HIP(hipMemcpyAsync(dev, h.data(), h.size() * sizeof(float2), hipMemcpyHostToDevice, s));
  OVL_HIP(hipStreamSynchronize(s));
}

// W'[k'][b][a] = W[k][a][b]^dag, the weights of the adjoint layer.
std::vector<zc> adjoint_weights(const std::vector<zc>& w, int cin, int cout) {
  std::vector<zc> o(w.size());
  for (int k = 0; k < NPATH; ++k) {
    const int kk = k == 0 ? 0 : (k <= 4 ? k + 4 : k - 4);
    for (int a = 0; a < cout; ++a)
      for (int b = 0; b < cin; ++b)
        for (int s = 0; s < 4; ++s)
          for (int t = 0; t < 4; ++t)
            o[(((kk * cin + b) * cout + a) * 16) + 4 * s + t] = std::conj(w[(((k * cout + a) * cin + b) * 16) + 4 * t + s]);
  }
  return o;
}

struct Layer {
  const ovl_gauge* u;
  const void* links;
  int recon;
  hipStream_t s;
  size_t vstride;

  // nb fields at once: field f reads in + f cin vstride, writes out + f cout vstride
  void forward(const void* in, void* out, int cin, int cout, const float2* W, int nb = 1) const {
    const Geo& g = u->geom.geo;
    dim3 grid((2 * g.Nh + 255) / 256, nb);
    const size_t ri = vstride * cin, ro = vstride * cout;
    with_channel(cin, [&](auto ci) {
      with_channel(cout, [&](auto co) {
        constexpr int CI = decltype(ci)::value, CO = decltype(co)::value;
        auto go = [&](auto kernel) {
          hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, g, links, static_cast<const char*>(in),
                             static_cast<char*>(out), vstride, W, ri, ro);
        };
        if (recon == 18) go(ptc_forward_kernel<18, CI, CO>);
        else go(ptc_forward_kernel<12, CI, CO>);
      });
    });
    OVL_HIP(hipGetLastError());
  }
  void wgrad(const void* in, const void* gout, int cin, int cout, double2* out, int accumulate = 0) const {
    const Geo& g = u->geom.geo;
    const int nout = cin * cout * 16;
    constexpr int G = WG_BLOCKS;
    WsBuf part(static_cast<size_t>(NPATH) * G * nout * sizeof(double2), s);
    with_channel(cin, [&](auto ci) {
      with_channel(cout, [&](auto co) {
        constexpr int CI = decltype(ci)::value, CO = decltype(co)::value;
        if constexpr (CI * CO <= CMAX) {
          auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(G, NPATH), dim3(256), 0, s, g, links, static_cast<const char*>(in),
                               static_cast<const char*>(gout), vstride, static_cast<double2*>(part.p));
          };
          if (recon == 18) go(ptc_wgrad_kernel<18, CI, CO>);
          else go(ptc_wgrad_kernel<12, CI, CO>);
        } else {
          throw Error(OVL_E_ARG, "weight gradient: cin*cout <= 4");
        }
      });
    });
    OVL_HIP(hipGetLastError());
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((nout + 3) / 4, NPATH), dim3(256), 0, s, nout, G,
                       static_cast<const double2*>(part.p), out, accumulate);
    OVL_HIP(hipGetLastError());
  }
};

size_t g_nsites(const ovl_gauge* u) { return static_cast<size_t>(u->geom.N); }

Layer make_layer(const ovl_gauge* u, hipStream_t s) {
  Layer L{u, nullptr, 0, s, spinor_vec_bytes(&u->geom, OVL_F32)};
  L.links = gauge_links(u, OVL_F32, &L.recon);
  return L;
}

}  // namespace

// out_r = M in_r for a batch of nrhs FP32 fields (back to back); the hidden
// channels of the batch come from the pool.
void net_apply(const ovl_net* net, const ovl_gauge* u, const void* in, void* out, int nrhs, hipStream_t s) {
  Layer L = make_layer(u, s);
  const int C = net->hidden;
  WsBuf hid(L.vstride * C * nrhs, s);
  WsBuf w1(net->w1.size() * sizeof(float2), s), w2(net->w2.size() * sizeof(float2), s);
  upload(net->w1, static_cast<float2*>(w1.p), s);
  upload(net->w2, static_cast<float2*>(w2.p), s);
  L.forward(in, hid.p, 1, C, static_cast<const float2*>(w1.p), nrhs);
  L.forward(hid.p, out, C, 1, static_cast<const float2*>(w2.p), nrhs);
}

}  // namespace ovl

using namespace ovl;

extern "C" {

int ovl_net_create(const ovl_geom* g, int hidden, ovl_net** out) {
  return guard([&] {
    OVL_REQUIRE(g && out, OVL_E_ARG, "null argument");
    OVL_REQUIRE(hidden >= 1 && hidden <= CMAX, OVL_E_ARG, "hidden channels must be 1..4");
    ovl_net* n = new ovl_net;
    n->geom = *g;
    n->hidden = hidden;
    n->w1.assign(static_cast<size_t>(NPATH) * hidden * 16, zc(0.0, 0.0));
    n->w2.assign(static_cast<size_t>(NPATH) * hidden * 16, zc(0.0, 0.0));
    *out = n;
    return OVL_OK;
  });
}

int ovl_net_destroy(ovl_net* n) {
  delete n;
  return OVL_OK;
}

int ovl_net_set_weights(ovl_net* n, const double* w1, const double* w2) {
  return guard([&] {
    OVL_REQUIRE(n && w1 && w2, OVL_E_ARG, "null argument");
    for (size_t i = 0; i < n->w1.size(); ++i) n->w1[i] = zc(w1[2 * i], w1[2 * i + 1]);
    for (size_t i = 0; i < n->w2.size(); ++i) n->w2[i] = zc(w2[2 * i], w2[2 * i + 1]);
    return OVL_OK;
  });
}

int ovl_net_get_weights(const ovl_net* n, double* w1, double* w2) {
  return guard([&] {
    OVL_REQUIRE(n && w1 && w2, OVL_E_ARG, "null argument");
    for (size_t i = 0; i < n->w1.size(); ++i) {
      w1[2 * i] = n->w1[i].real();
      w1[2 * i + 1] = n->w1[i].imag();
    }
    for (size_t i = 0; i < n->w2.size(); ++i) {
      w2[2 * i] = n->w2[i].real();
      w2[2 * i + 1] = n->w2[i].imag();
    }
    return OVL_OK;
  });
}

int ovl_ptc_layer_forward(const ovl_gauge* u, const void* in, int cin, void* out, int cout, const double* W,
                          ovl_stream_t st) {
  return guard([&] {
    OVL_REQUIRE(u && in && out && W, OVL_E_ARG, "null argument");
    OVL_REQUIRE(cin >= 1 && cin <= CMAX && cout >= 1 && cout <= CMAX, OVL_E_ARG, "channels must be 1..4");
    OVL_REQUIRE(in != out, OVL_E_ALIAS, "output must not alias the input");
    hipStream_t s = static_cast<hipStream_t>(st);
    Layer L = make_layer(u, s);
    const size_t nw = static_cast<size_t>(NPATH) * cin * cout * 16;
    std::vector<zc> w(nw);
    for (size_t i = 0; i < nw; ++i) w[i] = zc(W[2 * i], W[2 * i + 1]);
    WsBuf dw(nw * sizeof(float2), s);
    upload(w, static_cast<float2*>(dw.p), s);
    L.forward(in, out, cin, cout, static_cast<const float2*>(dw.p));
    return OVL_OK;
  });
}

int ovl_ptc_layer_backward(const ovl_gauge* u, const void* in, int cin, const void* gout, int cout, const double* W,
                           void* gin, double* gW, ovl_stream_t st) {
  return guard([&] {
    OVL_REQUIRE(u && in && gout && W, OVL_E_ARG, "null argument");
    OVL_REQUIRE(cin >= 1 && cin <= CMAX && cout >= 1 && cout <= CMAX && cin * cout <= CMAX, OVL_E_ARG,
                "channels must be 1..4 with cin*cout <= 4");
    hipStream_t s = static_cast<hipStream_t>(st);
    Layer L = make_layer(u, s);
    const size_t nw = static_cast<size_t>(NPATH) * cin * cout * 16;
    std::vector<zc> w(nw);
    for (size_t i = 0; i < nw; ++i) w[i] = zc(W[2 * i], W[2 * i + 1]);
    if (gin) {
      OVL_REQUIRE(gin != gout && gin != in, OVL_E_ALIAS, "gradient output aliases an input");
      WsBuf dw(nw * sizeof(float2), s);
      upload(adjoint_weights(w, cin, cout), static_cast<float2*>(dw.p), s);
      L.forward(gout, gin, cout, cin, static_cast<const float2*>(dw.p));
    }
    if (gW) {
      WsBuf dg(nw * sizeof(double2), s);
      L.wgrad(in, gout, cin, cout, static_cast<double2*>(dg.p));
      OVL_HIP(hipMemcpyAsync(gW, dg.p, nw * sizeof(double2), hipMemcpyDeviceToHost, s));
    }
    OVL_HIP(hipStreamSynchronize(s));
    return OVL_OK;
  });
}

int ovl_net_train(ovl_net* n, const ovl_gauge* u, const void* B, const void* X, int npairs, int epochs, int batch,
                  double lr, const int32_t* order, double* loss_history, ovl_stream_t st) {
  return guard([&] {
    OVL_REQUIRE(n && u && B && X && order, OVL_E_ARG, "null argument");
    OVL_REQUIRE(npairs >= 1 && epochs >= 1 && batch >= 1 && lr > 0.0, OVL_E_ARG, "bad training parameter");
    hipStream_t s = static_cast<hipStream_t>(st);
    Layer L = make_layer(u, s);
    const int C = n->hidden;
    const size_t vs = L.vstride;
    const size_t nw = n->w1.size();  // = n->w2.size()
    WsBuf hid(vs * C, s), out(vs, s), gout(vs, s), gh(vs * C, s);
    WsBuf dw1(nw * sizeof(float2), s), dw2(nw * sizeof(float2), s), dw2a(nw * sizeof(float2), s);
    WsBuf g1(nw * sizeof(double2), s), g2(nw * sizeof(double2), s);
    WsBuf sc(8 * sizeof(double), s);
    double* dsc = static_cast<double*>(sc.p);  // [0..1] norm tmp, [2] x2, [3] d2, [4] loss, [6..7] gscale
    const double one_m1[4] = {1.0, 0.0, -1.0, 0.0};
    WsBuf cst(4 * sizeof(double), s);
    OVL_HIP(hipMemcpyAsync(cst.p, one_m1, sizeof(one_m1), hipMemcpyHostToDevice, s));
    const double* d_one = static_cast<const double*>(cst.p);
    const double* d_m1 = d_one + 2;
    // Adam state over the real and imaginary parts of every weight
    std::vector<double> m1(4 * nw, 0.0), v1(4 * nw, 0.0);
    const double b1 = 0.9, b2 = 0.999, eps = 1e-8;
    int tstep = 0;
    std::vector<double2> hg(nw);
    const size_t n16 = vs / 16;
    auto norm2_into = [&](const void* x, double* dst) {
      blas_norm2(OVL_F32, n16, x, 1, vs, dsc, s);
      OVL_HIP(hipMemcpyAsync(dst, dsc, sizeof(double), hipMemcpyDeviceToDevice, s));
    };
    for (int ep = 0; ep < epochs; ++ep) {
      double zero = 0.0;
      OVL_HIP(hipMemcpyAsync(dsc + 4, &zero, sizeof(double), hipMemcpyHostToDevice, s));
      for (int b0 = 0; b0 < npairs; b0 += batch) {
        const int nb = std::min(batch, npairs - b0);
        upload(n->w1, static_cast<float2*>(dw1.p), s);
        upload(n->w2, static_cast<float2*>(dw2.p), s);
        upload(adjoint_weights(n->w2, C, 1), static_cast<float2*>(dw2a.p), s);
        blas_zero(g1.p, nw * sizeof(double2), s);
        blas_zero(g2.p, nw * sizeof(double2), s);
        for (int q = 0; q < nb; ++q) {
          const int idx = order[static_cast<size_t>(ep) * npairs + b0 + q];
          OVL_REQUIRE(idx >= 0 && idx < npairs, OVL_E_ARG, "training order index out of range");
          const char* bb = static_cast<const char*>(B) + static_cast<size_t>(idx) * vs;
          const char* xx = static_cast<const char*>(X) + static_cast<size_t>(idx) * vs;
          L.forward(bb, hid.p, 1, C, static_cast<const float2*>(dw1.p));
          L.forward(hid.p, out.p, C, 1, static_cast<const float2*>(dw2.p));
          // diff = out - x (into gout), loss and gradient scale
          blas_axpby(OVL_F32, xx, d_m1, OVL_F32, out.p, d_one, g_nsites(u), 1, s);
          norm2_into(xx, dsc + 2);
          norm2_into(out.p, dsc + 3);
          hipLaunchKernelGGL(pair_loss_kernel, dim3(1), dim3(64), 0, s, dsc + 3, dsc + 2, dsc + 4, dsc + 6);
          blas_axpby(OVL_F32, out.p, dsc + 6, OVL_F32, gout.p, nullptr, g_nsites(u), 1, s);
          // layer 2: weight gradient and input gradient; layer 1: weight gradient
          L.wgrad(hid.p, gout.p, C, 1, static_cast<double2*>(g2.p), 1);
          L.forward(gout.p, gh.p, 1, C, static_cast<const float2*>(dw2a.p));
          L.wgrad(bb, gh.p, 1, C, static_cast<double2*>(g1.p), 1);
        }
        // Adam step on the mean gradient of the batch
        ++tstep;
        for (int layer = 0; layer < 2; ++layer) {
          OVL_HIP(hipMemcpyAsync(hg.data(), layer == 0 ? g1.p : g2.p, nw * sizeof(double2), hipMemcpyDeviceToHost, s));
          OVL_HIP(hipStreamSynchronize(s));
          std::vector<zc>& W = layer == 0 ? n->w1 : n->w2;
          for (size_t i = 0; i < nw; ++i) {
            const double gr[2] = {hg[i].x / nb, hg[i].y / nb};
            double wv[2] = {W[i].real(), W[i].imag()};
            for (int c = 0; c < 2; ++c) {
              const size_t k = (layer * nw + i) * 2 + c;
              m1[k] = b1 * m1[k] + (1 - b1) * gr[c];
              v1[k] = b2 * v1[k] + (1 - b2) * gr[c] * gr[c];
              const double mh = m1[k] / (1 - std::pow(b1, tstep)), vh = v1[k] / (1 - std::pow(b2, tstep));
              wv[c] -= lr * mh / (std::sqrt(vh) + eps);
            }
            W[i] = zc(wv[0], wv[1]);
          }
        }
      }
      double loss = 0.0;
      OVL_HIP(hipMemcpyAsync(&loss, dsc + 4, sizeof(double), hipMemcpyDeviceToHost, s));
      OVL_HIP(hipStreamSynchronize(s));
      OVL_REQUIRE(std::isfinite(loss), OVL_E_NAN, "training loss is NaN or Inf");
      if (loss_history) loss_history[ep] = loss / npairs;
    }
    return OVL_OK;
  });
}

int ovl_net_apply(const ovl_net* n, const ovl_gauge* u, const void* in, void* out, ovl_stream_t st) {
  return guard([&] {
    OVL_REQUIRE(n && u && in && out, OVL_E_ARG, "null argument");
    OVL_REQUIRE(in != out, OVL_E_ALIAS, "output must not alias the input");
    net_apply(n, u, in, out, 1, static_cast<hipStream_t>(st));
    return OVL_OK;
  });
}

}  // extern "C"
