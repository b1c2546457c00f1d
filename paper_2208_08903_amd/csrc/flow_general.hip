// General flow kernels: every network without batch norm (any hidden_sizes, odd
// kernel 1 .. 7; paper Sec. 1, coupling-layer equation) on every lattice, with
// implicit-GEMM convolutions on the matrix cores (net_engine.hpp).
//
//   resident  samples whose field and activations fit the LDS: one workgroup per
//             sample runs all layers in one launch (kg_forward), and the backward's
//             recompute, affine backward and data gradients of a group of layers in
//             one launch (kg_backward)
//   staged    larger samples: one launch per convolution over the whole batch,
//             activations in HBM (kg_staged)
//
// Which of the two runs depends, in BF16, on the shape alone, and in FP32 both add in
// the same order, so a sample's result does not depend on the batch it is in.  Either
// backward leaves the hidden activations and the gradients of every convolution's output
// in HBM for a group of layers, and one launch forms all their weight gradients
// (kg_wgrad_slab, kg_wgrad).
//
// Small samples are bound by latency: 64 samples of 64 sites keep 64 of the 256 CUs
// busy with a chain of N n_conv dependent convolutions.  What counts is the time from
// one barrier to the next, hence one launch for all layers instead of one per
// convolution, fragments fetched a layer ahead, neighbours from a table and gathers
// without branches.  Training step of the 2D L = 8 flow with hidden [16, 16, 16], 16
// layers, batch 64, FP32: 3400 us with a launch per convolution and direct sums, 465 so
// (forward 121, backward 246, weight gradients 85).  3D L = 12, hidden 16, 12 layers,
// batch 50, FP32, where a sample does not fit: 47.1 -> 2.57 ms (a hidden convolution of
// 86400 sites 25 us, its data gradient 24 us; direct sums: 294 and 257).
#include "general_wgrad.hpp"

namespace lfs {
namespace {

// LDS of a resident workgroup, byte offsets.
struct ResLds {
  int ps;  // plane stride
  int xs, xm, gy, go, slot[LFS_MAX_HIDDEN], red, nbr;  // xm: the field at the frozen sites
  int ls;                     // forward: every active site's sum of s over the layers
  int frags[2];               // a layer's weight fragments (lf), see kg_forward and kg_backward
  bool lf;
  int total;
};

// of `waves` waves, with the fragments in LDS where they fit and lf asks for it.
ResLds res_lds(const NetDev& d, bool bwd, int waves = kResWaves, bool lf = true) {
  ResLds r{};
  const int V = d.lat.V;
  r.ps = lds_plane_stride(V);
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    const int64_t o = off;
    off += (bytes + 15) / 16 * 16;
    return (int)std::min<int64_t>(o, 1 << 30);
  };
  r.xs = take(4ll * V);
  r.xm = take(4ll * (V + 1));
  if (bwd) {
    r.gy = take(4ll * V);
    r.go = take(4ll * r.ps);
    for (int i = 0; i + 1 < d.n_conv; ++i) r.slot[i] = take(4ll * r.ps * cdiv(d.cout[i], 4));
  } else {
    int q = 0;
    for (int i = 0; i + 1 < d.n_conv; ++i) q = std::max(q, cdiv(d.cout[i], 4));
    const int a = take(4ll * r.ps * q), b = d.n_conv > 2 ? take(4ll * r.ps * q) : a;
    for (int i = 0; i + 1 < d.n_conv; ++i) r.slot[i] = i & 1 ? b : a;
  }
  r.red = take(waves == kResWaves ? 1024ll * kResWaves : 0);
  r.nbr = take(nbr_bytes(d.T, V));
  if (!bwd) r.ls = take(4ll * V);
  // fragments: two layers' in the forward, one layer's forward and transposed ones in the
  // backward
  const int64_t fr = off;
  const int64_t f0 = d.frags_fwd * 1024ll, f1 = (bwd ? d.frags_all - d.frags_fwd : d.frags_fwd) * 1024ll;
  r.lf = lf && fr + f0 + f1 <= (int64_t)kLdsMax;
  if (r.lf) {
    r.frags[0] = take(f0);
    r.frags[1] = take(f1);
  }
  r.total = (int)std::min<int64_t>(off, 1 << 30);
  return r;
}

// Tables of a resident workgroup, and the zero site after the field and every plane.
template <int DIM>
__device__ __forceinline__ void build_tables(const NetDev& d, const ResLds& S, unsigned char* smem, bool bwd) {
  build_nbr<DIM>(d, reinterpret_cast<uint16_t*>(smem + S.nbr));
  const int V = d.lat.V;
  if (threadIdx.x == 0) reinterpret_cast<float*>(smem + S.xm)[V] = 0.f;
  if (bwd && threadIdx.x < 4) reinterpret_cast<float*>(smem + S.go)[4 * V + threadIdx.x] = 0.f;
  for (int i = 0; i + 1 < d.n_conv; ++i)
    for (int k = threadIdx.x; k < (d.cout[i] + 3) / 4 * 4; k += blockDim.x)
      reinterpret_cast<float*>(smem + S.slot[i])[(k >> 2) * S.ps + 4 * V + (k & 3)] = 0.f;
}

// The hidden convolutions of one layer from the masked field into the slots.  store(i, plane,
// site, values) also receives every quad of activation i.  frags: the layer's forward
// fragments.
template <int MODE, bool FEW, class Store>
__device__ __forceinline__ void hidden_convs(const NetDev& d, const ResLds& S, unsigned char* smem,
                                             const u32x4* frags, Store&& store) {
  const Lat& lat = d.lat;
  const int lane = threadIdx.x & 63, j = lane >> 4, m = lane & 15;
  f32x4* red = reinterpret_cast<f32x4*>(smem + S.red);
  const uint16_t* nbr = reinterpret_cast<const uint16_t*>(smem + S.nbr);
  const int tiles = (lat.V + 15) >> 4;
  for (int i = 0; i + 1 < d.n_conv; ++i) {
    const ConvDir& c = d.f[i];
    float* out = reinterpret_cast<float*>(smem + S.slot[i]);
    const int rows = c.rows;
    auto epi = [&](int tile, int ct, const f32x4& acc) {
      const int n = tile * 16 + m, pl = ct * 4 + j;
      if (n < lat.V && 4 * pl < rows) {
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = masked(leaky(acc[r]), (4 * pl + r - rows) >> 31);
        *reinterpret_cast<f32x4*>(out + pl * S.ps + 4 * n) = v;
        store(i, pl, n, v);
      }
    };
    if (i == 0) {
      conv_pass<MODE, false, FEW>(tiles, c, frags + c.off * 64, red, [&](int tile) {
        return lds_field(d, nbr, reinterpret_cast<const float*>(smem + S.xm), min(tile * 16 + m, lat.V - 1));
      }, epi);
    } else {
      const float* in = reinterpret_cast<const float*>(smem + S.slot[i - 1]);
      conv_pass<MODE, false, FEW>(tiles, c, frags + c.off * 64, red, [&](int tile) {
        return lds_planes<false>(d, nbr, S.ps, in, min(tile * 16 + m, lat.V - 1));
      }, epi);
    }
    lds_barrier();
  }
}

// The last convolution at the active sites: f(a, site, o_0, o_1) for the a-th of them.
template <int DIM, int MODE, bool FEW, class F>
__device__ __forceinline__ void last_conv(const NetDev& d, const ResLds& S, unsigned char* smem, const u32x4* frags,
                                          int apar, F&& f) {
  const Lat& lat = d.lat;
  const int lane = threadIdx.x & 63, j = lane >> 4, m = lane & 15, i = d.n_conv - 1, half = lat.V / 2;
  const ConvDir& c = d.f[i];
  const uint16_t* nbr = reinterpret_cast<const uint16_t*>(smem + S.nbr);
  const float* in = reinterpret_cast<const float*>(smem + S.slot[i - 1]);
  conv_pass<MODE, false, FEW>((half + 15) >> 4, c, frags + c.off * 64, reinterpret_cast<f32x4*>(smem + S.red),
                                    [&](int tile) {
    return lds_planes<false>(d, nbr, S.ps, in, half_site<DIM>(lat, min(tile * 16 + m, half - 1), apar));
  }, [&](int tile, int, const f32x4& acc) {
    const int a = tile * 16 + m;
    if (j == 0 && a < half) f(a, half_site<DIM>(lat, a, apar), acc[0], acc[1]);
  });
}

// ---- log q ---------------------------------------------------------------------
// s is summed in FP64: the a-th active site's over the layers, then over the sites in the
// order of 256 threads.  Resident and staged kernels add in this order.  (FP32 sums over all
// layers left the log-det of 12^3 sites and 12 layers off by 6e-5.  The 16 sites of a tile
// added in every layer, by lane exchanges, took 0.25 us a layer more.)

// ---- resident forward ----------------------------------------------------------

// Layers [l0, l1), whose fragments frags are: all of them, or, where the workspace does not
// hold as many, group after group (z of a later one is the earlier one's phi; log r waits in
// logq, the sites' sums in carry [B][V / 2]).
// LF: a layer's fragments are read from LDS, the next layer's copied there meanwhile.
template <int DIM, int MODE, bool LF, bool FEW>
__global__ void __launch_bounds__(64 * kResWaves) kg_forward(NetDev d, ResLds S, const u32x4* __restrict__ frags,
                                                             int l0, int l1, int B, const float* z, float* phi,
                                                             float* __restrict__ saved, double* logq,
                                                             double* __restrict__ logdet, double* carry) {
  using R = std::conditional_t<MODE == kBf16, double, float>;
  extern __shared__ __align__(16) unsigned char smem[];
  const int V = d.lat.V, half = V / 2, F = d.frags_fwd, lane = threadIdx.x & 63;
  const bool sums = fused::wave_id() == (int)(blockDim.x >> 6) - 1;  // the wave that makes the sample's sums
  float* xs = reinterpret_cast<float*>(smem + S.xs);
  float* xm = reinterpret_cast<float*>(smem + S.xm);
  double* ls = reinterpret_cast<double*>(smem + S.ls);
  if constexpr (LF) copy_frags(frags, smem + S.frags[0], F);
  build_tables<DIM>(d, S, smem, false);
  const size_t BV = (size_t)B * V;
  int cur = 0;
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    for (int n = threadIdx.x; n < V; n += blockDim.x) {
      const float v = z[(size_t)b * V + n];
      xs[n] = v;
      xm[n] = masked(v, (parity_of<DIM>(site_of<DIM>(d.lat, n)) ^ ((l0 + d.parity0) & 1)) - 1);
      if (saved && l0 == 0) saved[(size_t)b * V + n] = v;
    }
    double* cb = carry + (size_t)b * half;
    for (int a = threadIdx.x; a < half; a += blockDim.x) ls[a] = l0 > 0 ? cb[a] : 0.0;
    if constexpr (LF) wait_copies();
    lds_barrier();
    double logr = 0.0;
    if (sums)
      logr = l0 > 0 ? logq[b] : log_prior(V, sum_of_256<R>(V, [&](int n) { return (R)xs[n] * xs[n]; }));
    for (int l = l0; l < l1; ++l) {
      const int fpar = (l + d.parity0) & 1;
      const u32x4* fr;
      if constexpr (LF) {
        fr = reinterpret_cast<const u32x4*>(smem + S.frags[cur]);
        cur ^= 1;
        copy_frags(frags + (size_t)(l + 1 < l1 ? l + 1 - l0 : 0) * F * 64, smem + S.frags[cur], F);
      } else {
        fr = frags + (size_t)(l - l0) * F * 64;
      }
      hidden_convs<MODE, FEW>(d, S, smem, fr, [](int, int, int, const f32x4&) {});
      last_conv<DIM, MODE, FEW>(d, S, smem, fr, fpar ^ 1, [&](int a, int n, float o0, float o1) {
        const double ld = ls[a];  // (the a-th site is the same lane's in every layer)
        const float s = d.final_tanh ? tanhf(o0) : o0;
        const float xn = xs[n] * expf(s) + o1;
        xs[n] = xn;
        xm[n] = xn;  // frozen in the next layer, and its partner active
        xm[half_site<DIM>(d.lat, a, fpar)] = 0.f;
        ls[a] = ld + (double)s;
      });
      if constexpr (LF) wait_copies();
      lds_barrier();
      if (saved) {
        float* sv = saved + (size_t)(l + 1) * BV + (size_t)b * V;
        for (int n = threadIdx.x; n < V; n += blockDim.x) sv[n] = xs[n];
      }
    }
    for (int n = threadIdx.x; n < V; n += blockDim.x) phi[(size_t)b * V + n] = xs[n];
    if (l1 < d.N) {
      for (int a = threadIdx.x; a < half; a += blockDim.x) cb[a] = ls[a];
      if (sums && lane == 0) logq[b] = logr;
    } else if (sums) {
      const double ld = sum_of_256<double>(half, [&](int a) { return ls[a]; });
      if (lane == 0) {
        logq[b] = logr - ld;
        if (logdet) logdet[b] = ld;
      }
      // (the sums are cleared for the next sample by other waves, behind this one's reads)
    }
    lds_barrier();
  }
}

// ---- resident backward ---------------------------------------------------------

// A layer's activations and gradients in HBM for the weight gradients: planes of
// [V][4] floats, per (layer of the group, sample): the hidden activations, the
// gradients of the hidden convolutions' outputs in the same order, the gradient of
// the last one's (one plane).
__host__ __device__ inline int store_planes(const NetDev& d) { return 2 * d.hplanes + 1; }

// Layers [l0, l1) of every sample, last to first: g_in is the cotangent of layer l1 - 1's
// output, g_out receives that of layer l0's input.  LF: the layer's forward fragments
// and its transposed ones each have a place in LDS; one is filled while the other is used.
template <int DIM, int MODE, bool LF, bool FEW>
__global__ void __launch_bounds__(64 * kResWaves) kg_backward(NetDev d, ResLds S, const u32x4* __restrict__ frags,
                                                              int B, int l0, int l1, const float* __restrict__ saved,
                                                              const float* g_in, float g_ld,
                                                              const double* __restrict__ g_ld_vec, float* g_out,
                                                              float* __restrict__ store) {
  extern __shared__ __align__(16) unsigned char smem[];
  const Lat& lat = d.lat;
  const int V = lat.V, lane = threadIdx.x & 63, j = lane >> 4, m = lane & 15;
  const int F = d.frags_fwd, FT = d.frags_all - F;
  float* xs = reinterpret_cast<float*>(smem + S.xs);
  float* xm = reinterpret_cast<float*>(smem + S.xm);
  float* gy = reinterpret_cast<float*>(smem + S.gy);
  float* go = reinterpret_cast<float*>(smem + S.go);
  const uint16_t* nbr = reinterpret_cast<const uint16_t*>(smem + S.nbr);
  f32x4* red = reinterpret_cast<f32x4*>(smem + S.red);
  if constexpr (LF) copy_frags(frags + (size_t)(l1 - 1) * d.frags_all * 64, smem + S.frags[0], F);
  build_tables<DIM>(d, S, smem, true);
  const size_t BV = (size_t)B * V;
  const int PL = store_planes(d), HP = d.hplanes;
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    const float gld = g_ld_vec ? (float)(-g_ld_vec[b]) : g_ld;
    for (int n = threadIdx.x; n < V; n += blockDim.x) gy[n] = g_in[(size_t)b * V + n];
    // a layer's field: the thread's first site is loaded a layer ahead
    const float* xb = saved + (size_t)b * V;
    const bool own = threadIdx.x < V;
    float xpre = own ? xb[(size_t)(l1 - 1) * BV + threadIdx.x] : 0.f;
    for (int l = l1 - 1; l >= l0; --l) {
      const int fpar = (l + d.parity0) & 1, apar = fpar ^ 1;
      float* st = store + ((size_t)(l - l0) * B + b) * PL * V * 4;
      auto put = [&](int plane, int n, const f32x4& v) {
        *reinterpret_cast<f32x4*>(st + ((size_t)plane * V + n) * 4) = v;
      };
      auto put_x = [&](int n, float v) {
        xs[n] = v;
        xm[n] = masked(v, (parity_of<DIM>(site_of<DIM>(lat, n)) ^ fpar) - 1);
      };
      if (own) put_x(threadIdx.x, xpre);
      for (int n = threadIdx.x + blockDim.x; n < V; n += blockDim.x) put_x(n, xb[(size_t)l * BV + n]);
      if constexpr (LF) wait_copies();
      lds_barrier();
      const u32x4 *ff, *ft;
      if constexpr (LF) {
        ff = reinterpret_cast<const u32x4*>(smem + S.frags[0]);
        ft = reinterpret_cast<const u32x4*>(smem + S.frags[1]);
        copy_frags(frags + ((size_t)l * d.frags_all + F) * 64, smem + S.frags[1], FT);
      } else {
        ff = frags + (size_t)l * d.frags_all * 64;
        ft = ff + F * 64;
      }
      hidden_convs<MODE, FEW>(d, S, smem, ff, [&](int i, int pl, int n, const f32x4& v) { put(d.hplane[i] + pl, n, v); });
      last_conv<DIM, MODE, FEW>(d, S, smem, ff, apar, [&](int a, int n, float o0, float) {
        const int nf = half_site<DIM>(lat, a, fpar);
        float go0, gx;
        const float g = gy[n];
        affine_bwd(d.final_tanh, o0, xs[n], g, gld, go0, gx);
        gy[n] = gx;
        const f32x4 v{go0, g, 0.f, 0.f}, zero{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f32x4*>(go + 4 * n) = v;
        *reinterpret_cast<f32x4*>(go + 4 * nf) = zero;
        put(2 * HP, n, v);
        put(2 * HP, nf, zero);
      });
      if constexpr (LF) wait_copies();
      lds_barrier();
      const int ln = l > l0 ? l - 1 : l1 - 1;
      xpre = own ? xb[(size_t)ln * BV + threadIdx.x] : 0.f;
      if constexpr (LF) copy_frags(frags + (size_t)ln * d.frags_all * 64, smem + S.frags[0], F);
      // data gradients, last convolution to first; a hidden gradient takes the place of
      // its activation
      for (int i = d.n_conv - 1; i > 0; --i) {
        const ConvDir& c = d.t[i];
        const float* in = i + 1 == d.n_conv ? go : reinterpret_cast<const float*>(smem + S.slot[i]);
        float* h = reinterpret_cast<float*>(smem + S.slot[i - 1]);
        const int rows = c.rows;
        conv_pass<MODE, true, FEW>((V + 15) >> 4, c, ft + (c.off - F) * 64, red, [&](int tile) {
          return lds_planes<true>(d, nbr, S.ps, in, min(tile * 16 + m, V - 1));
        }, [&](int tile, int ct, const f32x4& acc) {
          const int n = tile * 16 + m, pl = ct * 4 + j;
          if (n < V && 4 * pl < rows) {
            f32x4* p = reinterpret_cast<f32x4*>(h + pl * S.ps + 4 * n);
            const f32x4 hv = *p;
            f32x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r)
              v[r] = masked(acc[r] * leaky_grad_from_out(hv[r]), (4 * pl + r - rows) >> 31);
            *p = v;
            put(HP + d.hplane[i - 1] + pl, n, v);
          }
        });
        lds_barrier();
      }
      {
        const int half = V / 2;
        const float* in = reinterpret_cast<const float*>(smem + S.slot[0]);
        const ConvDir& c = d.t[0];
        conv_pass<MODE, true, FEW>((half + 15) >> 4, c, ft + (c.off - F) * 64, red, [&](int tile) {
          return lds_planes<true>(d, nbr, S.ps, in, half_site<DIM>(lat, min(tile * 16 + m, half - 1), fpar));
        }, [&](int tile, int, const f32x4& acc) {
          const int a = tile * 16 + m;
          if (j == 0 && a < half) gy[half_site<DIM>(lat, a, fpar)] += acc[0];
        });
      }
      // the next layer's xs may be written at once: its readers are behind the barriers above
    }
    lds_barrier();
    for (int n = threadIdx.x; n < V; n += blockDim.x) g_out[(size_t)b * V + n] = gy[n];
    lds_barrier();
  }
  if constexpr (LF) wait_copies();  // none may land in the LDS of the next workgroup
}

// ---- staged kernels --------------------------------------------------------------

// log q = log r - the sum of the active sites' sums (one block per sample).
__global__ void __launch_bounds__(256) kg_end(int half, const double* __restrict__ ld, const double* __restrict__ logr,
                                              double* __restrict__ logq, double* __restrict__ logdet) {
  __shared__ double sh[16];
  const int b = blockIdx.x;
  double acc = 0;
  for (int a = threadIdx.x; a < half; a += blockDim.x) acc += ld[(size_t)b * half + a];
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) {
    logq[b] = logr[b] - acc;
    if (logdet) logdet[b] = acc;
  }
}

enum class Op { First, Hidden, Couple, Affine, Grad, GradField };

struct StagedArgs {
  int i, B, fpar;
  int ct0, ct1;      // row tiles of this launch; frags are theirs
  const float* in;   // planes of the input (sample stride in_ss floats), or the layer's field (i = 0 forward)
  size_t in_ss;
  float* out;        // planes of the output; Grad: over the gradients, h holds the activations
  size_t out_ss;
  const float* h;
  size_t h_ss;
  const float* x;    // Couple: the layer's field; Affine: likewise
  float* xout;       // Couple: the next field (may be x); Affine: g_x
  float* xout2;      // Couple: a second copy of the next field, or null
  double* ld;        // Couple: per active site sums of s, [B][V / 2]
  int first;         // Couple: the sums start here
  const float* gy;   // Affine: the cotangent of the layer's output; GradField: unused
  float gld;
  const double* gld_vec;
};

// One convolution of one layer over the whole batch: a workgroup takes 64 sites and a row
// tile, 16 sites a wave, of one sample after the other; the sites' neighbours and, where they
// fit (LF), the weights are laid out in its LDS once.
//   First      h = leaky(conv) of the masked field       all sites
//   Hidden     h = leaky(conv)                          all sites
//   Couple     the last convolution and the affine update   active sites
//   Affine     the last convolution and its affine backward  active sites
//   Grad       g_h = conv^T(g) leaky'(h)                all sites
//   GradField  g_x += conv^T(g)                         frozen sites
template <int DIM, int MODE, Op OP, bool LF>
__global__ void __launch_bounds__(256) kg_staged(NetDev d, StagedArgs A, const u32x4* frags) {
  constexpr bool TR = OP == Op::Grad || OP == Op::GradField;
  constexpr bool HALF = OP == Op::Couple || OP == Op::Affine || OP == Op::GradField;
  extern __shared__ __align__(16) unsigned char smem[];
  const Lat& lat = d.lat;
  const ConvDir c = TR ? d.t[A.i] : d.f[A.i];
  const int V = lat.V, half = V / 2, lane = threadIdx.x & 63, j = lane >> 4, m = lane & 15;
  const int sites = HALF ? half : V, par = OP == Op::GradField ? A.fpar : A.fpar ^ 1;
  const int groups = (sites + kTileSites - 1) / kTileSites, group = blockIdx.x % groups;
  auto site = [&](int k) {
    const int a = min(group * kTileSites + k, sites - 1);
    return HALF ? half_site<DIM>(lat, a, par) : a;
  };
  uint32_t* nbr = reinterpret_cast<uint32_t*>(smem);
  const int ct = blockIdx.y, k16 = fused::wave_id() * 16 + m, a = group * kTileSites + k16, n = site(k16);
  const bool valid = a < sites;
  Weights W{frags + (size_t)ct * c.per_ct() * 64, c.per_ct(), lane};
  if constexpr (LF) {
    copy_frags(W.frags, smem + tile_table_bytes(d.T), W.per_ct);
    W.frags = reinterpret_cast<const u32x4*>(smem + tile_table_bytes(d.T));
  }
  build_tile<DIM>(d, TR ? -1 : 1, OP == Op::First ? A.fpar : -1, nbr, site);
  if constexpr (LF) wait_copies();
  __syncthreads();
  for (int b = blockIdx.x / groups; b < A.B; b += gridDim.x / groups) {
    const f32x4 bias = __builtin_bit_cast(f32x4, W.at(0, -1));
    f32x4 acc;
    auto conv = [&](const auto& rd) {
      if constexpr (MODE == kTree) {
        acc = tree<false>(rd, c, W, 0, j, 0);
        if constexpr (!TR) acc += bias;
      } else {
        acc = chain<MODE, TR>(rd, c, W, 0, j, 0, c.nb, bias);
      }
    };
    if constexpr (OP == Op::First)
      conv(Field<false>{nbr + k16, A.in + (size_t)b * V, kTileSites, d.T});
    else
      conv(Planes<false, false>{nbr + k16, A.in + (size_t)b * A.in_ss, kTileSites, 4 * V, d.T});
    const int pl = (A.ct0 + ct) * 4 + j;
    if constexpr (OP == Op::First || OP == Op::Hidden || OP == Op::Grad) {
      if (valid && 4 * pl < c.rows) {
        f32x4 v, hv{};
        if (OP == Op::Grad) hv = *reinterpret_cast<const f32x4*>(A.h + (size_t)b * A.h_ss + ((size_t)pl * V + n) * 4);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          v[k] = masked(OP != Op::Grad ? leaky(acc[k]) : acc[k] * leaky_grad_from_out(hv[k]),
                        (4 * pl + k - c.rows) >> 31);
        *reinterpret_cast<f32x4*>(A.out + (size_t)b * A.out_ss + ((size_t)pl * V + n) * 4) = v;
      }
    } else if (valid && j == 0) {
      const size_t o = (size_t)b * V + n;
      if constexpr (OP == Op::GradField) {
        A.xout[o] += acc[0];
      } else {
        const size_t of = (size_t)b * V + half_site<DIM>(lat, a, A.fpar);
        if constexpr (OP == Op::Couple) {
          double* ld = A.ld + (size_t)b * half + a;
          const double l = A.first ? 0.0 : *ld;
          const float sv = d.final_tanh ? tanhf(acc[0]) : acc[0];
          const float xn = A.x[o] * expf(sv) + acc[1], xf = A.x[of];
          A.xout[o] = xn;
          if (A.xout != A.x) A.xout[of] = xf;
          if (A.xout2) A.xout2[o] = xn, A.xout2[of] = xf;
          *ld = l + (double)sv;
        } else {
          float go0, gx;
          const float g = A.gy[o];
          affine_bwd(d.final_tanh, acc[0], A.x[o], g, A.gld_vec ? (float)(-A.gld_vec[b]) : A.gld, go0, gx);
          A.xout[o] = gx;
          A.xout[of] = A.gy[of];
          float* go = A.out + (size_t)b * A.out_ss;
          *reinterpret_cast<f32x4*>(go + 4 * n) = f32x4{go0, g, 0.f, 0.f};
          *reinterpret_cast<f32x4*>(go + 4 * half_site<DIM>(lat, a, A.fpar)) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
  }
}

// ---- host ------------------------------------------------------------------------

// Whether B samples are run by the resident kernels: a sample's forward (backward) state has
// to fit the LDS (the neighbour table holds 16-bit sites).  In FP32, where the staged kernels
// give the same bits, they take over where most CUs would be idle and a sample is many tiles
// to eight waves.  8 layers, resident and staged, us forward (backward):
//   34 x 34, hidden [4], 1 sample 149 and 82 (385 and 173), 64 150 and 136 (460 and 385), 128
//     150 and 187 (518 and 607)
//   24 x 24, hidden [16, 16, 16], 16 samples 276 and 185 (691 and 491), 64 274 and 272 (877
//     and 839); [8, 8], kernel 3, 16 samples 109 and 126 (316 and 298)
//   20 x 20, hidden [16, 16], kernel 3, 16 samples 117 and 137 (311 and 312)
bool resident(const NetDev& d, int B, bool bwd) {
  int widest = 0;
  for (int i = 0; i + 1 < d.n_conv; ++i) widest = std::max(widest, d.cout[i]);
  const int V = d.lat.V, few = V >= 900 || (bwd && widest >= 12) ? 64 : bwd || widest >= 12 ? 16 : 0;
  if (d.mode != kBf16 && V >= 512 && B <= few) return false;
  return V < 65536 && (size_t)res_lds(d, bwd).total <= kLdsMax;
}

size_t frag_bytes(const NetDev& d, bool bwd) {
  return (size_t)d.N * (bwd ? d.frags_all : d.frags_fwd) * 1024;
}

// Workgroups of a resident launch.  A sample per CU or less: eight waves each, whose latency is
// what counts.  More: the number of waves per workgroup, and fragments in LDS or read from the
// L2, that give a CU the most waves with a unit of their own, within its LDS, the registers
// (12 to 24 waves) and its share of the samples; of as many, fragments in LDS first, then
// the smaller workgroups.  Forward of 8 layers, hidden 8, FP32, 4096 samples of 4 x 4: 422 us
// with eight waves and one workgroup a CU, 65 with one wave and 16; of 6 x 6: 427 and 121; 523
// of 24 x 24: 301, 237 with two workgroups whose fragments stay in the L2.  The sums' orders do
// not depend on it.
struct ResGrid {
  ResLds S;
  int waves, blocks;
};
ResGrid res_grid(const NetDev& d, int B, bool bwd) {
  const int cus = num_cus(), per = cdiv(B, cus);
  ResGrid best{res_lds(d, bwd), kResWaves, std::min(B, cus)};
  if (per == 1) return best;
  int units = 1;
  for (int i = 0; i < d.n_conv; ++i)
    units = std::max(units, cdiv(d.lat.V, 16) * std::max(d.f[i].nct, bwd ? d.t[i].nct : 0));
  // (in BF16 eight waves share a CU's few units; with many samples they are better apart)
  const bool apart = d.mode != kBf16 || per >= 8;
  const int cap = d.mode == kTree ? (bwd ? 16 : 12) : d.mode == kBf16 && !bwd ? 20 : 24;
  int most = 0;
  for (const bool lf : {true, false})
    for (int waves = 1; waves <= kResWaves; waves *= 2) {
      const ResLds S = res_lds(d, bwd, waves, lf);
      if ((size_t)S.total > kLdsMax || (lf && !S.lf)) continue;
      const int wgs = std::min({per, std::max(1, cap / waves), 160 * 1024 / (S.total + 1024)});
      const int busy = wgs * (apart ? std::min(waves, units) : waves);
      if (busy <= most) continue;
      most = busy;
      best = ResGrid{S, waves, std::min(B, cus * wgs)};
    }
  return best;
}

struct BwdWs {
  u32x4* frags;
  float *gA, *gB, *store;
  double* partial;
};
BwdWs carve_bwd(const NetDev& d, int B, char* base, size_t* total) {
  BwdWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align_up(bytes);
    return p;
  };
  const size_t BV = (size_t)B * d.lat.V;
  const int group = layer_group(d, B, store_planes(d));
  w.frags = (u32x4*)take(frag_bytes(d, true));
  w.gA = (float*)take(4 * BV);
  w.gB = (float*)take(4 * BV);
  w.store = (float*)take((size_t)group * B * store_planes(d) * d.lat.V * 16);
  w.partial = (double*)take(partial_bytes(d, B, group, store_planes(d)));
  *total = off;
  return w;
}

// Where a staged convolution's fragments come from: prepared for all layers (count
// per layer), or, with count = 0, prepared launch by launch into room bytes.
struct FragSrc {
  u32x4* buf;
  int count;
  size_t room;
  const float* params;
};

template <int DIM, int MODE, Op OP>
int32_t staged(const NetDev& d, StagedArgs a, int layer, const FragSrc& src, hipStream_t st) {
  constexpr bool TR = OP == Op::Grad || OP == Op::GradField;
  const ConvDir& c = TR ? d.t[a.i] : d.f[a.i];
  const size_t one = (size_t)c.per_ct() * 1024;  // a row tile's fragments
  const int step = src.count ? c.nct : (int)std::min<size_t>(c.nct, src.room / one);
  if (step < 1) return LFS_EWORKSPACE;
  for (int ct = 0; ct < c.nct; ct += step) {
    a.ct0 = ct;
    a.ct1 = std::min(ct + step, c.nct);
    const int nct = a.ct1 - a.ct0;
    const u32x4* frags = src.buf;
    if (src.count)
      frags += ((size_t)layer * src.count + c.off) * 64;
    else
      prep<MODE>(d, src.params + (size_t)layer * d.P_layer, 1, c.off + ct * c.per_ct(), nct * c.per_ct(), src.buf, st);
    const int tab = tile_table_bytes(d.T);
    const bool lf = tab + one <= 78 * 1024;  // two workgroups per CU
    const int lds = tab + (lf ? (int)one : 0);
    const bool half = OP == Op::Couple || OP == Op::Affine || OP == Op::GradField;
    // as many workgroups as the chip holds at once, each with an equal number of samples
    const int groups = cdiv(half ? d.lat.V / 2 : d.lat.V, kTileSites);
    const int64_t fit = (int64_t)num_cus() * std::min(6, 158 * 1024 / lds) / ((int64_t)groups * nct);
    const int per = cdiv(a.B, (int)std::max<int64_t>(1, std::min<int64_t>(fit, a.B)));
    const dim3 grid((unsigned)(groups * cdiv(a.B, per)), (unsigned)nct);
    LFS_TRY(with_lf(lf, [&](auto l) {
      constexpr auto k = kg_staged<DIM, MODE, OP, decltype(l)::value>;
      if (!set_lds_limit<k>(kLdsMax)) return (int32_t)LFS_EDEVICE;
      hipLaunchKernelGGL(k, grid, dim3(256), lds, st, d, a, frags);
      return (int32_t)LFS_OK;
    }));
  }
  return LFS_OK;
}

// Bytes of the staged forward of B samples beside the fragments: log r, the log-det
// sums of the active sites and the hidden activations (two sets of planes, the
// convolutions alternating between them).
struct StagedWs {
  double *logr, *ld;
  float* planes[2];
  size_t bytes;
};
StagedWs staged_ws(const NetDev& d, int B, char* base) {
  StagedWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align_up(bytes);
    return p;
  };
  const size_t BV = (size_t)B * d.lat.V;
  int q[2] = {0, 0};
  for (int i = 0; i + 1 < d.n_conv; ++i) q[i & 1] = std::max(q[i & 1], cdiv(d.cout[i], 4));
  w.logr = (double*)take(sizeof(double) * B);
  w.ld = (double*)take(sizeof(double) * (BV / 2));
  for (int k = 0; k < 2; ++k) w.planes[k] = (float*)take(BV * 16 * q[k]);
  w.bytes = off;
  return w;
}

// The staged forward of samples [0, B) of arrays whose layers are BV_all floats apart.
template <int DIM, int MODE>
int32_t forward_staged(const FlowGeom& g, const NetDev& d, int B, const float* z, float* phi, double* logq,
                       double* logdet, float* saved, size_t BV_all, const StagedWs& w, const FragSrc& src,
                       hipStream_t st) {
  using R = std::conditional_t<MODE == kBf16, double, float>;
  const int V = g.V;
  float* x = saved ? saved : phi;
  hipLaunchKernelGGL((kg_begin<R>), dim3(B), dim3(256), 0, st, V, z, x, w.logr);
  for (int l = 0; l < d.N; ++l) {
    float* xn = saved ? saved + (size_t)(l + 1) * BV_all : phi;
    StagedArgs a{};
    a.B = B;
    a.fpar = g.frozen_parity(l);
    for (int i = 0; i < d.n_conv; ++i) {
      a.i = i;
      a.in = i == 0 ? x : w.planes[(i - 1) & 1];
      a.in_ss = i == 0 ? 0 : (size_t)cdiv(d.cout[i - 1], 4) * V * 4;
      if (i + 1 < d.n_conv) {
        a.out = w.planes[i & 1];
        a.out_ss = (size_t)cdiv(d.cout[i], 4) * V * 4;
        LFS_TRY(i == 0 ? (staged<DIM, MODE, Op::First>(d, a, l, src, st))
                       : (staged<DIM, MODE, Op::Hidden>(d, a, l, src, st)));
      }
    }
    a.x = x;
    a.xout = xn;
    a.xout2 = saved && l + 1 == d.N ? phi : nullptr;
    a.ld = w.ld;
    a.first = l == 0;
    LFS_TRY((staged<DIM, MODE, Op::Couple>(d, a, l, src, st)));
    x = xn;
  }
  hipLaunchKernelGGL(kg_end, dim3(B), dim3(256), 0, st, V / 2, w.ld, w.logr, logq, logdet);
  return launch_status();
}

template <int DIM, int MODE>
int32_t forward_impl(const FlowGeom& g, const float* params, int B, const float* z, float* phi, double* logq,
                     double* logdet, float* saved, char* ws, size_t ws_bytes, hipStream_t st) {
  const NetDev d = make_net(g);
  const size_t fb = frag_bytes(d, false), BV = (size_t)B * g.V;
  // the static scratch may be smaller than general_ws_bytes
  if (resident(d, B, false)) {
    const ResGrid R = res_grid(d, B, false);
    const size_t layer = (size_t)d.frags_fwd * 1024, cb = align_up(sizeof(double) * (BV / 2));
    const bool whole = ws_bytes >= fb;
    const int group = whole ? d.N : ws_bytes < cb ? 0 : (int)std::min<size_t>(d.N, (ws_bytes - cb) / layer);
    double* carry = whole ? nullptr : reinterpret_cast<double*>(ws);
    u32x4* frags = reinterpret_cast<u32x4*>(ws + (whole ? 0 : cb));
    for (int l0 = 0; group > 0 && l0 < d.N; l0 += group) {
      const int l1 = std::min(l0 + group, d.N);
      prep<MODE>(d, params + (size_t)l0 * d.P_layer, l1 - l0, 0, d.frags_fwd, frags, st);
      LFS_TRY(with_lf(R.S.lf, R.waves < kResWaves, [&](auto lf, auto few) {
        constexpr auto k = kg_forward<DIM, MODE, decltype(lf)::value, decltype(few)::value>;
        if (!set_lds_limit<k>(kLdsMax)) return (int32_t)LFS_EDEVICE;
        hipLaunchKernelGGL(k, dim3((unsigned)R.blocks), dim3(64 * R.waves), R.S.total, st, d, R.S, frags,
                           l0, l1, B, l0 > 0 ? phi : z, phi, saved, logq, logdet, carry);
        return launch_status();
      }));
    }
    if (group > 0) return LFS_OK;
  } else if (ws_bytes >= fb + staged_ws(d, B, nullptr).bytes) {
    u32x4* frags = reinterpret_cast<u32x4*>(ws);
    prep<MODE>(d, params, d.N, 0, d.frags_fwd, frags, st);
    return forward_staged<DIM, MODE>(g, d, B, z, phi, logq, logdet, saved, BV, staged_ws(d, B, ws + fb),
                                     FragSrc{frags, d.frags_fwd, fb, params}, st);
  }
  // no room for a layer's fragments (FP32: the sums' order is that of the resident kernels),
  // or for the whole batch's activations: the staged kernels on as many samples at a time as
  // leave room for a row tile's fragments
  size_t one = 0;
  for (int i = 0; i < d.n_conv; ++i) one = std::max(one, (size_t)d.f[i].per_ct() * 1024);
  int step = B;
  while (step > 1 && staged_ws(d, step, nullptr).bytes + one > ws_bytes) step = (step + 1) / 2;
  const StagedWs w = staged_ws(d, step, ws);
  if (w.bytes + one > ws_bytes) return LFS_EWORKSPACE;
  const FragSrc src{reinterpret_cast<u32x4*>(ws + w.bytes), 0, ws_bytes - w.bytes, params};
  for (int b = 0; b < B; b += step) {
    const size_t o = (size_t)b * g.V;
    LFS_TRY((forward_staged<DIM, MODE>(g, d, std::min(step, B - b), z + o, phi + o, logq + b,
                                       logdet ? logdet + b : nullptr, saved ? saved + o : nullptr, BV, w, src, st)));
  }
  return LFS_OK;
}

template <int DIM, int MODE>
int32_t backward_impl(const FlowGeom& g, const float* params, int B, const float* saved, const float* g_phi,
                      double g_logq, const double* g_logq_vec, float* g_params, float* g_z, char* ws,
                      hipStream_t st) {
  const NetDev d = make_net(g);
  const int V = g.V, PL = store_planes(d), HP = d.hplanes, group = layer_group(d, B, PL);
  const size_t BV = (size_t)B * V, ss = (size_t)PL * V * 4;
  size_t total;
  const BwdWs w = carve_bwd(d, B, ws, &total);
  prep<MODE>(d, params, d.N, 0, d.frags_all, w.frags, st);
  const FragSrc src{w.frags, d.frags_all, frag_bytes(d, true), params};
  const bool res = resident(d, B, true);
  const float* gy = g_phi;
  float* bufs[2] = {w.gA, w.gB};
  int which = 0;
  for (int l1 = d.N; l1 > 0;) {
    const int l0 = l1 > group ? l1 - group : 0;
    if (res) {
      const ResGrid R = res_grid(d, B, true);
      float* gx = bufs[which];
      LFS_TRY(with_lf(R.S.lf, R.waves < kResWaves, [&](auto lf, auto few) {
        constexpr auto k = kg_backward<DIM, MODE, decltype(lf)::value, decltype(few)::value>;
        if (!set_lds_limit<k>(kLdsMax)) return (int32_t)LFS_EDEVICE;
        hipLaunchKernelGGL(k, dim3((unsigned)R.blocks), dim3(64 * R.waves), R.S.total, st, d, R.S, w.frags,
                           B, l0, l1, saved, gy, (float)(-g_logq), g_logq_vec, gx, w.store);
        return (int32_t)LFS_OK;
      }));
      gy = gx;
      which ^= 1;
    } else {
      for (int l = l1 - 1; l >= l0; --l) {
        float* gx = bufs[which];
        float* st_l = w.store + (size_t)(l - l0) * B * ss;
        auto plane = [&](int p) { return st_l + (size_t)p * V * 4; };
        StagedArgs a{};
        a.B = B;
        a.fpar = g.frozen_parity(l);
        a.in_ss = a.out_ss = a.h_ss = ss;
        for (int i = 0; i + 1 < d.n_conv; ++i) {
          a.i = i;
          a.in = i == 0 ? saved + (size_t)l * BV : plane(d.hplane[i - 1]);
          a.out = plane(d.hplane[i]);
          LFS_TRY(i == 0 ? (staged<DIM, MODE, Op::First>(d, a, l, src, st))
                         : (staged<DIM, MODE, Op::Hidden>(d, a, l, src, st)));
        }
        a.i = d.n_conv - 1;
        a.in = plane(d.hplane[a.i - 1]);
        a.out = plane(2 * HP);
        a.x = saved + (size_t)l * BV;
        a.xout = gx;
        a.gy = gy;
        a.gld = (float)(-g_logq);
        a.gld_vec = g_logq_vec;
        LFS_TRY((staged<DIM, MODE, Op::Affine>(d, a, l, src, st)));
        for (int i = d.n_conv - 1; i > 0; --i) {
          a.i = i;
          a.in = i + 1 == d.n_conv ? plane(2 * HP) : plane(HP + d.hplane[i]);
          a.out = plane(HP + d.hplane[i - 1]);
          a.h = plane(d.hplane[i - 1]);
          LFS_TRY((staged<DIM, MODE, Op::Grad>(d, a, l, src, st)));
        }
        a.i = 0;
        a.in = plane(HP);
        LFS_TRY((staged<DIM, MODE, Op::GradField>(d, a, l, src, st)));
        gy = gx;
        which ^= 1;
      }
    }
    LFS_TRY((run_wgrad<DIM, MODE>(d, B, l0, l1 - l0, PL, w.store, saved, w.partial, g_params, st)));
    l1 = l0;
  }
  if (g_z)
    hipLaunchKernelGGL(kg_gz, dim3(blocks((int64_t)BV)), dim3(256), 0, st, (int64_t)BV, gy, saved, (float)g_logq,
                       g_logq_vec, (int64_t)V, g_z);
  return launch_status();
}

// f(integral constants of the dimension and the mode).
template <class F>
int32_t dispatch(const FlowGeom& g, F&& f) {
  auto mode = [&](auto dim) {
    if (g.bf16()) return f(dim, std::integral_constant<int, kBf16>{});
    if (g.net_default) return f(dim, std::integral_constant<int, kSeq>{});
    return f(dim, std::integral_constant<int, kTree>{});
  };
  return g.dim == 2 ? mode(std::integral_constant<int, 2>{}) : mode(std::integral_constant<int, 3>{});
}

}  // namespace

size_t general_ws_bytes(const FlowGeom& g, int B, int for_backward) {
  const NetDev d = make_net(g);
  if (!for_backward)
    return kWsAlign + frag_bytes(d, false) + (resident(d, B, false) ? 0 : staged_ws(d, B, nullptr).bytes);
  size_t total;
  carve_bwd(d, B, nullptr, &total);
  return kWsAlign + total;
}

int32_t general_forward(const FlowGeom& g, const float* params, int B, const float* z, float* phi, double* logq,
                        double* logdet, float* saved, char* ws, size_t ws_bytes, hipStream_t st) {
  ws = aligned_ws(ws, &ws_bytes);
  return dispatch(g, [&](auto dim, auto mode) {
    return forward_impl<decltype(dim)::value, decltype(mode)::value>(g, params, B, z, phi, logq, logdet, saved, ws,
                                                                     ws_bytes, st);
  });
}

int32_t general_backward(const FlowGeom& g, const float* params, int B, const float* saved, const float* g_phi,
                         double g_logq, const double* g_logq_vec, float* g_params, float* g_z, char* ws,
                         hipStream_t st) {
  size_t unused = kWsAlign;
  ws = aligned_ws(ws, &unused);
  return dispatch(g, [&](auto dim, auto mode) {
    return backward_impl<decltype(dim)::value, decltype(mode)::value>(g, params, B, saved, g_phi, g_logq, g_logq_vec,
                                                                      g_params, g_z, ws, st);
  });
}

}  // namespace lfs
