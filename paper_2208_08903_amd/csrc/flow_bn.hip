// Batch-norm flows (the parameter file's use_bn) whose sample fits the LDS: one launch per
// convolution and direction, a workgroup per sample, with everything between two
// convolutions folded into the launches on its sides.
//
// Batch statistics couple the samples at every hidden convolution, so a launch is the
// shortest unit of the chain; what can be saved is the number of launches.  A forward
// launch first merges the per-workgroup sums that the previous one left (each workgroup
// all of them: a few KB), normalises the sample's activations on their way into LDS,
// convolves, and leaves the sums of its own outputs; the last one of a layer also makes
// the affine update or its backward.  A backward launch likewise turns g_y into g_a on its
// way in and leaves the sums the next one needs.  Per layer of n convolutions that is n
// launches forward and 2 n backward where one operation per launch took 5 n - 2 and
// 11 n - 8.  2D L = 8, hidden [8, 8], 16 layers, batch 64, FP32 training step: 2877 -> 930 us.
//
// Statistics are FP64: per sample the sum and the squared deviations from the sample's
// own mean, merged by count (Chan, Golub and LeVeque's update) in a fixed order.
#include "general_wgrad.hpp"

namespace lfs {
namespace {

constexpr double kBnEps = 1e-5;
constexpr int kMaxC = 64;  // hidden_sizes entries are at most 64

__device__ __forceinline__ float bn_xhat(float a, double mean, double r) { return (float)(((double)a - mean) * r); }

// LDS of a workgroup, byte offsets: the masked field, the input and output planes of a
// convolution, tables, per-channel numbers and the convolution's fragments (lf).
struct BnLds {
  int ps, xs, in, out, red, nbr, st, ab, frags, total;
  bool lf;
};
BnLds bn_lds(const NetDev& d) {
  BnLds r{};
  const int V = d.lat.V;
  r.ps = lds_plane_stride(V);
  int64_t off = 0;
  auto take = [&](int64_t bytes) {
    const int64_t o = off;
    off += (bytes + 15) / 16 * 16;
    return (int)std::min<int64_t>(o, 1 << 30);
  };
  int q = 1, f = 0;
  for (int i = 0; i < d.n_conv; ++i) {
    if (i + 1 < d.n_conv) q = std::max(q, cdiv(d.cout[i], 4));
    f = std::max(f, std::max(d.f[i].nct * d.f[i].per_ct(), d.t[i].nct * d.t[i].per_ct()));
  }
  r.xs = take(4ll * (V + 1));
  r.in = take(4ll * r.ps * q);
  r.out = take(4ll * r.ps * q);
  r.red = take(1024ll * kResWaves);
  r.nbr = take(nbr_bytes(d.T, V));
  r.st = take(8ll * 6 * kMaxC);
  r.ab = take(4ll * 2 * kMaxC);
  r.lf = off + f * 1024ll <= (int64_t)kLdsMax;
  if (r.lf) r.frags = take(f * 1024ll);
  r.total = (int)std::min<int64_t>(off, 1 << 30);
  return r;
}

template <int DIM>
__device__ __forceinline__ void bn_tables(const NetDev& d, const BnLds& S, unsigned char* smem) {
  build_nbr<DIM>(d, reinterpret_cast<uint16_t*>(smem + S.nbr));
  const int V = d.lat.V;
  if (threadIdx.x == 0) reinterpret_cast<float*>(smem + S.xs)[V] = 0.f;
  const int q = (S.out - S.in) / (4 * S.ps);
  for (int k = threadIdx.x; k < 4 * q; k += blockDim.x)
    reinterpret_cast<float*>(smem + S.in)[(k >> 2) * S.ps + 4 * V + (k & 3)] = 0.f;
}

// The sites of workgroup g's samples when G workgroups take B samples in turn.
__device__ __forceinline__ double wg_sites(int g, int G, int B, int V) { return (double)((B - g + G - 1) / G) * V; }

// How hidden activation i - 1 is normalised on its way into convolution i.
struct BnIn {
  int batch;                       // statistics of the batch, else running
  const float* running;            // running: mean[c], var[c]
  float* update;                   // batch: running statistics to update, or null
  float momentum;
  const float *gamma, *beta;
  double inv_n, inv_cnt[2];        // 1 / (B V), 1 / wg_sites of the first workgroup and of the last
  const double* part;              // batch: sums of the previous launch, s[c][G] then m2[c][G]
  double* mr;                      // mean[c], r[c] for later launches
};

// Loads one value per thread of a buffer that the kernel's end will read, so that it is in
// the L1 by then; keep() takes the values where their latency has passed.
__device__ __forceinline__ float touch(const float* p, int n) { return threadIdx.x < n ? p[threadIdx.x] : 0.f; }
__device__ __forceinline__ void keep(float a, float b) { asm volatile("" ::"v"(a), "v"(b)); }

// The sums of this wave's first channel, one workgroup's per lane (loaded early).
struct BnPart {
  double a, b;
};
__device__ __forceinline__ BnPart first_part(const double* part, int c, int G) {
  const int lane = threadIdx.x & 63, ch = threadIdx.x >> 6;
  BnPart p{0.0, 0.0};
  if (ch < c && lane < G) {
    p.a = part[ch * G + lane];
    p.b = part[(c + ch) * G + lane];
  }
  return p;
}

// mean and r = 1 / sqrt(var + eps) of c channels into ms, a wave per channel.  The squared
// deviations are taken from the first workgroup's mean and moved to the mean afterwards,
// so that one pass sums both (the two differ by the spread of a workgroup's mean, a
// fraction of the standard deviation: nothing cancels).
__device__ __forceinline__ void bn_merge(const BnIn& in, BnPart p, int c, int G, int B, int V, double* ms) {
  const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const double n = (double)B * V;
  for (int ch = fused::wave_id(); ch < c; ch += nw) {
    double mu, var;
    if (in.batch) {
      double s = 0.0, sq = 0.0, pivot = 0.0;
      for (int g0 = 0; g0 < G; g0 += 64) {
        const int g = g0 + lane;
        if (ch >= nw || g0 > 0) {
          p.a = g < G ? in.part[ch * G + g] : 0.0;
          p.b = g < G ? in.part[(c + ch) * G + g] : 0.0;
        }
        const double cnt = wg_sites(min(g, G - 1), G, B, V);
        const double mg = p.a * (min(g, G - 1) <= (B - 1) % G ? in.inv_cnt[0] : in.inv_cnt[1]);
        if (g0 == 0) pivot = __longlong_as_double(__shfl(__double_as_longlong(mg), 0, 64));
        const double dev = mg - pivot;
        s += p.a;
        sq += g < G ? p.b + cnt * dev * dev : 0.0;
      }
      s = wave_sum(s);
      sq = wave_sum(sq);
      mu = s * in.inv_n;
      var = sq * in.inv_n - (mu - pivot) * (mu - pivot);
    } else {
      mu = (double)in.running[ch];
      var = (double)in.running[c + ch];
    }
    if (lane == 0) {
      const double r = rsqrt(var + kBnEps);
      ms[ch] = mu;
      ms[kMaxC + ch] = r;
      if (blockIdx.x == 0) {
        in.mr[ch] = mu;
        in.mr[c + ch] = r;
        if (in.batch && in.update) {
          const double m = (double)in.momentum;
          in.update[ch] = (float)((1.0 - m) * (double)in.update[ch] + m * mu);
          in.update[c + ch] = (float)((1.0 - m) * (double)in.update[c + ch] + m * var * (n / (n - 1.0)));
        }
      }
    }
  }
}

enum class Kind { Hidden, Couple, Affine };

struct BnConvArgs {
  int i, B, fpar;
  BnIn in;
  double* part;         // Hidden: this launch's sums
  const float* x;       // the layer's field
  float* store;         // planes of every sample, ss floats apart
  size_t ss;
  int ain, hin, aout;   // planes: input a, where the normalised input goes (-1: nowhere), output a
  float *xout, *xout2;  // Couple: the next field, and a second copy or null; Affine: g_x
  double* ld;           // Couple: the layer's log-det per sample
  const float* gy;      // Affine: the cotangent of the layer's output
  float gld;
  const double* gld_vec;
  int go;               // Affine: plane of g_o
};

template <int DIM, int MODE, bool LF, bool FEW, Kind KIND>
__global__ void __launch_bounds__(64 * kResWaves) kb_conv(NetDev d, BnLds S, BnConvArgs A, const u32x4* frags) {
  extern __shared__ __align__(16) unsigned char smem[];
  const Lat& lat = d.lat;
  const ConvDir& c = d.f[A.i];
  const int V = lat.V, half = V / 2, lane = threadIdx.x & 63, j = lane >> 4, m = lane & 15, w = fused::wave_id(),
            nw = blockDim.x >> 6, G = gridDim.x;
  float* xs = reinterpret_cast<float*>(smem + S.xs);
  float* in = reinterpret_cast<float*>(smem + S.in);
  float* out = reinterpret_cast<float*>(smem + S.out);
  f32x4* red = reinterpret_cast<f32x4*>(smem + S.red);
  const uint16_t* nbr = reinterpret_cast<const uint16_t*>(smem + S.nbr);
  double* ms = reinterpret_cast<double*>(smem + S.st);  // mean, r of the input channels
  double* acc = ms + 2 * kMaxC;                         // s, m2 of the output channels
  if constexpr (LF) {
    copy_frags(frags, smem + S.frags, c.nct * c.per_ct());
    frags = reinterpret_cast<const u32x4*>(smem + S.frags);
  }
  const int cin = c.ck, cout = c.rows, qin = (cin + 3) >> 2;
  // what the first sample's normalisation reads is under way while the statistics are
  // merged: gamma and beta, and the thread's first quad
  float* ab = reinterpret_cast<float*>(smem + S.ab);
  f32x4 pre{};
  float ga = 0.f, be = 0.f, t0 = 0.f, t1 = 0.f;
  BnPart part{0.0, 0.0};
  if (A.i > 0) {
    if (A.in.batch) part = first_part(A.in.part, cin, G);
    if (threadIdx.x < cin) {
      ga = A.in.gamma[threadIdx.x];
      be = A.in.beta[threadIdx.x];
    }
    if (threadIdx.x < qin * V)
      pre = *reinterpret_cast<const f32x4*>(A.store + (size_t)blockIdx.x * A.ss + ((size_t)A.ain * V + threadIdx.x) * 4);
  }
  t0 = touch(A.x + (size_t)blockIdx.x * V, V);
  if constexpr (KIND == Kind::Affine) t1 = touch(A.gy + (size_t)blockIdx.x * V, V);
  bn_tables<DIM>(d, S, smem);
  keep(t0, t1);
  if (A.i > 0) {
    if (threadIdx.x < cin) {
      ab[threadIdx.x] = ga;
      ab[kMaxC + threadIdx.x] = be;
    }
    bn_merge(A.in, part, cin, G, A.B, V, ms);
  }
  __syncthreads();
  if constexpr (LF) wait_copies();
  for (int b = blockIdx.x, k = 0; b < A.B; b += G, ++k) {
    float* st = A.store + (size_t)b * A.ss;
    const float* xb = A.x + (size_t)b * V;
    if (A.i == 0) {
      for (int n = threadIdx.x; n < V; n += blockDim.x)
        xs[n] = masked(xb[n], (parity_of<DIM>(site_of<DIM>(lat, n)) ^ A.fpar) - 1);
    } else {
      for (int e = threadIdx.x; e < qin * V; e += blockDim.x) {
        const int q = fdiv(e, lat.dV), n = e - q * V;
        f32x4 a = pre, h;
        if (k > 0 || e >= blockDim.x)
          a = *reinterpret_cast<const f32x4*>(st + ((size_t)(A.ain + q) * V + n) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ch = min(4 * q + r, cin - 1);
          const float y = ab[ch] * bn_xhat(a[r], ms[ch], ms[kMaxC + ch]) + ab[kMaxC + ch];
          h[r] = masked(leaky(y), (4 * q + r - cin) >> 31);
        }
        *reinterpret_cast<f32x4*>(in + q * S.ps + 4 * n) = h;
        if (A.hin >= 0) *reinterpret_cast<f32x4*>(st + ((size_t)(A.hin + q) * V + n) * 4) = h;
      }
    }
    lds_barrier();
    if constexpr (KIND == Kind::Hidden) {
      auto epi = [&](int tile, int ct, const f32x4& v) {
        const int n = tile * 16 + m, pl = ct * 4 + j;
        if (n < V && 4 * pl < cout) {
          f32x4 a;
#pragma unroll
          for (int r = 0; r < 4; ++r) a[r] = masked(v[r], (4 * pl + r - cout) >> 31);
          *reinterpret_cast<f32x4*>(out + pl * S.ps + 4 * n) = a;
          *reinterpret_cast<f32x4*>(st + ((size_t)(A.aout + pl) * V + n) * 4) = a;
        }
      };
      if (A.i == 0) {
        conv_pass<MODE, false, FEW>((V + 15) >> 4, c, frags, red, [&](int tile) {
          return lds_field(d, nbr, xs, min(tile * 16 + m, V - 1));
        }, epi);
      } else {
        conv_pass<MODE, false, FEW>((V + 15) >> 4, c, frags, red, [&](int tile) {
          return lds_planes<false>(d, nbr, S.ps, in, min(tile * 16 + m, V - 1));
        }, epi);
      }
      lds_barrier();
      for (int ch = w; ch < cout; ch += nw) {
        const float* a = out + (ch >> 2) * S.ps + (ch & 3);
        double s = 0.0, sq = 0.0;
        for (int n = lane; n < V; n += 64) s += (double)a[4 * n];
        s = wave_sum(s);
        const double mu = s / V;
        for (int n = lane; n < V; n += 64) {
          const double t = (double)a[4 * n] - mu;
          sq += t * t;
        }
        sq = wave_sum(sq);
        if (lane == 0) {
          if (k > 0) {
            const double n1 = (double)k * V, dev = mu - acc[ch] / n1;
            sq += acc[kMaxC + ch] + dev * dev * (n1 * V / (n1 + V));
            s += acc[ch];
          }
          acc[ch] = s;
          acc[kMaxC + ch] = sq;
        }
      }
    } else {
      const size_t o = (size_t)b * V;
      const int apar = A.fpar ^ 1;
      const float gld = KIND == Kind::Affine && A.gld_vec ? (float)(-A.gld_vec[b]) : A.gld;
      conv_pass<MODE, false, FEW>((half + 15) >> 4, c, frags, red, [&](int tile) {
        return lds_planes<false>(d, nbr, S.ps, in, half_site<DIM>(lat, min(tile * 16 + m, half - 1), apar));
      }, [&](int tile, int, const f32x4& v) {
        const int a = tile * 16 + m;
        if (j != 0 || a >= half) return;
        const int n = half_site<DIM>(lat, a, apar), nf = half_site<DIM>(lat, a, A.fpar);
        if constexpr (KIND == Kind::Couple) {
          const float s = d.final_tanh ? tanhf(v[0]) : v[0];
          const float xn = xb[n] * expf(s) + v[1], xf = xb[nf];
          out[a] = s;
          A.xout[o + n] = xn;
          if (A.xout != A.x) A.xout[o + nf] = xf;
          if (A.xout2) A.xout2[o + n] = xn, A.xout2[o + nf] = xf;
        } else {
          float go0, gx;
          const float g = A.gy[o + n];
          affine_bwd(d.final_tanh, v[0], xb[n], g, gld, go0, gx);
          A.xout[o + n] = gx;
          A.xout[o + nf] = A.gy[o + nf];
          float* go = st + (size_t)A.go * V * 4;
          *reinterpret_cast<f32x4*>(go + 4 * n) = f32x4{go0, g, 0.f, 0.f};
          *reinterpret_cast<f32x4*>(go + 4 * nf) = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      });
      if constexpr (KIND == Kind::Couple) {
        lds_barrier();
        if (w == 0) {
          const double ld = sum_of_256<double>(half, [&](int a) { return (double)out[a]; });
          if (lane == 0) A.ld[b] = ld;
        }
      }
    }
    lds_barrier();
  }
  if constexpr (KIND == Kind::Hidden)
    for (int ch = threadIdx.x; ch < cout; ch += blockDim.x) {
      A.part[ch * G + blockIdx.x] = acc[ch];
      A.part[(cout + ch) * G + blockIdx.x] = acc[kMaxC + ch];
    }
}

struct BnGradArgs {
  int i, B, fpar, batch;
  // normalisation of hidden activation i (not of the last convolution's output): its
  // mean and r, gamma, the previous launch's sums of g xhat and g, their gradients
  const double *mr, *part;
  const float* gamma;
  float* gg;
  float* store;
  size_t ss;
  int gin, ain;               // planes: gradient of convolution i's output, a of hidden i
  int gout, hout, aout;       // planes of hidden i - 1: gradient, h, a
  const double* mr_out;       // its mean and r
  double* part_out;           // and the sums of this launch
  float* gx;                  // i = 0: the field's gradient
};

template <int DIM, int MODE, bool LF, bool FEW, bool FIELD>
__global__ void __launch_bounds__(64 * kResWaves) kb_grad(NetDev d, BnLds S, BnGradArgs A, const u32x4* frags) {
  extern __shared__ __align__(16) unsigned char smem[];
  const Lat& lat = d.lat;
  const ConvDir& c = d.t[A.i];
  const int V = lat.V, half = V / 2, lane = threadIdx.x & 63, j = lane >> 4, m = lane & 15, w = fused::wave_id(),
            nw = blockDim.x >> 6, G = gridDim.x;
  float* in = reinterpret_cast<float*>(smem + S.in);
  float* out = reinterpret_cast<float*>(smem + S.out);
  f32x4* red = reinterpret_cast<f32x4*>(smem + S.red);
  const uint16_t* nbr = reinterpret_cast<const uint16_t*>(smem + S.nbr);
  double* ms = reinterpret_cast<double*>(smem + S.st);  // sums of g xhat and g of hidden i
  double* acc = ms + 2 * kMaxC;                         // and of hidden i - 1
  if constexpr (LF) {
    copy_frags(frags, smem + S.frags, c.nct * c.per_ct());
    frags = reinterpret_cast<const u32x4*>(smem + S.frags);
  }
  const bool norm = A.i + 1 < d.n_conv;
  const int cg = c.ck, cx = c.rows, qin = norm ? (cg + 3) >> 2 : 1;
  const double n_all = (double)A.B * V;
  // as in kb_conv: mean, r and gamma of hidden i, the thread's first quads
  double* mr = ms + 4 * kMaxC;
  float* ab = reinterpret_cast<float*>(smem + S.ab);
  f32x4 pg{}, pa{};
  float ga = 0.f, t0 = 0.f, t1 = 0.f;
  double mrv = 0.0;
  BnPart part{0.0, 0.0};
  if (norm) part = first_part(A.part, cg, G);
  if (threadIdx.x < qin * V) {
    const float* st = A.store + (size_t)blockIdx.x * A.ss;
    pg = *reinterpret_cast<const f32x4*>(st + ((size_t)A.gin * V + threadIdx.x) * 4);
    if (norm) pa = *reinterpret_cast<const f32x4*>(st + ((size_t)A.ain * V + threadIdx.x) * 4);
  }
  if (norm && threadIdx.x < 2 * cg) mrv = A.mr[threadIdx.x];
  if (norm && threadIdx.x < cg) ga = A.gamma[threadIdx.x];
  if constexpr (FIELD) {
    t0 = touch(A.gx + (size_t)blockIdx.x * V, V);
  } else {
    const float* st = A.store + (size_t)blockIdx.x * A.ss;
    const int n = ((cx + 3) >> 2) * V;  // every sixteenth byte
    if (threadIdx.x < n) {
      t0 = st[((size_t)A.hout * V + threadIdx.x) * 4];
      t1 = st[((size_t)A.aout * V + threadIdx.x) * 4];
    }
  }
  bn_tables<DIM>(d, S, smem);
  keep(t0, t1);
  if (norm) {
    if (threadIdx.x < 2 * cg) mr[threadIdx.x] = mrv;
    if (threadIdx.x < cg) ab[threadIdx.x] = ga;
    for (int ch = w; ch < cg; ch += nw) {
      double s0 = ch < nw ? part.a : 0.0, s1 = ch < nw ? part.b : 0.0;
      for (int g = ch < nw ? lane + 64 : lane; g < G; g += 64) {
        s0 += A.part[ch * G + g];
        s1 += A.part[(cg + ch) * G + g];
      }
      s0 = wave_sum(s0);
      s1 = wave_sum(s1);
      if (lane == 0) {
        ms[ch] = s0;
        ms[kMaxC + ch] = s1;
        if (blockIdx.x == 0) {
          A.gg[ch] = (float)s0;
          A.gg[cg + ch] = (float)s1;
        }
      }
    }
  }
  if constexpr (!FIELD)
    for (int ch = threadIdx.x; ch < 2 * kMaxC; ch += blockDim.x) acc[ch] = 0.0;
  __syncthreads();
  if constexpr (LF) wait_copies();
  for (int b = blockIdx.x; b < A.B; b += G) {
    float* st = A.store + (size_t)b * A.ss;
    for (int e = threadIdx.x; e < qin * V; e += blockDim.x) {
      const int q = fdiv(e, lat.dV), n = e - q * V;
      f32x4* gp = reinterpret_cast<f32x4*>(st + ((size_t)(A.gin + q) * V + n) * 4);
      const bool far = b != (int)blockIdx.x || e >= blockDim.x;
      f32x4 g = pg;
      if (far) g = *gp;
      if (norm) {
        f32x4 a = pa;
        if (far) a = *reinterpret_cast<const f32x4*>(st + ((size_t)(A.ain + q) * V + n) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ch = min(4 * q + r, cg - 1);
          const double mu = mr[ch], rs = mr[cg + ch];
          double ga = (double)g[r];
          if (A.batch) ga -= ms[kMaxC + ch] / n_all + (double)bn_xhat(a[r], mu, rs) * (ms[ch] / n_all);
          g[r] = masked((float)((double)ab[ch] * rs * ga), (4 * q + r - cg) >> 31);
        }
        *gp = g;
      }
      *reinterpret_cast<f32x4*>(in + q * S.ps + 4 * n) = g;
    }
    lds_barrier();
    if constexpr (FIELD) {
      float* gx = A.gx + (size_t)b * V;
      conv_pass<MODE, true, FEW>((half + 15) >> 4, c, frags, red, [&](int tile) {
        return lds_planes<true>(d, nbr, S.ps, in, half_site<DIM>(lat, min(tile * 16 + m, half - 1), A.fpar));
      }, [&](int tile, int, const f32x4& v) {
        const int a = tile * 16 + m;
        if (j == 0 && a < half) gx[half_site<DIM>(lat, a, A.fpar)] += v[0];
      });
    } else {
      conv_pass<MODE, true, FEW>((V + 15) >> 4, c, frags, red, [&](int tile) {
        return lds_planes<true>(d, nbr, S.ps, in, min(tile * 16 + m, V - 1));
      }, [&](int tile, int ct, const f32x4& v) {
        const int n = tile * 16 + m, pl = ct * 4 + j;
        if (n < V && 4 * pl < cx) {
          const f32x4 h = *reinterpret_cast<const f32x4*>(st + ((size_t)(A.hout + pl) * V + n) * 4);
          f32x4 g;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            g[r] = masked(v[r] * leaky_grad_from_out(h[r]), (4 * pl + r - cx) >> 31);
          *reinterpret_cast<f32x4*>(out + pl * S.ps + 4 * n) = g;
          *reinterpret_cast<f32x4*>(st + ((size_t)(A.gout + pl) * V + n) * 4) = g;
        }
      });
      lds_barrier();
      for (int ch = w; ch < cx; ch += nw) {
        const float* g = out + (ch >> 2) * S.ps + (ch & 3);
        const float* a = st + ((size_t)(A.aout + (ch >> 2)) * V) * 4 + (ch & 3);
        const double mu = A.mr_out[ch], rs = A.mr_out[cx + ch];
        double s0 = 0.0, s1 = 0.0;
        for (int n = lane; n < V; n += 64) {
          const double gv = (double)g[4 * n];
          s0 += gv * (double)bn_xhat(a[4 * n], mu, rs);
          s1 += gv;
        }
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        if (lane == 0) {
          acc[ch] += s0;
          acc[kMaxC + ch] += s1;
        }
      }
    }
    lds_barrier();
  }
  if constexpr (!FIELD)
    for (int ch = threadIdx.x; ch < cx; ch += blockDim.x) {
      A.part_out[ch * G + blockIdx.x] = acc[ch];
      A.part_out[(cx + ch) * G + blockIdx.x] = acc[kMaxC + ch];
    }
}

// log q = log r - the layers' log-dets in order.
__global__ void __launch_bounds__(256) kb_end(int B, int N, const double* __restrict__ logr,
                                              const double* __restrict__ ld, double* __restrict__ logq,
                                              double* __restrict__ logdet) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  double s = 0.0;
#pragma unroll 8
  for (int l = 0; l < N; ++l) s += ld[(size_t)l * B + b];
  logq[b] = logr[b] - s;
  if (logdet) logdet[b] = s;
}

// ---- host ------------------------------------------------------------------------

struct BnWs {
  u32x4* frags;
  double *logr, *ld, *part[2], *mr;  // mr: 2 kMaxC per hidden convolution
  float *store, *gA, *gB;
  double* partial;
};
// Workgroups of a launch.  Up to one sample per CU: eight waves each.  More samples: two such
// workgroups per CU; 16 and more samples per CU of a narrow network: four of four waves (4096
// samples of 8 x 8, hidden [8, 8], 4 layers: 533 us forward with one workgroup per CU, 390
// with two, 381 with four; hidden [32, 32], whose merges are longer, 2048 samples: 601, 536
// and 1122).
struct BnGrid {
  int blocks, waves;
};
BnGrid bn_grid(const NetDev& d, int B) {
  const int cus = num_cus();
  int widest = 0;
  for (int i = 0; i + 1 < d.n_conv; ++i) widest = std::max(widest, d.cout[i]);
  if (B <= cus) return BnGrid{B, kResWaves};
  if (B < 16 * cus || widest > 8) return BnGrid{std::min(B, 2 * cus), kResWaves};
  return BnGrid{4 * cus, kResWaves / 2};
}

constexpr int kBnPlanes(int hp, bool bwd) { return bwd ? 3 * hp + 1 : hp; }

BnWs bn_carve(const NetDev& d, int B, bool bwd, char* base, size_t* total) {
  BnWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align_up(bytes);
    return p;
  };
  const size_t BV = (size_t)B * d.lat.V;
  const int planes = kBnPlanes(d.hplanes, bwd), group = bwd ? layer_group(d, B, planes) : 1;
  w.frags = (u32x4*)take((size_t)d.N * (bwd ? d.frags_all : d.frags_fwd) * 1024);
  w.logr = (double*)take(sizeof(double) * B);
  w.ld = (double*)take(bwd ? 0 : sizeof(double) * B * d.N);
  for (auto& p : w.part) p = (double*)take(sizeof(double) * 2 * kMaxC * (size_t)bn_grid(d, B).blocks);
  w.mr = (double*)take(sizeof(double) * 2 * kMaxC * LFS_MAX_HIDDEN);
  w.store = (float*)take((size_t)group * BV * planes * 16);
  if (bwd) {
    w.gA = (float*)take(4 * BV);
    w.gB = (float*)take(4 * BV);
    w.partial = (double*)take(partial_bytes(d, B, group, planes));
  }
  *total = off;
  return w;
}

void set_counts(BnIn& in, int B, int V, int G) {
  in.inv_n = 1.0 / ((double)B * V);
  in.inv_cnt[0] = 1.0 / ((double)((B + G - 1) / G) * V);
  in.inv_cnt[1] = 1.0 / ((double)((B - (G - 1) + G - 1) / G) * V);
}

template <int DIM, int MODE, Kind KIND>
int32_t launch_conv(const NetDev& d, const BnLds& S, const BnConvArgs& a, const u32x4* layer_frags, hipStream_t st) {
  const BnGrid G = bn_grid(d, a.B);
  return with_lf(S.lf, G.waves < kResWaves, [&](auto lf, auto few) {
    constexpr auto k = kb_conv<DIM, MODE, decltype(lf)::value, decltype(few)::value, KIND>;
    if (!set_lds_limit<k>(kLdsMax)) return (int32_t)LFS_EDEVICE;
    hipLaunchKernelGGL(k, dim3((unsigned)G.blocks), dim3(64 * G.waves), S.total, st, d, S, a,
                       layer_frags + (size_t)d.f[a.i].off * 64);
    return (int32_t)LFS_OK;
  });
}

// The convolutions of one layer in order, the last one as KIND (a.xout .. set by the caller).
template <int DIM, int MODE, Kind KIND>
int32_t run_layer(const NetDev& d, const BnLds& S, BnConvArgs a, const float* p, const BnWs& w, int aplane, int hplane,
                  const float* running, float* update, const size_t* offS, const u32x4* layer_frags, hipStream_t st) {
  for (int i = 0; i < d.n_conv; ++i) {
    a.i = i;
    a.part = w.part[i & 1];
    a.aout = i + 1 < d.n_conv ? aplane + d.hplane[i] : 0;
    if (i > 0) {
      a.in.gamma = p + d.offg[i - 1];
      a.in.beta = a.in.gamma + d.cout[i - 1];
      a.in.part = w.part[(i - 1) & 1];
      a.in.mr = w.mr + (i - 1) * 2 * kMaxC;
      a.in.running = running ? running + offS[i - 1] : nullptr;
      a.in.update = update ? update + offS[i - 1] : nullptr;
      a.ain = aplane + d.hplane[i - 1];
      a.hin = hplane < 0 ? -1 : hplane + d.hplane[i - 1];
    }
    LFS_TRY(i + 1 < d.n_conv ? (launch_conv<DIM, MODE, Kind::Hidden>(d, S, a, layer_frags, st))
                             : (launch_conv<DIM, MODE, KIND>(d, S, a, layer_frags, st)));
  }
  return LFS_OK;
}

template <int DIM, int MODE>
int32_t forward_impl(const FlowGeom& g, const float* params, int B, const float* z, float* phi, double* logq,
                     double* logdet, float* saved, int bn_mode, float* stats, float momentum, char* ws,
                     hipStream_t st) {
  using R = std::conditional_t<MODE == kBf16, double, float>;
  const NetDev d = make_net(g);
  const BnLds S = bn_lds(d);
  const int V = g.V;
  const size_t BV = (size_t)B * V;
  size_t total;
  const BnWs w = bn_carve(d, B, false, ws, &total);
  prep<MODE>(d, params, d.N, 0, d.frags_fwd, w.frags, st);
  float* x = saved ? saved : phi;
  hipLaunchKernelGGL((kg_begin<R>), dim3(B), dim3(256), 0, st, V, z, x, w.logr);
  for (int l = 0; l < d.N; ++l) {
    BnConvArgs a{};
    a.B = B;
    a.fpar = g.frozen_parity(l);
    a.in.batch = bn_mode == LFS_BN_BATCH;
    set_counts(a.in, B, V, bn_grid(d, B).blocks);
    a.in.momentum = momentum;
    a.x = x;
    a.store = w.store;
    a.ss = (size_t)d.hplanes * V * 4;
    a.xout = saved ? saved + (size_t)(l + 1) * BV : phi;
    a.xout2 = saved && l + 1 == d.N ? phi : nullptr;
    a.ld = w.ld + (size_t)l * B;
    float* sl = stats ? stats + (size_t)l * g.S_layer : nullptr;
    LFS_TRY((run_layer<DIM, MODE, Kind::Couple>(d, S, a, params + (size_t)l * g.P_layer, w, 0, -1, sl, sl, g.offS,
                                                w.frags + (size_t)l * d.frags_fwd * 64, st)));
    x = a.xout;
  }
  hipLaunchKernelGGL(kb_end, dim3(blocks(B)), dim3(256), 0, st, B, d.N, w.logr, w.ld, logq, logdet);
  return launch_status();
}

template <int DIM, int MODE>
int32_t backward_impl(const FlowGeom& g, const float* params, int B, const float* saved, const float* g_phi,
                      double g_logq, const double* g_logq_vec, int bn_mode, const float* stats, float* g_params,
                      float* g_z, char* ws, hipStream_t st) {
  const NetDev d = make_net(g);
  const BnLds S = bn_lds(d);
  const int V = g.V, HP = d.hplanes, PL = kBnPlanes(HP, true), group = layer_group(d, B, PL);
  const size_t BV = (size_t)B * V, ss = (size_t)PL * V * 4;
  size_t total;
  const BnWs w = bn_carve(d, B, true, ws, &total);
  prep<MODE>(d, params, d.N, 0, d.frags_all, w.frags, st);
  const float* gy = g_phi;
  float* bufs[2] = {w.gA, w.gB};
  int which = 0;
  for (int l1 = d.N; l1 > 0;) {
    const int l0 = l1 > group ? l1 - group : 0;
    for (int l = l1 - 1; l >= l0; --l) {
      const float* p = params + (size_t)l * g.P_layer;
      const u32x4* lf = w.frags + (size_t)l * d.frags_all * 64;
      float* sl = w.store + (size_t)(l - l0) * B * ss;
      float* gx = bufs[which];
      const int fpar = g.frozen_parity(l);
      const bool batch = bn_mode == LFS_BN_BATCH;
      BnConvArgs a{};
      a.B = B;
      a.fpar = fpar;
      a.in.batch = batch;
      set_counts(a.in, B, V, bn_grid(d, B).blocks);
      a.x = saved + (size_t)l * BV;
      a.store = sl;
      a.ss = ss;
      a.xout = gx;
      a.gy = gy;
      a.gld = (float)(-g_logq);
      a.gld_vec = g_logq_vec;
      a.go = 2 * HP;
      LFS_TRY((run_layer<DIM, MODE, Kind::Affine>(d, S, a, p, w, 2 * HP + 1, 0,
                                                  batch ? nullptr : stats + (size_t)l * g.S_layer, nullptr, g.offS, lf,
                                                  st)));
      for (int i = d.n_conv - 1; i >= 0; --i) {
        const bool last = i + 1 == d.n_conv;
        BnGradArgs q{};
        q.i = i;
        q.B = B;
        q.fpar = fpar;
        q.batch = batch;
        q.store = sl;
        q.ss = ss;
        q.gin = last ? 2 * HP : HP + d.hplane[i];
        if (!last) {
          q.ain = 2 * HP + 1 + d.hplane[i];
          q.mr = w.mr + i * 2 * kMaxC;
          q.gamma = p + d.offg[i];
          q.part = w.part[i & 1];
          q.gg = g_params + (size_t)l * g.P_layer + d.offg[i];
        }
        if (i > 0) {
          q.gout = HP + d.hplane[i - 1];
          q.hout = d.hplane[i - 1];
          q.aout = 2 * HP + 1 + d.hplane[i - 1];
          q.mr_out = w.mr + (i - 1) * 2 * kMaxC;
          q.part_out = w.part[(i - 1) & 1];
        }
        q.gx = gx;
        const u32x4* fr = lf + (size_t)d.t[i].off * 64;
        auto launch = [&](auto field) {
          const BnGrid G = bn_grid(d, B);
          return with_lf(S.lf, G.waves < kResWaves, [&](auto in_lds, auto few) {
            constexpr auto k = kb_grad<DIM, MODE, decltype(in_lds)::value, decltype(few)::value, decltype(field)::value>;
            if (!set_lds_limit<k>(kLdsMax)) return (int32_t)LFS_EDEVICE;
            hipLaunchKernelGGL(k, dim3((unsigned)G.blocks), dim3(64 * G.waves), S.total, st, d, S, q, fr);
            return (int32_t)LFS_OK;
          });
        };
        LFS_TRY(i == 0 ? launch(std::true_type{}) : launch(std::false_type{}));
      }
      gy = gx;
      which ^= 1;
    }
    LFS_TRY((run_wgrad<DIM, MODE>(d, B, l0, l1 - l0, PL, w.store, saved, w.partial, g_params, st)));
    l1 = l0;
  }
  if (g_z)
    hipLaunchKernelGGL(kg_gz, dim3(blocks((int64_t)BV)), dim3(256), 0, st, (int64_t)BV, gy, saved, (float)g_logq,
                       g_logq_vec, (int64_t)V, g_z);
  return launch_status();
}

// f(integral constants of the dimension and the mode); with batch norm no network is the
// default one, so FP32 is Tree.
template <class F>
int32_t bn_dispatch(const FlowGeom& g, F&& f) {
  auto mode = [&](auto dim) {
    return g.bf16() ? f(dim, std::integral_constant<int, kBf16>{}) : f(dim, std::integral_constant<int, kTree>{});
  };
  return g.dim == 2 ? mode(std::integral_constant<int, 2>{}) : mode(std::integral_constant<int, 3>{});
}

}  // namespace

bool bn_resident(const FlowGeom& g) { return g.V < 65536 && (size_t)bn_lds(make_net(g)).total <= kLdsMax; }

size_t bn_ws_bytes(const FlowGeom& g, int B, int for_backward) {
  size_t total;
  bn_carve(make_net(g), B, for_backward != 0, nullptr, &total);
  return kWsAlign + total;
}

int32_t bn_forward(const FlowGeom& g, const float* params, int B, const float* z, float* phi, double* logq,
                   double* logdet, float* saved, int bn_mode, float* stats, float momentum, char* ws,
                   hipStream_t st) {
  size_t unused = kWsAlign;
  ws = aligned_ws(ws, &unused);
  return bn_dispatch(g, [&](auto dim, auto mode) {
    return forward_impl<decltype(dim)::value, decltype(mode)::value>(g, params, B, z, phi, logq, logdet, saved, bn_mode,
                                                                     stats, momentum, ws, st);
  });
}

int32_t bn_backward(const FlowGeom& g, const float* params, int B, const float* saved, const float* g_phi,
                    double g_logq, const double* g_logq_vec, int bn_mode, const float* stats, float* g_params,
                    float* g_z, char* ws, hipStream_t st) {
  size_t unused = kWsAlign;
  ws = aligned_ws(ws, &unused);
  return bn_dispatch(g, [&](auto dim, auto mode) {
    return backward_impl<decltype(dim)::value, decltype(mode)::value>(g, params, B, saved, g_phi, g_logq, g_logq_vec,
                                                                      bn_mode, stats, g_params, g_z, ws, st);
  });
}

}  // namespace lfs
